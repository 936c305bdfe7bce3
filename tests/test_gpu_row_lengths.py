"""GPU parity over row lengths: heads per row that do and do not fill a wave's span, token counts at the edges of the
units that rows of 1, 2, 4 and 8 heads are cut into, layer counts whose last plane group is a smaller one (5 layers of 4
heads: groups of 4, 4 and 2 planes; 10 and 11 of 5 heads: 7, 7, 6 and 8, 8, 6).  Bit equality with the oracle throughout (the
definition fixes every bit)."""
import numpy as np
import pytest

import kv_inputs as gen
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TDT = {gen.F16: torch.float16, gen.BF16: torch.bfloat16}
CASES = [(heads, l, dt) for heads, l, dt in (
    (1, 2, gen.BF16), (1, 5, gen.F16), (2, 1, gen.F16), (2, 9, gen.BF16), (3, 3, gen.BF16), (4, 4, gen.F16), (4, 5, gen.BF16), (5, 7, gen.BF16),
    (5, 10, gen.F16), (5, 11, gen.BF16),
    (6, 2, gen.F16), (7, 1, gen.BF16), (8, 2, gen.F16), (10, 2, gen.BF16), (12, 1, gen.F16), (16, 1, gen.BF16))]


@pytest.fixture(scope="module")
def kvh():
    import paper_2509_00105_amd as m

    m.lib()
    return m


def device(bits, dt):
    return torch.from_numpy(bits.view(np.int16)).cuda().view(TDT[dt])


def host(t):
    return t.contiguous().view(torch.int16).cpu().numpy().view(np.uint16)


@pytest.mark.parametrize("heads,l,dt", CASES)
def test_row_lengths(kvh, heads, l, dt):
    c = 128 * heads
    for i, n in enumerate((1, 15, 33, 63, 64, 65, 127, 128, 129, 255, 300, 513)):
        level, to = i % 4, (i + 1) % 3
        k, v = gen.make_kv(l, n, c, dt, seed=100 * heads + i)
        if i % 3 == 0:  # groups whose maximum is close to zero take the explicit top-code rule
            k = np.where(k & 0x7fff, k | 0x8000, k)
        want = oracle.encode(k, v, dt, level)
        blob = kvh.encode(device(k, dt), device(v, dt), level)
        status = torch.zeros(1, dtype=torch.int32, device="cuda")
        out = torch.full((2, l, n + 3, c + 8), 7.0, dtype=TDT[dt], device="cuda")
        kvh.decode(blob, level, n, out[0, :, :, :c], out[1, :, :, :c], dst_token0=2, status=status)
        table = torch.randperm(-(-n // 16) + 1, generator=torch.Generator().manual_seed(i)).to(torch.int32)
        pk = np.zeros((l, len(table) + 1, 16, c), np.uint16)
        pv = np.zeros_like(pk)
        paged = torch.zeros((2, l, len(table) + 1, 16, c), dtype=TDT[dt], device="cuda")
        kvh.decode(blob, level, n, paged[0], paged[1], dst_token0=5, page_table=table.cuda(), block_tokens=16, status=status)
        low = kvh.transcode(blob, dt, l, n, c, level, to, status=status) if level < 3 else None
        torch.cuda.synchronize()
        assert np.array_equal(blob.cpu().numpy(), want), ("encode", n, level)
        wk, wv = oracle.decode(want, dt, l, n, c, level)
        got = host(out)
        assert status.item() == 0 and np.array_equal(got[0, :, 2:2 + n, :c], wk) and np.array_equal(got[1, :, 2:2 + n, :c], wv), ("decode", n, level)
        got[:, :, 2:2 + n, :c] = got[0, 0, 0, 0]
        assert (got == got[0, 0, 0, 0]).all(), ("decode wrote outside its rows", n, level)
        assert oracle.decode_into(want, dt, l, n, c, level, pk, pv, dst_token0=5, page_table=table.numpy(), block_tokens=16) == 0
        assert np.array_equal(host(paged[0]), pk) and np.array_equal(host(paged[1]), pv), ("paged", n, level)
        if low is not None:
            assert np.array_equal(low.cpu().numpy(), oracle.transcode(want, dt, l, n, c, level, to)), ("transcode", n, level, to)


@pytest.mark.parametrize("heads", (1, 5, 8))
def test_row_lengths_batch(kvh, heads):
    """Items of mixed lengths and levels in one launch, the header of one of them broken."""
    l, c, dt = 5, 128 * heads, gen.BF16
    lengths, levels = [1, 300, 64, 129, 700, 65], [0, 1, 2, 3, 2, 0]
    total = sum(lengths)
    k, v = gen.make_kv(l, total, c, dt, seed=heads)
    starts = np.concatenate([[0], np.cumsum(lengths)[:-1]])
    sizes = [kvh.blob_size(l, n, c, lv) for n, lv in zip(lengths, levels)]
    offs = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    buf = torch.zeros(int(offs[-1]), dtype=torch.uint8, device="cuda")
    ptrs = [buf.data_ptr() + int(o) for o in offs[:-1]]
    kvh.encode_batch(kvh.make_enc_items(ptrs, starts, lengths, levels, "cuda"), len(lengths), 700, device(k, dt), device(v, dt))
    torch.cuda.synchronize()
    buf[int(offs[2])] = 0
    out = torch.zeros((2, l, total, c), dtype=TDT[dt], device="cuda")
    status = torch.zeros(len(lengths), dtype=torch.int32, device="cuda")
    kvh.decode_batch(kvh.make_dec_items(ptrs, lengths, levels, starts, [0] * len(lengths), "cuda"), len(lengths), 700, out[0], out[1],
                     status=status)
    torch.cuda.synchronize()
    assert status.tolist() == [0, 0, 1, 0, 0, 0]
    got, blobs = host(out), buf.cpu().numpy()
    for i, (t0, n, lv) in enumerate(zip(starts, lengths, levels)):
        want = oracle.encode(np.ascontiguousarray(k[:, t0:t0 + n]), np.ascontiguousarray(v[:, t0:t0 + n]), dt, lv)
        if i == 2:
            assert (got[:, :, t0:t0 + n] == 0).all()
            continue
        assert np.array_equal(blobs[offs[i]:offs[i + 1]], want), ("encode", i)
        wk, wv = oracle.decode(want, dt, l, n, c, lv)
        assert np.array_equal(got[0, :, t0:t0 + n], wk) and np.array_equal(got[1, :, t0:t0 + n], wv), ("decode", i)


@pytest.mark.parametrize("l,n", [(9, 8191), (20, 15000)])
def test_launch_sizes(kvh, l, n):
    """Whole spans on both sides of the sizes at which the decoder changes its layout, block order and occupancy: 288 MiB of rows walk
    turns of 4 planes, the last of 2, 1.1 GiB plane by plane, the pieces of 22 MiB are units of slots, those of 50 MiB spans with two
    blocks a compute unit.  Every row equals what 640-token pieces of the entry give."""
    c = 1024
    kv = gen.make_kv_device(l, n, c, gen.BF16, seed=n)
    for level in range(4):
        out, ref = torch.zeros_like(kv), torch.zeros_like(kv)
        kvh.decode(kvh.encode(kv[0], kv[1], level), level, n, out[0], out[1])
        starts = list(range(0, n, 640))  # pieces of whole token-groups, so that their K statistics are the entry's
        for t0 in starts:
            m = min(640, n - t0)
            kvh.decode(kvh.encode(kv[0][:, t0:t0 + m], kv[1][:, t0:t0 + m], level), level, m, ref[0], ref[1], dst_token0=t0)
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), ref.view(torch.int16)), (l, n, level)


@pytest.mark.parametrize("heads", (1, 4, 5, 8, 16))
def test_layers_side_by_side(kvh, heads):
    """[tokens][layers][channels] sources and destinations: the layer stride is below the token stride, and the decoder walks
    all planes instead of groups of them."""
    l, n, c, dt = 5, 300, 128 * heads, gen.BF16
    k, v = gen.make_kv(l, n, c, dt, seed=heads)
    src = torch.stack([device(k, dt).transpose(0, 1), device(v, dt).transpose(0, 1)]).contiguous().transpose(1, 2)
    for level in range(4):
        blob = kvh.encode(src[0], src[1], level)
        out = torch.zeros((2, n + 3, l, c), dtype=TDT[dt], device="cuda").transpose(1, 2)
        status = torch.zeros(1, dtype=torch.int32, device="cuda")
        kvh.decode(blob, level, n, out[0], out[1], dst_token0=2, status=status)
        torch.cuda.synchronize()
        want = oracle.encode(k, v, dt, level)
        wk, wv = oracle.decode(want, dt, l, n, c, level)
        got = host(out)
        assert status.item() == 0 and np.array_equal(blob.cpu().numpy(), want), level
        assert np.array_equal(got[0, :, 2:2 + n], wk) and np.array_equal(got[1, :, 2:2 + n], wv), level
        assert not got[:, :, :2].any() and not got[:, :, 2 + n:].any(), level


def test_row_tiles_with_a_remainder(kvh):
    """A batch of whole spans above 896 MiB over planes more than 1 GiB apart: row tiles of 4 blocks, and 300 tokens are 5
    blocks, so that the last tile holds one.  Every row equals what the items give one at a time."""
    l, m, items, c = 9, 300, 100, 1024
    kv = gen.make_kv_device(l, m * items, c, gen.BF16, seed=3)
    starts, lengths, levels = [m * i for i in range(items)], [m] * items, [i % 4 for i in range(items)]
    offs = np.concatenate([[0], np.cumsum([kvh.blob_size(l, m, c, lv) for lv in levels])]).astype(np.int64)
    blobs = torch.zeros(int(offs[-1]), dtype=torch.uint8, device="cuda")
    ptrs = [blobs.data_ptr() + int(o) for o in offs[:-1]]
    kvh.encode_batch(kvh.make_enc_items(ptrs, starts, lengths, levels, "cuda"), items, m, kv[0], kv[1])
    out, ref = torch.zeros_like(kv), torch.zeros_like(kv)
    status = torch.zeros(items, dtype=torch.int32, device="cuda")
    kvh.decode_batch(kvh.make_dec_items(ptrs, lengths, levels, starts, [0] * items, "cuda"), items, m, out[0], out[1], status=status)
    for i, lv in enumerate(levels):
        kvh.decode(blobs[int(offs[i]):int(offs[i + 1])], lv, m, ref[0], ref[1], dst_token0=starts[i])
    torch.cuda.synchronize()
    assert not status.any() and torch.equal(out.view(torch.int16), ref.view(torch.int16))
    assert out.any()


@pytest.mark.parametrize("l,items,m", [(11, 8, 300), (31, 13, 600), (57, 10, 660)])
def test_turns_of_planes_through_all_items(kvh, l, items, m):
    """Batches of whole spans of 103 MiB to 1.4 GiB: planes 4 or 8 at a time through all items, the last turn a smaller one.  Every
    row equals what the items give one at a time."""
    c = 1024
    kv = gen.make_kv_device(l, m * items, c, gen.BF16, seed=l)
    starts, lengths, levels = [m * i for i in range(items)], [m - i for i in range(items)], [i % 4 for i in range(items)]
    offs = np.concatenate([[0], np.cumsum([kvh.blob_size(l, n, c, lv) for n, lv in zip(lengths, levels)])]).astype(np.int64)
    blobs = torch.zeros(int(offs[-1]), dtype=torch.uint8, device="cuda")
    ptrs = [blobs.data_ptr() + int(o) for o in offs[:-1]]
    kvh.encode_batch(kvh.make_enc_items(ptrs, starts, lengths, levels, "cuda"), items, m, kv[0], kv[1])
    out, ref = torch.zeros_like(kv), torch.zeros_like(kv)
    status = torch.zeros(items, dtype=torch.int32, device="cuda")
    kvh.decode_batch(kvh.make_dec_items(ptrs, lengths, levels, starts, [0] * items, "cuda"), items, m, out[0], out[1], status=status)
    for i, lv in enumerate(levels):
        kvh.decode(blobs[int(offs[i]):int(offs[i + 1])], lv, lengths[i], ref[0], ref[1], dst_token0=starts[i])
    torch.cuda.synchronize()
    assert not status.any() and torch.equal(out.view(torch.int16), ref.view(torch.int16))
    assert out.any()


# heads -> items of 2 layers x 300 tokens in launches of up to 144, 256 and 400 blocks of strips, and more
ENCODER_ITEMS = {heads: items for group, items in (((3, 4), (1, 13, 22, 40)), ((5, 6, 7, 8), (1, 7, 11, 20)), ((9, 10, 12), (1, 5, 8, 14)),
                                                   ((16,), (1, 4, 6, 10)), ((17,), (1, 3, 5, 7))) for heads in group}


@pytest.mark.parametrize("dt", [gen.F16, gen.BF16])
@pytest.mark.parametrize("heads", list(ENCODER_ITEMS))
def test_encode_forms(kvh, heads, dt):
    """The same rows encoded as often as it takes for the launch to go through slots in blocks of 4 waves and through the layouts
    of middling and of large launches.  Every blob equals the oracle's, and nothing is written between them."""
    l, n, c = 2, 300, 128 * heads
    k, v = gen.make_kv(l, n, c, dt, seed=heads)
    kd, vd = device(k, dt), device(v, dt)
    for level in range(4):
        want = torch.from_numpy(oracle.encode(k, v, dt, level)).cuda()
        for items in ENCODER_ITEMS[heads]:
            out = torch.full((items, want.numel() + 32), 0xAB, dtype=torch.uint8, device="cuda")
            ptrs = [out.data_ptr() + i * out.shape[1] for i in range(items)]
            kvh.encode_batch(kvh.make_enc_items(ptrs, [0] * items, [n] * items, [level] * items, "cuda"), items, n, kd, vd)
            torch.cuda.synchronize()
            assert torch.equal(out[:, : want.numel()], want.expand(items, -1)), (level, items)
            assert (out[:, want.numel():] == 0xAB).all(), (level, items)


@pytest.mark.parametrize("dt", [gen.F16, gen.BF16])
@pytest.mark.parametrize("heads,copies", [(8, 1), (8, 96), (16, 48)])
def test_one_blob_many_times(kvh, heads, copies, dt):
    """One blob decoded once (units of slots) and so often that the launch takes spans (225 MiB): groups whose maximum is close
    to zero (the explicit top-code rule) among others, 300 tokens (a last block of 44 rows), contiguous, paged, and token-dropped
    with the kept tokens back in their places.  Every copy equals the oracle."""
    l, n, c = 2, 300, 128 * heads
    k, v = gen.make_kv(l, n, c, dt, seed=heads + copies)
    half = np.arange(c) < c // 2
    k, v = np.where(half & (k & 0x7fff != 0), k | 0x8000, k), np.where(~half & (v & 0x7fff != 0), v | 0x8000, v)
    orig, sink, window = 340, 100, 200
    words = np.array([orig, sink, window], np.uint32).view(np.uint8)
    pages = -(-n // 16)
    for level in range(4):
        blob = oracle.encode(k, v, dt, level)
        wk, wv = (device(x, dt).view(torch.int16) for x in oracle.decode(blob, dt, l, n, c, level))
        src, dropped = torch.from_numpy(blob).cuda(), torch.from_numpy(blob).cuda()
        dropped[32:44] = torch.from_numpy(words).cuda()
        status = torch.zeros(copies, dtype=torch.int32, device="cuda")
        one = lambda x: [x] * copies

        def check(out, at):
            torch.cuda.synchronize()
            assert not status.any(), (level, at)
            got = out.view(torch.int16).view(2, l, copies, -1, c)
            if at == "dropped":
                assert not got[:, :, :, sink:orig - window].any()
                got = torch.cat([got[:, :, :, :sink], got[:, :, :, orig - window:orig]], dim=3)
            got = got[:, :, :, :n]
            assert torch.equal(got[0], wk[:, None].expand_as(got[0])) and torch.equal(got[1], wv[:, None].expand_as(got[1])), (level, at)

        out = torch.zeros((2, l, copies * n, c), dtype=TDT[dt], device="cuda")
        kvh.decode_batch(kvh.make_dec_items(one(src.data_ptr()), one(n), one(level), [i * n for i in range(copies)], one(0), "cuda"), copies, n,
                         out[0], out[1], status=status)
        check(out, "contiguous")
        out = torch.zeros((2, l, copies * pages, 16, c), dtype=TDT[dt], device="cuda")
        tables = torch.arange(copies * pages, dtype=torch.int32, device="cuda").view(copies, pages)
        kvh.decode_batch(kvh.make_dec_items(one(src.data_ptr()), one(n), one(level), one(0), [t.data_ptr() for t in tables], "cuda"), copies, n,
                         out[0], out[1], paged=True, status=status)
        check(out, "paged")
        out = torch.zeros((2, l, copies * orig, c), dtype=TDT[dt], device="cuda")
        kvh.decode_kept_batch(kvh.make_kept_items(one(dropped.data_ptr()), one(n), one(level), [i * orig for i in range(copies)], one(0), one(orig),
                                                  one(sink), one(window), one(0), "cuda"), copies, n, out[0], out[1], status=status)
        check(out, "dropped")


@pytest.mark.parametrize("heads", (1, 2, 3, 5, 6, 12))
def test_refused_items(kvh, heads):
    """Items that break a batched call's limits are refused as a whole in the layouts of these rows too: more tokens than the
    launch covers, rows outside the 31-bit range, a bad level.  Their buffers keep every byte."""
    l, c, dt, bound = 3, 128 * heads, gen.F16, 200
    lengths, levels, starts = [200, 201, 70, 64, 65], [0, 1, 2, 3, 1], [0, 200, 420, 500, 600]
    k, v = gen.make_kv(l, 700, c, dt, seed=heads)
    kd, vd = device(k, dt), device(v, dt)
    wants = [oracle.encode(np.ascontiguousarray(k[:, t:t + n]), np.ascontiguousarray(v[:, t:t + n]), dt, lv)
             for t, n, lv in zip(starts, lengths, levels)]
    bufs = [torch.full((w.size,), 0xA7, dtype=torch.uint8, device="cuda") for w in wants]
    ptrs = [b.data_ptr() for b in bufs]
    kvh.encode_batch(kvh.make_enc_items(ptrs, starts, lengths, [0, 1, 7, 3, 1], "cuda"), 5, bound, kd, vd)
    torch.cuda.synchronize()
    for i, (b, w) in enumerate(zip(bufs, wants)):
        assert (b.cpu().numpy() == 0xA7).all() if i in (1, 2) else np.array_equal(b.cpu().numpy(), w), ("encode", i)
    blobs = [torch.from_numpy(w).cuda() for w in wants]
    out = torch.full((2, l, 700, c), 9.0, dtype=TDT[dt], device="cuda")
    rows = [0, 200, 420, 2**31 - 60, -8]
    status = torch.zeros(5, dtype=torch.int32, device="cuda")
    kvh.decode_batch(kvh.make_dec_items([b.data_ptr() for b in blobs], lengths, levels, rows, [0] * 5, "cuda"), 5, bound, out[0], out[1],
                     status=status)
    torch.cuda.synchronize()
    assert status.tolist() == [0, 1, 0, 1, 1]
    got, untouched = host(out), np.ones(700, bool)
    for i in (0, 2):
        wk, wv = oracle.decode(wants[i], dt, l, lengths[i], c, levels[i])
        at = slice(rows[i], rows[i] + lengths[i])
        assert np.array_equal(got[0, :, at], wk) and np.array_equal(got[1, :, at], wv), ("decode", i)
        untouched[at] = False
    assert (got[:, :, untouched] == got[0, 0, 699, 0]).all() and got[0, 0, 699, 0] == np.float16(9.0).view(np.uint16)
    lows = [torch.full((kvh.blob_size(l, n, c, 2),), 0x3C, dtype=torch.uint8, device="cuda") for n in lengths]
    status.zero_()
    kvh.transcode_batch(kvh.make_tc_items([b.data_ptr() for b in blobs], [b.data_ptr() for b in lows], lengths, levels, [2, 2, 2, 2, 9], "cuda"),
                        5, bound, dt, l, c, status=status)
    torch.cuda.synchronize()
    assert status.tolist() == [0, 1, 0, 1, 1]
    for i, low in enumerate(lows):
        want = oracle.transcode(wants[i], dt, l, lengths[i], c, levels[i], 2) if i in (0, 2) else 0x3C
        assert (low.cpu().numpy() == want).all(), ("transcode", i)


@pytest.mark.parametrize("heads", (1, 2, 3, 5, 6))
def test_non_finite_rows_stay_inside_the_blob(kvh, heads):
    """Codes of non-finite input are unspecified, but nothing is written outside the blob, the header is as for finite input,
    and a V group of finite values is stored as the oracle stores it."""
    l, n, c = 2, 129, 128 * heads
    for dt, bad in ((gen.F16, (0x7C00, 0xFC00, 0x7E00)), (gen.BF16, (0x7F80, 0xFF80, 0x7FC0))):
        k, v = gen.make_kv(l, n, c, dt, seed=heads)
        hit = np.random.default_rng(heads).random(v.shape) < 1 / 256
        k0, v0 = np.where(hit, 0, k).astype(np.uint16), np.where(hit, 0, v).astype(np.uint16)
        values = np.resize(np.array(bad, np.uint16), v.shape)
        k, v = np.where(hit, values, k), np.where(hit, values, v)
        clean = ~hit.reshape(l, n, heads, 128).any(-1)
        for level in range(3):
            size, bits = kvh.blob_size(l, n, c, level), kvh.level_bits(level)
            buf = torch.full((size + 8192,), 0xEE, dtype=torch.uint8, device="cuda")
            kvh.encode(device(k, dt), device(v, dt), level, blob=buf[4096:4096 + size])
            torch.cuda.synchronize()
            got, want = buf.cpu().numpy(), oracle.encode(k0, v0, dt, level)
            assert (got[:4096] == 0xEE).all() and (got[4096 + size:] == 0xEE).all(), (dt, level)
            got = got[4096:4096 + size]
            assert np.array_equal(got[:64], want[:64])
            for lam in range(l):
                off = oracle.section_offsets(l, n, c, level, lam)
                for section, width in (("vcodes", 16 * bits), ("vmeta", 4)):
                    a, b = (x[off[section]:off[section] + n * heads * width].reshape(n, heads, width) for x in (got, want))
                    assert np.array_equal(a[clean[lam]], b[clean[lam]]), (dt, level, lam, section)
        assert 0.3 < clean.mean() < 0.9
