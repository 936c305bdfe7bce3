"""GPU parity over row lengths: heads per row that do and do not fill a wave's span, token counts at the edges of the
units that rows of 1, 2, 4 and 8 heads are cut into, layer counts that split unevenly into plane groups.  Bit equality
with the oracle throughout (the definition fixes every bit)."""
import numpy as np
import pytest

import kv_inputs as gen
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TDT = {gen.F16: torch.float16, gen.BF16: torch.bfloat16}
CASES = [(heads, l, dt) for heads, l, dt in (
    (1, 2, gen.BF16), (1, 5, gen.F16), (2, 1, gen.F16), (2, 9, gen.BF16), (3, 3, gen.BF16), (4, 4, gen.F16), (5, 7, gen.BF16),
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
    """Whole spans on both sides of the sizes at which the decoder changes its block order and occupancy (288 MiB and 1.1 GiB
    of rows here; the other tests decode less than 256 MiB): every row equals what 640-token pieces of the entry give."""
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
