"""GPU parity of the transcoder's large launches, in both block sizes and all layouts of K, against the CPU oracle.  Bar: blobs byte for byte."""
import numpy as np
import pytest

import kv_inputs as gen
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

F16, BF16 = gen.F16, gen.BF16
TDT = {F16: torch.float16, BF16: torch.bfloat16}


@pytest.fixture(scope="module")
def kvh():
    import paper_2509_00105_amd as m

    m.lib()
    return m


def awkward(k, v, dt, rng):
    """Some groups with a maximum close to zero against the range, far from zero, and constant."""
    n, c = k.shape[1:]
    x = oracle.t16_to_f32_array(k.ravel(), dt).reshape(k.shape)
    y = oracle.t16_to_f32_array(v.ravel(), dt).reshape(v.shape)
    for ch in rng.integers(0, c, 12):
        x[:, :, ch] = -np.abs(x[:, :, ch])
        x[:, 0, ch] = np.float32(2.0 ** -13)
    for ch in rng.integers(0, c, 12):
        x[:, :, ch] = x[:, :, ch] * np.float32(2.0 ** -6) + np.float32(rng.choice([1.0, 40.0]))
    x[:, :, rng.integers(0, c)] = 0.5
    for t in rng.integers(0, n, max(1, n // 8)):
        h = int(rng.integers(0, c // 128)) * 128
        y[:, t, h:h + 128] = y[:, t, h:h + 128] * np.float32(2.0 ** -5) + np.float32(8.0)
    return tuple(oracle.f32_to_t16_array(t.ravel(), dt).reshape(k.shape) for t in (x, y))


# heads: items of the 300-token entry below, so that launches of 1 layer take blocks of up to 8 waves and (5 to 8 heads) of up to 4
ITEMS = {1: (500,), 2: (250,), 3: (340,), 4: (260,), 5: (100, 160), 6: (95, 140), 7: (60, 300), 8: (60, 250), 9: (40,), 10: (40,), 11: (35,),
         12: (30,), 13: (20, 50), 16: (20,), 20: (4,), 24: (4,), 25: (3, 30)}


@pytest.mark.parametrize("dt", [F16, BF16])
@pytest.mark.parametrize("heads", sorted(ITEMS))
def test_large_launches_match_oracle(kvh, heads, dt):
    l, c, lens = 1, 128 * heads, (300, 129, 64, 1)
    rng = np.random.default_rng(heads)
    entries = [awkward(*gen.make_kv(l, n, c, dt, seed=heads + n), dt, rng) for n in lens]
    for a, b in ((0, 1), (0, 2), (1, 2), (2, 0), (1, 1)):
        srcs = [oracle.encode(k, v, dt, a) for k, v in entries]
        wants = [oracle.transcode(s, dt, l, n, c, a, b) for s, n in zip(srcs, lens)]
        dev = [torch.from_numpy(s).cuda() for s in srcs]
        for count in ITEMS[heads]:
            which = [i % len(lens) for i in range(count)]
            at = np.concatenate([[0], np.cumsum([wants[w].size for w in which])])
            out = torch.full((int(at[-1]) + 64,), 0xAB, dtype=torch.uint8, device="cuda")
            status = torch.zeros(count, dtype=torch.int32, device="cuda")
            items = kvh.make_tc_items([dev[w].data_ptr() for w in which], [out.data_ptr() + int(o) for o in at[:-1]], [lens[w] for w in which],
                                      [a] * count, [b] * count, out.device)
            kvh.transcode_batch(items, count, max(lens), TDT[dt], l, c, status=status)
            torch.cuda.synchronize()
            assert int(status.abs().sum()) == 0
            got = out.cpu().numpy()
            for i, w in enumerate(which):
                assert np.array_equal(got[at[i]:at[i + 1]], wants[w]), (heads, count, i, lens[w], "%d->%d" % (a, b))
            assert (got[at[-1]:] == 0xAB).all()


@pytest.mark.parametrize("dt", [F16, BF16])
def test_large_launches_of_short_items_of_one_head(kvh, dt):
    """Items of two token-groups, which fill half of a block."""
    l, c, lens, count = 4, 128, (256, 129, 1), 640
    entries = [awkward(*gen.make_kv(l, n, c, dt, seed=n), dt, np.random.default_rng(n)) for n in lens]
    for a, b in ((0, 1), (0, 2), (1, 2)):
        srcs = [oracle.encode(k, v, dt, a) for k, v in entries]
        wants = [oracle.transcode(s, dt, l, n, c, a, b) for s, n in zip(srcs, lens)]
        dev = [torch.from_numpy(s).cuda() for s in srcs]
        pitch = max(w.size for w in wants) + 16
        out = torch.full((count, pitch), 0xAB, dtype=torch.uint8, device="cuda")
        items = kvh.make_tc_items([dev[i % 3].data_ptr() for i in range(count)], [o.data_ptr() for o in out], [lens[i % 3] for i in range(count)],
                                  [a] * count, [b] * count, out.device)
        kvh.transcode_batch(items, count, 256, TDT[dt], l, c)
        got = out.cpu().numpy()
        for i in range(count):
            w = wants[i % 3]
            assert np.array_equal(got[i, :w.size], w) and (got[i, w.size:] == 0xAB).all(), (i, a, b)
