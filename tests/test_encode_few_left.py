"""The encoder's launches that leave a few blocks over once the chip has been filled: the rule, on the CPU, and the blobs, on the GPU."""
import numpy as np
import pytest

import kv_inputs as gen
import oracle
from test_launch_plans import plans  # noqa: F401  (the fixture)

# heads, layers, items, tokens: 513 to 575 and 1,025 to 1,087 blocks of strips, and just outside
LEFT = [(8, 10, 1, 1627), (8, 1, 44, 300), (16, 1, 11, 700), (12, 1, 30, 300), (8, 1, 130, 129), (15, 1, 17, 500)]
EVEN = [(8, 4, 1, 4096), (8, 4, 1, 4603), (8, 4, 1, 8192), (8, 4, 1, 8700)]


def test_rule(plans):  # noqa: F811
    """8 heads, 10 x 1,627 tokens at 2 bits: 520 blocks of strips 20.7 us, blocks of 4 waves 18.9; 4 x 5,083 (640): 21.4 and 22.1."""
    form = lambda a, known=False: plans("enc_units", a[0], a[1], a[2], a[3], known=known)[0]
    assert all(form(a) == 4 for a in LEFT) and not any(form(a) for a in EVEN)
    assert form((15, 1, 17, 500), True) == 0 and form((8, 10, 1, 1627), True) == 4  # raw rows that are no whole strips
    # three turns; items that do not fill a token-group, whose raw rows lie in few blocks (8 heads, 135 x 2 x 28 raw: 0.56 of the speed of strips)
    assert not form((8, 1, 1, 49209)) and not any(form((8, 2, 135, n)) for n in (28, 68, 127)) and form((8, 2, 135, 128)) == 4
    assert not any(form((8, l, items, n)) for l, items, n in ((33, 4, 28), (8, 17, 68))) and form((8, 32767, 65535, 2**31 - 1)) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("dt", [gen.F16, gen.BF16])
@pytest.mark.parametrize("shape", LEFT[1:])
def test_blobs(shape, dt):
    import torch

    import paper_2509_00105_amd as kvh

    heads, l, items, n = shape
    c = 128 * heads
    k, v = gen.make_kv(l, n, c, dt, seed=heads)
    tdt = torch.float16 if dt == gen.F16 else torch.bfloat16
    kd, vd = (torch.from_numpy(x.view(np.int16)).cuda().view(tdt) for x in (k, v))
    for level in range(4):
        want = oracle.encode(k, v, dt, level)
        out = torch.full((items, want.size), 0xAB, dtype=torch.uint8, device="cuda")
        jobs = kvh.make_enc_items([out[i].data_ptr() for i in range(items)], [0] * items, [n] * items, [level] * items, out.device)
        kvh.encode_batch(jobs, items, n, kd, vd)
        got = out.cpu().numpy()
        assert all(np.array_equal(g, want) for g in got), (shape, level)
