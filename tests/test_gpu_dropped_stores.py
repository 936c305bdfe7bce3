"""Token-dropped entries on both sides of the size up to which their codes are stored plainly, in device and in pinned host memory: the blob is that of the
kept rows encoded by themselves (which other tests hold against the oracle), with the token-dropping words in its header, and nothing beyond it is written."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# layers, channels, level, kept tokens: blobs just below and just above 96 MiB in strips and in slots, small ones, raw ones
CASES = [(32, 1024, 1, 2889), (32, 1024, 1, 2890), (40, 640, 0, 1906), (40, 640, 0, 1907), (32, 1024, 2, 700), (3, 640, 1, 129), (4, 1024, 3, 200), (3, 640, 3, 129)]


@pytest.mark.parametrize("l, c, level, kept", CASES)
def test_blobs(l, c, level, kept):
    import paper_2509_00105_amd as kvh

    n, sink = kept + 37, 5
    g = torch.Generator(device="cuda")
    g.manual_seed(kept)
    kv = torch.randn((2, l, n, c), generator=g, device="cuda").to(torch.bfloat16)
    size = kvh.blob_size(l, kept, c, level)
    want = kvh.encode(*[torch.cat([x[:, :sink], x[:, n - kept + sink:]], dim=1) for x in kv], level).clone()
    want[32:44] = torch.from_numpy(np.array([n, sink, kept - sink], np.uint32).view(np.uint8)).cuda()
    for out in (torch.full((size + 64,), 0xAB, dtype=torch.uint8, device="cuda"), torch.full((size + 64,), 0xAB, dtype=torch.uint8).pin_memory()):
        kvh.encode_kept(kv[0], kv[1], sink, kept - sink, level, blob=out)
        torch.cuda.synchronize()
        got = out.cuda()
        assert torch.equal(got[:size], want[:size]) and (got[size:] == 0xAB).all()


def test_the_sizes_lie_on_both_sides():
    import paper_2509_00105_amd as kvh

    assert [kvh.blob_size(l, kept, c, level) <= 96 << 20 for l, c, level, kept in CASES[:4]] == [True, False, True, False]
