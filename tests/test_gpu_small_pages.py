"""2-bit entries into small pages, whose stores take another form in launches of slots: the rows are those of a contiguous decode of the same blobs
(which other tests hold against the oracle), bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("l, c, lens, page", [(32, 1024, [256] * 17 + [203], 16), (4, 1024, [256, 100, 1], 16), (3, 640, [300, 129], 32), (5, 128, [515], 16),
                                              (40, 640, [256] * 9, 16), (80, 640, [256] * 20 + [203], 16)])
@pytest.mark.parametrize("dt", [torch.float16, torch.bfloat16])
def test_rows_of_small_pages(l, c, lens, page, dt):
    import paper_2509_00105_amd as kvh

    total = sum(lens)
    g = torch.Generator(device="cuda")
    g.manual_seed(l + c)
    kv = torch.randn((2, l, total, c), generator=g, device="cuda").to(dt)
    kv[0, :, :, 5] = -kv[0, :, :, 5].abs()  # a few groups that need the rule for top codes
    kv[0, :, 0, 5] = 2.0 ** -13
    kv[1, :, 3::50] = -kv[1, :, 3::50].abs()
    kv[1, :, 3::50, 7::128] = 2.0 ** -13
    sizes = [kvh.blob_size(l, n, c, 2) for n in lens]
    at = np.concatenate([[0], np.cumsum(sizes)])
    first = np.concatenate([[0], np.cumsum(lens)])[:-1].tolist()
    blobs = torch.empty(int(at[-1]), dtype=torch.uint8, device="cuda")
    ptrs = [blobs.data_ptr() + int(o) for o in at[:-1]]
    kvh.encode_batch(kvh.make_enc_items(ptrs, first, lens, [2] * len(lens), kv.device), len(lens), max(lens), kv[0], kv[1])
    dense = torch.zeros_like(kv)
    kvh.decode_batch(kvh.make_dec_items(ptrs, lens, [2] * len(lens), first, [0] * len(lens), kv.device), len(lens), max(lens), dense[0], dense[1])
    pages = -(-total // page) + 3
    table = torch.from_numpy(np.random.default_rng(c).permutation(pages).astype(np.int32)).cuda()
    cache = torch.full((2, l, pages, page, c), -7.0, dtype=dt, device="cuda")
    kvh.decode_batch(kvh.make_dec_items(ptrs, lens, [2] * len(lens), first, [table.data_ptr()] * len(lens), kv.device), len(lens), max(lens), cache[0],
                     cache[1], paged=True, block_tokens=page)
    pos = torch.arange(pages * page, device="cuda")
    row = table.long()[pos // page] * page + pos % page
    flat = cache.view(2, l, pages * page, c)
    for which in range(2):
        for lam in range(l):
            got = flat[which, lam][row]
            assert torch.equal(got[:total].view(torch.int16), dense[which, lam].view(torch.int16)), (which, lam)
            assert (got[total:] == -7.0).all()
    assert not torch.equal(dense, torch.zeros_like(dense))
