"""The per-chunk and batched calls through the native call module against the same calls through ctypes: equal results for ordinary
arguments, and what is not ordinary is left to the ctypes way, which accepts or refuses it as it did."""
import numpy as np
import pytest

import kv_inputs as gen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def kvh():
    import paper_2509_00105_amd as m

    m.lib()
    assert m.binding._fast is not None
    return m


def both(kvh, monkeypatch, call):
    """call() by the native module and by ctypes: their results, or the type and text of what they raise."""
    out = []
    for fast in (kvh.binding._fast, None):
        with monkeypatch.context() as m:
            m.setattr(kvh.binding, "_fast", fast)
            try:
                out.append(call())
            except Exception as e:
                out.append((type(e), str(e)))
        torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("dt", [torch.float16, torch.bfloat16])
def test_results_are_those_of_the_ctypes_calls(kvh, monkeypatch, dt):
    l, n, c = 3, 200, 256
    kv = gen.make_kv_device(l, n, c, gen.F16 if dt == torch.float16 else gen.BF16, seed=1)
    side = torch.cuda.Stream()
    table = torch.randperm(13, device="cuda").to(torch.int32)
    for level in range(4):
        for stream in (None, side):
            size = kvh.blob_size(l, n, c, level)

            def encode():
                torch.cuda.synchronize()
                blob = torch.zeros(size, dtype=torch.uint8, device="cuda")
                torch.cuda.synchronize()
                assert kvh.encode(kv[0], kv[1], level, blob=blob, stream=stream) is blob
                return blob

            a, b = both(kvh, monkeypatch, encode)
            assert torch.equal(a, b) and a.any()
            blob = a
            items = kvh.make_enc_items([blob.data_ptr()], [0], [n], [level], "cuda")

            def encode_batch():
                blob.zero_()
                torch.cuda.synchronize()
                assert kvh.encode_batch(items, 1, n, kv[0], kv[1], stream=stream) is None
                torch.cuda.synchronize()
                return blob.clone()

            a2, b2 = both(kvh, monkeypatch, encode_batch)
            assert torch.equal(a2, a) and torch.equal(b2, a)

            def decode(paged, batch, wrong=False):
                shape = (2, l, 14, 16, c) if paged else (2, l, n + 5, c)
                out, status = torch.zeros(shape, dtype=dt, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
                torch.cuda.synchronize()
                lv = (level + 1) % 4 if wrong else level
                src = torch.cat([blob, torch.zeros(1 << 20, dtype=torch.uint8, device="cuda")])
                torch.cuda.synchronize()
                if batch:
                    it = kvh.make_dec_items([src.data_ptr()], [n], [lv], [3], [table.data_ptr() if paged else 0], "cuda")
                    kvh.decode_batch(it, 1, n, out[0], out[1], paged=paged, status=status, stream=stream)
                else:
                    kvh.decode(src, lv, n, out[0], out[1], dst_token0=3, page_table=table if paged else None, status=status, stream=stream)
                torch.cuda.synchronize()
                assert status.item() == int(wrong)
                return out

            for paged in (False, True):
                for batch in (False, True):
                    a, b = both(kvh, monkeypatch, lambda: decode(paged, batch))
                    assert torch.equal(a.view(torch.int16), b.view(torch.int16)) and a.any()
            a, b = both(kvh, monkeypatch, lambda: decode(False, False, wrong=True))
            assert not a.any() and not b.any()

            def kept():
                m = kvh.kept_tokens(n, 8, 50)
                small = torch.zeros(kvh.blob_size(l, m, c, level), dtype=torch.uint8, device="cuda")
                outs = [torch.zeros((2, l, m, c), dtype=dt, device="cuda"), torch.zeros((2, l, n, c), dtype=dt, device="cuda")]
                torch.cuda.synchronize()
                assert kvh.encode_kept(kv[0], kv[1], 8, 50, level, blob=small, stream=stream) is small
                for compact, out in zip((True, False), outs):
                    kvh.decode_kept(small, level, n, 8, 50, out[0], out[1], compact=compact, stream=stream)
                torch.cuda.synchronize()
                return torch.cat([t.view(torch.uint8).flatten() for t in (small, *outs)])

            a, b = both(kvh, monkeypatch, kept)
            assert torch.equal(a, b)


def test_what_is_not_ordinary_is_accepted_or_refused_as_by_ctypes(kvh, monkeypatch):
    l, n, c = 2, 64, 128
    kv = gen.make_kv_device(l, n, c, gen.BF16, seed=2)
    k, v = kv[0], kv[1]
    size = kvh.blob_size(l, n, c, 1)
    blob = kvh.encode(k, v, 1)
    out = torch.zeros_like(kv)
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    table = torch.arange(4, dtype=torch.int32, device="cuda")
    paged = torch.zeros((2, l, 4, 16, c), dtype=kv.dtype, device="cuda")
    host = torch.empty(size, dtype=torch.uint8, pin_memory=True)
    items = kvh.make_dec_items([blob.data_ptr()], [n], [1], [0], [0], "cuda")

    class Sub(torch.Tensor):
        pass

    f = kvh.binding._fast
    gone = lambda *a: f.decode(*a) is None  # left to ctypes
    d = dict(dst_token0=0, page_table=None, block_tokens=16, status=status, stream=None)
    calls = [
        lambda: kvh.decode(blob, 1, n, out[0].float(), out[1].float()), lambda: kvh.decode(blob, 1, n, out[0], out[1].half()),
        lambda: kvh.decode(blob, 1, n, out[0].cpu(), out[1].cpu()), lambda: kvh.decode(blob.cpu(), 1, n, out[0], out[1]),
        lambda: kvh.decode(blob, 1, n, out[0], out[1][:, :-1]), lambda: kvh.decode(blob, 1, n, out[0].transpose(1, 2), out[1].transpose(1, 2)),
        lambda: kvh.decode(blob, 1, n, out[0], out[1], page_table=table), lambda: kvh.decode(blob, 1, n, paged[0], paged[1]),
        lambda: kvh.decode(blob, 1, n, paged[0], paged[1], page_table=table.long()),
        lambda: kvh.decode(blob, 1, n, paged[0][:, :, :8], paged[1][:, :, :8], page_table=table),
        lambda: kvh.decode(blob, 1, n, out[0], out[1], status=status.long()), lambda: kvh.decode(blob, 1, n, out[0], out[1], status=status.cpu()),
        lambda: kvh.decode(blob, 1, n, out[0], out[1], dst_token0=-1), lambda: kvh.decode(blob, 9, n, out[0], out[1]),
        lambda: kvh.decode(blob, 1, 0, out[0], out[1]), lambda: kvh.decode(blob[1:], 1, n, out[0], out[1]),
        lambda: kvh.decode(blob, 1.0, n, out[0], out[1]), lambda: kvh.decode(blob, 1, "64", out[0], out[1]),
        lambda: kvh.decode(blob, 1, n, out[0], out[1], stream=7), lambda: kvh.decode(None, 1, n, out[0], out[1]),
        lambda: kvh.decode_batch(items, 1, n, out[0], out[1], status=status[:0]), lambda: kvh.decode_batch(items, 0, n, out[0], out[1]),
        lambda: kvh.decode_batch(items.cpu(), 1, n, out[0], out[1]), lambda: kvh.decode_batch(items, 70000, n, out[0], out[1]),
        lambda: kvh.encode(k, v, 1, blob=blob[:-16]), lambda: kvh.encode(k, v, 1, blob=host[:-16]), lambda: kvh.encode(k, v.half(), 1, blob=blob),
        lambda: kvh.encode(k, v, 1, blob=torch.empty(size, dtype=torch.uint8)), lambda: kvh.encode(k, v, 5, blob=blob),
        lambda: kvh.encode(k[:, :, :100], v[:, :, :100], 1, blob=blob), lambda: kvh.encode_batch(items.cpu(), 1, n, k, v),
        lambda: kvh.encode_kept(k, v, -1, 5, 1, blob=blob), lambda: kvh.encode_kept(k, v, 4, 5, 1, blob=blob[:16]),
        lambda: kvh.decode_kept(blob, 1, n, 4, 5, out[0], out[1].half()), lambda: kvh.decode_kept(blob, 1, n, 0, 0, out[0], out[1]),
    ]
    for i, call in enumerate(calls):
        a, b = both(kvh, monkeypatch, call)
        assert isinstance(a, tuple) and issubclass(a[0], Exception) and a == b, (i, a, b)
    accepted = [
        lambda: kvh.decode(blob, np.int64(1).item(), n, out[0], out[1], **d), lambda: kvh.decode(blob, True, n, out[0], out[1], **d),
        lambda: kvh.decode(blob.as_subclass(Sub), 1, n, out[0].as_subclass(Sub), out[1].as_subclass(Sub), **d),
        lambda: kvh.encode(k, v, 1, blob=host), lambda: kvh.decode_batch(items, 1, n, out[0], out[1], paged=0, status=status),
        lambda: kvh.decode(blob, 1, n, torch.nn.Parameter(out[0], requires_grad=False), out[1], **d),
    ]
    for call in accepted:
        a, b = both(kvh, monkeypatch, call)
        assert not isinstance(a, tuple) and type(a) is type(b)
    assert gone(blob, True, n, out[0], out[1], 0, None, 16, status, None) and gone(blob, 1, 2**40, out[0], out[1], 0, None, 16, status, None)
    assert gone(blob, 1, n, out[0], out[1], 2**70, None, 16, status, None) and gone(host, 1, n, out[0], out[1], 0, None, 16, status, None)
    assert f.decode(blob, 1, n, out[0], out[1], 0, None, 16, status, None) == 0
    torch.cuda.synchronize()
    assert not status.any() and torch.equal(kvh.encode(k, v, 1), blob)


def test_an_interrupt_is_not_dropped(kvh):
    """Python code runs while the native module asks for the current stream.  What it raises as an error of the call is left to the
    ctypes way, an interrupt or an exit comes out."""
    k = torch.zeros((1, 128, 128), dtype=torch.float16, device="cuda")
    blob = torch.zeros(kvh.blob_size(1, 128, 128, 0), dtype=torch.uint8, device="cuda")

    def raising(what):
        def current_device():
            raise what

        return type(kvh.binding._fast)(current_device, kvh.binding._raw_stream, 0, 0, 0, 0, 0, 0)  # no call gets as far as its function

    assert raising(RuntimeError()).encode(k, k, 0, blob, None, None) is None
    for what in (KeyboardInterrupt, SystemExit):
        with pytest.raises(what):
            raising(what()).encode(k, k, 0, blob, None, None)
        with pytest.raises(what):
            raising(what()).decode(blob, 0, 128, k, k, 0, None, 16, None, None)
