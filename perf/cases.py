"""The work that users of the KV-cache level codec have it do, as cases that can be timed and compared.

A case is a plain dict:

  kind    "encode"        kvh.encode: one entry (a chunk as prefill produces it, or a whole short context) -> one blob
          "decode"        kvh.decode: one blob -> rows of the serving cache
          "encode_batch"  kvh.encode_batch: all chunks of a context -> blobs, one launch
          "decode_batch"  kvh.decode_batch: all chunks of one or several requests -> the serving cache, one launch
          "transcode"     kvh.transcode_batch: stored chunks are compressed further (the policy's step under pressure)
          "kept"          kvh.encode_kept and kvh.decode_kept: token dropping, there and back into a dense cache
          "load"          kvh.Loader.run: blobs in pinned host memory -> staging slots -> the serving cache
  l, n, c layers, tokens, channels.  1024 channels are 8 KV heads of 128 (the 8B- and 70B-shaped models of this
          repository); 128, 256 and 512 are what one rank of a model split by KV heads over 8, 4 or 2 GPUs holds; 640,
          1280 and 2048 stand for models with other head counts
  dt      "bf16" or "fp16"
  level   0 / 1 / 2 = 8 / 4 / 2 bits, 3 = full quality (raw), -1 = a level per chunk as the policy left them
  to      transcode: the level to go to
  chunk   tokens per chunk; requests = requests of mixed lengths that share the n tokens
  page    tokens per page of the destination cache, 0 for a contiguous one; pages are handed out in random order
  sink, window   token dropping: tokens kept at the beginning and at the end

Keys, values and lengths have the distributions of kv_inputs.py: a wide spread of per-channel scales, 1 % outlier
channels, a rotary-like drift on K, request lengths lognormal.  Values and page tables are made from the seed.
"""
import math

import numpy as np
import torch

import paper_2509_00105_amd as kvh

_DT = {"bf16": torch.bfloat16, "fp16": torch.float16}
_BITS = {0: 8, 1: 4, 2: 2, 3: 16}
_TEMPLATE = dict(kind="", l=32, n=8192, c=1024, dt="bf16", level=0, to=0, chunk=256, requests=1, page=0, sink=0, window=0)


def _case(**kw):
    return dict(_TEMPLATE, **kw)


def listed():
    return [
        # The smallest call there is: one chunk of a small model's cache goes back into a paged cache.
        _case(name="decode one chunk, 4 layers", kind="decode", l=4, n=256, dt="fp16", level=0, page=16),
        # One 256-token chunk of the 8B-shaped model as prefill produces it, and one as a cache hit brings it back.
        _case(name="encode one chunk, 8B", kind="encode", n=256, level=1),
        _case(name="decode one chunk, 8B paged", kind="decode", n=256, level=2, page=16),
        # An 8K-token context of the 8B-shaped model is stored, and read back: one batched launch each.
        _case(name="encode 8K context, 8B", kind="encode_batch", level=0),
        _case(name="decode 8K context, 8B", kind="decode_batch", level=1),
        # Requests of mixed lengths and levels are restored into a paged cache at once (the largest case).
        _case(name="decode mixed requests, paged", kind="decode_batch", n=65536, level=-1, requests=16, page=16),
        # One rank of the 70B-shaped model split by KV heads: over 8 GPUs (1 head) and over 4 GPUs (2 heads).
        _case(name="encode 8K, 70B 1 head", kind="encode_batch", l=80, c=128, chunk=512, level=2),
        _case(name="decode 8K, 70B 2 heads", kind="decode_batch", l=80, c=256, chunk=512, level=0, page=16),
        # A context of odd length of a model with 5 KV heads, stored as one entry.
        _case(name="encode 3001 tokens, 5 heads", kind="encode", l=20, n=3001, c=640, dt="fp16", level=1, chunk=3001),
        # The policy lowers a stored 8K-token context from 8 to 4 bits.
        _case(name="transcode 8K context 8->4", kind="transcode", level=0, to=1),
        # The second method of the paper: the beginning and the end of a long context are kept, at two bits.
        _case(name="drop tokens of 16K context", kind="kept", n=16000, dt="fp16", level=2, chunk=16000, sink=64, window=4000),
        # A cache hit in the DRAM tier: 2K tokens at mixed levels travel over the host bus into the paged cache.
        _case(name="load 2K tokens from host", kind="load", n=2048, level=-1, page=16),
    ]


def draw(rng):
    def spread(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["encode", "decode", "encode_batch", "encode_batch", "decode_batch", "decode_batch", "transcode",
                       "transcode", "kept", "load"])
    c = rng.choice([128, 256, 512, 640, 1024, 1024, 1024, 1280, 2048])
    l = spread(4, 80)
    dt = rng.choice(["bf16", "bf16", "fp16"])
    page = rng.choice([0, 16, 16, 32])
    level = rng.choice([-1, 0, 1, 2, 0, 1, 2, 3])
    one = kind in ("encode", "decode", "kept")
    n = spread(200, 32768) if one else spread(1024, 65536)
    most = 1 << 28 if kind == "load" else 1 << 32  # bytes of 16-bit KV
    n = max(256, min(n, most // (4 * l * c)))
    case = _case(kind=kind, l=l, n=n, c=c, dt=dt, level=level, page=0, chunk=n if one else rng.choice([256, 256, 512, 1024, 2048]))
    if one and level == -1:
        case["level"] = rng.randrange(3)
    if kind in ("decode", "decode_batch", "load"):
        case["page"] = page
    if kind == "decode_batch" and n >= 4096:
        case["requests"] = rng.choice([1, 1, max(2, n // 4096)])
    if kind == "transcode":
        case["level"], case["to"] = rng.choice([(0, 1), (0, 2), (1, 2)])
    if kind == "kept":
        case["sink"], case["window"] = rng.choice([4, 16, 64, 128]), max(1, n // rng.choice([2, 4, 8]))
    return case


# ---- inputs -------------------------------------------------------------------------------------------------
def _make_kv(g, l, n, c, dt):
    """[2][l][n][c] of the 16-bit type: K with a rotary-like drift, V without."""
    dev = torch.device("cuda")
    kv = torch.empty((2, l, n, c), dtype=_DT[dt], device=dev)
    ch = torch.arange(c, device=dev)
    theta = 10000.0 ** (-2.0 * torch.floor((ch % 128) / 2.0) / 128.0)
    token = torch.arange(n, device=dev, dtype=torch.float32)[:, None]
    n_out = int(math.ceil(0.01 * c))
    for which in range(2):
        for lam in range(l):
            sigma = torch.exp(torch.randn(c, generator=g, device=dev))
            sigma[torch.randperm(c, generator=g, device=dev)[:n_out]] *= 10.0
            x = torch.randn((n, c), generator=g, device=dev)
            if which == 0:
                phi = torch.rand(c, generator=g, device=dev) * (2.0 * math.pi)
                x += 2.0 * torch.sin(theta[None, :] * token + phi[None, :])
            kv[which, lam] = (x * sigma[None, :]).to(_DT[dt])
    return kv


def _requests(rng, case):
    """Lengths of the requests that share the case's tokens: lognormal, sigma 0.8, none below 16 tokens."""
    if case["requests"] == 1:
        return [case["n"]]
    w = np.exp(rng.normal(0.0, 0.8, size=case["requests"]))
    lengths = np.maximum(16, np.floor(w / w.sum() * case["n"]).astype(np.int64))
    return [int(x) for x in lengths]


def _plan(case):
    """Chunks of the case: (request, first token in the request, first token over all, tokens, level), byte offsets.
    Lengths and levels belong to the case, so that its outputs have one shape whatever the seed."""
    rng = np.random.default_rng(case["n"])
    chunks, start = [], 0
    for r, length in enumerate(_requests(rng, case)):
        for t0 in range(0, length, case["chunk"]):
            level = case["level"] if case["level"] >= 0 else int(rng.integers(0, 3))
            chunks.append((r, t0, start + t0, min(case["chunk"], length - t0), level))
        start += length
    sizes = [kvh.blob_size(case["l"], m, case["c"], lv) for _, _, _, m, lv in chunks]
    offs = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    return chunks, offs[:-1], int(offs[-1]), start


def _store(case, kv, chunks, offs, total):
    """The chunks of kv as stored blobs, in one device buffer."""
    dev = kv.device
    blobs = torch.empty(total, dtype=torch.uint8, device=dev)
    ptrs = [blobs.data_ptr() + int(o) for o in offs]
    items = kvh.make_enc_items(ptrs, [a for _, _, a, _, _ in chunks], [m for _, _, _, m, _ in chunks],
                               [lv for _, _, _, _, lv in chunks], dev)
    kvh.encode_batch(items, len(chunks), max(m for _, _, _, m, _ in chunks), kv[0], kv[1])
    torch.cuda.synchronize()
    return blobs, ptrs, items


def _cache(rng, case, chunks, tokens):
    """The destination: a zeroed cache, contiguous or paged, and for a paged one the page table of every request."""
    dev, l, c, page = torch.device("cuda"), case["l"], case["c"], case["page"]
    if page == 0:
        return torch.zeros((2, l, tokens, c), dtype=_DT[case["dt"]], device=dev), None
    need = {}
    for r, t0, _, m, _ in chunks:
        need[r] = max(need.get(r, 0), -(-(t0 + m) // page))
    order = torch.from_numpy(rng.permutation(sum(need.values())).astype(np.int32)).to(dev)
    tables, at = [], 0
    for r in sorted(need):
        tables.append(order[at:at + need[r]].clone())
        at += need[r]
    return torch.zeros((2, l, at, page, c), dtype=_DT[case["dt"]], device=dev), tables


def prepare(case, seed):
    dev = torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    rng = np.random.default_rng(seed)
    l, n, c, kind = case["l"], case["n"], case["c"], case["kind"]
    if kind == "kept":
        kv = _make_kv(g, l, n, c, case["dt"])
        m = kvh.kept_tokens(n, case["sink"], case["window"])
        return {"case": case, "kv": kv, "blob": torch.empty(kvh.blob_size(l, m, c, case["level"]), dtype=torch.uint8, device=dev),
                "cache": torch.zeros((2, l, m, c), dtype=kv.dtype, device=dev), "status": torch.zeros(1, dtype=torch.int32, device=dev)}
    chunks, offs, total, tokens = _plan(case)
    kv = _make_kv(g, l, tokens, c, case["dt"])
    blobs, ptrs, items = _store(case, kv, chunks, offs, total)
    state = {"case": case, "chunks": chunks, "offs": offs, "blobs": blobs, "count": len(chunks),
             "most": max(m for _, _, _, m, _ in chunks), "status": torch.zeros(len(chunks), dtype=torch.int32, device=dev)}
    lengths, levels = [m for _, _, _, m, _ in chunks], [lv for _, _, _, _, lv in chunks]
    if kind in ("encode", "encode_batch"):
        blobs.zero_()
        state.update(kv=kv, items=items)
    elif kind == "transcode":
        sizes = [kvh.blob_size(l, m, c, case["to"]) for m in lengths]
        at = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
        out = torch.zeros(int(at[-1]), dtype=torch.uint8, device=dev)
        state.update(out=out, items=kvh.make_tc_items(ptrs, [out.data_ptr() + int(o) for o in at[:-1]], lengths, levels,
                                                      [case["to"]] * len(chunks), dev))
    else:
        del kv
        state["cache"], state["tables"] = _cache(rng, case, chunks, tokens)
        paged = state["tables"] is not None
        first = [t0 if paged else a for _, t0, a, _, _ in chunks]
        if kind == "decode_batch":
            state["items"] = kvh.make_dec_items(ptrs, lengths, levels, first,
                                                [state["tables"][r].data_ptr() for r, _, _, _, _ in chunks] if paged else [0] * len(chunks), dev)
        elif kind == "load":
            host = torch.empty(total, dtype=torch.uint8, pin_memory=True)
            host.copy_(blobs)
            ends = list(offs[1:]) + [total]
            state["host"] = [host[int(a):int(b)] for a, b in zip(offs, ends)]
            slot = 4 * max(kvh.blob_size(l, state["most"], c, lv) for lv in levels) + 4096
            state["loader"] = kvh.Loader(torch.empty(2 * slot, dtype=torch.uint8, device=dev), n_slots=2)
            state.update(lengths=lengths, levels=levels, first=first,
                         per_chunk=[state["tables"][r] for r, _, _, _, _ in chunks] if paged else None)
    return state


# ---- one pass -----------------------------------------------------------------------------------------------
def run(state):
    case = state["case"]
    kind, level = case["kind"], case["level"]
    if kind == "encode":
        return kvh.encode(state["kv"][0], state["kv"][1], level, blob=state["blobs"])
    if kind == "encode_batch":
        kvh.encode_batch(state["items"], state["count"], state["most"], state["kv"][0], state["kv"][1])
        return state["blobs"]
    if kind == "transcode":
        kvh.transcode_batch(state["items"], state["count"], state["most"], _DT[case["dt"]], case["l"], case["c"], status=state["status"])
        return [state["out"], state["status"]]
    k, v = state["cache"][0], state["cache"][1]
    if kind == "kept":
        kvh.encode_kept(state["kv"][0], state["kv"][1], case["sink"], case["window"], level, blob=state["blob"])
        kvh.decode_kept(state["blob"], level, case["n"], case["sink"], case["window"], k, v, compact=True, status=state["status"])
        return [state["cache"], state["status"], state["blob"]]
    page, tables = case["page"] or 16, state["tables"]
    if kind == "decode":
        kvh.decode(state["blobs"], level, case["n"], k, v, page_table=tables[0] if tables else None, block_tokens=page, status=state["status"])
    elif kind == "decode_batch":
        kvh.decode_batch(state["items"], state["count"], state["most"], k, v, paged=tables is not None, block_tokens=page, status=state["status"])
    else:
        state["loader"].run(state["host"], state["lengths"], state["levels"], state["first"], k, v, page_tables=state["per_chunk"],
                            block_tokens=page, status=state["status"])
    return [state["cache"], state["status"]]


# ---- what a pass cannot do without --------------------------------------------------------------------------
def work(case):
    """Bytes: the 16-bit rows once and the blobs once, in whichever direction.  Operations: what the definition asks of
    an element (two comparisons, a subtraction and a product to encode, one fused multiply-add to decode)."""
    l, c = case["l"], case["c"]
    if case["kind"] == "kept":
        m = kvh.kept_tokens(case["n"], case["sink"], case["window"])
        values, blob = 2 * l * m * c, kvh.blob_size(l, m, c, case["level"])
        return {"bytes": 2 * (2 * values + blob), "flops": 6 * values}
    # levels and lengths drawn at random: priced at their average
    n, levels = case["n"], [case["level"]] if case["level"] >= 0 else [0, 1, 2]
    values = 2 * l * n * c

    def stored(level):
        whole, rest = divmod(n, case["chunk"])
        return whole * kvh.blob_size(l, case["chunk"], c, level) + (kvh.blob_size(l, rest, c, level) if rest else 0)

    blob = sum(stored(lv) for lv in levels) // len(levels)
    if case["kind"] == "transcode":
        return {"bytes": blob + stored(case["to"]), "flops": 4 * values}
    return {"bytes": 2 * values + blob, "flops": (4 if case["kind"].startswith("encode") else 2) * values}


def tolerance(case):
    """The format fixes every bit: codes and metadata as bytes, decoded values as 16-bit patterns."""
    return "exact"


# ---- the same in 64 bits ------------------------------------------------------------------------------------
def _values64(blob, l, n, c, level, dt):
    """[2][l][n][c]: what a stored blob stands for, each code as minimum + code * range / levels."""
    bits = _BITS[level]
    body = blob[64:].view(l, -1)
    if bits == 16:
        return body.contiguous().view(_DT[dt]).view(l, 2, n, c).transpose(0, 1).double()

    def pad(x):
        return (x + 15) // 16 * 16

    groups = -(-n // 128)
    at, out = 0, []
    for which in range(2):
        meta_bytes = groups * c * 4 if which == 0 else n * (c // 128) * 4
        meta = body[:, at:at + meta_bytes].contiguous().view(_DT[dt]).double()
        at += pad(meta_bytes)
        code_bytes = n * c * bits // 8
        packed = body[:, at:at + code_bytes].contiguous()
        at += pad(code_bytes)
        q = torch.stack([(packed >> s) & ((1 << bits) - 1) for s in range(0, 8, bits)], dim=-1).view(l, n, c).double()
        if which == 0:
            mn, mx = (t.repeat_interleave(128, dim=1)[:, :n] for t in meta.view(l, groups, c, 2).unbind(-1))
        else:
            mn, mx = (t.repeat_interleave(128, dim=2) for t in meta.view(l, n, c // 128, 2).unbind(-1))
        out.append(mn + q * ((mx - mn) / float((1 << bits) - 1)))
    return torch.stack(out)


def _round_trip64(kv, level):
    """What [2][l][n][c] rows are after quantisation, each group of 128 (K: tokens, V: channels) in 64 bits."""
    if _BITS[level] == 16:
        return kv.double()
    top, (k, v), n = float((1 << _BITS[level]) - 1), kv.double(), kv.shape[2]

    def quantised(x, mn, mx):
        step = (mx - mn) / top
        return mn + torch.round((x - mn) / torch.where(step > 0, step, 1.0)) * step

    out = torch.empty(kv.shape, dtype=torch.float64, device=kv.device)
    for t0 in range(0, n, 128):
        x = k[:, t0:t0 + 128]
        out[0, :, t0:t0 + 128] = quantised(x, x.amin(1, keepdim=True), x.amax(1, keepdim=True))
    v = v.unflatten(-1, (-1, 128))
    out[1] = quantised(v, v.amin(-1, keepdim=True), v.amax(-1, keepdim=True)).flatten(-2)
    return out


def exact(case, seed):
    """Decoded rows in 64 bits.  Blobs are packed bytes and have no 64-bit value: None in their place."""
    if case["kind"] in ("encode", "encode_batch", "transcode"):
        return None
    if case["kind"] == "kept":
        kv = prepare(case, seed)["kv"]
        at = torch.arange(kvh.kept_tokens(case["n"], case["sink"], case["window"]), device="cuda")
        at = torch.where(at < case["sink"], at, at + (case["n"] - len(at)))
        return [_round_trip64(kv[:, :, at], case["level"]), None, None]
    state = prepare(case, seed)
    page = case["page"]
    out = torch.zeros(state["cache"].shape, dtype=torch.float64, device="cuda")
    sizes = list(state["offs"][1:]) + [state["blobs"].numel()]
    for (r, t0, first, m, level), a, b in zip(state["chunks"], state["offs"], sizes):
        rows = _values64(state["blobs"][int(a):int(b)], case["l"], m, case["c"], level, case["dt"])
        if page == 0:
            out[:, :, first:first + m] = rows
        else:
            at = torch.arange(t0, t0 + m, device="cuda")
            row = state["tables"][r].long()[at // page] * page + at % page
            out.view(2, case["l"], -1, case["c"])[:, :, row] = rows
    return [out, None]
