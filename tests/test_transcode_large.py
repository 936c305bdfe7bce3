"""Large launches of the transcoder, on the CPU: the launcher's rule covers every (row, head) slot once, the code that a top code becomes
needs no rule of its own, and the maps that are not evaluated are those of the definition."""
import ctypes
import subprocess

import numpy as np
import pytest

import kv_inputs as gen
import oracle
from test_launch_plans import CSRC, ceil

F16, BF16 = gen.F16, gen.BF16
SHIM = r"""
#include "kvh_plan.hpp"
extern "C" void stream(int heads, int l, int items, int tokens, int64_t* o) {
  const kvh::TcStream p = kvh::transcode_stream_plan(heads, l, items, tokens);
  o[0] = p.log_s; o[1] = p.in.period; o[2] = p.in.units; o[3] = p.in.parts; o[4] = p.in.groups; o[5] = p.in.waves; o[6] = p.in.blocks;
}
"""


@pytest.fixture(scope="module")
def stream(tmp_path_factory):
    d = tmp_path_factory.mktemp("stream")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, "-o", str(d / "s.so"), str(d / "shim.cpp")], check=True)
    lib = ctypes.CDLL(str(d / "s.so"))

    def call(*args):
        out = (ctypes.c_int64 * 8)()
        lib.stream(*args, out)
        return list(out)[:7]

    return call


@pytest.mark.parametrize("heads", list(range(1, 26)) + [33, 64, 65, 72])
def test_units_cover_every_slot_once(stream, heads):
    """The kernel's arithmetic, repeated here, for both block sizes: every slot of a K and of a V section is in one unit, a lane of a K unit
    keeps its head, its parameters are among those the block prepares, and its accesses stay in the token-group."""
    for l, items in ((1, 1), (32, 200)):
        for n in (1, 63, 127, 129, 300, 385):
            log_s, period, units, parts, groups, waves, blocks = stream(heads, l, items, n)
            total = n * heads
            assert waves <= 8 and (log_s >= 0) == (heads > 8)
            v = np.zeros(total, int)
            for u in range(blocks * waves):
                v[u * 128:min(total, u * 128 + 128)] += 1
            assert (v == 1).all()
            seen, words = np.zeros(total, int), set()
            for bx in range(blocks):
                for w in range(waves):
                    if log_s >= 0:
                        sets, s = ceil(heads, 1 << log_s), 1 << log_s
                        half = log_s == 3 and waves == 4  # a set is two blocks
                        i = bx >> 1 if half else bx * (waves >> log_s) + (w >> log_s)
                        g, head0 = i // sets, i % sets * s
                        if half and g * 128 + (bx & 1) * 64 >= n:
                            continue
                        s0, step = (g * 128 + (w % s + (bx & half) * 4) * (128 >> log_s)) * heads + head0, heads << (3 - log_s)
                        lane = [(x >> log_s) * heads + x % s if head0 + x % s < heads else None for x in range(8)]
                        prepared = {(g, head0 + x) for x in range(s)}
                        assert s * 64 <= 2 * 64 * waves
                        if g * 128 < n and not (bx & half):
                            words.update((g, h) for _, h in prepared if h < heads)
                    else:
                        q, gi = bx // parts, w // units
                        first = (bx - q * parts) * waves
                        u, g = first + w - gi * units, q * groups + gi
                        if u >= units or (first and q * groups * 128 * heads + first // period * 128 * period >= total):
                            continue
                        r, j = u % period, u // period
                        s0, step = g * 128 * heads + 8 * r + j * 16 * 8 * period, 8 * period
                        lane = list(range(8))
                        prepared = {(q * groups + x, h) for x in range(groups) for h in range(heads)}
                        assert groups * heads * 64 <= 2 * 64 * waves  # two pairs of channels a thread
                        if first == 0:
                            words.update((x, h) for x, h in prepared if x * 128 < n)
                    for k in range(16):
                        for x in lane:
                            if x is not None and s0 + x + k * step < total:
                                at = s0 + x + k * step
                                assert at // (128 * heads) == g and (g, at % heads) in prepared and at % heads == (s0 + x) % heads
                                seen[at] += 1
            assert (seen == 1).all(), (l, items, n)
            assert words == {(g, h) for g in range(ceil(n, 128)) for h in range(heads)}


def test_blocks_are_small_where_that_measured_faster(stream):
    waves = lambda heads, l, items, n=512: stream(heads, l, items, n)[5]
    assert [waves(h, 32, 16) for h in (1, 2, 3, 4, 5, 6, 7, 8)] == [4, 4, 3, 4, 3, 3, 4, 4]
    assert [waves(h, 4, 2) for h in (1, 2, 3, 4, 5, 6, 7, 8)] == [4, 4, 3, 4, 5, 6, 7, 8]
    assert [waves(h, 32, 16) for h in (9, 10, 11, 12, 13, 16, 20, 25, 33)] == [4] * 9
    assert [waves(h, 2, 14, 300) for h in (13, 15, 16, 24, 25, 33)] == [8, 8, 4, 4, 4, 4]
    assert stream(2**24 - 4, 1, 1, 128)[0] == 3  # rows this long: the slots of an access stay within 32 bits


def groups(dt, count, seed):
    """Pairs (minimum, maximum) of finite 16-bit values: anything, close together, and one close to zero against the range."""
    rng = np.random.default_rng(seed)
    a, b = rng.integers(0, 1 << 16, (2, count)).astype(np.uint16)
    kind = rng.integers(0, 4, count)
    b = np.where(kind == 1, a + rng.integers(0, 256, count).astype(np.uint16), b).astype(np.uint16)
    b = np.where(kind == 2, (a ^ 0x8000) + rng.integers(0, 1024, count).astype(np.uint16) - 512, b).astype(np.uint16)
    b = np.where(kind == 3, (a ^ 0x8000) - rng.integers(0, 6000, count).astype(np.uint16), b).astype(np.uint16)
    x, y = (oracle.t16_to_f32_array(t, dt) for t in (a, b))
    ok = np.isfinite(x) & np.isfinite(y)
    mn, mx = np.minimum(x, y)[ok], np.maximum(x, y)[ok]
    with np.errstate(over="ignore"):
        r = mx - mn
    keep = np.isfinite(r) & (r >= np.float32(2.0 ** -100))
    return mn[keep], mx[keep], r[keep]


def value(q, s, mn, dt):  # of code q: fma in fp32, then the 16-bit type (a product of 8 and 24 bits and the sum are exact in 64 bits but for far apart terms)
    y = (np.float64(q) * s.astype(np.float64) + mn.astype(np.float64)).astype(np.float32)
    return oracle.t16_to_f32_array(oracle.f32_to_t16_array(y, dt), dt)


@pytest.mark.parametrize("dt", [F16, BF16])
def test_top_codes_and_usual_maps(dt):
    mn, mx, r = groups(dt, 200000, 1 + dt)
    for bi in (8, 4, 2):
        li = (1 << bi) - 1
        s = (r / np.float32(li)).astype(np.float32)
        for bo in (8, 4, 2):
            lo = (1 << bo) - 1
            inv = (np.float32(lo) / r).astype(np.float32)
            code = lambda x: np.rint((x - mn) * inv)
            assert (code(value(li, s, mn, dt)) == lo).all() and (code(mx) == lo).all()  # reconstructed like any other code
            if (1 << bi) * bo > 32:
                continue
            most = np.maximum(np.abs(mn), np.abs(mx))
            off = most * np.float32(2.0 ** -11) + np.float32(2.0 ** -25) if dt == F16 else most * np.float32(2.0 ** -8)
            margin = 0.1 if bi == 4 else 0.5
            with np.errstate(over="ignore"):
                usual = (off < r * np.float32(margin / lo * 63 / 64)) & (most < r * np.float32(16)) & (r < np.float32(2.0 ** 120))
            assert usual.mean() > 0.1 or (dt == BF16 and bo == 8)  # (bf16 is too coarse for 8-bit results)
            for q in range(li + 1):
                got = code(mx if q == li else value(q, s, mn, dt))
                assert (got[usual] == (2 * q * lo + li) // (2 * li)).all(), (bi, bo, q)
