"""The launchers' rules (csrc/kvh_plan.hpp), compiled for the host: every row and head of an item is covered, and the
layouts that measured slower than another one are not chosen again."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_00105_amd", "csrc")
SHIM = r"""
#include "kvh_plan.hpp"
using namespace kvh;
extern "C" void tc_stream(int heads, int l, int items, int tokens, int64_t* o) {
  const TcStream p = transcode_stream_plan(heads, l, items, tokens);
  o[0] = p.log_s; o[1] = p.in.waves; o[2] = p.in.parts;
}
extern "C" void tc_units(int heads, int l, int items, int tokens, int64_t* o) {
  const TcUnits u = transcode_units_plan(heads, l, items, tokens);
  o[0] = u.accesses; o[1] = u.period; o[2] = u.units; o[3] = u.parts; o[4] = u.groups; o[5] = u.waves; o[6] = u.blocks;
}
extern "C" void enc_plan(int heads, int l, int items, int tokens, int64_t* o) {
  const EncPlan p = encode_plan(heads, l, items, tokens);
  o[0] = p.slots; o[1] = p.k_slots; o[2] = p.waves; o[3] = p.blocks;
}
extern "C" void enc_units(int heads, int l, int items, int tokens, int64_t* o) {
  const EncUnits u = encode_units_plan(heads, l, items, tokens, o[0] != 0);
  o[0] = u.waves; o[1] = u.blocks;
}
extern "C" void enc_keeps(int bits, int mib, int more, int64_t* o) { o[0] = encode_keeps(bits, ((uint64_t)mib << 20) + (int64_t)more); }
extern "C" void dec_plan(int heads, int l, int items, int tokens, int64_t layer_stride, int64_t token_stride, int64_t* o) {
  const DecPlan p = decode_plan(heads, l, items, tokens, layer_stride, token_stride);
  o[0] = p.slots; o[1] = p.short_launch; o[2] = p.waves; o[3] = p.blocks; o[4] = p.plane_group; o[5] = p.row_tile;
  o[6] = grid_fits(p.blocks, p.plane_group, p.waves);
}
extern "C" void dec_units(int heads, int l, int items, int tokens, int64_t layer_stride, int64_t token_stride, int64_t* o) {
  const DecUnits u = decode_units_plan(heads, l, items, tokens, layer_stride, token_stride, o[0] != 0);
  o[0] = u.blocks; o[1] = u.plane_group;
}
extern "C" void dec_launch(int heads, int l, int items, int tokens, int64_t layer_stride, int64_t token_stride, int64_t* o) {
  const DecLaunch d = decode_launch(heads, l, items, tokens, layer_stride, token_stride, o[0] != 0);
  o[0] = d.slots; o[1] = d.short_launch; o[2] = d.waves; o[3] = d.blocks; o[4] = d.plane_group; o[5] = d.row_tile;
  o[6] = d.page_through;
}
"""


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    d = tmp_path_factory.mktemp("plans")
    (d / "shim.cpp").write_text(SHIM)
    so = str(d / "plans.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, "-o", so, str(d / "shim.cpp")], check=True)
    lib = ctypes.CDLL(so)

    def call(name, *args, known=False):  # known: that all items are raw
        out = (ctypes.c_int64 * 8)(known)
        wide = 4 if name in ("dec_plan", "dec_units", "dec_launch") else len(args)  # the strides
        getattr(lib, name)(*[ctypes.c_int64(a) if i >= wide else a for i, a in enumerate(args)], out)
        return list(out)

    return call


def ceil(a, b):
    return -(-a // b)


@pytest.mark.parametrize("heads", list(range(1, 26)) + [33, 64, 255])
def test_encode_plan_covers_rows_and_heads(plans, heads):
    for l, items in ((1, 1), (4, 1), (32, 1), (32, 16)):
        for n in (1, 127, 128, 129, 256, 300, 3001, 40003):
            slots, k_slots, waves, blocks = plans("enc_plan", heads, l, items, n)[:4]
            assert waves in (4, 8) and (k_slots or waves == 8) and (slots or not k_slots)
            if k_slots:  # 2 S waves a set of S heads x a token-group
                s = 1 if heads & 1 else 2
                assert waves % (2 * s) == 0 and blocks * (waves // (2 * s)) >= ceil(n, 128) * (heads // s)
            else:
                assert blocks >= ceil(n, 128) * ceil(heads, 4)
            assert not slots or blocks * waves * 64 >= n * heads


def test_encode_blocks_of_few_heads_are_small(plans):
    """With 8 waves a block of 2 heads held 256 tokens: 4 layers of 3,001 tokens made 96 blocks for 256 compute units (raw
    8.5 us, 6.8 in strips), 32 of 256 tokens 64 (7.6 and 7.1).  Only items that fill such a block keep it."""
    for heads in (1, 2):
        assert plans("enc_plan", heads, 4, 1, 3001)[2:4] == [4, 12 * heads]
        assert plans("enc_plan", heads, 32, 1, 256)[2:4] == [4, heads]
        assert plans("enc_plan", heads, 32, 16, 512)[2:4] == [4, 2 * heads]
        assert plans("enc_plan", heads, 32, 8, 256)[2:4] == [4 * heads, 1]


def test_encode_slots_only_where_they_are_the_faster_form(plans):
    """Rows of 3 heads stay in one strip: slots were down to 0.89 of it (raw), never above 1.14."""
    assert [h for h in range(1, 25) if plans("enc_plan", h, 32, 16, 512)[0]] == [h for h in range(1, 25) if h % 4 and h != 3]
    assert [h for h in range(1, 25) if plans("enc_plan", h, 32, 16, 512)[1]] == [1, 2, 5, 6]


def dense(c, tokens):
    return tokens * c, c


@pytest.mark.parametrize("heads", list(range(1, 26)) + [33, 64, 255])
def test_decode_plan_covers_rows_and_planes(plans, heads):
    """The kernel's own block -> (plane, block of the plane) arithmetic, repeated here, reaches every block of every plane
    once, whatever the last plane group and the last row tile are."""
    c = 128 * heads
    for l in (1, 3, 4, 5, 6, 9, 10, 11, 13):
        for n, items in ((1, 1), (129, 2), (300, 1), (3001, 1)):
            for strides in (dense(c, n), dense(c, 40000), (c, l * c)):
                slots, _, waves, blocks, group, tile = plans("dec_plan", heads, l, items, n, *strides)[:6]
                s = 1 << (heads & -heads).bit_length() - 1
                if slots:
                    assert blocks * waves >= ceil(n, 64 // s) * (heads // s) and blocks * waves * 64 >= n * heads and tile == 1
                else:
                    assert blocks >= ceil(n, 64) * (heads // 8)
                if blocks > 400:
                    continue
                seen = set()
                for z in range(ceil(2 * l, group)):
                    first = z * group
                    planes = min(2 * l - first, group)
                    for lin in range(blocks * planes):
                        rt = min(tile, blocks)
                        full, t = blocks // rt, lin // (rt * planes)
                        size, start = (rt, t * rt) if t < full else (blocks - full * rt, full * rt)
                        j = lin - start * planes
                        seen.add((first + j // size, start + j % size))
                assert seen == {(p, b) for p in range(2 * l) for b in range(blocks)}


def test_decode_grid_fits_the_dispatcher(plans):
    for heads, l, n in ((8, 32767, 64), (1, 32767, 100000), (8, 80, 2**28), (5, 80, 2**26)):
        slots, _, waves, blocks, group, _, fits = plans("dec_plan", heads, l, 65535, n, *dense(128 * heads, n))[:7]
        assert ceil(2 * l, group) <= 65535 and fits and blocks * group * 64 * waves < 2**32
    for heads, n in ((8, 2**31 - 1), (9, 2**31 - 1), (1025, 2**31 - 1), (2**24 - 1, 2**31 - 1)):  # refused, not cut down to 32 bits
        assert not plans("dec_plan", heads, 1, 1, n, *dense(128 * heads, 1))[6]


def test_decode_takes_all_planes_where_layers_lie_side_by_side(plans):
    """[tokens][layers][channels]: plane groups leave holes between the rows that consecutive blocks write."""
    for heads in (1, 2, 4, 5, 8, 16):
        c = 128 * heads
        for n, items in ((256, 1), (256, 8), (8192, 1)):
            small = plans("dec_plan", heads, 32, items, n, c, 32 * c)[2] == 1
            assert plans("dec_plan", heads, 32, items, n, c, 32 * c)[4:6] == ([4, 1] if heads == 4 and small else [64, 1])
            assert plans("dec_plan", heads, 32, items, n, *dense(c, n))[4] <= 8 or (heads % 8 == 0 and n * heads > 7 * 8192)


def test_decode_whole_spans_take_groups_of_eight_planes_or_none(plans):
    """Groups of 5 to 7 planes put every plane on all XCDs: 6 layers in two groups of 6 took up to a third longer."""
    for l in range(1, 81):
        for n in (128, 512, 2048, 4096):
            mib = l * n / 256
            group, tile = plans("dec_plan", 8, l, 1, n, *dense(1024, n))[4:6]
            assert group in (4, 8, 2 * l)
            turned = mib > 80 and n >= 2048 and (l > 5 if mib <= 896 else True)  # planes of 4 to 8 MiB in turns
            turned = turned and (mib > 896 or n * 2 / 1024 >= 4.5)
            grouped = turned or (mib <= 896 and (l % 4 == 0 or (l > 8 and mib > 80)))
            assert group == (4 if turned else 8 if grouped else 2 * l) and (not grouped or tile == 1), (l, n)


def test_decode_two_blocks_per_cu_only_for_small_launches(plans):
    """Above 80 MiB of rows a second block per CU costs up to 8 %."""
    for heads, l in ((8, 4), (8, 32), (16, 4), (32, 80), (16, 24)):
        row_mib = 4 * l * heads * 128 / 2**20
        for mib in (16, 48, 79, 81, 96, 128, 255):
            n = int(mib / row_mib)
            if n:
                assert plans("dec_plan", heads, l, 1, n, *dense(128 * heads, n))[1] == int(n * row_mib <= 80), (heads, l, mib)
    assert not any(plans("dec_plan", heads, 4, 1, 256, *dense(128 * heads, 256))[1] for heads in (1, 2, 4, 5, 12))


def test_decode_launches_the_form_that_is_planned(plans):
    """Units of slots, one wave a block, for launches of whole spans of up to 48 MiB, beyond which spans win (4 bits, 48 to 192 MiB:
    units 0.96 of their speed); two blocks per CU for spans of up to 80 MiB (24 x 752 tokens of 3,760 at 8 bits: 22.4 us, with one block 24.6)."""
    at = lambda heads, l, items, n, strides=None: plans("dec_launch", heads, l, items, n, *(strides or dense(128 * heads, n * items)))[:6]
    assert at(8, 32, 1, 256) == [1, 0, 1, 32, 8, 1] and at(8, 32, 1, 256, dense(1024, 8192)) == [1, 0, 1, 32, 64, 1]
    for strides in (None, dense(1024, 8192)):
        assert at(8, 32, 1, 384, strides)[0] == 1 and at(8, 32, 1, 385, strides)[:2] == [0, 1]
        assert at(8, 32, 1, 640, strides)[:2] == [0, 1] and at(8, 32, 1, 641, strides)[:2] == [0, 0]
    assert at(8, 24, 1, 752, dense(1024, 3760)) == [0, 1, 8, 12, 8, 1]
    for heads, l, items, n in ((8, 32, 7, 256), (8, 80, 16, 256), (5, 32, 1, 256), (8, 20, 1, 15000), (8, 48, 1, 6000)):
        strides = dense(128 * heads, items * n)
        slots, _, waves, blocks, group, tile, fits = plans("dec_plan", heads, l, items, n, *strides)[:7]
        assert fits and at(heads, l, items, n) == [slots, 0, waves, blocks, group, tile]
    assert not any(at(8, 1, 1, 2**31 - 1, dense(1024, 1))[:4])  # refused


def test_decode_2_bit_rows_of_whole_spans_are_stored_alike_everywhere(plans):
    """With device scope, pages of 32 KiB and less: 600 to 1,000 MiB 0.96 in random order, 0.93 to 0.95 in order."""
    through = lambda heads, l, items, n: plans("dec_launch", heads, l, items, n, *dense(128 * heads, n * items))[6]
    assert not any(through(8, l, items, 256) for l, items in ((32, 2), (32, 18), (32, 32), (80, 256)))


def test_decode_2_bit_slots_take_device_scope_into_pages_in_small_and_large_launches_only(plans):
    """4 heads, 100 to 1,000 MiB: 0.93 to 0.97 in random order (48 x 10 x 512 tokens, 480 MiB: 88 us, 91 with device scope)."""
    through = lambda heads, l, items, n: plans("dec_launch", heads, l, items, n, *dense(128 * heads, n * items))[6]
    assert through(8, 32, 1, 256) and through(8, 32, 1, 320) and not through(8, 32, 1, 321)
    assert through(2, 80, 2, 256) and through(5, 4, 1, 300) and not through(4, 48, 10, 512) and not through(2, 80, 16, 512) and not through(5, 40, 9, 256)
    assert through(2, 80, 27, 512) and through(5, 80, 21, 256) and not through(5, 80, 20, 256)


def test_decode_raw_launches_of_up_to_one_block_of_spans_a_compute_unit_stay_in_spans(plans):
    """32 x 256 raw tokens into an 8,192-token cache: 15.6 us in spans, 17.1 in units.  With more blocks than compute units, or with
    many of them idle, units win."""
    def slots(l, n, strides, heads=8, items=1, raw=True):
        return plans("dec_launch", heads, l, items, n, *strides, known=raw)[0]

    cache = dense(1024, 8192)
    assert [slots(32, n, cache) for n in (64, 128, 129, 192, 256, 257, 384)] == [1, 1, 0, 0, 0, 1, 1]
    assert slots(20, 256, cache) == 1 and slots(21, 256, cache) == 0 and slots(24, 301, dense(1024, 301)) == 0
    assert slots(8, 256, cache, items=4) == 0 and slots(16, 256, dense(2048, 8192), heads=16) == 0
    assert all(slots(32, n, cache, raw=False) for n in (64, 129, 192, 256, 257, 384))


def test_decode_small_launches_of_slots_take_small_blocks(plans):
    """Blocks of 8 waves left compute units idle: 32 layers x 256 tokens of 2 heads made 64 blocks (raw 6.3 us, 5.4 in spans)."""
    for heads, l, n in ((1, 4, 256), (2, 32, 256), (3, 32, 256), (5, 4, 256), (6, 4, 3001), (10, 32, 256), (3, 80, 256)):
        waves, blocks = plans("dec_plan", heads, l, 1, n, *dense(128 * heads, n))[2:4]
        assert waves == 1 and blocks * 64 >= n * heads, (heads, l, n)
    for heads, l, items, n in ((2, 32, 8, 256), (2, 80, 16, 512), (10, 32, 8, 256), (5, 80, 1, 256)):
        assert plans("dec_plan", heads, l, items, n, *dense(128 * heads, n * items))[2] == 8, (heads, l, items, n)
    assert all(plans("dec_plan", h, 4, 1, 256, *dense(128 * h, 256))[2] == 8 for h in (8, 16, 24))


def test_gpu_tests_reach_the_orders_they_name(plans):
    """The shapes of tests/test_gpu_row_lengths.py: uneven last plane groups, row tiles with a remainder, plane by plane."""
    groups = {(h, l): plans("dec_plan", h, l, 1, 300, *dense(128 * h, 300))[4] for h, l in ((4, 5), (5, 10), (5, 11))}
    assert groups == {(4, 5): 4, (5, 10): 7, (5, 11): 8}                                     # of 10, 20 and 22 planes
    assert plans("dec_plan", 8, 9, 1, 8191, *dense(1024, 8191))[4:6] == [4, 1]               # of 18 planes
    assert plans("dec_plan", 8, 20, 1, 15000, *dense(1024, 15000))[4:6] == [40, 0x7fffffff]
    slots, short, _, blocks, group, tile = plans("dec_plan", 8, 9, 100, 300, *dense(1024, 30000))[:6]
    assert (slots, short, blocks, group, tile) == (0, 0, 5, 18, 4)


def test_decode_turns(plans):
    """Turns of 4 or 8 planes where a launch is large and its planes are neither small nor large."""
    def turn(heads, l, items, n, strides=None):
        group, tile = plans("dec_plan", heads, l, items, n, *(strides or dense(128 * heads, n * items)))[4:6]
        assert tile == 1 or group == 2 * l
        return group

    assert turn(8, 40, 28, 256) == 4 and turn(8, 80, 28, 256) == 8        # 1.1 and 2.2 GiB
    assert [turn(8, l, 40, 250) for l in (30, 31, 32, 33, 34, 35)] == [4, 62, 64, 66, 68, 4]  # an item of 248 to 272 blocks
    assert turn(8, 40, 56, 128) == 80 and turn(8, 40, 56, 129) == 4
    assert turn(8, 32, 32, 256) == 64 and turn(8, 32, 64, 256) == 64    # layers 16 and 32 MiB apart
    assert turn(8, 32, 16, 512) == 4 and turn(8, 80, 16, 256) == 4        # 16 MiB, longer items; 8 MiB
    assert turn(8, 32, 128, 256) == 64                                           # planes of 64 MiB
    assert turn(8, 32, 48, 512) == 8 and turn(8, 32, 64, 512) == 64 and turn(8, 32, 64, 1024) == 8 and turn(8, 32, 256, 1024) == 64
    assert turn(8, 48, 1, 6000) == 4 and turn(8, 80, 1, 8192) == 8 and turn(8, 80, 1, 8193) == 160
    assert turn(8, 11, 8, 300) == 4 and turn(8, 11, 1, 2400) == 4
    assert turn(8, 8, 16, 256) == 4 and turn(8, 40, 16, 256) == 4 and turn(8, 7, 16, 256) == 14 and turn(8, 7, 4, 1024) == 4
    assert turn(8, 32, 4, 256) == 8 and turn(16, 32, 2, 1024) == 8
    assert turn(8, 32, 32, 256, (1024, 32 * 1024)) == 64 and turn(5, 32, 32, 256) == 8


def test_gpu_tests_reach_the_turns_they_name(plans):
    for l, items, n, group in ((11, 8, 300, 4), (31, 13, 600, 4), (57, 10, 660, 8)):
        assert plans("dec_plan", 8, l, items, n, *dense(1024, n * items))[4] == group and 2 * l % group
    assert plans("dec_plan", 8, 9, 1, 8191, *dense(1024, 8191))[4] == 4 and 18 % 4


@pytest.mark.parametrize("heads", range(1, 17))
def test_transcode_units_cover_every_slot_once(plans, heads):
    """The kernel's arithmetic, repeated here: the units of V and of K hold every (row, head) slot once, a lane of a K unit keeps its
    head from access to access, and the parameters fit a block's threads."""
    forms = set()
    for l, items, n in ((1, 1, 1), (1, 1, 127), (1, 1, 300), (2, 1, 385), (2, 2, 129), (200 // heads, 1, 129), (150 // heads, 1, 300)):
        acc, period, units, parts, groups, waves, blocks = plans("tc_units", heads, max(1, l), items, n)[:7]
        if not acc:
            continue
        forms.add(acc)
        total, step_k = n * heads, 8 * period
        assert units * acc == 16 * heads and step_k % heads == 0 and waves <= 8
        assert groups * heads * 64 <= 2 * 64 * waves  # two pairs of channels a thread
        for is_v in (True, False):
            seen, stored = [0] * total, set()
            for bx in range(blocks):
                for w in range(waves):
                    if is_v:
                        s0, step, g = (bx * waves + w) * acc * 8, 8, None
                    else:
                        q = bx // parts
                        gi, first = w // units, (bx - q * parts) * waves
                        u, g = first + w - gi * units, q * groups + gi
                        if q * groups * 128 >= n or u >= units:
                            continue
                        s0, step = g * 128 * heads + 8 * (u % period) + u // period * acc * step_k, step_k
                        if first == 0:
                            stored.update(x for x in range(q * groups, q * groups + groups) if x * 128 < n)
                    rem = max(0, min(total - s0, acc * step))
                    count = -(-rem // 8) if is_v else (rem + step - 1) // 8 // period
                    for k in range(acc):
                        for slot in range(8):
                            if slot + k * step < rem:
                                x = s0 + k * step + slot
                                assert k < count
                                seen[x] += 1
                                assert is_v or (x // (128 * heads) == g and x % heads == (8 * u + slot) % heads)
            assert all(x == 1 for x in seen)
            assert is_v or stored == set(range(ceil(n, 128)))
    assert forms == {4, 8}


def test_transcode_units_only_where_they_are_the_faster_form(plans):
    """Against units of 16 accesses: 1 head in 256-token items beyond 5,000 waves 1.00 / 0.96 / 0.89 (8 -> 4, 8 -> 2, 4 -> 2 bits), 5 heads between 1,700 and 2,000
    0.97 / 0.85 / 1.00, 13 heads between 900 and 1,100 0.95 / 0.89 / 1.02."""
    acc = lambda *a: plans("tc_units", *a)[0]
    assert [acc(8, l, 1, 300) for l in (10, 11, 22, 23)] == [4, 8, 8, 0]
    assert [acc(5, l, 1, 300) for l in (17, 18, 56, 57)] == [4, 8, 8, 0] and [acc(4, l, 1, 300) for l in (83, 84)] == [8, 0]
    assert [acc(1, 32, i, 256) for i in (39, 40)] == [8, 0] and [acc(1, 32, i, 257) for i in (10, 11)] == [8, 0] and [acc(2, 32, i, 256) for i in (7, 8)] == [8, 0]
    assert [acc(13, l, 1, 300) for l in (11, 12)] == [8, 0] and [acc(11, l, 1, 300) for l in (30, 31)] == [8, 0]
    assert acc(6, 20, 1, 400) == 8 and acc(16, 2, 1, 300) == 4 and acc(17, 1, 1, 1) == 0 and acc(8, 32, 32, 256) == 0 and acc(1, 32, 100, 256) == 0
    assert acc(2**24 - 1, 32767, 65535, 2**31 - 1) == 0


def test_gpu_tests_reach_the_transcoder_forms_they_name(plans):
    import test_gpu_transcode as t

    for heads, items in t.FORMS.items():
        assert [plans("tc_units", heads, 2, i, 300)[0] for i in items] == ([4, 8, 0] if heads <= 16 else [0])


def test_decode_units_of_whole_spans(plans):
    """Launches of whole spans of up to 48 MiB: enough one-wave blocks for K's sets of 4 heads x 16 rows and for V's 64 slots."""
    for heads in (8, 16, 24, 64):
        for l, items, n in ((1, 1, 1), (4, 1, 256), (3, 2, 17), (32, 1, 256), (80, 1, 33), (2, 1, 4001)):
            if l * items * n * heads > 48 * 2048:
                continue
            blocks, group = plans("dec_units", heads, l, items, n, *dense(128 * heads, n * items))[:2]
            assert blocks >= ceil(n, 16) * (heads // 4) and blocks * 64 >= n * heads and 1 <= group <= 2 * l
    at = lambda heads, l, items, n, strides=None: plans("dec_units", heads, l, items, n, *(strides or dense(128 * heads, n * items)))[:2]
    assert at(8, 32, 3, 128) == [16, 8] and at(8, 32, 1, 384) == [48, 8] and at(8, 2, 1, 256)[1] == 4
    assert at(8, 32, 3, 129)[0] == 0 and at(16, 32, 1, 193)[0] == 0 and at(8, 32767, 65535, 2**31 - 1)[0] == 0
    assert at(8, 32, 1, 256, (1024, 32 * 1024)) == [32, 64]
    assert at(8, 32, 1, 256, dense(1024, 8192)) == [32, 64] and at(8, 32, 1, 256, dense(1024, 512)) == [32, 64]   # half a plane and less
    assert at(8, 32, 1, 256, dense(1024, 511)) == [32, 8] and at(8, 32, 1, 384, dense(1024, 768)) == [48, 64]
    assert at(8, 32, 1, 385, dense(1024, 8192))[0] == 0 and at(8, 1, 1, 1, (2**62, 2**31))[0] == 2
    assert not any(at(h, 1, 1, 1)[0] for h in (1, 2, 3, 4, 5, 6, 7, 9, 12, 20))
    # what tests/test_gpu_row_lengths.py decodes in units and in spans
    assert at(8, 2, 1, 300)[0] and not at(8, 2, 96, 300)[0] and not at(16, 2, 48, 300)[0] and at(8, 9, 1, 640)[0] and not at(8, 9, 1, 8191)[0]


@pytest.mark.parametrize("heads", list(range(1, 26)) + [33, 64])
def test_encode_units_cover_rows_and_heads(plans, heads):
    s, strips = (1 if heads & 1 else 2), ceil(heads, 4)
    for l, items in ((1, 1), (4, 1), (7, 3), (32, 16)):
        for n in (1, 127, 129, 300, 3001):
            waves, blocks = plans("enc_units", heads, l, items, n)[:2]
            b = 2 * l * items * ceil(n, 128) * strips
            assert (waves != 0) == (heads >= 3 and not 144 < b <= 256 and (b <= 400 or (heads % 4 != 0 and heads < 15))), (l, items, n)
            if waves:  # sets of s heads x a token-group take 2 s waves; V and raw 64 slots a wave
                assert waves == 4 and blocks * (waves // (2 * s)) >= ceil(n, 128) * (heads // s) and blocks * waves * 64 >= n * heads
    assert plans("enc_units", 2**24 - 4, 32767, 65535, 2**31 - 1)[0] == 0


def test_encode_raw_slots_of_one_block_a_compute_unit_keep_their_blocks(plans):
    """9 heads, 4 x 1,536 tokens: 288 blocks of strips, but 216 of slots in blocks of 8 waves; raw 11.1 us in those, 12.6 in blocks of 4."""
    waves = lambda *a: (plans("enc_units", *a)[0], plans("enc_units", *a, known=True)[0])
    assert waves(9, 4, 1, 1536) == (4, 0) and waves(17, 4, 1, 960) == (4, 0) and waves(5, 12, 1, 748) == (4, 0)
    assert waves(9, 6, 1, 1152) == (4, 0) and waves(9, 8, 1, 1024) == (4, 4) and waves(10, 16, 1, 128) == (4, 4)
    assert waves(3, 20, 1, 876) == (4, 4) and waves(8, 17, 1, 477) == (4, 4)  # in strips before
    assert all(waves(h, 20, 1, 3001) == (0, 0) for h in (15, 17, 19, 22, 25, 33)) and waves(14, 20, 1, 3001) == (4, 4)
    assert [waves(h, 32, 32, 256)[0] for h in (7, 9, 10, 11, 13)] == [4, 0, 0, 0, 4]  # above 1 GiB in short items
    assert waves(10, 32, 25, 256) == (4, 4) and waves(10, 32, 16, 513) == (4, 4) and waves(10, 32, 1, 1024) == (4, 4)


def test_dropped_entries_are_stored_plainly_only_where_storing_alone_is_as_fast(plans):
    """Where nothing reads them back, raw blobs lost 3 to 7 % and quantised ones of more than 100 MB 1.5 to 2."""
    keeps = lambda bits, mib, more=0: plans("enc_keeps", bits, mib, more)[0]
    assert all(keeps(b, 0, 64) and keeps(b, 96) and not keeps(b, 96, 1) and not keeps(b, 262) for b in (8, 4, 2))
    assert not keeps(16, 0, 64) and not keeps(16, 48) and not keeps(16, 96)


def test_gpu_tests_reach_the_encoder_forms_they_name(plans):
    import test_gpu_row_lengths as t

    for heads, items in t.ENCODER_ITEMS.items():
        taken = [plans("enc_units", heads, 2, i, 300)[0] for i in items]
        assert taken == ([4, 0, 4, 0] if heads % 4 == 0 or heads >= 15 else [4, 0, 4, 4]), heads


def test_gpu_tests_reach_the_transcoder_streams_they_name(plans):
    """tests/test_gpu_transcode_large.py: units of 16 accesses, for 5 to 8 heads in one block and in two, for 13 and 25 in blocks of 8 waves and of 4."""
    import test_gpu_transcode_large as t

    assert not any(plans("tc_units", h, 1, n, 300)[0] for h, items in t.ITEMS.items() for n in items) and plans("tc_units", 1, 4, 640, 256)[0] == 0
    forms = {h: [plans("tc_stream", h, 1, n, 300)[:3] for n in items] for h, items in t.ITEMS.items()}
    assert forms == {1: [[-1, 3, 1]], 2: [[-1, 4, 1]], 3: [[-1, 3, 1]], 4: [[-1, 4, 1]], 5: [[-1, 5, 1], [-1, 3, 2]], 6: [[-1, 6, 1], [-1, 3, 2]],
                     7: [[-1, 7, 1], [-1, 4, 2]], 8: [[-1, 8, 1], [-1, 4, 2]], 9: [[0, 4, 1]], 10: [[1, 4, 1]], 11: [[0, 4, 1]], 12: [[2, 4, 1]],
                     13: [[3, 8, 1], [3, 4, 1]], 16: [[3, 4, 1]], 20: [[2, 4, 1]], 24: [[3, 4, 1]], 25: [[3, 8, 1], [3, 4, 1]]}


def test_gpu_tests_reach_the_large_forms_they_name(plans):
    import test_gpu_large_forms as t

    def spans(heads, items, rows):  # [slots, two blocks a compute unit]
        c = 128 * heads
        return plans("dec_launch", heads, t.L, items, t.N, items * rows * (c + 8), c + 8)[:2]

    assert [spans(h, n, 304) for h, n in t.DECODE] == [[0, 1], [0, 0], [0, 0]]
    assert all(plans("tc_units", h, t.L, n, t.N)[0] == 0 for h, n in t.TRANSCODE.items())
    forms = {h: plans("tc_stream", h, t.L, n, t.N)[:3] for h, n in t.TRANSCODE.items()}  # log2 of the heads of a set (-1: every P-th access), waves, blocks a token-group
    assert forms == {1: [-1, 3, 1], 2: [-1, 4, 1], 5: [-1, 5, 1], 8: [-1, 8, 1], 12: [2, 4, 1], 16: [3, 4, 1], 17: [0, 4, 1], 25: [3, 4, 1]}
    assert not any(plans("enc_units", h, t.L, n, 129)[0] for h, n in t.ENCODE)
    assert [plans("enc_plan", h, t.L, n, 129)[:2] for h, n in t.ENCODE] == [[0, 0], [1, 1], [0, 0], [0, 0], [1, 0], [1, 0]]
    for h, l, n in t.RAW:
        name, args = ("dec_launch", dense(128 * h, 4 * n)) if h % 8 == 0 else ("enc_units", ())
        a, b = (plans(name, h, l, 1, n, *args, known=known)[0] for known in (False, True))
        assert (a, b) == ((1, 0) if h % 8 == 0 else (4, 0)), (h, l, n)
