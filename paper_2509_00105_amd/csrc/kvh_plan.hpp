// What the launchers decide before a launch: the layout a kernel works in, its blocks and their order.  Plain host
// arithmetic over sizes, with no HIP in it, so that the rules can be checked without a GPU.
#pragma once

#include <stdint.h>

namespace kvh {

inline int lowest_bit(int x) { return __builtin_ctz((unsigned)x); }

// A grid's x dimension counts threads in 32 bits.  A launch beyond that is refused by its launcher: cut down to 32 bits the
// block count could pass for a small one that covers a part of the rows.
inline bool grid_fits(int64_t blocks, int planes, int waves) { return blocks <= 0xffffffffLL / (64LL * waves * planes); }

// ---- decoder ----------------------------------------------------------------------------------------------------
struct DecPlan {
  bool slots;           // rows in units of 64 (row, head) slots, otherwise in 1024-channel spans
  bool short_launch;    // spans with two blocks per CU
  int waves;            // of a block
  int64_t blocks;       // of a (layer, K|V) plane
  int plane_group, row_tile;  // block order, see decode_kernel
};

// Rows of whole 1024-channel spans: a block is 64 rows of a span.  Any other row length: units of 64 (row, head) slots, a
// wave each; the K units, whose row blocks are rounded up per set of heads, are the more numerous.
// Waves of a block of slots.  The waves are independent of each other.  With 8 a block holds 512 (row, head) pairs, four
// times what a block of spans holds of 2 heads, and a small launch leaves compute units without one.  Below 384 such blocks
// (three for two compute units) a block is one wave: 1 to 12 heads, 4 x 256 to 4 x 3,001 and 80 x 256 tokens, all levels
// 0.96 to 1.5 times as fast as blocks of 8 (2 heads 4 x 256 raw 5.2 -> 3.9 us, 3 heads 80 x 256 at 4 bits 10.9 -> 8.3); from
// 384 blocks on 0.87 to 1.06 (2 heads 32 x 2,048 raw 27 -> 31).
//
// Row tile.  Destination planes within 1 GiB of each other: planes first (one block per plane and turn), worth
// 1-2 % there over anything longer.  Beyond that: four blocks (256 rows) per plane and turn for items of up to
// 8,192 tokens, plane by plane for longer ones.  Measured on ten tensors of 2.5 to 16 GiB (8 to 80 layers, 8K to
// 128K tokens) against walking plane by plane, the kernel alone, 8 / 4 / 2 bits in points of HBM peak: items of 512
// tokens -1.4 to +3.9 / -1.6 to +5.3 / -0.4 to +4.9, of 1,024 tokens +0.9 to +8.9 / +1.0 to +11.8 / +2.2 to +9.2
// (walking plane by plane has a hole there, 67-69 % on most tensors), of 4,096 tokens -1.8 to +5.1 / -1.0 to +6.9 /
// -3.6 to +6.2; one item of 16,384 tokens +0.8 to +4.3 / -6.3 to +1.0 / -3.4 to +1.1, hence the limit.  Tiles of
// 2 are a point below tiles of 4, tiles of 8 two to four, tiles of 16 are the hole again.
// Plane group.  Groups of 8 planes, one block per plane and turn, through all items before the next group; or all planes,
// i.e. item by item in the row tiles above.  The dispatcher deals consecutive blocks to the 8 XCDs in turn, so that with 8
// planes each XCD writes one plane and keeps to its address translations.
//   Slots always take groups, of one size: against item by item, 40 shapes (128 to 2560 channels, 2,048 to 24,000 tokens,
//   chunks of 256 tokens to one item) 8 % faster on average, between -1 (512 channels) and +19 %; groups of 4 +7.6 %, but
//   better by 1 to 3 % for 512 channels, plane by plane +4.6 %.  With 10 planes two groups of 5 are 15 % (128 channels) to
//   4 % (640) faster than 8 and 2.
//   Whole spans take groups for launches of up to 896 MiB of 16-bit rows.  32 layers x 1024 channels in 256-token items,
//   five mixes of levels and destinations: 512 tokens +2 to +10 %, 1,024 +2 to +7, 2,048 +4 to +12, 4,096 +1 to +5,
//   6,144 (768 MiB) 0 to +4, 8,192 (1 GiB) -8 to -2.  Here it has to be 8: groups of 5 to 7 planes spread each plane over
//   all XCDs (6 layers in two groups of 6: 0.75 to 1.0 of the speed of all planes at once).  Where 8 does not divide the
//   planes, the smaller last group costs what the others gain unless there are two full groups before it and the launch
//   is over 80 MiB (13 layer counts from 5 to 42 that are no multiple of 4, 1024 to 4096 channels, 16 to 400 MiB: with this
//   rule 0.91 to 1.25 of the speed of all planes, 1.02 on average; groups of one size 0.75 to 1.2).
//   A destination in which a token's rows of all layers lie side by side (layer stride below token stride) always takes all
//   planes: consecutive blocks then fill a token's rows, groups leave holes between them.  32 layers, 256 to 8,192 tokens,
//   1 to 16 heads, all levels: groups 0.74 to 1.07 times as fast on all but the smallest launches (1024 channels, 2,048
//   tokens at 8 bits 77 us, in groups 88; 640 channels, 8,192 tokens at 2 bits 108 and 145).  Only small launches of 4 heads
//   (blocks of one wave) keep groups of 4: 32 x 256, 80 x 256 and 4 x 1,000 tokens 1.04 of the speed of all planes on
//   average, 0.92 to 1.24.
// Turns of whole spans.  Above 80 MiB the planes of a launch are better taken 4 (up to 1,400 MiB) or 8 at a time, one block
// each, than 8 or all, where a plane is neither small nor large: what is written at one time then lies close together,
// which counts most for pages of 16 tokens (32 KiB of 1024 channels, in random order).  Against groups of 8 or the row tiles below,
// inputs in no cache, 8 / 4 / 2 bits:
//   above 896 MiB, planes of up to 40 MiB (items of less than 512 tokens), 60 MiB (1,024) or 128 MiB.  50 launches of 256- and 384-token items
//   over 16 to 80 layers 0.98 to 1.10 / 0.98 to 1.11 / 0.98 to 1.15 (48 x 6,000 1.02 / 1.03 / 1.10, in pages 1.06 / 1.07 / 1.08; 80 x 3,727 in
//   pages 1.10 / 1.11 / 1.12); 512- to 2,048-token items of 24 to 80 layers x 4,096 to 40,000 tokens 0.98 to 1.09 at 8 bits, 0.99 to 1.1 at 4,
//   0.99 to 1.2 at 2 (below 1 where layers lie a multiple of 32 MiB apart), of 6 to 18 layers 0.98 to 1.15, 1.03 on average (11 layers in
//   512-token items 0.93 to 1.02), one item of 4,000 to 8,192 tokens 1.06 to 1.14 / 1.09 to 1.12 / 1.11 to 1.19;
//   larger planes 0.97 to 1.02 (32 x 32,768 in 512-token items 0.97 / 1.00 / 0.99);
//   80 to 896 MiB, 1024 channels, more than 10 planes of 4.5 to 16 MiB, turns of 4: items of 1,024 tokens and more, 60 launches 0.98 to 1.09
//   at 8 bits, 0.96 to 1.2 at 4, 1.0 to 1.29 at 2 (48 x 4,255 1.05 / 1.20 / 1.25); shorter items of 8 to 16 layers 0.98 to 1.12, 1.03 on average, of
//   20 to 80 0.96 to 1.09, 1.01 on average (30 x 4,128 in 512-token items in pages at 2 bits 94.4 -> 89.2 us), but of 6 and 7 layers 0.93 to 1.04.
// Not for items of less than 512 tokens where layers lie a multiple of 16 MiB apart (8,192 tokens x 1024 channels: 32 x 8,192 0.98 / 1.04 / 0.93, in
// pages 1.01 / 1.01 / 0.98; 32 x 16,384 0.99 / 1.02 / 0.94), nor of up to 128 tokens (ten launches 0.97 to 1.05 / 0.91 to 1.04 /
// 0.89 to 1.10, 0.99 on average).  Not where an item has just the blocks that run at a time, so that the previous order writes it all at
// once: 32 and 33 layers in 256-token items, 40 lengths from 7,400 to 9,200 tokens, 0.95 to 1.05 at 8 bits, 1.0 to 1.05 at 4 and 0.90 to 1.04 at 2,
// 0.96 on average there, three lengths apart (7,680 1.07, 8,128 1.22 and 8,256 1.28, whose previous order is as slow); 34 layers 0.99 to 1.01 and 0.94
// to 0.99, 30 layers 0.98 to 1.01 and 1.04 to 1.1; 16 layers in 512-token items 1.00 to 1.02 / 1.00 to 1.06 / 0.97 to 1.03.
// Items of more than 8,192 tokens that are alone stay plane by plane (1.00 to 1.1).
// Launches of whole spans of up to 80 MiB get two blocks per CU where they are not in units of slots (decode_units_plan): what they write
// is gone before the write stream has settled, and more waves in flight hide the start.  Nine layer counts from 2 to 80, 1024 to
// 4096 channels, all levels, two blocks against one in the same order: 48 MiB +3 to +8 % on average, 64 MiB +1 to +4, 80 MiB -1, 96
// MiB -1 to -3, 128 MiB 0 to -2, 192 and 256 MiB -1 to -2 (single cases down to -8 %).  Chunks of 48 to 80 MiB that go back into a
// cache of 2 to 8 times their size, one block against two: 8 bits 0.92 to 1.06, 0.94 on average, 4 bits 0.91 to 1.04, 0.96, 2 bits
// 0.97 to 1.07, raw 0.97 to 1.12 (24 x 752 of 3,760 tokens in pages, 8 bits: 22.4 us and 24.6).
inline DecPlan decode_plan(int heads, int l, int n_items, int max_tokens, int64_t layer_stride, int64_t token_stride) {
  DecPlan p;
  p.slots = heads % 8 != 0;
  p.waves = 8;
  if (p.slots) {
    const int log_s = lowest_bit(heads);
    const int64_t units = (((int64_t)max_tokens + (64 >> log_s) - 1) / (64 >> log_s)) * (heads >> log_s);
    p.blocks = (units + p.waves - 1) / p.waves;
    if ((double)p.blocks * 2 * l * n_items < 384) {
      p.waves = 1;
      p.blocks = units;
    }
  } else {
    p.blocks = (((int64_t)max_tokens + 63) / 64) * (heads / 8);
  }
  const int planes = 2 * l;
  const bool near = (int64_t)l * layer_stride * 2 <= ((int64_t)1 << 29);
  const bool side_by_side = layer_stride < token_stride;
  const double mib = 4.0 * l * heads * 128 * max_tokens * n_items / (1 << 20);  // of 16-bit rows
  p.short_launch = !p.slots && mib <= 80;
  p.row_tile = near || side_by_side || p.slots ? 1 : max_tokens <= 8192 ? 4 : 0x7fffffff;
  p.plane_group = planes;
  if (p.slots && (!side_by_side || (heads == 4 && p.waves == 1))) {
    const int most = heads == 4 ? 4 : 8, groups = (planes + most - 1) / most;
    p.plane_group = (planes + groups - 1) / groups;
  } else if (!p.slots && !side_by_side && mib <= 896 && (planes % 8 == 0 || (planes > 16 && mib > 80))) {
    p.row_tile = 1;
    p.plane_group = 8;
  }
  int turn = 0;
  if (!p.slots && !side_by_side && mib > 80) {
    const double plane = mib / planes;
    const int64_t item = p.blocks * planes;
    if (mib <= 896)
      turn = heads == 8 && plane >= 4.5 && plane <= 16 && planes > (max_tokens >= 1024 ? 10 : 14) ? 4 : 0;
    else if ((max_tokens < 512 && (max_tokens <= 128 || layer_stride % ((int64_t)8 << 20) == 0)) || (item >= 248 && item <= 272))
      turn = 0;
    else if (plane <= (max_tokens < 512 ? 40 : max_tokens < 1024 ? 60 : 128))
      turn = mib <= 1400 ? 4 : 8;
  }
  if (turn > 0 && turn < planes && (n_items > 1 || max_tokens <= 8192)) {
    p.row_tile = 1;
    p.plane_group = turn;
  }
  while (p.plane_group > 1 && !grid_fits(p.blocks, p.plane_group, p.waves)) p.plane_group = (p.plane_group + 1) / 2;
  return p;
}

// Whole spans, small launches.  A block of spans is 64 rows, 8 waves and (at 8 bits) a barrier, and its waves write 16 KiB a
// piece: 4 layers x 256 tokens make 32 blocks.  Up to 48 MiB of rows they run in units of slots, one wave a block (4 heads x 16
// rows, or 64 slots in memory order), which start sooner and spread evenly.  320 streams of launches over 2 to 80 layers, 8 and 16
// heads, all levels, inputs changing from launch to launch, against spans (two blocks per CU up to 80 MiB): up to 20 MiB 0.99 to 1.44
// times as fast (raw 0.92 to 1.21), 20 to 34 MiB 0.97 to 1.5 (raw 0.91 to 1.26), 34 to 48 MiB 1.0 to 1.4, 1.2 on average; beyond, spans win:
// 48 to 64 MiB 1.02 / 0.96 / 1.00 / 0.99 on average at 8 / 4 / 2 bits and raw, 100 to 130 MiB 1.01 / 0.97 / 1.00 / 1.01, 130 to 192
// MiB 0.99 / 0.96 / 0.98 / 0.99.  (4 x 256 tokens at 8 bits, pages: 6.9 -> 4.2 us by the kernel's own events.)
// Planes 8 at a time (4 at a time 0.96 to 1.0 of that), all at once where the layers of a token lie side by side (66 x 279 raw: 8 at
// a time 0.88, all 1.02), and where a launch fills no more than half of its planes (a chunk that goes back into a longer cache):
// planes a power of two apart then meet on the same memory channels when few of them are taken at a time.  32 x 256 tokens of
// an 8,192-token cache at 8 / 4 / 2 bits 11.7 / 9.8 / 9.1 us in spans, 12.4 / 11.0 / 10.7 in units with planes 8 at a time, 11.0 / 9.1 / 8.4
// with all; 50 such streams of 10 to 48 MiB into caches of 4,096 to 16,384 tokens 0.98 to 1.45 times as fast as spans.
// The raw level has no parameters to prepare and no barrier in spans, whose blocks only have to find a compute unit each: with more
// than 160 and up to 256 of them spans are the faster form.  Chunks into a longer cache by their blocks in spans, spans against units:
// 144 to 160 0.98 to 1.06, 168 to 256 0.99 to 1.1 (32 x 256 tokens of 8,192: 15.6 us and 17.1; 24 x 256 of 4,096 1.10), 280 to 384 0.82
// to 1.02; tensors of the launch's own size, inputs changing, 168 to 256 0.95 to 1.05, 264 and more 0.79 to 0.95.
// `raw`: every item is known to be of that level, as for a single blob; the descriptors of a batch are out of the launcher's sight.
struct DecUnits {
  int64_t blocks;   // of a (layer, K|V) plane, a wave each; 0: the layouts above
  int plane_group;
};
inline DecUnits decode_units_plan(int heads, int l, int n_items, int max_tokens, int64_t layer_stride, int64_t token_stride, bool raw) {
  DecUnits u{};
  const double mib = 4.0 * l * heads * 128 * max_tokens * n_items / (1 << 20);  // of 16-bit rows
  const bool sparse = 2.0 * n_items * max_tokens * token_stride <= layer_stride;
  if (heads % 8 != 0 || mib > 48) return u;
  const int64_t spans = ((int64_t)max_tokens + 63) / 64 * (heads / 8) * 2 * l * n_items;  // blocks of them
  if (raw && spans > 160 && spans <= 256) return u;
  u.blocks = ((int64_t)max_tokens + 15) / 16 * (heads / 4);  // K: sets of 4 heads x 16 rows; V has no more units
  const int most = sparse || layer_stride < token_stride ? 2 * l : 8;
  u.plane_group = most < 2 * l ? most : 2 * l;
  return u;
}

// What launch_decode launches.
struct DecLaunch {
  bool slots, short_launch;   // as in DecPlan: short_launch counts for spans alone
  int waves;
  int64_t blocks;             // of a (layer, K|V) plane; 0: refused, the grid would not fit
  int plane_group, row_tile;
  bool page_through;          // 2-bit rows into pages are stored with device scope
};
// Rows of 2 bits: whole spans are stored without device scope, into pages as elsewhere.  32 KiB pages (1024 channels x 16 tokens) and smaller ones, 1,130
// launches of 100 MiB to 4 GiB over buffers in turn, device scope against none: pages in random order 0.92 to 0.96 times as fast up to 1,000 MiB, 1.02 to
// 1.5 GiB and 0.995 beyond; in order 0.93 to 0.95, 1.00 and 0.97; in runs of 8 pages 0.94 to 0.98, 1.03 and 1.00.  200 launches of 4 to 14 GiB 1.01, 0.99 and 1.00,
// of mixed levels 1.00.  (A launch that the card is idle before and after is 1.1 times as fast on 32 x 8,192: what it leaves in the memory-side cache is
// written back in the time of what follows.)
// Slots of 2 bits into pages take device scope in small launches, whose rows are out before the kernel ends, and in large ones.  6,400 launches of 4 to 80
// layers, 128 to 3072 channels, pages of 8 to 64 tokens in random order and in order: up to 16 MiB 1.02 to 1.10, 16 to 40 MiB 0.99 to 1.04, 40 to 48 0.99; 48 to
// 100 MiB 0.98 to 0.995, 100 to 1,000 MiB 0.93 to 0.97 and 0.95 to 0.975; 1 to 1.5 GiB 1.02 and 1.03, beyond 1.01 to 1.03 and 1.03.
inline bool decode_page_through(double mib) { return mib <= 40 || mib >= 1024; }  // of 16-bit rows
inline DecLaunch decode_launch(int heads, int l, int n_items, int max_tokens, int64_t layer_stride, int64_t token_stride, bool raw) {
  const DecPlan p = decode_plan(heads, l, n_items, max_tokens, layer_stride, token_stride);
  if (!grid_fits(p.blocks, p.plane_group, p.waves)) return DecLaunch{};
  const DecUnits u = decode_units_plan(heads, l, n_items, max_tokens, layer_stride, token_stride, raw);
  const bool through = decode_page_through(4.0 * l * heads * 128 * max_tokens * n_items / (1 << 20));
  if (u.blocks != 0) return DecLaunch{true, false, 1, u.blocks, u.plane_group, 1, through};
  return DecLaunch{p.slots, p.short_launch, p.waves, p.blocks, p.plane_group, p.row_tile, p.slots && through};
}

// ---- transcoder -------------------------------------------------------------------------------------------------
// Small launches: units of 4 or 8 accesses (see transcode_units).
struct TcUnits {
  int accesses;    // of a unit, 0: units of 16, see transcode_stream_plan
  int period;      // accesses (of 8 slots) after which the heads repeat
  int units;       // of a token-group
  int parts;       // blocks of a token-group
  int groups;      // token-groups of a block
  int waves;       // of a block
  int64_t blocks;  // of a (layer, K|V) plane
};

// A wave of a large launch takes 16 accesses, and small launches then have few waves.  Units of 4 accesses, all requested at once, make 4 times the waves,
// but prepare K's parameters up to 4 times over (8 heads, 3 x 512 tokens bf16, 8 -> 4 bits: 9.7 / 7.1 / 5.5 us in units of 16 / 8 / 4).
// 19,000 launches of 1 to 80 layers and 200 to 3,001 tokens an item, buffers in turn, by w, the number of 16-access waves a launch takes.  Speed on average at
// 8 -> 4 / 8 -> 2 / 4 -> 2 bits, of units of 8 over units of 16:
//   w                up to 512            512 to 900           900 to 1,100         1,100 to 1,700       1,700 to 2,000       2,000 to 2,500
//   1 head           1.19 / 1.34 / 1.22   1.15 / 1.25 / 1.19   1.11 / 1.18 / 1.17   1.04 / 1.09 / 1.12   1.01 / 1.04 / 1.07   0.97 / 0.93 / 1.01 *
//   2                as 1                 as 1                 as 1                 1.02 / 1.08 / 1.11   1.00 / 1.05 / 1.08   0.99 / 0.97 / 1.03
//   4                1.14 / 1.31 / 1.17   1.10 / 1.22 / 1.14   1.05 / 1.15 / 1.11   1.01 / 1.08 / 1.11   1.01 / 1.08 / 1.11   0.99 / 0.99 / 1.06
//   11               1.16 / 1.12 / 1.20   1.10 / 1.08 / 1.16   1.00 / 1.02 / 1.08   1.10 / 1.09 / 1.20   1.08 / 1.06 / 1.16   1.10 / 1.05 / 1.17
//   3 and 5          1.14 / 1.31 / 1.17   1.10 / 1.22 / 1.14   1.05 / 1.15 / 1.11   1.04 / 1.04 / 1.09   0.98 / 0.88 / 1.00   0.89 / 0.82 / 0.90
//   9 and 10         1.16 / 1.12 / 1.20   1.10 / 1.08 / 1.16   1.00 / 1.02 / 1.08   1.07 / 1.03 / 1.17   0.98 / 0.90 / 1.00   1.05 / 0.91 / 1.08
//   6, 7, 8 and 12   1.39 / 1.35 / 1.34   1.24 / 1.25 / 1.27   1.08 / 1.12 / 1.13   0.99 / 1.02 / 1.06   1.04 / 0.99 / 1.08   1.03 / 0.94 / 1.07
//   15 and 16        1.21 / 1.12 / 1.20   1.17 / 1.08 / 1.19   1.11 / 1.03 / 1.14   0.99 / 0.91 / 1.05   1.02 / 0.90 / 1.06   1.01 / 0.85 / 1.03
//   13 and 14        1.23 / 1.08 / 1.23   1.19 / 1.05 / 1.21   0.95 / 0.89 / 1.02   as 15
// * 1 head in items of up to 256 tokens, which fill half a block of units of 16: 1.03 / 0.97 / 1.02 from 2,000 to 5,000, 1.00 / 0.96 / 0.89 beyond.
// Units of 4 over units of 8: 1.26 / 1.14 / 1.14 up to 512, 1.10 / 1.02 / 0.95 from there to 1,100.
// 2,700 launches of items of 8 to 128 tokens, units as taken over units of 16: 1.1 to 1.7 up to 512, 1.04 to 1.4 up to 1,100, 0.92 to 1.26 beyond (1 head).
// The limits are where the three pairs together no longer gain.  (Gains that are left: 11 heads beyond 2,000, 6, 7, 8 and 12 heads between 1,400 and 2,500.)
inline TcUnits transcode_units_plan(int heads, int l, int n_items, int max_tokens) {
  const int64_t groups = ((int64_t)max_tokens + 127) / 128;
  const double w = 2.0 * l * n_items * (double)groups * heads;
  double most = 1100;
  switch (heads) {
    case 1: most = max_tokens <= 256 ? 5000 : 2000; break;
    case 2: case 4: case 11: most = 2000; break;
    case 3: case 5: case 9: case 10: most = 1700; break;
    case 13: case 14: most = 900; break;
  }
  TcUnits u{};
  if (heads > 16 || w > most) return u;  // (16: what a block's threads prepare and its LDS holds)
  u.accesses = w <= 512 ? 4 : 8;
  const int log_g = lowest_bit(heads) < 3 ? lowest_bit(heads) : 3;
  u.period = heads >> log_g;
  u.units = 16 * heads / u.accesses;
  u.parts = (u.units + 7) / 8;
  u.groups = u.parts > 1 ? 1 : 8 / u.units;
  if (u.groups > groups) u.groups = (int)groups;
  u.waves = u.parts > 1 ? (u.units + u.parts - 1) / u.parts : u.units * u.groups;
  u.blocks = u.parts > 1 ? groups * u.parts : (groups + u.groups - 1) / u.groups;
  return u;
}

// All other launches: units of 16 accesses, in blocks of 3 to 8 waves.  130 launches of 4 to 65 layers, 256- to 2,048-token items, by w as above.  Speeds at 8 -> 4 /
// 8 -> 2 / 4 -> 2 bits, each over the same launches in a kernel with blocks of 8 waves and 4 accesses at a time, which is no longer there; the form taken comes first.
//   1 to 4 heads           every P-th access, up to 4 waves       0.97 to 1.45 / 1.05 to 1.47 / 1.04 to 1.56
//                          up to 8 waves                          0.96 to 1.39 / 1.05 to 1.46 / 1.00 to 1.30
//   5 and 6, w < 3,500     one block of all units                 1.01 to 1.25 / 1.04 to 1.20 / 1.00 to 1.13
//                          two blocks                             1.01 to 1.23 / 0.97 to 1.05 / 0.97 to 1.07
//            beyond        two blocks                             1.20 to 1.35 / 1.00 to 1.21 / 1.02 to 1.23
//                          one block                              1.08 to 1.35 / 0.96 to 1.14 / 0.93 to 1.13
//   7 and 8, w < 10,000    one block of all units                 1.00 to 1.34 / 1.05 to 1.15 / 0.99 to 1.04
//                          two blocks                             1.02 to 1.32 / 0.96 to 1.05 / 0.92 to 1.10
//            beyond        two blocks                             1.11 to 1.16 / 1.02 to 1.05 / 1.04
//                          one block                              1.06 to 1.14 / 1.04 to 1.07 / 0.99 to 1.02
//   16, 24 heads           sets of 8 heads, two blocks each       1.04 to 1.35 / 1.00 to 1.19 / 1.08 to 1.27
//                          one block each                         1.02 to 1.18 / 1.05 to 1.11 / 1.05 to 1.09
//                          sets of 4                              0.97 to 1.30 / 1.03 to 1.23 / 1.05 to 1.25
//   12, 20                 sets of 4                              1.04 to 1.29 / 1.06 to 1.27 / 1.06 to 1.24
//   10, 14, 18             pairs                                  1.00 to 1.23 / 1.10 to 1.28 / 1.06 to 1.23
//                          every P-th access                      0.90 to 1.00 / 0.73 to 0.93 / 0.79 to 1.00 (each block prepares all heads)
//   9, 11, 17              single heads                           1.02 to 1.25 / 1.04 to 1.23 / 0.96 to 1.37
//                          sets of 8, lanes idle                  0.80 to 1.15 / 0.76 to 1.14 / 0.78 to 1.08
//   13, 15, 25, 33         sets of 8, lanes idle, two blocks      1.12 to 1.31 / 1.03 to 1.20 / 1.12 to 1.26
//                          single heads                           1.02 to 1.31 / 1.00 to 1.29 / 0.91 to 1.19
//            w < 3,500     sets of 8 in one block                 1.19 / 1.13 / 1.12 (13 heads)
//                          two blocks                             1.31 / 0.96 / 1.16
// Blocks of two halves prepare the parameters twice, which 8 -> 2 bits feels in small launches.  More than 64 heads are sets of 8; the distance between the
// rows of an access then stays within 32 bits.
struct TcStream {
  int log_s;   // K: sets of 2^log_s heads x a token-group, a unit for each head (8 units are two blocks of 4 waves or one of 8); -1: every period-th access
  TcUnits in;  // with sets of heads only accesses, waves and blocks count
};

inline TcStream transcode_stream_plan(int heads, int l, int n_items, int max_tokens) {
  const int64_t groups = ((int64_t)max_tokens + 127) / 128;
  const double w = 2.0 * l * n_items * (double)groups * heads;
  const int lanes = (heads + 7) / 8 * 8, idle = lanes - heads, low = lowest_bit(heads);
  TcStream p{};
  TcUnits& u = p.in;
  u.accesses = 16;
  u.period = u.units = u.parts = u.groups = 1;
  if (heads <= 8) {
    const int most = heads > 4 && w < (heads < 7 ? 3500 : 10000) ? 8 : 4;
    p.log_s = -1;
    u.period = heads >> (low < 3 ? low : 3);
    u.units = heads;
    u.parts = (heads + most - 1) / most;
    u.groups = u.parts > 1 ? 1 : most / heads;
    if (u.groups > groups) u.groups = (int)groups;
    u.waves = u.parts > 1 ? (heads + u.parts - 1) / u.parts : heads * u.groups;
    u.blocks = u.parts > 1 ? groups * u.parts : (groups + u.groups - 1) / u.groups;
  } else {
    p.log_s = heads > 64 || low > 2 || (low == 0 && 4 * idle <= lanes) ? 3 : low;
    u.waves = p.log_s == 3 && idle > 0 && w < 3500 ? 8 : 4;
    const int64_t sets = groups * ((heads + (1 << p.log_s) - 1) >> p.log_s), per_block = u.waves >> p.log_s;
    u.blocks = per_block == 0 ? 2 * sets : (sets + per_block - 1) / per_block;
  }
  return p;
}

// ---- encoder ----------------------------------------------------------------------------------------------------
struct EncPlan {
  bool slots;      // V and raw rows in units of 64 (row, head) slots, otherwise in 512-channel strips
  bool k_slots;    // K in sets of slots (then `slots` holds), otherwise in strips
  bool plain_stores;  // with k_slots: single heads out of longer rows, see encode_kernel
  int waves;       // of a block
  int64_t blocks;  // of a (layer, K|V) plane
};

// The layouts of launches that encode_units_plan does not take: all of 1 and 2 heads, those of one block of strips a compute unit, and
// large ones of whole strips, of 15 heads and more and of 9 to 11 in short items above 1 GiB.
// Rows of whole strips, and of 3 heads: a block is one token-group of a strip.  Any other row length: V and raw blocks are
// units of slots, a wave each, in blocks of 8.  K slots in blocks of 8 take idle lanes away but read and write single heads or pairs: taken where more than
// a quarter of the strips' lanes idle, or a quarter and the heads come in pairs.  32 layers x 2,048 to 16,384 tokens in
// items of 256 to 12,000, strips (with slots for V) against slots: 1 head 1.35 to 2.3 times faster, 2 heads 1.1 to 1.25, 5
// heads 1.02 to 1.24, 6 heads 0.99 to 1.16, 3 heads 0.9 to 0.95, 7 to 18 heads 0.89 to 1.01.  With 3 heads slots in blocks of 8 bring V
// and the raw level nothing either (15 shapes, all levels: strips 1.00 to 1.11 times as fast as before slots, slots 0.89 to
// 1.14: 4 x 3,001 raw 8.9 -> 10.0 us, 32 x 1,024 in 256-token items raw 19.2 -> 21.0).
// Waves of a block: a set of slots takes 2 a head, so that the token-group of 1 or 2 heads is 2 or 4 waves.  Blocks of 8
// hold several token-groups of them, which leaves compute units without a block in small launches and half a block empty in
// short items; blocks of 4 are 0.97 to 1.37 times as fast on 19 shapes from 4 x 256 to 80 x 4,096 tokens (2 heads 4 x 3,001
// raw: 8.5 -> 6.3 us, 32 x 256 at 4 bits: 8.0 -> 6.6, 32 x 8,192 raw: 105.6 -> 97.9).  Items of up to 256 tokens keep one
// block an item where the launch is not small (2 heads, 32 x 2,048 in 256-token items with K and V rows in turn: blocks of 4
// 0.81 to 0.89; 80 x 256: 0.96 to 1.0; 32 x 256 and 4 x 256 on the other hand 1.15 to 1.34).
inline EncPlan encode_plan(int heads, int l, int n_items, int max_tokens) {
  const int strips = (heads + 3) / 4, lanes = strips * 4, idle = lanes - heads;
  const int64_t groups = ((int64_t)max_tokens + 127) / 128;
  EncPlan p;
  p.k_slots = 4 * idle > lanes || (4 * idle == lanes && heads % 2 == 0);
  p.slots = p.k_slots || (idle > 0 && heads > 3);
  p.plain_stores = p.k_slots && heads % 2 == 1 && heads > 1;
  p.waves = 8;
  p.blocks = groups * strips;  // never fewer than the blocks of slots in memory order
  if (p.k_slots) {
    const int s = (heads & 1) ? 1 : 2;
    auto blocks = [&](int waves) { return (groups * (heads / s) + waves / (2 * s) - 1) / (waves / (2 * s)); };
    if (heads <= 2) p.waves = max_tokens <= 256 && (double)blocks(8) * 2 * l * n_items >= 160 ? 4 * heads : 4;
    p.blocks = blocks(p.waves);
  }
  return p;
}

// Slots in blocks of 4 waves for rows of 3 heads and more.  A block of 4 waves is a K set of 2 heads (or two of one head) x a
// token-group, half a strip: twice the blocks, each half as long.  250 launches of 0.5 MiB to 1.3 GiB, 2 to 80 layers, against
// the layouts above, by the blocks of strips B a launch has:
//   rows that are not whole strips (3, 5, 6, 7, 9, 10, 11, 14 heads): 0.93 to 1.49 times as fast, 1.10 on average (5 heads, 20 x 3,001 at 4
//   bits 39.6 -> 37.3 us, 32 x 8,192 at 2 bits 150 -> 137; 10 heads, 14 x 220 raw 9.6 -> 7.0; least: 14 heads, 20 x 367), but with B from
//   145 to 256, where a block of strips finds a compute unit for itself, 0.85 to 1.11, 1.01 on average; large launches (200 to 3,000 MiB, inputs
//   changing) at 8 / 4 / 2 bits and raw on average: 5 and 6 heads 1.04 / 1.04 / 1.06 / 1.01, 7 1.00 / 1.01 / 1.07 / 1.00, 13 and 14 1.03 / 1.03 / 1.06 / 1.00, 9 and 10
//   1.02 / 1.02 / 1.07 / 1.01 and 11 0.98 / 0.99 / 1.05 / 1.01, but above 1 GiB in items of up to 512 tokens, where planes are taken 8 at a time, 9 to 11 heads 0.96
//   / 0.97 / 1.00 / 0.99 (64 x 6,000 of 10 heads 0.98 at every level, 48 x 8,192 of 9 0.91 / 0.97 / 0.99 / 0.96): these stay as they are;
//   whole strips: B up to 144 0.99 to 1.39 (8 heads, 24 x 83 at 8 bits 8.6 -> 7.2), 257 to 400, where some compute units get a second
//   block, 1.03 to 1.36 (17 x 477 raw 16.2 -> 11.9); 145 to 256 0.87 to 1.07 (one raw 1.27), beyond 400 0.94 to 1.06, but where a few blocks are
//   left over (few_left) when the chip, which holds 512, has been filled once or twice.  3,800 launches of 4 to 33 heads over 1 to 33 layers, 1 to 63 left over,
//   batches of one length and of mixed ones, at 8 / 4 / 2 bits and raw on average: whole strips after one turn 1.05 / 1.07 / 1.10 / 1.05, after two 1.03 / 1.05 /
//   1.09 / 1.05 (three 1.03 / 1.04 / 1.07 / 1.04, six 1.01 / 1.01 / 1.03 / 1.03; not taken), a tenth of them below 1.00 / 1.02 / 1.03 / 0.98; 15 heads and more that are no
//   whole strips 1.05 / 1.11 / 1.12 and 1.01 / 1.045 / 1.085, raw 1.03 and 1.08 in batches, 0.98 and 1.02 as single blobs, which stay (8 heads, 10 x 1,627, B = 520: 24.6 /
//   21.6 / 20.7 / 27.6 -> 23.7 / 20.2 / 18.9 / 27.2 us).  Raw items of less than 128 tokens have all their rows in the first blocks of a token-group: 0.90 on average, down to
//   0.49 (8 heads, 135 items of 2 x 28 tokens 0.56), and a batch's levels are out of the launcher's sight;
//   from 15 heads on few lanes of strips idle, and rows that are no whole strips follow the same limits: up to 144 and 257 to 400 0.98 to
//   1.46, 1.15 on average over 85 launches (66 heads, 4 x 128 at 8 bits 0.93); beyond, at 8 / 4 / 2 bits and raw, 0.91 to 1.04 / 0.92 to 1.07 / 0.98
//   to 1.11 / 0.97 to 1.01 (20 x 3,001 in one item at 8 bits: 15 to 33 heads but 21 and 23 0.91 to 0.94).
// Raw rows that are no whole strips were in slots before, in blocks of 8 waves, which they fill: where these are 145 to 256, blocks of 4
// lose as well (4 to 14 heads, B 264 to 320 0.87 to 0.98; 17 heads, 4 x 960 0.80).  `raw`: every item is known to be of that level, as for a
// single blob; the descriptors of a batch are out of the launcher's sight.
struct EncUnits {
  int waves;       // of a block, 0: the layouts above
  int64_t blocks;  // of a (layer, K|V) plane
};
inline EncUnits encode_units_plan(int heads, int l, int n_items, int max_tokens, bool raw) {
  const int64_t groups = ((int64_t)max_tokens + 127) / 128;
  const double planes = 2.0 * l * n_items;
  const bool whole = heads % 4 == 0;
  auto one_a_unit = [](double blocks) { return blocks > 144 && blocks <= 256; };
  const double b = planes * (double)groups * ((heads + 3) / 4);
  EncUnits u{};
  const bool far_apart = heads >= 9 && heads <= 11 && max_tokens <= 512 && planes * heads * 256 * max_tokens > ((int64_t)1 << 30);
  constexpr int kChip = 512, kTurns = 2;  // blocks of strips that run at a time; turns after which a few left over count
  const int turns = b < (kTurns + 1) * kChip ? (int)b / kChip : 0;
  const double left = b - turns * kChip;
  const bool few_left = turns >= 1 && left > 0 && left < 64 && max_tokens >= 128 && (whole || !raw);
  if (heads < 3 || one_a_unit(b) || far_apart || ((whole || heads >= 15) && b > 400 && !few_left)) return u;
  if (raw && !whole && heads > 3 && one_a_unit(planes * (double)(((int64_t)max_tokens * heads + 511) / 512))) return u;
  u.waves = 4;
  u.blocks = (groups * heads + 1) / 2;
  return u;
}

// Stores of the codes.  A blob is written once and read later, if at all on this device, so that its codes are stored non-temporally: on
// buffers in no cache 1.01 to 1.15 times as fast as plain stores.  The blob of one token-dropped entry (kvh_encode_kept; the items of a batch are out of
// the launcher's sight) may go back into the cache at once, compacted: stored plainly it stays in the 256 MiB of the memory-side cache, where
// kvh_decode_kept finds it.  That is taken as far as it costs next to nothing where the blob is not read again.  2,048 entries of 4 to 80 layers and 128 to 2048
// channels, blobs in turn over 1.5 GB so that what is written back later is in the time, speed of plain stores over non-temporal ones on average, of
// kvh_encode_kept alone / with a decode of other data behind it / with a copy / with kvh_decode_kept of the blob / with that and a decode behind it:
//   blob            quantised levels                          raw
//   up to 16 MB     0.99 / 1.00 / 0.99 / 1.05 / 1.02          0.97 / 0.99 / 0.98 / 1.11 / 1.04 (up to 24 MB)
//   16 to 48        1.01 / 0.995 / 1.00 / 1.09 / 1.05         0.98 / 0.98 / 0.98 / 1.13 / 1.06
//   48 to 100       0.99 / 0.99 / 1.00 / 1.09 / 1.06          0.96 / 0.97 / 0.98 / 1.14 / 1.08
//   100 to 170      0.985 / 0.985 / 1.01 / 1.07 / 1.05        0.935 / 0.95 / 0.98 / 1.12 / 1.07
//   170 to 268      0.98 / 0.98 / 1.02 / 1.06 / 1.06          0.93 / 0.94 / 0.98 / 1.12 / 1.10
// Beyond the size of the cache both lose (0.95).  Into pinned host memory plain stores are the faster ones (28 MB 527 us, non-temporal 729).
inline bool encode_keeps(int bits, uint64_t blob_bytes) { return bits <= 8 && blob_bytes <= (uint64_t)96 << 20; }

}  // namespace kvh
