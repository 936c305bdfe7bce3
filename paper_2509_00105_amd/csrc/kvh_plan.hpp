// What the launchers decide before a launch: the layout a kernel works in, its blocks and their order.  Plain host
// arithmetic over sizes, with no HIP in it, so that the rules can be checked without a GPU.
#pragma once

#include <stdint.h>

namespace kvh {

inline int lowest_bit(int x) { return __builtin_ctz((unsigned)x); }

// ---- transcoder -------------------------------------------------------------------------------------------------
struct TcPlan {
  bool slots;      // (row, head) slots; otherwise 1024-channel spans, in which the lanes beyond the row idle
  int log_s;       // K sets are 2^log_s heads (3: a span)
  int64_t sets;    // K sets of a token-group
  int64_t blocks;  // of a (layer, K|V) plane
};

// Slots take idle lanes away, but a K set of few heads reads and writes small pieces (128 * bits / 8 bytes a head).  32
// layers x 256 to 12,000 tokens, 4 x 3,001 and 80 x 1,000, slots against spans over the pairs of levels: 1 to 4, 9, 10 and
// 12 heads 1.0 to 4.9 times as fast but for small launches (below; least otherwise: 12 heads, 4 x 3,001 tokens, 4 to 8
// bits, 0.90); 5 heads 0.65 to 1.12, 6 heads 0.82 to 1.16, 7 heads 0.66 to 0.96, 11 heads 0.93 to 1.17, 13 heads 0.74 to
// 1.04, 17 heads 0.90 to 1.14, 33 heads 0.86 to 1.02.  So the share of idle lanes has to be the larger the smaller the
// pieces are: over 3/8 of a row's lanes with single heads, over 1/4 with pairs, 1/4 with fours.  (V alone in slots, K in
// spans: 5 to 33 heads 0.82 to 1.3.)
// A small launch of slots has an eighth to a half of the blocks that spans have: below 128 blocks rows of 3 heads and more
// keep spans (4 x 3,001 tokens x 384 channels, 8 -> 4 bits: spans 13.2 us, slots 14.6; 32 x 256: 12.4 and 13.3; rows of 1
// and 2 heads are 0.96 to 1.8 times as fast in slots even there).
inline TcPlan transcode_plan(int heads, int l, int n_items, int max_tokens) {
  const int spans = (heads + 7) / 8, lanes = spans * 8, idle = lanes - heads;
  const int s = 1 << lowest_bit(heads);
  const int64_t groups = ((int64_t)max_tokens + 127) / 128;
  TcPlan p;
  p.slots = 8 * idle > 3 * lanes || (s >= 2 && 4 * idle > lanes) || (s >= 4 && 4 * idle >= lanes);
  if (p.slots && heads > 2 && (double)((groups * heads + 7) / 8) * 2 * l * n_items < 128) p.slots = false;
  p.log_s = p.slots ? lowest_bit(heads) : 3;
  p.sets = p.slots ? heads >> p.log_s : spans;
  const int per_block = 8 >> p.log_s;
  p.blocks = (groups * p.sets + per_block - 1) / per_block;
  return p;
}

}  // namespace kvh
