// Level transcoder: re-compress a stored blob from b_in to b_out bits per element without ever
// writing 16-bit KV to memory (the policy's step that compresses a stored entry further; Design section,
// marginal utility drop).  The result is, byte for byte, encode(decode(blob)).
//
// Why no statistics pass is needed: in a blob written by the encoder (or by this kernel) every
// group holds code 0 and code L.  Code 0 decodes to the stored minimum exactly, code L to the
// stored maximum, and every other code to something in between, so the minimum and maximum of
// the decoded group are the stored ones and the re-encoded group keeps its metadata word.  The
// one exception is a degenerate group (range below 2^-100): all its elements decode to the
// minimum, so its new word is (mn, mn).  With the statistics known up front the kernel is a
// pure stream: code in -> fp32 reconstruction -> rounding to the 16-bit type -> position in the
// same range at the new rate -> code out.
//
// The (row, head) slots of a section are consecutive in memory.  A lane owns 16 consecutive channels, 8 lanes a slot, so that an
// access of a wave moves 8 slots (16 / 8 / 4 bytes per lane at 8 / 4 / 2 bits); a wave takes a unit of 16 accesses, of 4 or 8 in small
// launches (see transcode_units).  K parameters (per channel) are prepared once per block, two channels per thread, and shared
// through LDS; V parameters (per token and head) are prepared by one lane per group and broadcast inside the wave.  When
// the whole code -> code map of a group fits one register (4 -> 2 and the pairs that start from 2 bits) the "parameters"
// are that map, and an element costs a shift and a funnel shift.
#include <algorithm>
#include <type_traits>

#include "kvh_common.hpp"
#include "kvh_plan.hpp"

namespace kvh {

#ifndef KVH_TC_NT
#define KVH_TC_NT 1  // non-temporal stores of the output codes
#endif

#ifndef KVH_TC_WPE
#define KVH_TC_WPE 4  // waves per SIMD the register allocation is held to (0 = compiler's choice): two blocks per CU
#endif
#if KVH_TC_WPE
#define KVH_TC_OCC __attribute__((amdgpu_waves_per_eu(KVH_TC_WPE, KVH_TC_WPE)))
#else
#define KVH_TC_OCC
#endif

constexpr int kTcWaves = 8;                       // of a block, at most
constexpr int kTcThreads = kTcWaves * kWave;      // 512
constexpr int kTcLaneCh = 16;                     // channels per lane
constexpr int kTcBatch = 8;                       // accesses of a V wave whose groups its lanes prepare, one each
constexpr int kTcSpanHeads = kWave * kTcLaneCh / kGroup;  // 8 (row, head) slots per access
constexpr int kSlotLanes = kGroup / kTcLaneCh;    // 8 lanes per slot
static_assert(kTcBatch * kTcSpanHeads == kWave, "one lane per V group of a batch");

typedef uint32_t uintx2 __attribute__((ext_vector_type(2)));
typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

namespace {

template <typename T>
__device__ __forceinline__ T gload(const uint8_t* p) {
  return *reinterpret_cast<const __attribute__((address_space(1))) T*>(reinterpret_cast<uintptr_t>(p));
}
#ifndef KVH_TC_NTL
#define KVH_TC_NTL 1  // non-temporal loads of the input codes
#endif
template <typename T>
__device__ __forceinline__ T gload_codes(const uint8_t* p) {
#if KVH_TC_NTL
  return __builtin_nontemporal_load(reinterpret_cast<const __attribute__((address_space(1))) T*>(reinterpret_cast<uintptr_t>(p)));
#else
  return gload<T>(p);
#endif
}
template <typename T>
__device__ __forceinline__ void gstore(uint8_t* p, T v) {
  *reinterpret_cast<__attribute__((address_space(1))) T*>(reinterpret_cast<uintptr_t>(p)) = v;
}
template <typename T>
__device__ __forceinline__ void gstore_stream(uint8_t* p, T v) {
#if KVH_TC_NT
  __builtin_nontemporal_store(v, reinterpret_cast<__attribute__((address_space(1))) T*>(reinterpret_cast<uintptr_t>(p)));
#else
  gstore<T>(p, v);
#endif
}

// Two fp32 values -> two 16-bit values in one word, each rounded to nearest even.
template <int DT>
__device__ __forceinline__ uint32_t pack2(float a, float b) {
  floatx2 f = {a, b};
  if constexpr (DT == KVH_F16) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, halfx2));
  } else {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
  }
}

// fp32 reconstruction of a code.  The definition rounds twice (fma to fp32, then to the 16-bit
// type); the empty asm keeps the compiler from merging the two into one mixed-precision fma.
__device__ __forceinline__ float recon(float q, float scale, float mn) {
  float y = __builtin_fmaf(q, scale, mn);
  asm("" : "+v"(y));
  return y;
}

// The 16 input codes of a lane.  spread() lays them out one per byte (4 words), so that each code
// then costs a single byte->float convert; the empty asm keeps the compiler from undoing that
// into one bit-field extract plus one convert per code.
__device__ __forceinline__ uint32_t opaque(uint32_t x) {
  asm("" : "+v"(x));
  return x;
}
template <int BITS>
struct InCodes;
template <>
struct InCodes<8> {
  uintx4 w;
  __device__ __forceinline__ void load(const uint8_t* p) { w = gload_codes<uintx4>(p); }
  __device__ __forceinline__ float get(const uint32_t (&e)[4], int j) const { return (float)((e[j >> 2] >> (8 * (j & 3))) & 0xffu); }
  __device__ __forceinline__ void spread(uint32_t (&e)[4]) const {
    e[0] = w.x; e[1] = w.y; e[2] = w.z; e[3] = w.w;
  }
};
template <>
struct InCodes<4> {
  uintx2 w;
  __device__ __forceinline__ void load(const uint8_t* p) { w = gload_codes<uintx2>(p); }
  // e[0] / e[1] = even / odd nibbles of the first word, e[2] / e[3] of the second
  __device__ __forceinline__ void spread(uint32_t (&e)[4]) const {
    e[0] = opaque(w.x & 0x0f0f0f0fu);
    e[1] = opaque((w.x >> 4) & 0x0f0f0f0fu);
    e[2] = opaque(w.y & 0x0f0f0f0fu);
    e[3] = opaque((w.y >> 4) & 0x0f0f0f0fu);
  }
  __device__ __forceinline__ float get(const uint32_t (&e)[4], int j) const {
    return (float)((e[(j >> 3) * 2 + (j & 1)] >> (8 * ((j & 7) >> 1))) & 0xffu);
  }
};
template <>
struct InCodes<2> {
  uint32_t w;
  __device__ __forceinline__ void load(const uint8_t* p) { w = gload_codes<uint32_t>(p); }
  // e[k] holds codes k, k + 4, k + 8, k + 12 in its four bytes
  __device__ __forceinline__ void spread(uint32_t (&e)[4]) const {
#pragma unroll
    for (int k = 0; k < 4; ++k) e[k] = opaque((w >> (2 * k)) & 0x03030303u);
  }
  __device__ __forceinline__ float get(const uint32_t (&e)[4], int j) const {
    return (float)((e[j & 3] >> (8 * (j >> 2))) & 0xffu);
  }
};

// Four positions -> four code bytes in one word; the convert rounds to nearest even and
// saturates to [0, 255].
__device__ __forceinline__ uint32_t codes4(float t0, float t1, float t2, float t3) {
  uint32_t a = __builtin_amdgcn_cvt_pk_u8_f32(t0, 0, 0u);
  a = __builtin_amdgcn_cvt_pk_u8_f32(t1, 1, a);
  a = __builtin_amdgcn_cvt_pk_u8_f32(t2, 2, a);
  return __builtin_amdgcn_cvt_pk_u8_f32(t3, 3, a);
}

// Pack 16 positions into BITS-bit codes (channel order, LSB first) and store them.  The convert
// puts a code into any byte of a word, so narrow codes are routed at that point: word i receives,
// in its byte k, the code that belongs i fields above the bottom of output byte k, and the words
// are then merged with one shift-or each.  (For finite positions every code is <= L, so fields
// never overlap.)
template <int BITS>
__device__ __forceinline__ void store_codes16(uint8_t* p, const float (&t)[16]) {
  if constexpr (BITS == 8) {
    uintx4 o;
    o.x = codes4(t[0], t[1], t[2], t[3]);
    o.y = codes4(t[4], t[5], t[6], t[7]);
    o.z = codes4(t[8], t[9], t[10], t[11]);
    o.w = codes4(t[12], t[13], t[14], t[15]);
    gstore_stream<uintx4>(p, o);
  } else if constexpr (BITS == 4) {
    uintx2 o;
    o.x = codes4(t[0], t[2], t[4], t[6]) | codes4(t[1], t[3], t[5], t[7]) << 4;
    o.y = codes4(t[8], t[10], t[12], t[14]) | codes4(t[9], t[11], t[13], t[15]) << 4;
    gstore_stream<uintx2>(p, o);
  } else {
    uint32_t o = codes4(t[0], t[4], t[8], t[12]) | codes4(t[1], t[5], t[9], t[13]) << 2 |
                 codes4(t[2], t[6], t[10], t[14]) << 4 | codes4(t[3], t[7], t[11], t[15]) << 6;
    gstore_stream<uint32_t>(p, o);
  }
}

// Everything one group contributes to the arithmetic, as fp32.
struct TcParams {
  float mn;     // f32(mn)
  float scale;  // r / L_in, or 0 (degenerate)
  float inv;    // L_out / r, or 0 (degenerate)
  float top;    // what code L_in decodes to by definition: f32(mx), or f32(mn) (degenerate)
};

// Parameters of a group from its metadata word; also the word the re-encoded group stores.
template <int DT, int BI, int BO>
__device__ __forceinline__ TcParams tc_params(uint32_t meta, uint32_t& out_meta) {
  TcParams p;
  const uint32_t mn_bits = meta & 0xffffu, mx_bits = meta >> 16;
  p.mn = t16_to_f32<DT>(mn_bits);
  const float r = t16_to_f32<DT>(mx_bits) - p.mn;
  const bool degenerate = r < 0x1p-100f;
  p.scale = degenerate ? 0.0f : range_over_levels<BI>(r);  // correctly rounded quotients
  p.inv = degenerate ? 0.0f : levels_over_range<BO>(r);
  const uint32_t top_bits = degenerate ? mn_bits : mx_bits;
  p.top = t16_to_f32<DT>(top_bits);
  out_meta = mn_bits | top_bits << 16;
  return p;
}

// One row of a lane: 16 codes in, 16 codes out.  param(j) gives the parameters of channel j.
//
// The definition decodes code L_in to the stored maximum mx itself, here it is reconstructed like any other code: the new code is
// the same.  With r the range, y = fma(L_in, r / L_in, mn) is within r 2^-22 + |mx| 2^-24 of mx, and since mx is a 16-bit value,
// rounding y to the nearest one moves it by no more than that again.  Up to |mx| = 2^10 r the result is within r 2^-12 of mx,
// less than a tenth of a step at 8 bits; beyond, y is closer to mx than half a unit in its last place and becomes mx.  In either case the
// position rounds to L_out.  (A degenerate group has inv = 0 and only code 0.)
template <int DT, int BI, int BO, typename P>
__device__ __forceinline__ void transcode_row(uint8_t* out, const InCodes<BI>& cw, P&& param) {
  float t[kTcLaneCh];
  uint32_t e[4];
  cw.spread(e);
#pragma unroll
  for (int j = 0; j < kTcLaneCh; j += 2) {
    const TcParams& p0 = param(j);
    const TcParams& p1 = param(j + 1);
    const float q0 = cw.get(e, j), q1 = cw.get(e, j + 1);
    float x0, x1;
    if constexpr (DT == KVH_BF16) {
      // a bf16 value in the upper half of a word over a zero lower half is that value as fp32: one convert per
      // element rounds and widens at once (a pair packed together would need unpacking, half an operation more)
      x0 = __builtin_bit_cast(float, pack2<DT>(0.0f, recon(q0, p0.scale, p0.mn)));
      x1 = __builtin_bit_cast(float, pack2<DT>(0.0f, recon(q1, p1.scale, p1.mn)));
    } else {
      const uint32_t pk = pack2<DT>(recon(q0, p0.scale, p0.mn), recon(q1, p1.scale, p1.mn));
      x0 = t16_to_f32<DT>(pk & 0xffffu);
      x1 = t16_to_f32<DT>(pk >> 16);
    }
    // position in the range at the new rate: subtract, then multiply (two roundings)
    t[j] = (x0 - p0.mn) * p0.inv;
    t[j + 1] = (x1 - p1.mn) * p1.inv;
  }
  store_codes16<BO>(out, t);
}

// ---- narrow inputs: one small table per group ---------------------------------------------------
// With b_in <= 4 a group has at most 16 distinct input codes, so its whole code -> code map fits one
// register when 2^b_in * b_out <= 32 (4 -> 2, 2 -> 2, 2 -> 4, 2 -> 8).  The map is built by running
// the arithmetic above once per input code; an element then costs a shift and a funnel shift
// instead of seven floating-point instructions.
template <int BI, int BO>
constexpr bool kUseTable = (1 << BI) * BO <= 32;

// Where a group lies no further from zero than some multiple of its range, its map is the one of exact arithmetic, code q to the
// code nearest to q L_out / L_in, and needs no evaluation.  The quotient (never half-way between two codes) keeps a distance of
// kMargin from every half-way point, and what the definition adds to it is the rounding of the value to 16 bits, at most M 2^-8 (bf16) or
// M 2^-11 + 2^-25 (fp16) for a group whose values reach M, times L_out / r; the roundings to fp32 move the position
// by less than 20 L_out 2^-24 as long as M is below 2^4 r (the sum by M 2^-24 / r, its quotient, difference and product by 2^-24 each), at most 2^-10 of the margin
// (2 -> 8 bits), for which 1/64 is set aside.  From 4 to 2 bits that is M < 8.4 r in bf16: all groups but those of a large
// common offset.  32 layers x 8,192 tokens x 1024 channels, 4 -> 2 bits: 87.2 us with every
// table evaluated (16 times 7 operations), 77.5.
template <int BI, int BO>
constexpr uint32_t usual_table() {
  constexpr uint32_t LI = (1u << BI) - 1, LO = (1u << BO) - 1;
  uint32_t table = 0;
  for (uint32_t q = 0; q <= LI; ++q) table |= (2 * q * LO + LI) / (2 * LI) << (BO * q);
  return table;
}
template <int DT, int BI, int BO>
__device__ __forceinline__ bool usual_map(uint32_t meta) {
  static_assert(kUseTable<BI, BO>, "4 -> 2 bits, or from 2 bits");
  constexpr float LO = float((1 << BO) - 1);
  constexpr float kMargin = BI == 4 ? 0.1f : 0.5f;  // q / 5; otherwise a whole multiple of q
  const float mn = t16_to_f32<DT>(meta & 0xffffu), mx = t16_to_f32<DT>(meta >> 16), r = mx - mn;
  const float most = __builtin_fmaxf(__builtin_fabsf(mn), __builtin_fabsf(mx));
  const float off = DT == KVH_F16 ? __builtin_fmaf(most, 0x1p-11f, 0x1p-25f) : most * 0x1p-8f;
  return off < r * (kMargin / LO * (63.0f / 64.0f)) && most < r * 16.0f && r < 0x1p120f;
}

template <int DT, int BI, int BO>
__device__ __forceinline__ uint32_t code_table(uint32_t meta, uint32_t& out_meta) {
  constexpr int NQ = 1 << BI;
  const TcParams p = tc_params<DT, BI, BO>(meta, out_meta);
  const bool usual = usual_map<DT, BI, BO>(meta);
  uint32_t table = p.inv == 0.0f ? 0u : usual_table<BI, BO>();
  if (__builtin_amdgcn_ballot_w64(!usual && p.inv != 0.0f) == 0) return table;  // wave-uniform
  uint32_t other = 0;
#pragma unroll
  for (int q = 0; q < NQ; q += 2) {
    const uint32_t pk = pack2<DT>(recon((float)q, p.scale, p.mn), recon((float)(q + 1), p.scale, p.mn));
    const float x0 = t16_to_f32<DT>(pk & 0xffffu);
    const float x1 = q + 1 == NQ - 1 ? p.top : t16_to_f32<DT>(pk >> 16);  // the top code decodes to the stored maximum
    const uint32_t two = __builtin_amdgcn_cvt_pk_u8_f32((x1 - p.mn) * p.inv, 1,
                                                        __builtin_amdgcn_cvt_pk_u8_f32((x0 - p.mn) * p.inv, 0, 0u));
    other |= ((two & 0xffu) | ((two >> 8) & 0xffu) << BO) << (BO * q);
  }
  return usual ? table : other;
}

// Byte-wise shift amounts b_out * q for the 16 codes of a lane: code j sits in byte sh_byte(j) of
// e[sh_word(j)].
template <int BI, int BO>
struct Shifts;
template <int BO>
struct Shifts<4, BO> {
  static constexpr int S = BO == 2 ? 1 : BO == 4 ? 2 : 3;
  static constexpr uint32_t M = 0x0f0f0f0fu << S;
  static __device__ __forceinline__ void make(const InCodes<4>& cw, uint32_t (&e)[4]) {
    e[0] = opaque((cw.w.x << S) & M);
    e[1] = opaque((cw.w.x >> (4 - S)) & M);
    e[2] = opaque((cw.w.y << S) & M);
    e[3] = opaque((cw.w.y >> (4 - S)) & M);
  }
  static constexpr int word(int j) { return (j >> 3) * 2 + (j & 1); }
  static constexpr int byte(int j) { return (j & 7) >> 1; }
};
template <int BO>
struct Shifts<2, BO> {
  static constexpr int S = BO == 2 ? 1 : BO == 4 ? 2 : 3;
  static constexpr uint32_t M = 0x03030303u << S;
  static __device__ __forceinline__ void make(const InCodes<2>& cw, uint32_t (&e)[4]) {
#pragma unroll
    for (int k = 0; k < 4; ++k) e[k] = opaque((2 * k >= S ? cw.w >> (2 * k - S) : cw.w << (S - 2 * k)) & M);
  }
  static constexpr int word(int j) { return j & 3; }
  static constexpr int byte(int j) { return j >> 2; }
};

// One row of a lane through the tables.  table(j) gives the table of channel j.
template <int BI, int BO, typename T>
__device__ __forceinline__ void lookup_row(uint8_t* out, const InCodes<BI>& cw, T&& table) {
  using Sh = Shifts<BI, BO>;
  constexpr int kPer = 32 / BO;  // codes per output word
  uint32_t e[4];
  Sh::make(cw, e);
  uint32_t acc[kTcLaneCh / kPer] = {};
#pragma unroll
  for (int j = 0; j < kTcLaneCh; ++j) {
    const uint32_t x = table(j) >> ((e[Sh::word(j)] >> (8 * Sh::byte(j))) & 0xffu);
    // funnel shift: the low b_out bits of x enter at the top; after kPer steps code j sits at bit b_out * (j % kPer)
    acc[j / kPer] = __builtin_amdgcn_alignbit(x, acc[j / kPer], BO);
  }
  if constexpr (BO == 2) {
    gstore_stream<uint32_t>(out, acc[0]);
  } else if constexpr (BO == 4) {
    uintx2 o = {acc[0], acc[1]};
    gstore_stream<uintx2>(out, o);
  } else {
    uintx4 o = {acc[0], acc[1], acc[2], acc[3]};
    gstore_stream<uintx4>(out, o);
  }
}

// ---- 8 -> 2 bits: the code -> code map of a group as a polynomial of the input code ------------------
// The map f(q) of a group (reconstruct, round to the 16-bit type, re-position, round to a code) is a monotone step
// function of q with three steps, because every operation in it is monotone.  If some cheap monotone function
// g(q) is shown to round to f(q) at the last code before each step and at the first code of each step (and at both
// ends), the two agree at all 256 codes, and an element costs  byte -> float, g, float -> code  instead of the seven
// floating-point instructions of the definition.  Two forms of g are used:
//   standard  g(q) = q / 85: steps at 43, 128, 213, which is where the steps of a group lie unless the rounding to
//             the 16-bit type moves them (it does when the group sits far from zero compared with its range);
//             recognised by evaluating f at the six codes around those steps;
//   fitted    the parabola through the three step positions of the group, found by evaluating f itself, and
//             accepted only if evaluating it with the very instructions of the row loop reproduces f at the codes
//             around its steps and at both ends, with a slope that keeps it monotone.
// A group that passes neither test (a range of a few units in the last place, say) sends its block, or its batch
// of V rows, down the arithmetic route above.  Bit-exactness therefore never rests on the fit, only on the checks.
struct Quad {
  float a, b, c;  // g(q) = (a q + b) q + c
};
enum : uint32_t { kStandard = 0u, kFitted = 1u, kHard = 2u };

// f(q) by the definition (the top code decodes to the stored maximum).
template <int DT>
__device__ __forceinline__ uint32_t code82(float q, const TcParams& p) {
  const uint32_t pk = pack2<DT>(recon(q, p.scale, p.mn), 0.0f);
  float x = t16_to_f32<DT>(pk & 0xffffu);
  x = q == 255.0f ? p.top : x;
  return __builtin_amdgcn_cvt_pk_u8_f32((x - p.mn) * p.inv, 0, 0u);
}
// g(q) exactly as the row loop evaluates it
__device__ __forceinline__ float quad_value(float q, const Quad& g) { return __builtin_fmaf(__builtin_fmaf(g.a, q, g.b), q, g.c); }
__device__ __forceinline__ uint32_t quad_code(float q, const Quad& g) { return __builtin_amdgcn_cvt_pk_u8_f32(quad_value(q, g), 0, 0u); }

template <int DT>
__device__ __forceinline__ uint32_t classify82(const TcParams& p, Quad& g) {
  g = Quad{0.0f, 0.0f, 0.0f};
  if (p.inv == 0.0f) return kFitted;  // degenerate group: every code becomes 0, and so does g
  const bool standard = code82<DT>(42.0f, p) == 0u && code82<DT>(43.0f, p) == 1u && code82<DT>(127.0f, p) == 1u &&
                        code82<DT>(128.0f, p) == 2u && code82<DT>(212.0f, p) == 2u && code82<DT>(213.0f, p) == 3u;
  if (standard) {
    g.b = 1.0f / 85.0f;  // what a standard group contributes where its neighbours need the fitted form
    return kStandard;
  }
  // First code of each step.  The steps lie within a few codes of 43, 128, 213, so each is looked for from there,
  // one code at a time in the direction the two evaluations at the usual place point to; a step further away than
  // kReach codes makes the group a hard one.
  constexpr int kReach = 6;
  float t[3];
  bool found = true;
#pragma unroll
  for (int k = 1; k <= 3; ++k) {
    const float hi0 = k == 1 ? 43.0f : k == 2 ? 128.0f : 213.0f;
    const bool below = code82<DT>(hi0 - 1.0f, p) >= (uint32_t)k;  // the step is at or before the code below the usual place
    const bool above = code82<DT>(hi0, p) < (uint32_t)k;          // the step is after the usual place
    float tk = hi0;
    bool searching = below || above;
    const float dir = below ? -1.0f : 1.0f;
    float q = below ? hi0 - 1.0f : hi0;
#pragma unroll 1
    for (int step = 0; step < kReach && __builtin_amdgcn_ballot_w64(searching) != 0; ++step) {
      q += dir;
      const bool ge = code82<DT>(q, p) >= (uint32_t)k;
      if (searching && ge != below) {  // crossed the step: going up, q is its first code; going down, q + 1 is
        tk = below ? q + 1.0f : q;
        searching = false;
      }
    }
    found = found && !searching;
    t[k - 1] = tk;
  }
  if (!found || !(t[0] >= 1.0f && t[0] < t[1] && t[1] < t[2] && t[2] <= 255.0f)) return kHard;
  // parabola through (t_k - 1/2, k - 1/2); approximate reciprocals will do, the checks below are what counts
  const float x1 = t[0] - 0.5f, x2 = t[1] - 0.5f, x3 = t[2] - 0.5f;
  const float d1 = __builtin_amdgcn_rcpf(x2 - x1), d2 = __builtin_amdgcn_rcpf(x3 - x2);
  g.a = (d2 - d1) * __builtin_amdgcn_rcpf(x3 - x1);
  g.b = d1 - g.a * (x1 + x2);
  g.c = 0.5f - (g.a * x1 + g.b) * x1;
  bool ok = quad_code(0.0f, g) == 0u && quad_code(255.0f, g) == 3u;
#pragma unroll
  for (int k = 1; k <= 3; ++k) ok = ok && quad_code(t[k - 1] - 1.0f, g) == (uint32_t)(k - 1) && quad_code(t[k - 1], g) == (uint32_t)k;
  // slope at both ends well above what rounding errors in g could undo
  ok = ok && g.b >= 0x1p-9f && __builtin_fmaf(510.0f, g.a, g.b) >= 0x1p-9f;
  return ok ? kFitted : kHard;
}

// One row of a lane through g.  coef(j) gives the polynomial of channel j (unused when STANDARD).
template <bool STANDARD, typename C>
__device__ __forceinline__ void poly_row82(uint8_t* out, const InCodes<8>& cw, C&& coef) {
  constexpr float kStep = 1.0f / 85.0f;
  float t[kTcLaneCh];
  uint32_t e[4];
  cw.spread(e);
#pragma unroll
  for (int j = 0; j < kTcLaneCh; ++j) {
    const float q = cw.get(e, j);
    if constexpr (STANDARD) t[j] = q * kStep; else t[j] = quad_value(q, coef(j));
  }
  store_codes16<2>(out, t);
}

struct HeaderWords {
  uintx4 a, b, c;
};

// Header of the source blob against the call; the token-dropping words are accepted if they are
// all zero or describe an entry of which exactly n tokens are kept.
__device__ __forceinline__ bool source_header_ok(const HeaderWords& h, int dt, int bits, int l, int n, int c, size_t total) {
  const bool fields = h.a.x == kMagic && h.a.y == (1u | (uint32_t)dt << 16 | (uint32_t)bits << 24) && h.a.z == (uint32_t)l &&
                      h.a.w == (uint32_t)n && h.b.x == (uint32_t)c && h.b.y == ((uint32_t)kGroup | (uint32_t)kGroup << 16) &&
                      h.b.z == (uint32_t)total && h.b.w == (uint32_t)((uint64_t)total >> 32);
  const uint32_t orig = h.c.x, sink = h.c.y, window = h.c.z;
  const uint64_t sw = (uint64_t)sink + window;
  const bool plain = (orig | sink | window) == 0;
  const bool dropped = orig >= 1 && orig <= 0x7fffffffu && sw >= 1 && sw <= 0x7fffffffu &&
                       (sw >= orig ? orig : (uint32_t)sw) == (uint32_t)n;
  return fields && (plain || dropped);
}

// One word a thread of the header of the result; the token-dropping words are carried over.
template <int DT, int BO>
__device__ __forceinline__ void write_header(uint8_t* dst, const TranscodeParams& a, uint32_t n, const LayerGeom& go, const HeaderWords& hdr) {
  const uint64_t total = kHeaderBytes + (uint64_t)a.l * go.layer_bytes();
  uint32_t w = 0;
  switch (threadIdx.x) {
    case 0: w = kMagic; break;
    case 1: w = 1u | (uint32_t)DT << 16 | (uint32_t)BO << 24; break;
    case 2: w = (uint32_t)a.l; break;
    case 3: w = n; break;
    case 4: w = (uint32_t)a.c; break;
    case 5: w = (uint32_t)kGroup | (uint32_t)kGroup << 16; break;
    case 6: w = (uint32_t)total; break;
    case 7: w = (uint32_t)(total >> 32); break;
    case 8: w = hdr.c.x; break;
    case 9: w = hdr.c.y; break;
    case 10: w = hdr.c.z; break;
    default: break;
  }
  gstore<uint32_t>(dst + 4 * threadIdx.x, w);
}

// ---- units of slots ----------------------------------------------------------------------------------------------
// An access is 8 slots (1 KiB of 8-bit codes), and a unit, one wave, is ACC accesses.
//   V: consecutive slots.
//   K: a lane has to keep its channels, that is the head of its slot, from access to access.  Up to 8 heads, and in small launches: with H
//     heads a row the heads of consecutive accesses repeat after P = H / gcd(H, 8) of them, so that a unit takes every P-th access of its
//     token-group: unit u is accesses r + P (ACC j + i), i = 0 .. ACC - 1, with r = u mod P, j = u / P.  The 16 H / ACC units of a token-group
//     are waves of one block, or of a few, each of which prepares the parameters of all heads.  No lane is idle.
//     SETS, longer rows: a set is 2^log_s heads x a token-group and 2^log_s units; an access is 8 >> log_s rows of the set.  Sets of 8 heads
//     take in what lies beyond the row, as idle lanes, and are one block of 8 waves or two of 4, each of which prepares all of the set's parameters.
// What bounds it.  Small launches (ACC = 4 and 8): the chain of trips to memory, so that everything a unit reads is requested before
// anything of it is used (8 -> 4 bits bf16: 3 x 309 tokens of 8 heads 11.8 -> 5.8 us; an empty launch is 3.9).  Large ones
// (ACC = 16): memory, and beside it 6 to 7 operations an element, 0.6 of what the vector units do in the time memory takes, so that one
// has to run under the other.  8-bit codes come through a ring of 8 accesses (or 6): 4 are used while 4 are on their way, and those that follow
// are requested before the next stores are issued (a wait for a load is a wait for every store before it as well).  No register is spilled on the way of
// a row but one access of 8 -> 2 bits in fp16 (8 registers; all pairs of fp16 share the kernel and its 20 bytes of scratch a lane), and blocks are 3 or 4 waves where that is to be had: a block takes the place of one that has ended,
// and its start is hidden by the others of the compute unit, four and not one.  Before, a wave took 4 accesses, waited for its stores, and took the
// next 4, in blocks of 8 waves over 8 heads (or single heads, pairs and fours), with lanes idle for 3, 5, 6, 7, 11 and from 13 heads on.
//   32 layers x 8,192 tokens in 256-token items, 8 heads bf16, 8 -> 4 / 8 -> 2 / 4 -> 2 bits: 153.7 / 140.8 / 88.5 -> 142 / 130.7 / 77.5 us (5.9 TB/s; without
//   any arithmetic the same traffic takes 136 us at 8 -> 4 bits); 16 heads, 60 x 6,250: 510 / 474 / 291 -> 451 / 398 / 247; 5 heads, 7 x 20,000:
//   75.2 / 73.1 / 43.6 -> 56.0 / 56.7 / 33.3; 10 heads, 20 x 8,000: 129 / 118 / 74 -> 119 / 106 / 67; 4 heads, 20 x 9,000: 58.2 / 54.6 / 35.5 -> 51.9 / 48.3 / 31.3.
constexpr unsigned kUnitsHeadBytes = kGroup * 6 * sizeof(float);  // LDS for the parameters of a head: three values of a channel, and the 8 -> 2 polynomial
template <int DT, int BI, int BO, int ACC, bool SETS>
__device__ __forceinline__ void transcode_units(const TranscodeParams& a, const kvh_tc_item& it, int item_idx, int lay_kv,
                                                uint32_t bx, uint8_t* lds, uint32_t* kflags) {
  // Accesses whose codes a wave holds, and how many are requested again at a time as they are used up.
  // From 8 to 2 bits bf16 groups mostly need the fitted polynomial, whose coefficients leave registers for 6 (8 spilled one: 32 x 8,192 x 1024 135.7 -> 130.7 us);
  // fp16 groups are standard ones and run best with 8 (115.6 us, 120.6 with 6).
  constexpr bool kTight = DT == KVH_BF16 && BO == 2;
  constexpr int kRing = BI == 8 && ACC > kTcBatch ? (kTight ? 6 : kTcBatch) : ACC, kRefill = kRing < ACC ? (kTight ? 2 : kRing / 2) : ACC;
  // The search for the steps of an 8 -> 2 bit group needs registers of its own: half of the ring is requested behind it.
  constexpr int kEarly = BI == 8 && BO == 2 && kRing < ACC ? kRing / 2 : kRing;
  constexpr int kVBatch = ACC < kTcBatch ? ACC : kTcBatch;  // accesses whose V groups the lanes prepare at a time, one each
  static_assert(ACC % kRefill == 0 && ACC % kVBatch == 0 && kVBatch % kRefill == 0 || kRing == ACC, "whole batches");
  constexpr uint32_t kInBytes = kGroup * BI / 8, kOutBytes = kGroup * BO / 8;  // of a slot
  const int lane = threadIdx.x & (kWave - 1);
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t sub = lane % kSlotLanes, slot = lane / kSlotLanes;
  const uint32_t n = (uint32_t)it.n_tokens, heads = (uint32_t)a.c / kGroup;
  const int lam = lay_kv >> 1;
  const bool is_v = lay_kv & 1;
  const uint64_t total = (uint64_t)n * heads;

  // The unit: its first slot, the slots from one access to the next, how many slots it has at most, and where in an access the
  // lane's slot lies.
  uint32_t g0 = 0, gi = 0, block_unit = 0;  // K in accesses: first token-group of the block, this wave's among them, first unit of the block
  uint32_t par_head = 0;                    // K: which of the heads that the block prepares is the lane's
  uint64_t s0;
  uint32_t step = kTcSpanHeads, lane_slot = slot;
  bool live = true, active = true;
  const uint32_t half = (uint32_t)a.k_log_s == 3u && a.waves == 4 ? 1u : 0u;  // SETS: a set is two blocks
  auto set_of = [&](uint32_t i, uint32_t& g, uint32_t& head0) {  // the i-th set of the block
    const uint32_t set = half ? bx >> 1 : bx * ((uint32_t)a.waves >> a.k_log_s) + i;
    g = a.by_sets.quotient(set);
    head0 = (set - g * a.by_sets.d) << a.k_log_s;
  };
  if (is_v) {
    s0 = ((uint64_t)bx * (uint32_t)a.waves + wave) * (uint32_t)(ACC * kTcSpanHeads);
  } else if (SETS) {
    uint32_t g, head0;
    set_of(0, g, head0);
    if ((uint64_t)g * kGroup >= n) return;  // block-uniform
    const uint32_t log_s = (uint32_t)a.k_log_s, mask = (1u << log_s) - 1;
    set_of(wave >> log_s, g, head0);
    block_unit = (bx & half) * 4u;
    if ((uint64_t)g * kGroup + (block_unit << 4) >= n && half) return;  // block-uniform: the token-group ends in the first half
    s0 = ((uint64_t)g * kGroup + (((wave & mask) + block_unit) << (7 - log_s))) * heads + head0;
    step = heads << (3 - log_s);
    lane_slot = (slot >> log_s) * heads + (slot & mask);
    active = head0 + (slot & mask) < heads;
    par_head = (wave & ~mask) + (slot & mask);
  } else {
    const uint32_t q = a.by_parts.quotient(bx);
    g0 = q * (uint32_t)a.groups;
    if ((uint64_t)g0 * kGroup >= n) return;  // block-uniform
    gi = a.by_units.quotient(wave);
    block_unit = (bx - q * a.by_parts.d) * (uint32_t)a.waves;
    if (block_unit != 0) {  // block-uniform: the token-group is too short for this block
      const uint64_t from = (uint64_t)g0 * (kGroup * heads) + (uint64_t)a.by_period.quotient(block_unit) * (ACC * kTcSpanHeads * a.by_period.d);
      if (from >= total) return;
    }
    const uint32_t u = block_unit + wave - gi * a.by_units.d;
    live = u < a.by_units.d;
    const uint32_t j = a.by_period.quotient(u), r = u - j * a.by_period.d;
    step = kTcSpanHeads * a.by_period.d;
    s0 = (uint64_t)(g0 + gi) * (kGroup * heads) + kTcSpanHeads * r + (uint64_t)j * (ACC * step);
    const uint32_t x = kTcSpanHeads * r + slot;  // 8 P is a multiple of H
    par_head = gi * heads + x - a.by_heads.quotient(x) * heads;
  }
  uint32_t rem = 0;
  if (live && s0 < total) rem = total - s0 < ACC * step ? (uint32_t)(total - s0) : ACC * step;
  rem = (uint32_t)uniform((int32_t)rem);
  s0 = uniform(rem > 0 ? s0 : 0);
  // accesses with something to store
  const int count = (int)((is_v ? rem + kTcSpanHeads - 1 : a.by_step.quotient(rem + step - 1) * kTcSpanHeads) / kTcSpanHeads);

  const uint8_t* src = static_cast<const uint8_t*>(it.src);
  uint8_t* dst = static_cast<uint8_t*>(it.dst);
  const LayerGeom gin = layer_geom(it.n_tokens, a.c, BI), gout = layer_geom(it.n_tokens, a.c, BO);
  const HeaderWords hdr = {sload<uintx4>(src), sload<uintx4>(src + 16), sload<uintx4>(src + 32)};
  const uint8_t* in_layer = src + kHeaderBytes + (size_t)lam * gin.layer_bytes();
  uint8_t* out_layer = dst + kHeaderBytes + (size_t)lam * gout.layer_bytes();
  const uint8_t* in_codes = in_layer + gin.kmeta + (is_v ? gin.codes + gin.vmeta : 0) + s0 * kInBytes;  // wave-uniform
  uint8_t* out_codes = out_layer + gout.kmeta + (is_v ? gout.codes + gout.vmeta : 0) + s0 * kOutBytes;
  const uint32_t in_sub = sub * (kTcLaneCh * BI / 8), in_lane = lane_slot * kInBytes + in_sub;
  const uint32_t out_lane = lane_slot * kOutBytes + sub * (kTcLaneCh * BO / 8);

  InCodes<BI> cw[kRing];
  // The caller guarantees kvh_blob_size(l, n_tokens, c, level_in) readable bytes at the source, so the loads issued before the header verdict stay inside the
  // buffer whatever it says.  Accesses past the last re-read it; lanes whose slot lies past the end read the access's first slot.  Neither is stored.
  // lane_count: accesses in which the lane's slot is stored.
  const uint32_t lane_rem = active && rem > lane_slot ? rem - lane_slot : 0u;
  const int lane_count = (int)(is_v ? (lane_rem + kTcSpanHeads - 1) / kTcSpanHeads : lane_rem == 0 ? 0u : a.by_step.quotient(lane_rem + step - 1));
  auto stores = [&](int k) { return k < lane_count; };
  auto out_row = [&](int k) { return uniform(out_codes + (size_t)((uint32_t)k * step) * kOutBytes) + out_lane; };
  auto load_one = [&](InCodes<BI>& in, int i) {
    const int k = i < count ? i : count - 1;
    in.load(uniform(in_codes + (size_t)((uint32_t)k * step) * kInBytes) + (stores(k) ? in_lane : in_sub));
  };
  auto load = [&](int i) { load_one(cw[i % kRing], i); };
  // Accesses first .. first + number - 1, in whole batches of the ring: one(i, codes) for each, and what a batch leaves free is
  // requested again before the next batch is waited for.
  auto each = [&](auto first_tag, auto number_tag, auto&& one) {
    constexpr int kFirst = decltype(first_tag)::value, kNumber = decltype(number_tag)::value;
#pragma unroll
    for (int i = kFirst; i < kFirst + kNumber; ++i) {
      one(i, cw[i % kRing]);
      __builtin_amdgcn_sched_barrier(0);
      if ((i + 1) % kRefill == 0) {
#pragma unroll
        for (int f = 0; f < kRefill; ++f)
          if (i + 1 - kRefill + kRing + f < ACC) load(i + 1 - kRefill + kRing + f);
      }
    }
  };
  auto load_rest = [&] {
#pragma unroll
    for (int i = kEarly; i < kRing; ++i) load(i);
  };
  using First = std::integral_constant<int, 0>;
  using All = std::integral_constant<int, ACC>;
  using Yes = std::integral_constant<bool, true>;
  using No = std::integral_constant<bool, false>;

  // V metadata: lane l prepares the l-th slot of a batch.  The words are requested with the codes, and by every lane (lanes without a slot read the
  // unit's first), so that the wait for them, which takes in the codes, is on every path: a wait that some path skips is repeated before each access, where
  // it also waits for the stores before (4 -> 2 bits, 32 x 8,192 x 1024 in blocks of 8 waves: 100 us instead of 88).
  const uint8_t* in_vmeta = in_layer + gin.kmeta + gin.codes + s0 * 4;
  constexpr int kWords = ACC / kVBatch;
  auto owns = [&](int b) { return (uint32_t)(b * kVBatch * kTcSpanHeads + lane) < rem && lane < kVBatch * kTcSpanHeads; };
  uint32_t vm[kWords] = {};
  if (count > 0) {
#pragma unroll
    for (int i = 0; i < kEarly; ++i) load(i);
    if (is_v) {
#pragma unroll
      for (int b = 0; b < kWords; ++b) vm[b] = gload<uint32_t>(in_vmeta + (owns(b) ? (b * kWave + lane) * 4 : 0));
    }
  }
  // K: pairs of channels, this thread's first and second (all heads of the block's token-groups are 2 pairs a thread at most)
  const uint32_t threads = (uint32_t)a.waves * kWave, pairs = SETS ? threads << half : (uint32_t)a.groups * heads * (kGroup / 2);
  uintx2 km[2] = {};
  bool pact[2] = {false, false};
  size_t pmeta[2] = {0, 0};
  if (!is_v) {
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const uint32_t pr = threadIdx.x + e * threads;
      if (pr >= pairs) break;
      uint32_t g, first;  // the pair's token-group, its first channel
      if (SETS) {
        set_of(pr >> (6 + a.k_log_s), g, first);
        first = first * kGroup + (pr & ((64u << a.k_log_s) - 1)) * 2;
      } else {
        const uint32_t pg = a.by_heads.quotient(pr / (kGroup / 2));
        g = g0 + pg;
        first = (pr - pg * heads * (kGroup / 2)) * 2;
      }
      pact[e] = (uint64_t)g * kGroup < n && first < (uint32_t)a.c;
      pmeta[e] = ((size_t)g * (uint32_t)a.c + first) * 4;
      if (pact[e]) km[e] = gload<uintx2>(in_layer + pmeta[e]);
    }
  }

  // block-uniform verdict: every thread reads the same header
  if (!source_header_ok(hdr, DT, BI, a.l, it.n_tokens, a.c, kHeaderBytes + (size_t)a.l * gin.layer_bytes())) {
    if (a.status != nullptr && threadIdx.x == 0) a.status[item_idx] = KVH_DEV_HEADER_MISMATCH;
    return;
  }
  if (bx == 0 && lay_kv == 0 && threadIdx.x < kHeaderBytes / 4) write_header<DT, BO>(dst, a, n, gout, hdr);

  if (!is_v) {
    const uint32_t cols = pairs / (kTcLaneCh / 2);  // of the parameter tables, 16 channels each
    const uint32_t par_lane = par_head * kSlotLanes + sub;
    // one plane of LDS for each of the values of a channel: channels 4 m .. 4 m + 3 of all columns, then the next four
    const uint32_t plane = cols * kTcLaneCh;
    float* kpar = reinterpret_cast<float*>(lds);      // minima, scales, inverses; or tables
    [[maybe_unused]] float* kquad = kpar + 3 * plane;  // the 8 -> 2 polynomials
    auto pair_at = [&](uint32_t pr) { return pr / 2 % 4 * (cols * 4) + pr / 8 * 4 + pr % 2 * 2; };  // channels 2 pr, 2 pr + 1
    auto lane_values = [&](const float* from, float (&out)[kTcLaneCh]) {
#pragma unroll
      for (int m = 0; m < kTcLaneCh / 4; ++m) {
        const float4 f = *reinterpret_cast<const float4*>(from + m * (cols * 4) + par_lane * 4);
        out[4 * m] = f.x; out[4 * m + 1] = f.y; out[4 * m + 2] = f.z; out[4 * m + 3] = f.w;
      }
    };
    [[maybe_unused]] uint32_t worst = kStandard;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const uint32_t pr = threadIdx.x + e * threads;
      if (pr >= pairs) break;
      const uint32_t meta[2] = {km[e].x, km[e].y};
      uint32_t om[2];
      float* at = kpar + pair_at(pr);
      if constexpr (kUseTable<BI, BO>) {
        const uint32_t t0 = code_table<DT, BI, BO>(meta[0], om[0]), t1 = code_table<DT, BI, BO>(meta[1], om[1]);
        *reinterpret_cast<uint2*>(at) = make_uint2(t0, t1);
      } else {
        const TcParams p[2] = {tc_params<DT, BI, BO>(meta[0], om[0]), tc_params<DT, BI, BO>(meta[1], om[1])};
        *reinterpret_cast<float2*>(at) = make_float2(p[0].mn, p[1].mn);
        *reinterpret_cast<float2*>(at + plane) = make_float2(p[0].scale, p[1].scale);
        *reinterpret_cast<float2*>(at + 2 * plane) = make_float2(p[0].inv, p[1].inv);
        if constexpr (BI == 8 && BO == 2) {
          Quad gq[2];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const uint32_t cls = classify82<DT>(p[h], gq[h]);
            if (pact[e] && cls > worst) worst = cls;
          }
          float* quad = kquad + pair_at(pr);
          *reinterpret_cast<float2*>(quad) = make_float2(gq[0].a, gq[1].a);
          *reinterpret_cast<float2*>(quad + plane) = make_float2(gq[0].b, gq[1].b);
          *reinterpret_cast<float2*>(quad + 2 * plane) = make_float2(gq[0].c, gq[1].c);
        }
      }
      if (pact[e] && block_unit == 0) {
        uintx2 o = {om[0], om[1]};
        gstore<uintx2>(out_layer + pmeta[e], o);
      }
    }
    if constexpr (kUseTable<BI, BO>) {
      __syncthreads();
      if (count == 0) return;  // wave-uniform, after the barrier
      float tab[kTcLaneCh];
      lane_values(kpar, tab);
      each(First{}, All{}, [&](int i, const InCodes<BI>& in) {
        if (stores(i)) lookup_row<BI, BO>(out_row(i), in, [&tab](int j) { return __builtin_bit_cast(uint32_t, tab[j]); });
      });
      return;
    }
    if constexpr (BI == 8 && BO == 2) {  // block-wide verdicts through the barrier: every wave leaves its own in LDS
      const uint32_t mine = (__builtin_amdgcn_ballot_w64(worst != kStandard) != 0 ? 1u : 0u) |
                            (__builtin_amdgcn_ballot_w64(worst == kHard) != 0 ? 2u : 0u);
      if (lane == 0) kflags[wave] = mine;
    }
    __syncthreads();
    if (count == 0) return;  // wave-uniform, after the barrier
    load_rest();
    if constexpr (BI == 8 && BO == 2) {
      uint32_t all = 0;
      for (int w = 0; w < a.waves; ++w) all |= kflags[w];
      all = (uint32_t)__builtin_amdgcn_readfirstlane((int)all);
      if ((all & 2u) == 0) {  // no hard group in the block: the polynomial route
        auto poly_rows = [&](auto standard_tag) {
          constexpr bool STANDARD = decltype(standard_tag)::value;
          float ga[kTcLaneCh] = {}, gb[kTcLaneCh] = {}, gc[kTcLaneCh] = {};
          if constexpr (!STANDARD) {
            lane_values(kquad, ga);
            lane_values(kquad + plane, gb);
            lane_values(kquad + 2 * plane, gc);
          }
          each(First{}, All{}, [&](int i, const InCodes<BI>& in) {
            if (stores(i)) poly_row82<STANDARD>(out_row(i), in, [&](int j) { return Quad{ga[j], gb[j], gc[j]}; });
          });
        };
        if (all == 0) poly_rows(Yes{}); else poly_rows(No{});
        return;
      }
    }
    float mn[kTcLaneCh], scale[kTcLaneCh], inv[kTcLaneCh];
    lane_values(kpar, mn);
    lane_values(kpar + plane, scale);
    lane_values(kpar + 2 * plane, inv);
    each(First{}, All{}, [&](int i, const InCodes<BI>& in) {
      if (stores(i)) transcode_row<DT, BI, BO>(out_row(i), in, [&](int j) { return TcParams{mn[j], scale[j], inv[j], 0.0f}; });
    });
    return;
  }

  if (count == 0) return;  // wave-uniform; V waves never meet at a barrier
  uint8_t* out_vmeta = out_layer + gout.kmeta + gout.codes + s0 * 4;
  // zero the padding that rounds the vmeta section up to 16 bytes: the unit that holds the section's last slot
  if (s0 + rem == total && lane == 0) {
    for (size_t o = (size_t)total * 4; o < gout.vmeta; o += 4) gstore<uint32_t>(out_vmeta - s0 * 4 + o, 0u);
  }
  using Batch = std::integral_constant<int, kVBatch>;
  auto some = [&](auto b_tag) {  // kVBatch accesses: lane l prepares their l-th slot
    constexpr int b = decltype(b_tag)::value;
    using Start = std::integral_constant<int, b * kVBatch>;
    if (b * kVBatch >= count) return;  // wave-uniform
    const bool own = owns(b);
    auto owner = [&](int i) { return (i - b * kVBatch) * kTcSpanHeads + (int)slot; };
    uint32_t om;
    auto store_word = [&] {
      if (own) gstore<uint32_t>(out_vmeta + (b * kWave + lane) * 4, om);
    };
    if constexpr (kUseTable<BI, BO>) {
      const uint32_t mine = code_table<DT, BI, BO>(vm[b], om);
      store_word();
      each(Start{}, Batch{}, [&](int i, const InCodes<BI>& in) {
        if (i >= count) return;  // wave-uniform; the shuffle is taken with the whole wave enabled
        const uint32_t tab = __shfl(mine, owner(i));
        if (stores(i)) lookup_row<BI, BO>(out_row(i), in, [tab](int) { return tab; });
      });
    } else {
      const TcParams mine = tc_params<DT, BI, BO>(vm[b], om);
      store_word();
      if constexpr (BI == 8 && BO == 2) {
        Quad gq;
        uint32_t cls = classify82<DT>(mine, gq);
        if (!own) cls = kStandard;  // a lane without a group has no say
        if constexpr (b == 0) load_rest();
        if (__builtin_amdgcn_ballot_w64(cls == kHard) == 0) {
          const bool all_standard = __builtin_amdgcn_ballot_w64(cls != kStandard) == 0;
          each(Start{}, Batch{}, [&](int i, const InCodes<BI>& in) {
            if (i >= count) return;  // wave-uniform; the shuffles are taken with the whole wave enabled
            if (all_standard) {
              if (stores(i)) poly_row82<true>(out_row(i), in, [&gq](int) -> const Quad& { return gq; });
            } else {
              const Quad gr = {__shfl(gq.a, owner(i)), __shfl(gq.b, owner(i)), __shfl(gq.c, owner(i))};
              if (stores(i)) poly_row82<false>(out_row(i), in, [&gr](int) -> const Quad& { return gr; });
            }
          });
          return;
        }
      }
      each(Start{}, Batch{}, [&](int i, const InCodes<BI>& in) {
        if (i >= count) return;  // wave-uniform; the shuffles are taken with the whole wave enabled
        const TcParams p = {__shfl(mine.mn, owner(i)), __shfl(mine.scale, owner(i)), __shfl(mine.inv, owner(i)), 0.0f};
        if (stores(i)) transcode_row<DT, BI, BO>(out_row(i), in, [&p](int) -> const TcParams& { return p; });
      });
    }
  };
  some(First{});
  if constexpr (kWords > 1) some(std::integral_constant<int, 1>{});
  static_assert(kWords <= 2, "batches of a unit");
}

// The job of this block's item, for transcode_units_kernel; its level pair as bits in * 16 + bits out, or -1: nothing to do.
__device__ __forceinline__ int load_job(const TranscodeParams& a, kvh_tc_item& it) {
  if (a.items != nullptr) {
    const uint8_t* p = reinterpret_cast<const uint8_t*>(a.items + blockIdx.z);
    uintx4 lo = gload<uintx4>(p), hi = gload<uintx4>(p + 16);
    it.src = reinterpret_cast<const void*>((uint64_t)lo.x | (uint64_t)lo.y << 32);
    it.dst = reinterpret_cast<void*>((uint64_t)lo.z | (uint64_t)lo.w << 32);
    it.n_tokens = (int32_t)hi.x;
    it.level_in = (int32_t)hi.y;
    it.level_out = (int32_t)hi.z;
    it.reserved = 0;
  } else {
    it = a.one;
  }
  it.src = uniform(it.src);
  it.dst = uniform(it.dst);
  it.n_tokens = uniform(it.n_tokens);
  it.level_in = uniform(it.level_in);
  it.level_out = uniform(it.level_out);
  if (it.n_tokens < 1) return -1;
  const int bi = level_bits(it.level_in), bo = level_bits(it.level_out);
  // refused: a level out of range, the raw level (no codes to transcode), more tokens than the grid covers
  if (bi < 0 || bo < 0 || bi > 8 || bo > 8 || it.n_tokens > a.max_tokens) {
    if (a.status != nullptr && threadIdx.x == 0) a.status[blockIdx.z] = KVH_DEV_HEADER_MISMATCH;
    return -1;
  }
  return bi * 16 + bo;
}

}  // namespace

// grid = (blocks of a plane, 2 * l, items); a block is `waves` units
template <int DT, int ACC, bool SETS>
__global__ __launch_bounds__(kTcThreads) KVH_TC_OCC void transcode_units_kernel(TranscodeParams a) {
  extern __shared__ __align__(16) uint8_t units_lds[];  // K parameters, then the 8 -> 2 polynomials; kUnitsHeadBytes a head
  __shared__ uint32_t kflags[kTcWaves];
  kvh_tc_item it;
  const int pair = load_job(a, it);
  if (pair < 0) return;  // block-uniform
#define KVH_TC_CASE(BI, BO) \
  case BI * 16 + BO: transcode_units<DT, BI, BO, ACC, SETS>(a, it, blockIdx.z, blockIdx.y, blockIdx.x, units_lds, kflags); break;
  switch (pair) {
    KVH_TC_CASE(8, 8) KVH_TC_CASE(8, 4) KVH_TC_CASE(8, 2)
    KVH_TC_CASE(4, 8) KVH_TC_CASE(4, 4) KVH_TC_CASE(4, 2)
    KVH_TC_CASE(2, 8) KVH_TC_CASE(2, 4) KVH_TC_CASE(2, 2)
    default: break;
  }
#undef KVH_TC_CASE
}

int launch_transcode(const TranscodeParams& a, int dt, int n_items, int max_tokens, hipStream_t stream) {
  const int heads = a.c / kGroup;
  const TcStream plan = transcode_stream_plan(heads, a.l, n_items, max_tokens);
  const TcUnits units = transcode_units_plan(heads, a.l, n_items, max_tokens);
  const bool small = units.accesses != 0, sets = !small && plan.log_s >= 0;
  const TcUnits u = small ? units : plan.in;
  if (!grid_fits(u.blocks, 1, u.waves)) return KVH_E_HIP;
  TranscodeParams b = a;
  b.max_tokens = max_tokens;
  b.waves = u.waves;
  b.groups = u.groups;
  b.k_log_s = plan.log_s;
  b.by_heads = Divisor((uint32_t)heads);
  b.by_sets = Divisor((uint32_t)(sets ? (heads + (1 << plan.log_s) - 1) >> plan.log_s : 1));
  b.by_units = Divisor((uint32_t)u.units);
  b.by_parts = Divisor((uint32_t)u.parts);
  b.by_period = Divisor((uint32_t)u.period);
  b.by_step = Divisor((uint32_t)(sets ? heads << (3 - plan.log_s) : kTcSpanHeads * u.period));
  const unsigned lds = (unsigned)(sets ? std::max(u.waves, 1 << plan.log_s) : u.groups * heads) * kUnitsHeadBytes;
  const dim3 grid((unsigned)u.blocks, (unsigned)(2 * a.l), (unsigned)n_items);
  auto pick = [&](auto dt_tag) {
    constexpr int D = decltype(dt_tag)::value;
    return sets ? transcode_units_kernel<D, 16, true> : u.accesses == 4 ? transcode_units_kernel<D, 4, false>
                : u.accesses == 8 ? transcode_units_kernel<D, 8, false> : transcode_units_kernel<D, 16, false>;
  };
  auto kernel = dt == KVH_F16 ? pick(std::integral_constant<int, KVH_F16>{}) : pick(std::integral_constant<int, KVH_BF16>{});
  launch_kernel(kernel, grid, dim3((unsigned)(u.waves * kWave)), lds, stream, b);
  KVH_HIP_CHECK_LAUNCH();
  return KVH_OK;
}

}  // namespace kvh
