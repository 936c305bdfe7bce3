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
// Block = 8 waves x 16 token rows = one K token-group x a 1024-channel span; a lane owns 16
// consecutive channels, so a wave moves one whole code row of the span per access (16 / 8 / 4
// bytes per lane at 8 / 4 / 2 bits).  K parameters (per channel) are prepared once per block,
// two channels per thread, and shared through LDS; V parameters (per token and head) are
// prepared by one lane per group and broadcast inside the wave.  When the whole code -> code map
// of a group fits one register (4 -> 2 and the pairs that start from 2 bits) the "parameters"
// are that map, built by running the arithmetic once per input code, and an element costs a
// shift and a funnel shift.
//
// Rows that are not a multiple of 1024 channels leave lanes of the last span idle, 56 of 64 with 128 channels.  Where that
// costs more than it saves (transcode_plan has the rule and its figures) an access covers 8 (row, head) slots of 8 lanes
// each instead (SLOTS), 128 slots per wave: V slots are consecutive in memory; K slots are sets of 1, 2 or 4 heads x a
// token-group, several sets to a block, so that a lane keeps its channels.  32 layers, 8 -> 4 bits, 2,048 tokens x 128
// channels: 30.3 -> 13.2 us, 8,192 x 256: 115 -> 41 us; 4 -> 2 bits, 12,000 x 128: 101 -> 21 us, 8,192 x 1280: 157 -> 116 us.
//
// Small launches, where either layout makes few blocks, run in finer units of slots: see transcode_units.
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

constexpr int kTcWaves = 8;
constexpr int kTcThreads = kTcWaves * kWave;      // 512
constexpr int kTcLaneCh = 16;                     // channels per lane
constexpr int kTcSpanCh = kWave * kTcLaneCh;      // 1024 channels per wave access
constexpr int kTcRows = kGroup / kTcWaves;        // 16 accesses per wave
constexpr int kTcBatch = 8;                       // accesses in flight per wave
constexpr int kTcSpanHeads = kTcSpanCh / kGroup;  // 8 (row, head) slots per access
constexpr int kTcSlots = kTcRows * kTcSpanHeads;  // 128 slots per wave
constexpr int kSlotLanes = kGroup / kTcLaneCh;    // 8 lanes per slot
static_assert(kTcBatch * kTcSpanHeads == kWave, "one lane per V group of a batch");
static_assert(kTcThreads * 2 == kTcSpanCh, "two K channels per thread");

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
  float top;    // what code L_in decodes to: f32(mx), or f32(mn) (degenerate)
};

// Parameters of a group from its metadata word; also the word the re-encoded group stores and
// whether code L_in needs the explicit "decode to the stored maximum" rule.
template <int DT, int BI, int BO>
__device__ __forceinline__ TcParams tc_params(uint32_t meta, uint32_t& out_meta, bool& fix) {
  constexpr float LI = float((1 << BI) - 1), LO = float((1 << BO) - 1);
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
  fix = (pack2<DT>(recon(LI, p.scale, p.mn), 0.0f) & 0xffffu) != top_bits;
  return p;
}

// One row of a lane: 16 codes in, 16 codes out.  param(j) gives the parameters of channel j.
template <int DT, int BI, int BO, bool FIX, typename P>
__device__ __forceinline__ void transcode_row(uint8_t* out, const InCodes<BI>& cw, P&& param) {
  constexpr float LI = float((1 << BI) - 1);
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
    if constexpr (FIX) {
      x0 = q0 == LI ? p0.top : x0;
      x1 = q1 == LI ? p1.top : x1;
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

template <int DT, int BI, int BO>
__device__ __forceinline__ uint32_t code_table(uint32_t meta, uint32_t& out_meta) {
  constexpr int NQ = 1 << BI;
  bool fix;
  const TcParams p = tc_params<DT, BI, BO>(meta, out_meta, fix);
  uint32_t table = 0;
#pragma unroll
  for (int q = 0; q < NQ; q += 2) {
    const uint32_t pk = pack2<DT>(recon((float)q, p.scale, p.mn), recon((float)(q + 1), p.scale, p.mn));
    const float x0 = t16_to_f32<DT>(pk & 0xffffu);
    const float x1 = q + 1 == NQ - 1 ? p.top : t16_to_f32<DT>(pk >> 16);  // the top code decodes to the stored maximum
    const uint32_t two = __builtin_amdgcn_cvt_pk_u8_f32((x1 - p.mn) * p.inv, 1,
                                                        __builtin_amdgcn_cvt_pk_u8_f32((x0 - p.mn) * p.inv, 0, 0u));
    table |= ((two & 0xffu) | ((two >> 8) & 0xffu) << BO) << (BO * q);
  }
  return table;
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

// SLOTS: the lanes are cut into (row, head) slots (see the head of the file); otherwise a span's lanes keep its channels
// and those beyond the row idle.
template <int DT, int BI, int BO, bool SLOTS>
__device__ __forceinline__ void transcode_block(const TranscodeParams& a, const kvh_tc_item& it, int item_idx, int lay_kv,
                                                int bx, TcParams* kpar, float* kquad, uint32_t* kflags) {
  using Yes = std::integral_constant<bool, true>;
  using No = std::integral_constant<bool, false>;
  const int lane = threadIdx.x & (kWave - 1);
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t sub = lane % kSlotLanes, slot = lane / kSlotLanes;
  const uint32_t n = (uint32_t)it.n_tokens, c = (uint32_t)a.c, heads = c / kGroup;
  const int lam = lay_kv >> 1;
  const bool is_v = lay_kv & 1;

  // K: a set is 2^log_s heads (a span's 8 without SLOTS) x one token-group, shared by as many waves; a block holds
  // 8 >> log_s sets
  const uint32_t log_s = SLOTS ? (uint32_t)a.k_log_s : 3u;
  const uint32_t sets = SLOTS ? heads >> log_s : (heads + 7) >> 3;  // per token-group
  const uint32_t first_set = (uint32_t)bx * (8u >> log_s);
  const uint32_t first_g = a.by_sets.quotient(first_set);
  if ((!SLOTS || !is_v) && (uint64_t)first_g * kGroup >= n) return;  // block-uniform
  auto set_of = [&](uint32_t s, uint32_t& g, uint32_t& head0) {  // the s-th set of the block
    g = SLOTS ? a.by_sets.quotient(first_set + s) : first_g;
    head0 = (first_set + s - g * sets) << log_s;
  };
  // V: the wave's slots start at row t0, head y0.  In spans they are 16 rows x 8 heads, with SLOTS 128 in memory order;
  // access i is `v_step` slots of the section on.
  uint32_t t0 = 0, y0 = 0, left = 0;
  uint64_t left64 = 0;  // SLOTS: slots from the wave's first to the end of the section
  const uint32_t v_step = SLOTS ? (uint32_t)kTcSpanHeads : heads;
  if (is_v) {
    if constexpr (SLOTS) {
      const uint32_t unit = (uint32_t)bx * kTcWaves + wave;
      const uint32_t q = a.by_heads.quotient(unit), x = (unit - q * heads) * kTcSlots, xq = a.by_heads.quotient(x);
      t0 = q * kTcSlots + xq;
      y0 = x - xq * heads;
      if (t0 < n) left64 = (uint64_t)(n - t0) * heads - y0;
      left = left64 < kTcSlots ? (uint32_t)left64 : (uint32_t)kTcSlots;
    } else {
      t0 = first_g * kGroup + wave * kTcRows;
      y0 = (first_set - first_g * sets) << 3;
      left = t0 >= n ? 0 : n - t0 < kTcRows ? (n - t0) * kTcSpanHeads : (uint32_t)kTcSlots;
    }
  }

  const uint8_t* src = static_cast<const uint8_t*>(it.src);
  uint8_t* dst = static_cast<uint8_t*>(it.dst);
  const LayerGeom gi = layer_geom(it.n_tokens, a.c, BI), go = layer_geom(it.n_tokens, a.c, BO);
  const HeaderWords hdr = {gload<uintx4>(src), gload<uintx4>(src + 16), gload<uintx4>(src + 32)};
  const uint8_t* in_layer = src + kHeaderBytes + (size_t)lam * gi.layer_bytes();
  uint8_t* out_layer = dst + kHeaderBytes + (size_t)lam * go.layer_bytes();

  // A lane's codes: access i is i strides on; accesses beyond `last` (-1: none) re-read it and are not stored.  `count`
  // (wave-uniform) accesses have something to store.
  const uint8_t* in_codes;
  uint8_t* out_codes;
  const size_t in_stride_k = gi.row_bytes << (3 - log_s), out_stride_k = go.row_bytes << (3 - log_s);
  const size_t in_stride_v = (size_t)v_step * (kGroup * BI / 8), out_stride_v = (size_t)v_step * (kGroup * BO / 8);
  int last, count;
  bool active = true;  // without SLOTS: the lane's channels exist
  uint32_t par_lane = 0;  // K: where the parameters of this lane's channels lie in LDS
  if (!is_v) {
    const uint32_t sib = wave >> log_s;
    uint32_t g, head0;
    set_of(sib, g, head0);
    const uint32_t t_wave = g * kGroup + (wave & ((1u << log_s) - 1)) * (kGroup >> log_s);
    const uint32_t t = t_wave + (slot >> log_s), t_in = t < n ? t : n - 1;
    const uint32_t head = head0 + (slot & ((1u << log_s) - 1));
    if (!SLOTS) active = head < heads;
    const uint32_t ch = (active ? head : 0u) * kGroup + sub * kTcLaneCh;
    in_codes = in_layer + gi.kmeta + (size_t)t_in * gi.row_bytes + ch * BI / 8;
    out_codes = out_layer + go.kmeta + (size_t)t_in * go.row_bytes + ch * BO / 8;
    last = t < n ? (int)((n - 1 - t) >> (3 - log_s)) : -1;
    count = t_wave < n ? (int)((n - 1 - t_wave) >> (3 - log_s)) + 1 : 0;
    par_lane = (sib << (3 + log_s)) + ((uint32_t)lane & ((8u << log_s) - 1));
  } else {
    if (!SLOTS) active = y0 + slot < heads;
    const size_t first = left == 0 ? 0 : (size_t)t0 * heads + y0 + (!SLOTS ? (active ? slot : 0) : slot < left ? slot : left - 1);
    in_codes = in_layer + gi.kmeta + gi.codes + gi.vmeta + first * (kGroup * BI / 8) + sub * (kTcLaneCh * BI / 8);
    out_codes = out_layer + go.kmeta + go.codes + go.vmeta + first * (kGroup * BO / 8) + sub * (kTcLaneCh * BO / 8);
    count = (int)((left + kTcSpanHeads - 1) / kTcSpanHeads);
    last = !SLOTS ? count - 1 : slot < left ? (int)((left - 1 - slot) / kTcSpanHeads) : -1;
  }

  // Accesses in flight per wave.  Narrow codes (2 registers an access or less) are loaded for all 16 accesses of
  // the wave at once: one round trip to memory instead of two, and twice the bytes in flight.  With
  // 8-bit input an access takes 4 registers; a K wave also holds the parameters of its 16 channels
  // (48 registers), so it takes 4 at a time and a V wave 8.
  constexpr int kRowsK = BI == 8 ? kTcBatch / 2 : kTcRows;
  constexpr int kRowsV = BI == 8 ? kTcBatch : kTcRows;
  InCodes<BI> cw[kRowsV];
  auto stores = [&](int k) { return SLOTS ? k <= last : k < count && active; };
  auto load_batch = [&](int a0, auto rows_tag, size_t in_stride) {
#pragma unroll
    for (int i = 0; i < decltype(rows_tag)::value; ++i) {
      int k = a0 + i;
      k = k <= last ? k : last < 0 ? 0 : last;
      cw[i].load(in_codes + (size_t)(uint32_t)k * in_stride);
    }
  };
  // accesses a0 .. a0 + rows - 1, held in cw[first ..]
  auto run_batch = [&](int a0, auto first_tag, auto rows_tag, auto fix_tag, size_t out_stride, auto&& param_of) {
    constexpr bool FIX = decltype(fix_tag)::value;
    constexpr int kFirst = decltype(first_tag)::value;
#pragma unroll
    for (int i = 0; i < decltype(rows_tag)::value; ++i) {
      if (a0 + i < count) {  // wave-uniform
        auto param = param_of(i);  // may shuffle across lanes: taken with the whole wave enabled
        if (stores(a0 + i)) transcode_row<DT, BI, BO, FIX>(out_codes + (size_t)(uint32_t)(a0 + i) * out_stride, cw[kFirst + i], param);
      }
      __builtin_amdgcn_sched_barrier(0);  // one access at a time: keeps the temporaries of different ones apart
    }
  };
  using Zero = std::integral_constant<int, 0>;
  using Eight = std::integral_constant<int, kTcBatch>;
  using Batch = std::integral_constant<int, kTcBatch>;
  using RowsK = std::integral_constant<int, kRowsK>;
  using RowsV = std::integral_constant<int, kRowsV>;

  // The caller guarantees kvh_blob_size(l, n_tokens, c, level_in) readable bytes at the source,
  // so the loads issued before the header verdict stay inside the buffer whatever it says.
  // V metadata: lane l prepares the l-th of the 64 slots of a batch of 8 accesses.  On the table routes the words are
  // requested with the codes, and by every lane (lanes without a slot read the wave's first), so that the wait for
  // them, which takes in the codes, is on every path: a wait that some path skips is repeated before each access, where
  // it also waits for the stores before (4 -> 2: 100 instead of 88 us on 32 x 8192 x 1024).
  const uint32_t m_lane = ((uint32_t)lane / kTcSpanHeads * v_step + lane % kTcSpanHeads) * 4, m_batch = v_step * (kTcBatch * 4);
  const size_t vfirst = ((size_t)t0 * heads + y0) * 4;  // metadata word of the wave's first slot
  const uint8_t* in_vmeta = in_layer + gi.kmeta + gi.codes + vfirst;
  auto owns = [&](int batch) { return (uint32_t)(batch * kWave + lane) < left && (SLOTS || y0 + lane % kTcSpanHeads < heads); };
  [[maybe_unused]] uint32_t vm[2] = {0u, 0u};
  if (count > 0) {
    if (is_v) {
      load_batch(0, RowsV{}, in_stride_v);
      if constexpr (kUseTable<BI, BO>) {
#pragma unroll
        for (int sb = 0; sb < 2; ++sb) vm[sb] = gload<uint32_t>(in_vmeta + (owns(sb) ? (size_t)sb * m_batch + m_lane : 0));
      }
    } else {
      load_batch(0, RowsK{}, in_stride_k);
    }
  }

  // the two K channels this thread prepares
  uintx2 km = {0u, 0u};
  bool pact = false;
  size_t pmeta = 0;  // offset of their metadata words
  if (!is_v) {
    const uint32_t lc = threadIdx.x * 2;  // channel within the block's sets
    uint32_t g, head0;
    set_of(lc >> (7 + log_s), g, head0);
    const uint32_t pc = head0 * kGroup + (lc & ((128u << log_s) - 1));
    pact = (uint64_t)g * kGroup < n && (SLOTS || pc < c);
    pmeta = ((size_t)g * c + pc) * 4;
    if (pact) km = gload<uintx2>(in_layer + pmeta);
  }

  // block-uniform verdict: every thread reads the same header
  if (!source_header_ok(hdr, DT, BI, a.l, it.n_tokens, a.c, kHeaderBytes + (size_t)a.l * gi.layer_bytes())) {
    if (a.status != nullptr && threadIdx.x == 0) a.status[item_idx] = KVH_DEV_HEADER_MISMATCH;
    return;
  }
  if (bx == 0 && lay_kv == 0 && threadIdx.x < kHeaderBytes / 4) write_header<DT, BO>(dst, a, n, go, hdr);

  if (!is_v) {
    uint32_t om[2] = {0u, 0u};
    const uint32_t meta[2] = {km.x, km.y};
    if constexpr (kUseTable<BI, BO>) {
      uint32_t* ktab = reinterpret_cast<uint32_t*>(kpar);  // [slot][lane], one word per channel
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int lc = (int)threadIdx.x * 2 + e;
        ktab[(lc % kTcLaneCh) * kWave + lc / kTcLaneCh] = code_table<DT, BI, BO>(meta[e], om[e]);
      }
      if (pact) {
        uintx2 o = {om[0], om[1]};
        gstore<uintx2>(out_layer + pmeta, o);
      }
      __syncthreads();
      if (count == 0) return;  // wave-uniform, after the barrier
      uint32_t tab[kTcLaneCh];
#pragma unroll
      for (int j = 0; j < kTcLaneCh; ++j) tab[j] = ktab[j * kWave + par_lane];
#pragma unroll
      for (int i = 0; i < kRowsK; ++i) {  // kRowsK == kTcRows here: the wave's accesses are all loaded
        if (stores(i))
          lookup_row<BI, BO>(out_codes + (size_t)i * out_stride_k, cw[i], [&tab](int j) { return tab[j]; });
        __builtin_amdgcn_sched_barrier(0);
      }
      return;
    }
    bool fix = false;
    [[maybe_unused]] uint32_t worst = kStandard;  // 8 -> 2: the least tractable of this thread's channels
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      bool f;
      const TcParams p = tc_params<DT, BI, BO>(meta[e], om[e], f);
      fix |= pact && f;
      const int lc = (int)threadIdx.x * 2 + e;  // channel within the span; its user is lane lc / 16, slot lc % 16
      const int slot = (lc % kTcLaneCh) * kWave + lc / kTcLaneCh;
      kpar[slot] = p;
      if constexpr (BI == 8 && BO == 2) {
        Quad gq;
        const uint32_t cls = classify82<DT>(p, gq);
        if (pact && cls > worst) worst = cls;
        kquad[slot] = gq.a;
        kquad[kTcLaneCh * kWave + slot] = gq.b;
        kquad[2 * kTcLaneCh * kWave + slot] = gq.c;
      }
    }
    if (pact) {
      uintx2 o = {om[0], om[1]};
      gstore<uintx2>(out_layer + pmeta, o);
    }
    bool any_fix;
    if constexpr (BI == 8 && BO == 2) {
      // three block-wide verdicts through one barrier: every wave leaves its own in LDS
      const uint32_t mine = (__builtin_amdgcn_ballot_w64(fix) != 0 ? 1u : 0u) |
                            (__builtin_amdgcn_ballot_w64(worst != kStandard) != 0 ? 2u : 0u) |
                            (__builtin_amdgcn_ballot_w64(worst == kHard) != 0 ? 4u : 0u);
      if (lane == 0) kflags[wave] = mine;
      __syncthreads();
      uint32_t all = 0;
#pragma unroll
      for (int w = 0; w < kTcWaves; ++w) all |= kflags[w];
      all = (uint32_t)__builtin_amdgcn_readfirstlane((int)all);
      any_fix = (all & 1u) != 0;
      if ((all & 4u) == 0) {  // no hard group in the block: the polynomial route
        if (count == 0) return;  // wave-uniform, after the barrier
        auto poly_rows = [&](auto standard_tag) {
          constexpr bool STANDARD = decltype(standard_tag)::value;
          Quad gq[kTcLaneCh];
#pragma unroll
          for (int j = 0; j < kTcLaneCh; ++j) {
            gq[j].a = STANDARD ? 0.0f : kquad[j * kWave + par_lane];
            gq[j].b = STANDARD ? 0.0f : kquad[(kTcLaneCh + j) * kWave + par_lane];
            gq[j].c = STANDARD ? 0.0f : kquad[(2 * kTcLaneCh + j) * kWave + par_lane];
          }
#pragma unroll 1
          for (int a0 = 0;;) {
#pragma unroll
            for (int i = 0; i < kRowsK; ++i) {
              if (stores(a0 + i))
                poly_row82<STANDARD>(out_codes + (size_t)(uint32_t)(a0 + i) * out_stride_k, cw[i], [&gq](int j) -> const Quad& { return gq[j]; });
              __builtin_amdgcn_sched_barrier(0);
            }
            a0 += kRowsK;
            if (a0 >= kTcRows || a0 >= count) break;
            load_batch(a0, RowsK{}, in_stride_k);
          }
        };
        if ((all & 2u) == 0) poly_rows(Yes{}); else poly_rows(No{});
        return;
      }
    } else {
      any_fix = __syncthreads_or(fix);
    }
    if (count == 0) return;  // wave-uniform, after the barrier
    // The common path never touches `top`; reading it only where the rule is needed keeps that path's
    // register count down.
    auto k_rows = [&](auto fix_tag) {
      constexpr bool FIX = decltype(fix_tag)::value;
      TcParams p[kTcLaneCh];
#pragma unroll
      for (int j = 0; j < kTcLaneCh; ++j) {
        const TcParams& s = kpar[j * kWave + par_lane];
        p[j].mn = s.mn;
        p[j].scale = s.scale;
        p[j].inv = s.inv;
        p[j].top = FIX ? s.top : 0.0f;
      }
      auto param_of = [&](int) { return [&p](int j) -> const TcParams& { return p[j]; }; };
#pragma unroll 1
      for (int a0 = 0;;) {
        run_batch(a0, Zero{}, RowsK{}, fix_tag, out_stride_k, param_of);
        a0 += kRowsK;
        if (a0 >= kTcRows || a0 >= count) break;
        load_batch(a0, RowsK{}, in_stride_k);
      }
    };
    if (any_fix) k_rows(Yes{}); else k_rows(No{});
  } else {
    if (count == 0) return;  // wave-uniform; V waves never meet at a barrier
    uint8_t* out_vmeta = out_layer + go.kmeta + go.codes + vfirst;
    if constexpr (kUseTable<BI, BO>) {
      // the wave's 16 accesses are loaded; their groups are prepared 8 accesses (= 64 groups, one per lane) at a time
      asm volatile("" : "+v"(vm[0]), "+v"(vm[1]));  // both words, and with them all codes, have arrived from here on
      auto eight_rows = [&](auto sb_tag) {
        constexpr int sb = decltype(sb_tag)::value;
        constexpr int a0 = sb * kTcBatch;
        uint32_t om;
        const uint32_t mine = code_table<DT, BI, BO>(vm[sb], om);
        if (owns(sb)) gstore<uint32_t>(out_vmeta + (size_t)sb * m_batch + m_lane, om);
#pragma unroll
        for (int i = 0; i < kTcBatch; ++i) {
          if (a0 + i < count) {  // wave-uniform; the shuffle is taken with the whole wave enabled
            const uint32_t tab = __shfl(mine, i * kTcSpanHeads + (int)slot);
            if (stores(a0 + i))
              lookup_row<BI, BO>(out_codes + (size_t)(a0 + i) * out_stride_v, cw[a0 + i], [tab](int) { return tab; });
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      };
      eight_rows(std::integral_constant<int, 0>{});
      if (kTcBatch < count) eight_rows(std::integral_constant<int, 1>{});
    } else {
#pragma unroll 1
      for (int a0 = 0;;) {  // kRowsV accesses from a0 on are loaded
        auto eight_rows = [&](auto first_tag) {
          const int tb = a0 + decltype(first_tag)::value;
          const int batch = tb / kTcBatch;
          const bool own = owns(batch);
          TcParams mine = {0.0f, 0.0f, 0.0f, 0.0f};
          bool fix = false;
          if (own) {
            const size_t off = (size_t)(uint32_t)batch * m_batch + m_lane;
            uint32_t om;
            mine = tc_params<DT, BI, BO>(gload<uint32_t>(in_vmeta + off), om, fix);
            gstore<uint32_t>(out_vmeta + off, om);
          }
          const bool any_fix = __builtin_amdgcn_ballot_w64(fix) != 0;
          if constexpr (BI == 8 && BO == 2) {
            Quad gq;
            uint32_t cls = classify82<DT>(mine, gq);
            if (!own) cls = kStandard;  // a lane without a group has no say
            if (__builtin_amdgcn_ballot_w64(cls == kHard) == 0) {
              const bool all_standard = __builtin_amdgcn_ballot_w64(cls != kStandard) == 0;
              constexpr int kFirst = decltype(first_tag)::value;
#pragma unroll
              for (int i = 0; i < kTcBatch; ++i) {
                if (tb + i < count) {  // wave-uniform; the shuffles are taken with the whole wave enabled
                  const int owner = i * kTcSpanHeads + (int)slot;
                  uint8_t* out_row = out_codes + (size_t)(uint32_t)(tb + i) * out_stride_v;
                  if (all_standard) {
                    if (stores(tb + i)) poly_row82<true>(out_row, cw[kFirst + i], [&gq](int) -> const Quad& { return gq; });
                  } else {
                    const Quad gr = {__shfl(gq.a, owner), __shfl(gq.b, owner), __shfl(gq.c, owner)};
                    if (stores(tb + i)) poly_row82<false>(out_row, cw[kFirst + i], [&gr](int) -> const Quad& { return gr; });
                  }
                }
                __builtin_amdgcn_sched_barrier(0);
              }
              return;
            }
          }
          auto param_of = [&](int i) {
            const int owner = i * kTcSpanHeads + (int)slot;
            TcParams p;
            p.mn = __shfl(mine.mn, owner);
            p.scale = __shfl(mine.scale, owner);
            p.inv = __shfl(mine.inv, owner);
            p.top = __shfl(mine.top, owner);
            return [p](int) -> const TcParams& { return p; };
          };
          if (any_fix) run_batch(tb, first_tag, Batch{}, Yes{}, out_stride_v, param_of); else run_batch(tb, first_tag, Batch{}, No{}, out_stride_v, param_of);
        };
        eight_rows(Zero{});
        if constexpr (kRowsV > kTcBatch) {
          if (a0 + kTcBatch < count) eight_rows(Eight{});
        }
        a0 += kRowsV;
        if (a0 >= kTcRows || a0 >= count) break;
        load_batch(a0, RowsV{}, in_stride_v);
      }
    }
    // zero the padding that rounds the vmeta section up to 16 bytes
    if (SLOTS ? left64 <= kTcSlots && lane == 0 : y0 == 0 && threadIdx.x == 0 && t0 + kGroup >= n) {
      for (size_t o = (size_t)n * heads * 4; o < go.vmeta; o += 4) gstore<uint32_t>(out_vmeta - vfirst + o, 0u);
    }
  }
}

// ---- units of slots ----------------------------------------------------------------------------------------------
// Any row length with every lane at work.  The (row, head) slots of a section are consecutive in memory, 8 lanes each; an
// access is 8 consecutive slots (1 KiB of 8-bit codes), and a unit, one wave, is ACC accesses.
//   V: consecutive accesses.
//   K: a lane has to keep its channels, that is the head of its slot, from access to access.  With H heads a row the heads of
//     consecutive accesses repeat after P = H / gcd(H, 8) of them, so that a unit takes every P-th access of its token-group: unit
//     u is accesses r + P (ACC j + i), i = 0 .. ACC - 1, with r = u mod P, j = u / P.  The 16 H / ACC units of a token-group are
//     waves of one block, or of a few.
// A block prepares the parameters of all heads of its token-groups.  Everything a unit reads is requested before anything of it is
// used: what bounds a small launch is its chain of trips to memory.  8 -> 4 bits bf16: 3 x 309 tokens of 8 heads 11.8 -> 5.8 us, 11 x
// 890 14.0 -> 12.0, 10 x 2,012 of 1 head in 512-token items 8 -> 8 bits 9.6 -> 5.5; an empty launch is 3.9.
constexpr unsigned kUnitsHeadBytes = kGroup * (sizeof(TcParams) + sizeof(Quad));  // LDS for the parameters of one head
template <int DT, int BI, int BO, int ACC>
__device__ __forceinline__ void transcode_units(const TranscodeParams& a, const kvh_tc_item& it, int item_idx, int lay_kv,
                                                uint32_t bx, uint8_t* lds, uint32_t* kflags) {
  static_assert(ACC <= kTcBatch, "one lane per V group of a unit");
  constexpr uint32_t kInBytes = kGroup * BI / 8, kOutBytes = kGroup * BO / 8;  // of a slot
  const int lane = threadIdx.x & (kWave - 1);
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t sub = lane % kSlotLanes, slot = lane / kSlotLanes;
  const uint32_t n = (uint32_t)it.n_tokens, heads = (uint32_t)a.c / kGroup;
  const int lam = lay_kv >> 1;
  const bool is_v = lay_kv & 1;
  const uint64_t total = (uint64_t)n * heads;

  // the unit: its first slot, the slots from one access to the next, and how many slots it has at most
  uint32_t g0 = 0, gi = 0, block_unit = 0;  // K: first token-group of the block, this wave's among them, first unit of the block
  uint64_t s0;
  uint32_t step = kTcSpanHeads;
  bool live = true;
  if (is_v) {
    s0 = ((uint64_t)bx * (uint32_t)a.waves + wave) * (uint32_t)(ACC * kTcSpanHeads);
  } else {
    const uint32_t q = a.by_parts.quotient(bx);
    g0 = q * (uint32_t)a.groups;
    if ((uint64_t)g0 * kGroup >= n) return;  // block-uniform
    gi = a.by_units.quotient(wave);
    block_unit = (bx - q * a.by_parts.d) * (uint32_t)a.waves;
    const uint32_t u = block_unit + wave - gi * a.by_units.d;
    live = u < a.by_units.d;
    const uint32_t j = a.by_period.quotient(u);
    step = kTcSpanHeads * a.by_period.d;
    s0 = (uint64_t)(g0 + gi) * (kGroup * heads) + kTcSpanHeads * (u - j * a.by_period.d) + (uint64_t)j * (ACC * step);
  }
  uint32_t rem = 0;
  if (live && s0 < total) rem = total - s0 < ACC * step ? (uint32_t)(total - s0) : ACC * step;
  rem = (uint32_t)uniform((int32_t)rem);
  s0 = uniform(rem > 0 ? s0 : 0);
  // accesses with something to store
  const int count = is_v ? (int)((rem + kTcSpanHeads - 1) / kTcSpanHeads) : (int)a.by_period.quotient((rem + step - 1) / kTcSpanHeads);

  const uint8_t* src = static_cast<const uint8_t*>(it.src);
  uint8_t* dst = static_cast<uint8_t*>(it.dst);
  const LayerGeom gin = layer_geom(it.n_tokens, a.c, BI), gout = layer_geom(it.n_tokens, a.c, BO);
  const HeaderWords hdr = {gload<uintx4>(src), gload<uintx4>(src + 16), gload<uintx4>(src + 32)};
  const uint8_t* in_layer = src + kHeaderBytes + (size_t)lam * gin.layer_bytes();
  uint8_t* out_layer = dst + kHeaderBytes + (size_t)lam * gout.layer_bytes();
  const uint8_t* in_codes = in_layer + gin.kmeta + (is_v ? gin.codes + gin.vmeta : 0) + s0 * kInBytes;  // wave-uniform
  uint8_t* out_codes = out_layer + gout.kmeta + (is_v ? gout.codes + gout.vmeta : 0) + s0 * kOutBytes;
  const uint32_t in_sub = sub * (kTcLaneCh * BI / 8), in_lane = slot * kInBytes + in_sub;
  const uint32_t out_lane = slot * kOutBytes + sub * (kTcLaneCh * BO / 8);

  InCodes<BI> cw[ACC];
  // Accesses past the last re-read it; lanes whose slot lies past the end read the access's first slot.  Neither is stored.
  auto stores = [&](int k) { return slot + (uint32_t)k * step < rem; };
  auto out_row = [&](int k) { return uniform(out_codes + (size_t)((uint32_t)k * step) * kOutBytes) + out_lane; };
  auto rows = [&](auto fix_tag, auto&& param_of) {
    constexpr bool FIX = decltype(fix_tag)::value;
#pragma unroll
    for (int i = 0; i < ACC; ++i) {
      if (i < count) {  // wave-uniform
        auto param = param_of(i);  // may shuffle across lanes: taken with the whole wave enabled
        if (stores(i)) transcode_row<DT, BI, BO, FIX>(out_row(i), cw[i], param);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  using Yes = std::integral_constant<bool, true>;
  using No = std::integral_constant<bool, false>;

  // V metadata: lane l prepares the l-th slot of the unit.  On the table routes every lane requests a word, and the wait for it
  // is on every path (see transcode_block).
  const uint8_t* in_vmeta = in_layer + gin.kmeta + gin.codes + s0 * 4;
  const bool owns = (uint32_t)lane < rem;
  uint32_t vm = 0;
  if (count > 0) {
#pragma unroll
    for (int i = 0; i < ACC; ++i) {
      const int k = i < count ? i : count - 1;
      cw[i].load(uniform(in_codes + (size_t)((uint32_t)k * step) * kInBytes) + (stores(k) ? in_lane : in_sub));
    }
    if (is_v) vm = gload<uint32_t>(in_vmeta + (owns ? lane * 4 : 0));
  }
  // K: pairs of channels, this thread's first and second (all heads of the block's token-groups are 2 pairs a thread at most)
  const uint32_t pairs = (uint32_t)a.groups * heads * (kGroup / 2), threads = (uint32_t)a.waves * kWave;
  uintx2 km[2] = {};
  bool pact[2] = {false, false};
  size_t pmeta[2] = {0, 0};
  if (!is_v) {
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const uint32_t pr = threadIdx.x + e * threads;
      const uint32_t pg = a.by_heads.quotient(pr / (kGroup / 2));
      pact[e] = pr < pairs && (uint64_t)(g0 + pg) * kGroup < n;
      pmeta[e] = ((size_t)(g0 + pg) * (uint32_t)a.c + (pr - pg * heads * (kGroup / 2)) * 2) * 4;
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
    const uint32_t cols = (uint32_t)a.groups * heads * kSlotLanes;  // of the parameter tables: [channel mod 16][column]
    const uint32_t col = gi * heads * kSlotLanes;                    // first column of the wave's token-group
    uint32_t head0;  // of the lane's slot
    {
      const uint32_t x = kTcSpanHeads * (block_unit + wave - gi * a.by_units.d) + slot;  // 8 u + slot: u = r mod P, and 8 P is a multiple of H
      head0 = x - a.by_heads.quotient(x) * heads;
    }
    const uint32_t par_lane = col + head0 * kSlotLanes + sub;
    TcParams* kpar = reinterpret_cast<TcParams*>(lds);
    [[maybe_unused]] uint32_t* ktab = reinterpret_cast<uint32_t*>(lds);
    [[maybe_unused]] float* kquad = reinterpret_cast<float*>(lds + (size_t)cols * kTcLaneCh * sizeof(TcParams));
    bool fix = false;
    [[maybe_unused]] uint32_t worst = kStandard;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const uint32_t pr = threadIdx.x + e * threads;
      if (pr >= pairs) break;
      const uint32_t meta[2] = {km[e].x, km[e].y};
      uint32_t om[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t lc = pr * 2 + h, at = lc % kTcLaneCh * cols + lc / kTcLaneCh;
        if constexpr (kUseTable<BI, BO>) {
          ktab[at] = code_table<DT, BI, BO>(meta[h], om[h]);
        } else {
          bool f;
          const TcParams p = tc_params<DT, BI, BO>(meta[h], om[h], f);
          fix |= pact[e] && f;
          kpar[at] = p;
          if constexpr (BI == 8 && BO == 2) {
            Quad gq;
            const uint32_t cls = classify82<DT>(p, gq);
            if (pact[e] && cls > worst) worst = cls;
            kquad[at] = gq.a;
            kquad[cols * kTcLaneCh + at] = gq.b;
            kquad[2 * cols * kTcLaneCh + at] = gq.c;
          }
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
      uint32_t tab[kTcLaneCh];
#pragma unroll
      for (int j = 0; j < kTcLaneCh; ++j) tab[j] = ktab[j * cols + par_lane];
#pragma unroll
      for (int i = 0; i < ACC; ++i) {
        if (stores(i)) lookup_row<BI, BO>(out_row(i), cw[i], [&tab](int j) { return tab[j]; });
        __builtin_amdgcn_sched_barrier(0);
      }
      return;
    }
    // block-wide verdicts through one barrier: every wave leaves its own in LDS
    const uint32_t mine = (__builtin_amdgcn_ballot_w64(fix) != 0 ? 1u : 0u) |
                          (__builtin_amdgcn_ballot_w64(worst != kStandard) != 0 ? 2u : 0u) |
                          (__builtin_amdgcn_ballot_w64(worst == kHard) != 0 ? 4u : 0u);
    if (lane == 0) kflags[wave] = mine;
    __syncthreads();
    uint32_t all = 0;
    for (int w = 0; w < a.waves; ++w) all |= kflags[w];
    all = (uint32_t)__builtin_amdgcn_readfirstlane((int)all);
    if (count == 0) return;  // wave-uniform, after the barrier
    if constexpr (BI == 8 && BO == 2) {
      if ((all & 4u) == 0) {  // no hard group in the block: the polynomial route
        auto poly_rows = [&](auto standard_tag) {
          constexpr bool STANDARD = decltype(standard_tag)::value;
          Quad gq[kTcLaneCh];
#pragma unroll
          for (int j = 0; j < kTcLaneCh; ++j) {
            gq[j].a = STANDARD ? 0.0f : kquad[j * cols + par_lane];
            gq[j].b = STANDARD ? 0.0f : kquad[(kTcLaneCh + j) * cols + par_lane];
            gq[j].c = STANDARD ? 0.0f : kquad[(2 * kTcLaneCh + j) * cols + par_lane];
          }
#pragma unroll
          for (int i = 0; i < ACC; ++i) {
            if (stores(i)) poly_row82<STANDARD>(out_row(i), cw[i], [&gq](int j) -> const Quad& { return gq[j]; });
            __builtin_amdgcn_sched_barrier(0);
          }
        };
        if ((all & 2u) == 0) poly_rows(Yes{}); else poly_rows(No{});
        return;
      }
    }
    auto k_rows = [&](auto fix_tag) {
      constexpr bool FIX = decltype(fix_tag)::value;
      TcParams p[kTcLaneCh];
#pragma unroll
      for (int j = 0; j < kTcLaneCh; ++j) {
        const TcParams& s = kpar[j * cols + par_lane];
        p[j].mn = s.mn;
        p[j].scale = s.scale;
        p[j].inv = s.inv;
        p[j].top = FIX ? s.top : 0.0f;
      }
      rows(fix_tag, [&](int) { return [&p](int j) -> const TcParams& { return p[j]; }; });
    };
    if ((all & 1u) != 0) k_rows(Yes{}); else k_rows(No{});
    return;
  }

  if (count == 0) return;  // wave-uniform; V waves never meet at a barrier
  uint8_t* out_vmeta = out_layer + gout.kmeta + gout.codes + s0 * 4;
  auto finish = [&](uint32_t om) {
    if (owns) gstore<uint32_t>(out_vmeta + lane * 4, om);
    // zero the padding that rounds the vmeta section up to 16 bytes: the unit that holds the section's last slot
    if (s0 + rem == total && lane == 0) {
      for (size_t o = (size_t)total * 4; o < gout.vmeta; o += 4) gstore<uint32_t>(out_vmeta - s0 * 4 + o, 0u);
    }
  };
  uint32_t om;
  if constexpr (kUseTable<BI, BO>) {
    const uint32_t mine = code_table<DT, BI, BO>(vm, om);
    finish(om);
#pragma unroll
    for (int i = 0; i < ACC; ++i) {
      if (i < count) {  // wave-uniform; the shuffle is taken with the whole wave enabled
        const uint32_t tab = __shfl(mine, i * kTcSpanHeads + (int)slot);
        if (stores(i)) lookup_row<BI, BO>(out_row(i), cw[i], [tab](int) { return tab; });
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  } else {
    bool fix;
    const TcParams mine = tc_params<DT, BI, BO>(vm, om, fix);
    finish(om);
    const bool any_fix = __builtin_amdgcn_ballot_w64(owns && fix) != 0;
    if constexpr (BI == 8 && BO == 2) {
      Quad gq;
      uint32_t cls = classify82<DT>(mine, gq);
      if (!owns) cls = kStandard;  // a lane without a group has no say
      if (__builtin_amdgcn_ballot_w64(cls == kHard) == 0) {
        const bool all_standard = __builtin_amdgcn_ballot_w64(cls != kStandard) == 0;
#pragma unroll
        for (int i = 0; i < ACC; ++i) {
          if (i < count) {  // wave-uniform; the shuffles are taken with the whole wave enabled
            const int owner = i * kTcSpanHeads + (int)slot;
            if (all_standard) {
              if (stores(i)) poly_row82<true>(out_row(i), cw[i], [&gq](int) -> const Quad& { return gq; });
            } else {
              const Quad gr = {__shfl(gq.a, owner), __shfl(gq.b, owner), __shfl(gq.c, owner)};
              if (stores(i)) poly_row82<false>(out_row(i), cw[i], [&gr](int) -> const Quad& { return gr; });
            }
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        return;
      }
    }
    auto param_of = [&](int i) {
      const int owner = i * kTcSpanHeads + (int)slot;
      TcParams p;
      p.mn = __shfl(mine.mn, owner);
      p.scale = __shfl(mine.scale, owner);
      p.inv = __shfl(mine.inv, owner);
      p.top = __shfl(mine.top, owner);
      return [p](int) -> const TcParams& { return p; };
    };
    if (any_fix) rows(Yes{}, param_of); else rows(No{}, param_of);
  }
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

// grid = (blocks of a plane, 2 * l, items)
template <int DT, bool SLOTS>
__global__ __launch_bounds__(kTcThreads) KVH_TC_OCC void transcode_kernel(TranscodeParams a) {
  __shared__ TcParams kpar[kTcLaneCh * kWave];  // 16 KiB, [slot][lane]
  __shared__ float kquad[3 * kTcLaneCh * kWave];  // 12 KiB, [coefficient][slot][lane]: the 8 -> 2 polynomials
  __shared__ uint32_t kflags[kTcWaves];
  kvh_tc_item it;
  // The steps of load_job, written out: through it the compiler needs some 280 instructions more for the layouts below, and
  // large launches take longer (4 -> 2 bits, 1024 channels: 80 layers x 8,192 tokens 211.5 us as it stands, 214.8 through it,
  // 32 x 32,768 334.4 and 338.2; 8 -> 4 bits no difference).
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
  const int bx = blockIdx.x, lay_kv = blockIdx.y;
  if (it.n_tokens < 1) return;  // block-uniform
  const int bi = level_bits(it.level_in), bo = level_bits(it.level_out);
  // refused: a level out of range, the raw level (no codes to transcode), more tokens than the grid covers
  if (bi < 0 || bo < 0 || bi > 8 || bo > 8 || it.n_tokens > a.max_tokens) {
    if (a.status != nullptr && threadIdx.x == 0) a.status[blockIdx.z] = KVH_DEV_HEADER_MISMATCH;
    return;
  }
#define KVH_TC_CASE(BI, BO) \
  case BI * 16 + BO: transcode_block<DT, BI, BO, SLOTS>(a, it, blockIdx.z, lay_kv, bx, kpar, kquad, kflags); break;
  switch (bi * 16 + bo) {
    KVH_TC_CASE(8, 8) KVH_TC_CASE(8, 4) KVH_TC_CASE(8, 2)
    KVH_TC_CASE(4, 8) KVH_TC_CASE(4, 4) KVH_TC_CASE(4, 2)
    KVH_TC_CASE(2, 8) KVH_TC_CASE(2, 4) KVH_TC_CASE(2, 2)
    default: break;
  }
#undef KVH_TC_CASE
}

// grid = (blocks of a plane, 2 * l, items); a block is `waves` units
template <int DT, int ACC>
__global__ __launch_bounds__(kTcThreads) KVH_TC_OCC void transcode_units_kernel(TranscodeParams a) {
  extern __shared__ __align__(16) uint8_t units_lds[];  // K parameters, then the 8 -> 2 polynomials; kUnitsHeadBytes a head
  __shared__ uint32_t kflags[kTcWaves];
  kvh_tc_item it;
  const int pair = load_job(a, it);
  if (pair < 0) return;  // block-uniform
#define KVH_TC_CASE(BI, BO) \
  case BI * 16 + BO: transcode_units<DT, BI, BO, ACC>(a, it, blockIdx.z, blockIdx.y, blockIdx.x, units_lds, kflags); break;
  switch (pair) {
    KVH_TC_CASE(8, 8) KVH_TC_CASE(8, 4) KVH_TC_CASE(8, 2)
    KVH_TC_CASE(4, 8) KVH_TC_CASE(4, 4) KVH_TC_CASE(4, 2)
    KVH_TC_CASE(2, 8) KVH_TC_CASE(2, 4) KVH_TC_CASE(2, 2)
    default: break;
  }
#undef KVH_TC_CASE
}

int launch_transcode(const TranscodeParams& a, int dt, int n_items, int max_tokens, bool narrow, hipStream_t stream) {
  const int heads = a.c / kGroup;
  TranscodeParams b = a;
  b.by_heads = Divisor((uint32_t)heads);
  const TcUnits u = transcode_units_plan(heads, a.l, n_items, max_tokens, narrow);
  if (u.accesses != 0) {
    b.max_tokens = max_tokens;
    b.waves = u.waves;
    b.groups = u.groups;
    b.by_units = Divisor((uint32_t)u.units);
    b.by_parts = Divisor((uint32_t)u.parts);
    b.by_period = Divisor((uint32_t)u.period);
    auto pick = [&](auto dt_tag) {
      constexpr int D = decltype(dt_tag)::value;
      return u.accesses == 4 ? transcode_units_kernel<D, 4> : transcode_units_kernel<D, 8>;
    };
    auto kernel = dt == KVH_F16 ? pick(std::integral_constant<int, KVH_F16>{}) : pick(std::integral_constant<int, KVH_BF16>{});
    const dim3 grid((unsigned)u.blocks, (unsigned)(2 * a.l), (unsigned)n_items);
    launch_kernel(kernel, grid, dim3((unsigned)(u.waves * kWave)), (unsigned)(u.groups * heads) * kUnitsHeadBytes, stream, b);
    KVH_HIP_CHECK_LAUNCH();
    return KVH_OK;
  }
  const TcPlan plan = transcode_plan(heads, a.l, n_items, max_tokens);
  if (!grid_fits(plan.blocks, 1, kTcWaves)) return KVH_E_HIP;
  b.max_tokens = max_tokens;
  b.k_log_s = plan.log_s;
  b.by_sets = Divisor((uint32_t)plan.sets);
  const dim3 grid((unsigned)plan.blocks, (unsigned)(2 * a.l), (unsigned)n_items);
  auto kernel = dt == KVH_F16 ? (plan.slots ? transcode_kernel<KVH_F16, true> : transcode_kernel<KVH_F16, false>)
                              : (plan.slots ? transcode_kernel<KVH_BF16, true> : transcode_kernel<KVH_BF16, false>);
  launch_kernel(kernel, grid, dim3(kTcThreads), 0u, stream, b);
  KVH_HIP_CHECK_LAUNCH();
  return KVH_OK;
}

}  // namespace kvh
