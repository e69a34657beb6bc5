// zc_quantize_pack: mixed-precision quantization and bit-packing of one cache
// tensor (Eq. 5, Eq. 6, Algorithm 1; the four quantizer calls of Algorithm 2).
//
// Channel statistics of a subset must be complete before any of its tokens can
// be quantized, so the work is two launches, one where the rows fit registers or
// the subsets are so short that every workgroup takes its statistics itself (k_short_kv):
//   1. k_columns        a workgroup owns a few channels of one subset: their minima
//                       and maxima over all its tokens, the parameters that follow
//                       (Eq. 5's R = max - min, 1/R and z, or Eq. 6's c and 1/c)
//                       and, for channelwise ROW codes that stay resident, the codes.
//                       Long subsets of few channels are cut into token ranges, whose
//                       minima k_column_params joins in a launch between the two.
//   2. k_pack_kv        (the paper's schemes and layouts) a few channels and tokens a thread;
//      k_quant_pack     (the others, and wide values) a team of waves (one thread per 8 channels) owns one to
//                       four word groups of a TGROUP block - the 32 / bits tokens
//                       whose codes share 32-bit words - and walks them in
//                       batches of 8 tokens, requesting batch i + 1 before it
//                       reduces and quantizes batch i: per-token range by DPP wave
//                       reduction (+ LDS across the team's waves) for the tokenwise
//                       schemes, tie-exact x (2^k-1) / R for the zero points and the
//                       plain tokenwise and channelwise codes, round half to even, + z,
//                       clamp, pack along channels (ROW layout) or along tokens (TGROUP).
// Every sweep reads 16 bytes per lane with consecutive lanes on consecutive
// addresses of a (token, head) row; the second sweep of a tensor that fits the
// 256 MB Infinity Cache does not reach HBM.
#include <type_traits>

#include "quant_math.hpp"

namespace zc {

struct QPArgs {
  const void* x;
  int64_t sB, sH, sL;
  int B, H, D, W, NV;          // NV = W / 8 channel vectors per token row
  const int32_t* idx[2];       // [B, n] token lists (salient, regular)
  int n[2];                    // tokens per subset
  int begin[2];                // first arena slot of this chunk
  int bits[2];
  int64_t cap[2];
  uint8_t* codes[2];
  float* tok_scale[2];
  float* tok_zero[2];
  int32_t* pos[2];
  float* chan_scale;           // this chunk: [2, B, W]
  float* chan_zero;
  float* params;               // workspace [B, 2, 3, W]: CHANNEL 1/R, z, R; CST 1/c, -, -; behind it (4 B W floats a subset on)
                               // the column sweep's [B, 2, split, W] (minimum, minimum of -x) where it goes by token ranges
  int32_t* chunk_row;          // device chunk_table row to fill
  int64_t pos_offset;
  int units[2];                // quantize sweep: word groups per subset (4 per TGROUP block)
  int upw, wgs[2];             // word groups per workgroup (1, 2 or 4: divides a block), workgroups per subset
  int scheme;
  int vl;                      // column sweep: lanes across a token row (8 channels each)
  int resident;                // column sweep: the subset's rows stay in registers and are packed there
};

constexpr int kStatBatch = 8;       // token rows requested at once where they do not stay resident
constexpr int kSplitLanes = 16, kSplitThreads = 512;      // shape of the split column sweep's workgroups
constexpr int kSplitRows = 16;      // least rows a thread of it takes

__device__ inline float2* range_minima(const QPArgs& a) { return reinterpret_cast<float2*>(a.params + (int64_t)a.B * 2 * a.W * 4); }

// Parameters of (batch element, subset), value v (0..2) of channel w.
__device__ inline float* param_row(const QPArgs& a, int b, int sub, int v) { return a.params + ((int64_t)(b * 2 + sub) * 3 + v) * a.W; }
__device__ inline void store_params(const QPArgs& a, int b, int sub, int w, float3 p) {
  param_row(a, b, sub, 0)[w] = p.x;
  if (a.scheme != ZC_SCHEME_CHANNEL) return;
  param_row(a, b, sub, 1)[w] = p.y;
  param_row(a, b, sub, 2)[w] = p.z;
}

struct QPPair { QPArgs t[2]; };   // keys and values of one cache, compressed by the same launches

// The bits of x as a number of their own: this file is compiled as if there were no NaN, and a test of a float's
// bits that only a NaN passes would be taken for the one it amounts to.
__device__ inline uint32_t bits_of(float x) {
  uint32_t b = __float_as_uint(x);
  asm("" : "+v"(b));
  return b;
}

// What the quantizer needs of a channel whose values span [lo, hi]; n tokens (0: defaults).  Channelwise, one without any
// number has NaN for its parameters.
__device__ inline float3 channel_params(int scheme, int n, float qmax, float lo, float hi, float* cs, float* cz) {
  *cs = 1.f; *cz = 0.f;
  if (n > 0 && scheme == ZC_SCHEME_CST) {
    float c = sqrtf(fmaxf(fabsf(lo), fabsf(hi)));       // Eq. 6
    if (c == 0.f) c = 1.f;
    *cs = c;
    return make_float3(1.f / c, 0.f, 1.f);
  }
  if (n > 0 && scheme == ZC_SCHEME_CHANNEL) {
    float R = hi - lo + 0.f;                               // Eq. 5: s = R / (2^k - 1)  (never -0)
    // Without a number the minimum and that of -x are where they began, or NaN: the range is -inf or NaN, and all bits are set.  (No
    // branch: it would be cold code in a chain that all workgroups of a small launch wait for.)
    uint32_t none = bits_of(R) > 0x7f800000u ? ~0u : 0u;
    asm("" : "+v"(none));
    if (R == 0.f) R = qmax;                                // max == min: s := 1
    const auto or_nan = [&](float x) { return __uint_as_float(__float_as_uint(x) | none); };
    *cs = or_nan(R / qmax);
    *cz = or_nan(-rintf(refined_ratio(lo, qmax, R, 1.f / R)));
    return make_float3(or_nan(1.f / R), *cz, or_nan(R));
  }
  return make_float3(1.f, 0.f, 1.f);
}

// ---- minima of N values over a wave at once -----------------------------------------
// Every lane brings N = 8 or 16 values (value j + N / 2 paired with value j in the first
// step); afterwards lane l holds the minimum over the wave of value number value_of_lane<N>(l).  Each step halves the values a lane still
// carries: two lanes that differ in one bit of the lane number exchange the half the
// other one keeps and reduce the half they keep themselves, so the whole reduction is
// about 2 N instructions instead of 6 per value.  Lane bit 4 and 5 (rows, halves of the
// wave) go through the register-pair swaps, bit 3 and 2 through DPP with a bank mask
// (one instruction per kept half), the last one or two steps (bits 0, 1, and 2 when
// N = 8) reduce the one remaining value over all lanes of a group.  All 64 lanes must
// be active.
__device__ inline float swap_min_rows(float a, float b) {      // rows 0, 2: a over the row pair; rows 1, 3: b
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return fminf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ inline float swap_min_halves(float a, float b) {    // lanes 0-31: a over both halves; lanes 32-63: b
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return fminf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
// (the two wait states are what a DPP read of a register needs after the vector
// instruction that wrote it; the compiler does not look inside the block)
__device__ inline float dpp_min_xor8_keep(float a, float b) {  // lanes 0-7 of a row: a; lanes 8-15: b
  asm volatile("s_nop 1\n\t"
               "v_min_f32_dpp %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
               "v_min_f32_dpp %0, %1, %1 row_ror:8 row_mask:0xf bank_mask:0xc" : "+v"(a) : "v"(b));
  return a;
}
__device__ inline float dpp_min_mirror8_keep(float a, float b) {  // lanes 0-3 of every eight: a; lanes 4-7: b
  asm volatile("s_nop 1\n\t"
               "v_min_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
               "v_min_f32_dpp %0, %1, %1 row_half_mirror row_mask:0xf bank_mask:0xa" : "+v"(a) : "v"(b));
  return a;
}
__device__ inline float dpp_min_mirror8(float a) {
  asm volatile("s_nop 1\n\tv_min_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf" : "+v"(a));
  return a;
}
__device__ inline float dpp_min_quad(float a) {
  asm volatile("s_nop 1\n\t"
               "v_min_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
               "s_nop 1\n\t"
               "v_min_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf" : "+v"(a));
  return a;
}
template <int N>
__device__ inline int value_of_lane(int lane) {
  const int b2 = (lane >> 2) & 1, b3 = (lane >> 3) & 1, b4 = (lane >> 4) & 1, b5 = (lane >> 5) & 1;
  return N == 16 ? 8 * b4 + 4 * b5 + 2 * b3 + b2 : 4 * b4 + 2 * b5 + b3;
}
// v[j] holds value j in the even rows of the wave and value j + N / 2 in the odd rows,
// already reduced over each row pair (swap_min_rows): the remaining steps.
template <int N>
__device__ inline float wave_min_rest(float (&v)[N / 2]) {
  static_assert(N == 8 || N == 16, "two values (min, -max) for 4 or 8 tokens");
#pragma unroll
  for (int j = 0; j < N / 4; ++j) v[j] = swap_min_halves(v[j], v[j + N / 4]);
#pragma unroll
  for (int j = 0; j < N / 8; ++j) v[j] = dpp_min_xor8_keep(v[j], v[j + N / 8]);
  float r;
  if constexpr (N == 16) r = dpp_min_mirror8_keep(v[0], v[1]);
  else r = dpp_min_mirror8(v[0]);
  return dpp_min_quad(r);
}

// x s rounded to an integer, plus 1.5 * 2^23 (exact for |x s| < 2^22); x s itself is rounded first.
constexpr float kRoundMagic = 12582912.f;
constexpr uint32_t kTameZero = 0x4a000000u;        // 2^21: zero points up to here keep every sum in range
__device__ inline float rounded_sum(float x, float s) {
#pragma clang fp contract(off)
  const float q = x * s;
  return q + kRoundMagic;
}

template <int BITS>
__device__ inline uint32_t shift_add(uint32_t acc, uint32_t x) {          // (written out: the compiler makes shifts and three-way sums of a chain)
  uint32_t r;
  asm("v_lshl_add_u32 %0, %1, %2, %3" : "=v"(r) : "v"(acc), "n"(BITS), "v"(x));
  return r;
}

__device__ inline int tile_of_field_group(int bits, int jf) {
  // Slot tile (16 slots) addressed by field group jf of a TGROUP word.
  return (bits == 2) ? ((jf & 1) * 2 + (jf >> 1)) : jf;
}

// ---- column sweep: statistics, parameters and - channelwise keys - codes in one launch ----
// A workgroup owns 8 vl channels of one subset of one batch element, vl lanes across a token
// row and THREADS / vl rows at a time.  With no partials to exchange the parameters are final
// when its own reduction is.  Channelwise codes in ROW layout need nothing else, so there
// (a.resident) the rows stay in registers between the reduction and the packing: the tensor
// is read from memory once and a launch does everything.  Bound by memory where the chip is
// full (16 x 4096 tokens of 5120 channels, fp16: keys packed and statistics of the values in
// 379 us, 517 as three launches that read the keys twice), by the latency of its two rounds
// of loads where it is not (one prompt of 4096 tokens, 1024 channels: 8 us for both tensors'
// statistics and parameters, 14 as two launches).
constexpr int64_t kPartBytes = 0xFFFFF000ll;                       // codes of a batch element: least size that a 32-bit offset does not reach
constexpr int kColRows(int dt) { return dt == ZC_F32 ? 10 : 20; }   // rows a thread can hold

template <int DT>
__device__ inline void widen8(const uint4 (&raw)[DT == ZC_F32 ? 2 : 1], float (&v)[8]) {
  if constexpr (DT == ZC_F32) {
    v[0] = __uint_as_float(raw[0].x); v[1] = __uint_as_float(raw[0].y); v[2] = __uint_as_float(raw[0].z); v[3] = __uint_as_float(raw[0].w);
    v[4] = __uint_as_float(raw[1].x); v[5] = __uint_as_float(raw[1].y); v[6] = __uint_as_float(raw[1].z); v[7] = __uint_as_float(raw[1].w);
  } else {
    const uint32_t w4[4] = {raw[0].x, raw[0].y, raw[0].z, raw[0].w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[2 * i] = half_bits_to_float<DT>(w4[i] & 0xffffu);
      v[2 * i + 1] = half_bits_to_float<DT>(w4[i] >> 16);
    }
  }
}

// The 8 codes of one token row, packed (ROW layout).
template <int DT, int BITS>
__device__ inline void row_codes(uint32_t (&code)[BITS == 8 ? 2 : 1], const float (&x)[8], const float (&p0)[8], const float (&p1)[8], const float (&p2)[8]) {
  constexpr float QMAX = (float)((1 << BITS) - 1);
  constexpr int FPG = 16 / BITS, NG = 8 / FPG;       // code fields per 16-bit group, groups
  uint32_t half[NG];
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    float acc = 0.f;
#pragma unroll
    for (int f = 0; f < FPG; ++f) {
      const int i = g * FPG + f;
      float qv;
      if constexpr (DT == ZC_F32) qv = rintf(refined_ratio(x[i], QMAX, p2[i], p0[i])) + p1[i];
      else qv = rintf(refined_div(x[i] * QMAX, p2[i], p0[i])) + p1[i];   // x * qmax is exact
      acc = fmaf(__builtin_amdgcn_fmed3f(qv, 0.f, QMAX), (float)(1 << (BITS * f)), acc);
    }
    half[g] = (uint32_t)acc;
  }
#pragma unroll
  for (int g = 0; g < NG; g += 2) code[g / 2] = half[g] | (g + 1 < NG ? half[g + 1] << 16 : 0u);
}
template <int DT, int BITS>
__device__ inline void store_row_codes(uint8_t* row, const float (&x)[8], const float (&p0)[8], const float (&p1)[8], const float (&p2)[8]) {
  uint32_t code[BITS == 8 ? 2 : 1];
  row_codes<DT, BITS>(code, x, p0, p1, p2);
  if constexpr (BITS == 8) *reinterpret_cast<uint2*>(row) = make_uint2(code[0], code[1]);
  else if constexpr (BITS == 4) *reinterpret_cast<uint32_t*>(row) = code[0];
  else *reinterpret_cast<uint16_t*>(row) = (uint16_t)code[0];
}

// ---- 2-bit codes of fp16 keys by thresholds ------------------------------------------------
// A channel's codes ascend with its values, so a 2-bit code is the number of three thresholds a value reaches:
// the least fp16 numbers whose code is 1, 2 and 3.  Two values at a time (the sign of x - t, which is exact), a code
// takes 4 instructions instead of 9.  (bf16 would take 5, with saturating differences of order-preserving integers: no
// faster where the chip is full, and finding the thresholds costs 0.6 us where it is not.)
// Ranges from 2^60 on or up to 2^-60 and zero points above 2^20, NaN among them (bits of larger ones are larger): the general path.
__device__ inline bool has_thresholds(float z, float R) {
  const uint32_t r = bits_of(R);
  return r > 0x21800000u && r < 0x5d800000u && (bits_of(z) & 0x7fffffffu) <= 0x49800000u;
}
typedef _Float16 half2v __attribute__((ext_vector_type(2)));

// Finding them is a chain of its own, which a thread with more rows than so many makes up for.  us for keys, dividing and by thresholds: 8 x
// 100 tokens of 8 heads of 128 channels 5.36 and 5.98, 4 x 1000 7.4 and 7.9 (4 to 6 rows), 4 x 2000 9.78 and 9.77 (9), 2 x 3000 of 32 heads
// 23.1 and 21.7, 4096 of 40 heads 26.8 and 24.7.
constexpr int kThresholdRows = 8;
// Order-preserving integer of a 16-bit float's bits, and back.
__device__ inline int ordered16(int bits) {
  const int s = (int)(int16_t)bits;
  return s ^ ((s >> 15) & 0x7fff);
}

// Negated threshold (bits) of code j (1 .. 3) of a channel with zero point z, range R and y = 1 / R.
__device__ inline uint16_t negated_threshold(int j, float z, float R, float y) {
  constexpr int inf = 0x7c00;
  const float at = ((float)j - 0.5f - z) * (R * (1.f / 3.f));     // where the rounding turns to j: the threshold is next to it
  const int g = ordered16((int)__builtin_bit_cast(uint16_t, (_Float16)at));
  int t = min(g + 2, inf);
#pragma unroll
  for (int d = 1; d >= -1; --d) {
    const int k = min(max(g + d, -inf - 1), inf);
    const float x = f16_bits_to_float((uint32_t)ordered16(k) & 0xffffu);
    if (k == inf || rintf(refined_div(x * 3.f, R, y)) + z >= (float)j) t = k;
  }
  return (uint16_t)(ordered16(t) ^ 0x8000);
}

// Bits of a where mask is set, of b elsewhere; the exclusive or of three.  (Written out: of constant masks the
// compiler makes ands and ors.)
__device__ inline uint32_t select_bits(uint32_t mask, uint32_t a, uint32_t b) { return __builtin_amdgcn_bitop3_b32(mask, a, b, 0xca); }
__device__ inline uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) { return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96); }
struct CodeMasks { uint32_t top, pair, quad; };          // of the bits 15; 14 and 15 of both halves; 2, 3, 6, 7, 10, 11, 14 and 15
__device__ inline CodeMasks code_masks() {
  CodeMasks m = {0x80008000u, 0xc000c000u, 0xccccu};
  asm("" : "+s"(m.top), "+s"(m.pair), "+s"(m.quad));
  return m;
}

// The 8 codes of one token row's channels, two bits each; t[j]: the negated thresholds of code j + 1, two to a word.
__device__ inline uint16_t threshold_codes(const uint4& raw, const uint4 (&t)[3], const CodeMasks& m) {
  const uint32_t x4[4] = {raw.x, raw.y, raw.z, raw.w};
  uint32_t w = 0u;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const auto below = [&](const uint4& v) {             // sign bits: below the threshold
      const uint32_t word = i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w;
      return __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2v, x4[i]) + __builtin_bit_cast(half2v, word));
    };
    const uint32_t b1 = below(t[0]), b2 = below(t[1]), b3 = below(t[2]);
    // the complement of a code: high bit "below 2", low bit the parity of the thresholds it is below
    const uint32_t c = select_bits(m.top, b2, xor3(b1, b2, b3) >> 1);
    w = i == 0 ? c : select_bits(m.pair, c, w >> 4);     // even channels' in the low half, four bits apart, odd ones' in the high half
  }
  return (uint16_t)__builtin_amdgcn_bitop3_b32(m.quad, w >> 16, w >> 2, 0x35);      // (the complement of select_bits)
}

// sum + 0 x for the 8 values of x, two at a time: not zero where one of them is a NaN.  (Written out: the compiler may drop
// arithmetic that only a NaN gets through.)
__device__ inline uint32_t plus_zero_times(uint32_t sum, const uint4& x) {
  const uint32_t x4[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) asm("v_pk_fma_f16 %0, %1, 0, %0" : "+v"(sum) : "v"(x4[i]));
  return sum;
}

template <int DT, int THREADS, bool SPLIT = false>       // SPLIT: `split` token ranges per subset, only their minima
__global__ __launch_bounds__(THREADS, 4) void k_columns(QPPair p, int tensors, int split) {
  constexpr int RAW = (DT == ZC_F32) ? 2 : 1, ESZ = (DT == ZC_F32) ? 4 : 2;
  constexpr int NR = kColRows(DT), NWAVE = THREADS / 64;
  __shared__ __align__(16) float red[NWAVE][2][128];
  __shared__ __align__(16) float prm[3][128];
  __shared__ __align__(16) uint16_t thr[3][128];         // thresholds of 2-bit codes
  __shared__ int wild;                                   // some channel has none

  // logical order: channel group fastest, then subset, tensor, batch element: the workgroups
  // that share a token row's cache lines run on one XCD at about the same time
  const int vl = p.t[0].vl, groups = ceil_div(p.t[0].NV, vl);
  int id = xcd_contiguous(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
  const int grp = id % groups; id /= groups;
  int part = 0;
  if constexpr (SPLIT) { part = id % split; id /= split; }
  const int sub = id & 1; id >>= 1;
  const int which = tensors == 2 ? id & 1 : 0, b = tensors == 2 ? id >> 1 : id;
  const QPArgs& a = which ? p.t[1] : p.t[0];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int x = tid & (vl - 1), y = tid / vl, step = THREADS / vl;
  const int y0 = __builtin_amdgcn_readfirstlane(y);             // the wave's first row
  const int n = a.scheme == ZC_SCHEME_TOKEN ? 0 : a.n[sub];     // (plain tokenwise: no channel statistics)
  const int vec = min(grp * vl + x, a.NV - 1);                  // (lanes past the row repeat its last vector)
  const int w = vec * 8, h = w / a.D, c = w % a.D;
  const char* base = reinterpret_cast<const char*>(a.x) + ((int64_t)b * a.sB + (int64_t)h * a.sH + c) * ESZ;
  const int64_t row_bytes = a.sL * ESZ;
  const int32_t* idx = a.idx[sub] + (int64_t)b * a.n[sub];

  float mn[8], mneg[8];                                         // minimum, minimum of -x
#pragma unroll
  for (int i = 0; i < 8; ++i) { mn[i] = INFINITY; mneg[i] = INFINITY; }
  uint4 raw[NR][RAW];
  auto reduce = [&](const uint4 (&rw)[RAW]) {
    float v[8];
    widen8<DT>(rw, v);
#pragma unroll
    for (int i = 0; i < 8; ++i) { mn[i] = fminf(mn[i], v[i]); mneg[i] = fminf(mneg[i], -v[i]); }
  };
  // Rows are requested before any is reduced, all of a resident subset or kStatBatch at a time;
  // rows past the end repeat the last one (minima do not care).
  if (!SPLIT && a.resident) {
    int32_t tok[NR];
    // (every wave takes a first row, if only the last one again: no branch in front of it)
    const auto has = [&](int r) { return r == 0 ? n > 0 : r * step + y0 < n; };
#pragma unroll
    for (int r = 0; r < NR; ++r)
      if (has(r)) tok[r] = idx[min(r * step + y, n - 1)];
#pragma unroll
    for (int r = 0; r < NR; ++r)
      if (has(r)) {
        const uint4* src = reinterpret_cast<const uint4*>(base + (int64_t)tok[r] * row_bytes);
#pragma unroll
        for (int q = 0; q < RAW; ++q) raw[r][q] = src[q];
      }
#pragma unroll
    for (int r = 0; r < NR; ++r)
      if (has(r)) reduce(raw[r]);
    // (all rows are here; the compiler, which does not see that a row that was requested has been reduced, would wait for
    // each again where it is packed - and with it for the codes stored before)
    __builtin_amdgcn_s_waitcnt(0x0F70);                        // vmcnt(0)
  } else {
    int first = 0, n1 = n;
    if constexpr (SPLIT) {
      const int per = ceil_div(n, split);
      first = part * per;
      n1 = min(n, first + per);
    }
    int32_t tok[kStatBatch];                     // of the next batch: looked up while the one before is on its way
    const auto look_up = [&](int t0) {
#pragma unroll
      for (int r = 0; r < kStatBatch; ++r) tok[r] = idx[min(t0 + r * step + y, n1 - 1)];
    };
    if (first < n1) look_up(first);
    for (int t0 = first; t0 < n1; t0 += kStatBatch * step) {
      uint4 rw[kStatBatch][RAW];
#pragma unroll
      for (int r = 0; r < kStatBatch; ++r) {
        const uint4* src = reinterpret_cast<const uint4*>(base + (int64_t)tok[r] * row_bytes);
#pragma unroll
        for (int q = 0; q < RAW; ++q) rw[r][q] = src[q];
      }
      if (t0 + kStatBatch * step < n1) look_up(t0 + kStatBatch * step);
#pragma unroll
      for (int r = 0; r < kStatBatch; ++r) reduce(rw[r]);
    }
  }
  // over the rows of a wave: (minimum, minimum of -x) split over its halves, channels 0..3 and
  // 4..7 over the rows of a half, the rest inside a row of 16 lanes
  {
    float u[4];
#pragma unroll
    for (int j = 0; j < 8; ++j) mn[j] = swap_min_halves(mn[j], mneg[j]);
#pragma unroll
    for (int j = 0; j < 4; ++j) u[j] = swap_min_rows(mn[j], mn[j + 4]);
    if (vl <= 8) {
#pragma unroll
      for (int j = 0; j < 4; ++j) u[j] = fminf(u[j], __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(u[j]), 0x128, 0xF, 0xF, true)));   // row_ror:8
    }
    if (vl <= 4) {
#pragma unroll
      for (int j = 0; j < 4; ++j) u[j] = fminf(u[j], __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(u[j]), 0x124, 0xF, 0xF, true)));   // row_ror:4
    }
    if (vl <= 2) {
#pragma unroll
      for (int j = 0; j < 4; ++j) u[j] = fminf(u[j], __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(u[j]), 0x122, 0xF, 0xF, true)));   // row_ror:2
    }
    if (tid == 0) wild = 0;
    if ((lane & 15) < vl)
      *reinterpret_cast<float4*>(&red[wave][lane >> 5][(lane & 15) * 8 + 4 * ((lane >> 4) & 1)]) = make_float4(u[0], u[1], u[2], u[3]);
  }
  __syncthreads();
  const int wc = grp * vl * 8 + tid;                            // channel of this thread in the parameter step
  const bool by_thresholds = DT == ZC_F16 && a.resident && a.bits[sub] == 2 && n > kThresholdRows * step;
  if (tid < vl * 8 && wc < a.W) {
    float lo = red[0][0][tid], neg = red[0][1][tid];
#pragma unroll
    for (int v = 1; v < NWAVE; ++v) { lo = fminf(lo, red[v][0][tid]); neg = fminf(neg, red[v][1][tid]); }
    if constexpr (SPLIT) {
      range_minima(a)[((int64_t)(b * 2 + sub) * split + part) * a.W + wc] = make_float2(lo, neg);
      return;
    }
    float cs, cz;
    const float3 pr = channel_params(a.scheme, n, (float)((1 << a.bits[sub]) - 1), lo, -neg, &cs, &cz);
    const int64_t o = (int64_t)(sub * a.B + b) * a.W + wc;
    a.chan_scale[o] = cs;
    a.chan_zero[o] = cz;
    if (!a.resident) store_params(a, b, sub, wc, pr);
    prm[0][tid] = pr.x; prm[1][tid] = pr.y; prm[2][tid] = pr.z;
    if (by_thresholds) {
      if (!has_thresholds(pr.y, pr.z)) wild = 1;
      else {
#pragma unroll 1
        for (int j = 0; j < 3; ++j) thr[j][tid] = negated_threshold(j + 1, pr.y, pr.z, pr.x);
      }
    }
  }
  if constexpr (SPLIT) return;
  if (grp == 0 && sub == 0 && b == 0 && tid == 0) {
    a.chunk_row[0] = a.begin[0]; a.chunk_row[1] = a.n[0];
    a.chunk_row[2] = a.begin[1]; a.chunk_row[3] = a.n[1];
  }
  if (!a.resident) return;
  __syncthreads();

  if (grp == 0 && a.pos[sub])
    for (int t = tid; t < n; t += THREADS) a.pos[sub][(int64_t)b * a.cap[sub] + a.begin[sub] + t] = (int32_t)(idx[t] + a.pos_offset);
  if (grp * vl + x >= a.NV) return;
  const int bits = a.bits[sub];
  // Codes of a row through a buffer descriptor over this batch element's, from the chunk's first slot on: rows past the
  // end are out of range (no branch), and the offset takes 32 bits.
  const int rowb = a.D * bits / 8;
  const uint32_t room = (uint32_t)(((int64_t)a.H * a.cap[sub] - a.begin[sub]) * rowb);      // (below kPartBytes: col_plan)
  const uint32_t at = (uint32_t)(((int64_t)h * a.cap[sub] + y) * rowb) + c * bits / 8;
  const auto rs_dst = __builtin_amdgcn_make_buffer_rsrc(a.codes[sub] + ((int64_t)b * a.H * a.cap[sub] + a.begin[sub]) * rowb, 0, room, 0x00020000);
  const auto offset_of = [&](int r) { return r * step + y < n ? (int)(at + (uint32_t)(r * step * rowb)) : (int)(uint32_t)kPartBytes; };
  if constexpr (DT == ZC_F16) {
    if (by_thresholds && !wild) {
      const CodeMasks m = code_masks();
      uint4 t[3];
#pragma unroll
      for (int j = 0; j < 3; ++j) t[j] = *reinterpret_cast<const uint4*>(&thr[j][x * 8]);
      uint32_t nan = 0u;
#pragma unroll
      for (int r = 0; r < NR; ++r)
        if (r * step + y0 < n) {
          __builtin_amdgcn_raw_buffer_store_b16((short)threshold_codes(raw[r][0], t, m), rs_dst, offset_of(r), 0, 0);
          nan = plus_zero_times(nan, raw[r][0]);
        }
      if (__builtin_amdgcn_ballot_w64((nan & 0x7fff7fffu) != 0u) == 0) return;      // (a NaN's code is what the general path makes of it)
    }
  }
  float p0[8], p1[8], p2[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) { p0[i] = prm[0][x * 8 + i]; p1[i] = prm[1][x * 8 + i]; p2[i] = prm[2][x * 8 + i]; }
  auto pack = [&](auto bits_c) {
    constexpr int BITS = decltype(bits_c)::value;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      if (r * step + y0 < n) {
        float v[8];
        uint32_t code[BITS == 8 ? 2 : 1];
        widen8<DT>(raw[r], v);
        row_codes<DT, BITS>(code, v, p0, p1, p2);
        if constexpr (BITS == 8) {
          typedef uint32_t u2 __attribute__((ext_vector_type(2)));
          __builtin_amdgcn_raw_buffer_store_b64(u2{code[0], code[1]}, rs_dst, offset_of(r), 0, 0);
        } else if constexpr (BITS == 4) {
          __builtin_amdgcn_raw_buffer_store_b32(code[0], rs_dst, offset_of(r), 0, 0);
        } else {
          __builtin_amdgcn_raw_buffer_store_b16((short)code[0], rs_dst, offset_of(r), 0, 0);
        }
      }
    }
  };
  if (bits == 4) pack(std::integral_constant<int, 4>{});
  else if (bits == 2) pack(std::integral_constant<int, 2>{});
  else pack(std::integral_constant<int, 8>{});
}

// Parameters from the minima of a subset's token ranges, a thread per channel; also those of the
// plain tokenwise scheme, which has no statistics (1 and 0).
// grid (ceil(W / 256), 2 subsets x tensors, B)
__global__ __launch_bounds__(256) void k_column_params(QPPair p, int split) {
  const QPArgs& a = blockIdx.y >> 1 ? p.t[1] : p.t[0];
  const int sub = blockIdx.y & 1, b = blockIdx.z, w = blockIdx.x * 256 + threadIdx.x;
  if (w >= a.W) return;
  float lo = INFINITY, neg = INFINITY;
  if (a.scheme != ZC_SCHEME_TOKEN) {
    const float2* src = range_minima(a) + (int64_t)(b * 2 + sub) * split * a.W + w;
    for (int t0 = 0; t0 < split; t0 += 16) {
      float2 v[16];
#pragma unroll
      for (int t = 0; t < 16; ++t) v[t] = src[(int64_t)min(t0 + t, split - 1) * a.W];
#pragma unroll
      for (int t = 0; t < 16; ++t) { lo = fminf(lo, v[t].x); neg = fminf(neg, v[t].y); }
    }
  }
  float cs, cz;
  const float3 pr = channel_params(a.scheme, a.n[sub], (float)((1 << a.bits[sub]) - 1), lo, -neg, &cs, &cz);
  const int64_t o = (int64_t)(sub * a.B + b) * a.W + w;
  a.chan_scale[o] = cs;
  a.chan_zero[o] = cz;
  store_params(a, b, sub, w, pr);
  if (sub == 0 && b == 0 && w == 0) {
    a.chunk_row[0] = a.begin[0]; a.chunk_row[1] = a.n[0];
    a.chunk_row[2] = a.begin[1]; a.chunk_row[3] = a.n[1];
  }
}

constexpr int kVPT = 1;  // channel vectors (8 channels each) per thread in the quantize sweep

// The quantize sweep of one workgroup: `ng` consecutive word groups of one TGROUP
// block.  A word group is the 32 / bits tokens whose codes share 32-bit words in
// the TGROUP layout (block blk, k-group kg); it is processed in batches of up to
// 8 tokens, a thread owning 8 channels of every token.  The rows of batch i + 1
// are requested before batch i is reduced and quantized.
//   tokenwise schemes: x' = x / c is kept in registers between the range pass and
//   the quantize pass; the per-token range goes through a DPP wave reduction,
//   then (teams of several waves) through LDS; lanes 0..7 then compute the
//   parameters of tokens 0..7 of the batch, once, and broadcast them.
//   codes are assembled in float: sum of code * 2^(bits * position) over a 16-bit
//   group is exact in fp32, so packing costs one FMA per code.
template <int DT, int BITS, int LAYOUT, bool TOKWISE, bool EXACT, bool PIPE>
__device__ inline void quant_units(const QPArgs& a, int sub, int g0, int ng, int b, float (*red)[16][16], int32_t* sidx) {
  constexpr int E = 32 / BITS;                       // tokens of a word group
  constexpr int TBAT = E < 8 ? E : 8;                // tokens per batch
  constexpr int NBAT = E / TBAT;                     // batches per word group
  constexpr int TB = 4 * E;                          // slots per TGROUP block
  constexpr int FPG = 16 / BITS;                     // code fields per 16-bit group
  constexpr float QMAX = (float)((1 << BITS) - 1);
  constexpr int RAW = (DT == ZC_F32) ? 2 : 1;        // 16-byte loads per channel vector
  constexpr int ESZ = (DT == ZC_F32) ? 4 : 2;

  const int n = a.n[sub];
  const int TX = blockDim.x, x = threadIdx.x;
  const int lane = x & 63, wave = x >> 6, nwaves = TX >> 6;
  const int32_t* idx = a.idx[sub] + (int64_t)b * n;
  const int blk = g0 >> 2;                           // every word group of this workgroup lies in this block

  // source positions of the block's slots (-1 past the end of the subset)
  if (x < TB) { const int rel = blk * TB + x; sidx[x] = rel < n ? idx[rel] : -1; }

  // parameters of the channels this thread owns
  // (the channelwise scheme needs no reduction over a token row, so its launches cut
  // the row into chunks of blockDim.x vectors along grid.z)
  const int vec = (int)blockIdx.z * TX + x;
  const bool vvalid = vec < a.NV;
  const int w = (vvalid ? vec : 0) * 8, h = w / a.D, c = w % a.D;
  const char* xbase = reinterpret_cast<const char*>(a.x) + ((int64_t)b * a.sB + (int64_t)h * a.sH + c) * ESZ;
  const int64_t row_bytes = a.sL * ESZ;
  float p0[8], p1[8], p2[8];
  {
    load8<ZC_F32>(param_row(a, b, sub, 0), w, p0);
    if constexpr (!TOKWISE) {
      load8<ZC_F32>(param_row(a, b, sub, 1), w, p1);
      load8<ZC_F32>(param_row(a, b, sub, 2), w, p2);
    }
  }
  __syncthreads();

  float neg_zero = -0.f;                             // (opaque: a known one would turn the fma back into a product)
  asm("" : "+s"(neg_zero));
  struct Batch { uint4 raw[TBAT][RAW]; };
  // batch q of the workgroup: word group g0 + q / NBAT, tokens (q % NBAT) * TBAT + t of it
  auto slot_of = [&](int q, int t) {                 // slot inside the block
    const int kg = (g0 + q / NBAT) & 3;
    const int e = (q % NBAT) * TBAT + t;
    return 16 * tile_of_field_group(BITS, e >> 2) + 4 * kg + (e & 3);
  };
  auto issue = [&](int q, Batch& bt) {
#pragma unroll
    for (int t = 0; t < TBAT; ++t) {
      const int pos = sidx[slot_of(q, t)];
#pragma unroll
      for (int r = 0; r < RAW; ++r) {
        bt.raw[t][r] = make_uint4(0u, 0u, 0u, 0u);
        if (pos >= 0 && vvalid) bt.raw[t][r] = *reinterpret_cast<const uint4*>(xbase + (int64_t)pos * row_bytes + 16 * r);
      }
    }
  };
  auto widen = [&](const Batch& bt, int t, float (&v)[8]) {
    if constexpr (DT == ZC_F32) {
      v[0] = __uint_as_float(bt.raw[t][0].x); v[1] = __uint_as_float(bt.raw[t][0].y);
      v[2] = __uint_as_float(bt.raw[t][0].z); v[3] = __uint_as_float(bt.raw[t][0].w);
      v[4] = __uint_as_float(bt.raw[t][RAW - 1].x); v[5] = __uint_as_float(bt.raw[t][RAW - 1].y);
      v[6] = __uint_as_float(bt.raw[t][RAW - 1].z); v[7] = __uint_as_float(bt.raw[t][RAW - 1].w);
    } else {
      const uint32_t w4[4] = {bt.raw[t][0].x, bt.raw[t][0].y, bt.raw[t][0].z, bt.raw[t][0].w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v[2 * i] = half_bits_to_float<DT>(w4[i] & 0xffffu);
        v[2 * i + 1] = half_bits_to_float<DT>(w4[i] >> 16);
      }
    }
  };

  uint32_t words[8];                                 // TGROUP: the word group's words of this thread's channels

  auto process = [&](int q, const Batch& bt, int parity) {
    const int kg = (g0 + q / NBAT) & 3, bi = q % NBAT;
    bool tv[TBAT];
#pragma unroll
    for (int t = 0; t < TBAT; ++t) tv[t] = blk * TB + slot_of(q, t) < n;
    if (LAYOUT == ZC_LAYOUT_TGROUP && bi == 0) {
#pragma unroll
      for (int i = 0; i < 8; ++i) words[i] = 0u;
    }
    // bookkeeping of the batch's tokens by lanes 0 .. TBAT-1 of the first wave
    const int my_t = lane < TBAT ? lane : 0;
    const int my_rel = blk * TB + slot_of(q, my_t);
    const bool my_live = x < TBAT && blockIdx.z == 0 && my_rel < n;
    const int64_t my_o = (int64_t)b * a.cap[sub] + a.begin[sub] + my_rel;
    if (my_live && a.pos[sub]) a.pos[sub][my_o] = (int32_t)(sidx[my_rel - blk * TB] + a.pos_offset);

    float xs[TBAT][8];                               // tokenwise: x' = x / c; channelwise: x
    float sinv[TBAT], zt[TBAT];
    float silane = 0.f, zlane = 0.f, low = 0.f, high = 0.f;      // of token (lane & 7): 1/s, z, the bounds of its rounded sums
    bool wild = false;                               // some token's zero point is out of their range
    float rt[TBAT], yt[TBAT];                        // EXACT (the plain tokenwise scheme) only: range and its reciprocal
#pragma unroll
    for (int t = 0; t < TBAT; ++t) {
      if constexpr (TOKWISE && DT == ZC_F16) {        // widened by the multiplication: v_fma_mix_f32 with an addend of -0
        typedef _Float16 h8v __attribute__((ext_vector_type(8)));
        const h8v hx = __builtin_bit_cast(h8v, bt.raw[t][0]);
#pragma unroll
        for (int i = 0; i < 8; ++i) xs[t][i] = fmaf((float)hx[i], p0[i], neg_zero);
        continue;
      }
      widen(bt, t, xs[t]);
      if constexpr (TOKWISE) {
#pragma unroll
        for (int i = 0; i < 8; ++i) xs[t][i] *= p0[i];
      }
    }
    if constexpr (TOKWISE) {
      // (min, -max) of every token over the wave: values 0 .. TBAT-1 the minima,
      // TBAT .. 2 TBAT-1 the negated maxima
      // (the first step - rows - pairs a token's minimum with its negated maximum, so
      // it is taken as soon as the two exist: TBAT registers live, not 2 TBAT)
      float mm[TBAT];
#pragma unroll
      for (int t = 0; t < TBAT; ++t) {
        float l = xs[t][0], hneg = -xs[t][0];
#pragma unroll
        for (int i = 1; i < 8; ++i) { l = fminf(l, xs[t][i]); hneg = fminf(hneg, -xs[t][i]); }
        if (!vvalid) { l = INFINITY; hneg = INFINITY; }
        mm[t] = swap_min_rows(l, hneg);
      }
      const float wmin = wave_min_rest<2 * TBAT>(mm);
      // through LDS: lane j < 16 ends up with value j (min of token j, or -max of token j - 8)
      // over all waves.  One barrier per batch: the scratch alternates, and the barrier
      // of the next batch separates these reads from the writes of the batch after it.
      float* mine = &red[parity][wave][0];
      if ((lane & 3) == 0) {
        const int vi = value_of_lane<2 * TBAT>(lane);
        mine[vi < TBAT ? vi : 8 + vi - TBAT] = wmin;
      }
      if (nwaves > 1) __syncthreads();
      float r = red[parity][0][lane & 15];
      for (int w2 = 1; w2 < nwaves; ++w2) r = fminf(r, red[parity][w2][lane & 15]);
      const float tmin = r;
      const float tmax = -__shfl(r, (lane & 7) + 8);
      // parameters of token (lane & 7), computed once per lane group
      float R = tmax - tmin;
      if (R == 0.f) R = QMAX;                        // max == min: s := 1
      const float y = __builtin_amdgcn_rcpf(R);
      const float z = -rintf(refined_ratio(tmin, QMAX, R, y));   // tie-exact: a whole row depends on it
      const float si = QMAX * y;
      silane = si; zlane = z;
      low = kRoundMagic - z;
      high = my_rel < n ? low + QMAX : low;
      wild = __ballot(lane < TBAT && (__float_as_uint(z) & 0x7fffffffu) > kTameZero) != 0;
      if (my_live) {
        a.tok_scale[sub][my_o] = R * (1.f / QMAX);
        a.tok_zero[sub][my_o] = z;
      }
#pragma unroll
      for (int t = 0; t < TBAT; ++t) {
        sinv[t] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(si), t));
        zt[t] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(z), t));
        if constexpr (EXACT) {
          rt[t] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(R), t));
          yt[t] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(y), t));
        }
      }
    }

    // Code of a tokenwise element before clipping.  With channel normalization x' = x / c is
    // not on a grid and a plain product decides the rounding; without it (the plain tokenwise
    // scheme, c = 1) 16-bit inputs sit on a grid where x (2^k - 1) / R hits n + 1/2 exactly
    // about once in 10^4 elements, so the quotient is the tie-exact one there.
    auto tok_code = [&](float xv, int t) {
      if constexpr (!EXACT) return rintf(xv * sinv[t]) + zt[t];
      else if constexpr (DT == ZC_F32) return rintf(refined_ratio(xv, QMAX, rt[t], yt[t])) + zt[t];
      else return rintf(refined_div(xv * QMAX, rt[t], yt[t])) + zt[t];      // x * qmax is exact
    };
    if (!vvalid) return;                             // (a row is whole heads of 64 or 128 channels: lanes 0..7, read below, stay or go together)
    if constexpr (LAYOUT == ZC_LAYOUT_ROW) {
      static_assert(TOKWISE, "channelwise codes in ROW layout are k_pack_kv's");
#pragma unroll
      for (int t = 0; t < TBAT; ++t) {
        // Eq. 5: round(x / s) first, then + z, then clip
        float code[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) code[i] = __builtin_amdgcn_fmed3f(tok_code(xs[t][i], t), 0.f, QMAX);
        if (!tv[t]) continue;
        // the 8 codes of this token, 16 bits at a time
        constexpr int NG = 8 / FPG;                  // 16-bit groups of the 8 codes (>= 1: bits >= 2)
        uint32_t half[NG];
#pragma unroll
        for (int g = 0; g < NG; ++g) {
          float acc = 0.f;
#pragma unroll
          for (int f = 0; f < FPG; ++f) acc = fmaf(code[g * FPG + f], (float)(1 << (BITS * f)), acc);
          half[g] = (uint32_t)acc;
        }
        const int64_t slot = a.begin[sub] + blk * TB + slot_of(q, t);
        uint8_t* row = a.codes[sub] + (((int64_t)b * a.H + h) * a.cap[sub] + slot) * (a.D * BITS / 8) + c * BITS / 8;
        if constexpr (BITS == 8) {
          *reinterpret_cast<uint2*>(row) = make_uint2(half[0] | (half[1] << 16), half[2] | (half[3] << 16));
        } else if constexpr (BITS == 4) {
          *reinterpret_cast<uint32_t*>(row) = half[0] | (half[1] << 16);
        } else {
          *reinterpret_cast<uint16_t*>(row) = (uint16_t)half[0];
        }
      }
    }
    if constexpr (LAYOUT == ZC_LAYOUT_TGROUP) {
      if constexpr (TOKWISE && !EXACT) {
        // Adding 1.5 * 2^23 rounds to the integers (half to even); clamped there to [-z, QMAX - z],
        // the sum's low bits are the code plus those of 1.5 * 2^23 - z, which come off once per word:
        // four instructions a code instead of five, and no conversion.  (A dead token's range is empty.)
        // Values of 16 x 4096 tokens of 40 heads, fp16, column sweep included: 320.6 -> 313.7 us.
        uint32_t word_part[8];
        float lo_t[TBAT], hi_t[TBAT];
        uint32_t off = 0u;
#pragma unroll
        for (int t = 0; t < TBAT; ++t) {
          const uint32_t u = (uint32_t)__builtin_amdgcn_readlane(__float_as_int(low), t);
          lo_t[t] = __uint_as_float(u);
          hi_t[t] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(high), t));
          off += u << (BITS * t);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          uint32_t acc = 0u;
#pragma unroll
          for (int t = TBAT - 1; t >= 0; --t)
            acc = shift_add<BITS>(acc, __float_as_uint(__builtin_amdgcn_fmed3f(rounded_sum(xs[t][i], sinv[t]), lo_t[t], hi_t[t])));
          word_part[i] = acc - off;
        }
        if (wild) {
          // A zero point out of that range (a row whose spread is a 10^-6 of its values, an infinity):
          // the batch again from memory, in a rolled loop that needs few registers.
#pragma unroll
          for (int i = 0; i < 8; ++i) word_part[i] = 0u;
#pragma unroll 1
          for (int t = 0; t < TBAT; ++t) {
            const int pos = sidx[slot_of(q, t)];
            if (pos < 0) continue;
            float v[8];
            load8<DT>(xbase + (int64_t)pos * row_bytes, 0, v);
            const float st = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(silane), t));
            const float zt = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(zlane), t));
#pragma unroll
            for (int i = 0; i < 8; ++i)
              word_part[i] |= (uint32_t)__builtin_amdgcn_fmed3f(rintf(v[i] * p0[i] * st) + zt, 0.f, QMAX) << (BITS * t);
          }
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) words[i] |= word_part[i] << (BITS * bi * TBAT);
      } else {
      // channel i: the batch's tokens, 16 bits (FPG tokens) at a time; dead tokens add nothing
      constexpr int NG = TBAT / FPG > 0 ? TBAT / FPG : 1;
      constexpr int TPG = TBAT < FPG ? TBAT : FPG;   // tokens per 16-bit group
      float mult[TBAT];
#pragma unroll
      for (int t = 0; t < TBAT; ++t) mult[t] = tv[t] ? (float)(1 << (BITS * (t % TPG))) : 0.f;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
#pragma unroll
        for (int g = 0; g < NG; ++g) {
          float acc = 0.f;
#pragma unroll
          for (int f = 0; f < TPG; ++f) {
            const int t = g * TPG + f;
            float qv;
            if constexpr (TOKWISE) qv = tok_code(xs[t][i], t);
            else if constexpr (DT == ZC_F32) qv = rintf(refined_ratio(xs[t][i], QMAX, p2[i], p0[i])) + p1[i];
            else qv = rintf(refined_div(xs[t][i] * QMAX, p2[i], p0[i])) + p1[i];
            acc = fmaf(__builtin_amdgcn_fmed3f(qv, 0.f, QMAX), mult[t], acc);
          }
          words[i] |= (uint32_t)acc << (BITS * (bi * TBAT + g * TPG));
        }
      }
      }
      if (bi == NBAT - 1) {
        const int64_t nblk = a.cap[sub] / TB;
        const int64_t gblk = a.begin[sub] / TB + blk;
        uint32_t* dst = reinterpret_cast<uint32_t*>(a.codes[sub]) + ((((int64_t)b * a.H + h) * nblk + gblk) * 4 + kg) * a.D + c;
        reinterpret_cast<uint4*>(dst)[0] = make_uint4(words[0], words[1], words[2], words[3]);
        reinterpret_cast<uint4*>(dst)[1] = make_uint4(words[4], words[5], words[6], words[7]);
      }
    }
  };

  const int nq = ng * NBAT;
  if constexpr (PIPE) {
    Batch b0, b1;
    issue(0, b0);
    for (int i = 0; i < nq; i += 2) {
      const bool second = i + 1 < nq;
      if (second) issue(i + 1, b1);
      process(i, b0, 0);
      if (second) {
        if (i + 2 < nq) issue(i + 2, b0);
        process(i + 1, b1, 1);
      }
    }
  } else {
    Batch b0;
    for (int i = 0; i < nq; ++i) {
      issue(i, b0);
      process(i, b0, i & 1);
    }
  }
}

// MAXT: most threads of a workgroup (W / 8 rounded up to a wave); it bounds the
// registers of a thread, and with them whether two batches of rows fit.
// EXACT: tokenwise without channel normalization (the plain tokenwise scheme): tie-exact codes.
template <int DT, int LAYOUT, bool TOKWISE, bool EXACT, int MAXT>
__global__ __launch_bounds__(MAXT) void k_quant_pack(QPArgs a) {
  constexpr bool PIPE = (DT != ZC_F32) && MAXT <= 768;
  __shared__ float red[2][16][16];   // [turn][wave][min of token 0..7, -max of token 0..7]
  __shared__ int32_t sidx[64];
  const int b = blockIdx.y;
  int wg = blockIdx.x;
  const int sub = wg >= a.wgs[0] ? 1 : 0;
  if (sub) wg -= a.wgs[0];
  const int g0 = wg * a.upw, ng = a.upw;
  const int bits = a.bits[sub];
  if (bits == 4) quant_units<DT, 4, LAYOUT, TOKWISE, EXACT, PIPE>(a, sub, g0, ng, b, red, sidx);
  else if (bits == 2) quant_units<DT, 2, LAYOUT, TOKWISE, EXACT, PIPE>(a, sub, g0, ng, b, red, sidx);
  else quant_units<DT, 8, LAYOUT, TOKWISE, EXACT, PIPE>(a, sub, g0, ng, b, red, sidx);
}

// ---- the paper's configuration: channelwise keys in ROW layout, channel-separable tokenwise
// values in TGROUP layout -------------------------------------------------------------------------
// Bound by latency for one prompt: the sweep above holds 8 tokens x 8 channels a thread in straight
// code, 5 KB for each of two alternating batches, which is fetched cold at every launch.  Here a thread
// takes 4 channels of a word group's 8 or 16 values, all requested at once, or 8 channels of 4 keys in
// a rolled loop: 1 to 4 KB, and twice the waves.  us per joint call (column sweep included), before ->
// here: 100 tokens of 8 heads of 128 channels, bf16: 12.1 -> 9.4; 1000: 13.2 -> 10.3; 4096: 16.3 -> 14.9;
// 32768: 70.3 -> 57.4; 2 x 32768 of 16 heads, fp16: 260 -> 253; 4 x 16384 of them, fp32: 452 -> 427.
// In fp32, workgroups of five and six waves (1088 to 1536 channels) need five waves a SIMD, so 96
// registers, for three or four of them a CU: 4 x 4096 tokens of 1280 channels 60.6 -> 60.5 (63.8 with
// four a SIMD), of 1536 68.6 -> 69.0; one prompt 28.8 -> 27.4 and 30.6 -> 30.3; but values alone of 4 x 4096
// tokens of 1536 channels lose 2 to 4 % (42.7 -> 43.4, at 8 and 4 bits 44.2 -> 46.0).  Keys
// alone, which need no more than their own rows, come here at any width: 2 x 9000 tokens of 40 heads with
// their values 210 -> 193.  Values wider than a workgroup takes go through quant_units.
constexpr int kPackThreads = 512, kPackCpt = 4;     // values: most threads of a workgroup, channels of a thread

// 4 consecutive elements.
template <int DT>
__device__ inline void load4(const void* p, float (&v)[4]) {
  if constexpr (DT == ZC_F32) {
    const float4 t = *reinterpret_cast<const float4*>(p);
    v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
  } else {
    const uint2 t = *reinterpret_cast<const uint2*>(p);
    v[0] = half_bits_to_float<DT>(t.x & 0xffffu);
    v[1] = half_bits_to_float<DT>(t.x >> 16);
    v[2] = half_bits_to_float<DT>(t.y & 0xffffu);
    v[3] = half_bits_to_float<DT>(t.y >> 16);
  }
}

// Token e of a word group of values: its index in the subset.
template <int BITS>
__device__ inline int value_token(int blk, int kg, int e) {       // (the word group's block, its group in it)
  constexpr int TB = 4 * (32 / BITS);
  return blk * TB + 16 * tile_of_field_group(BITS, e >> 2) + 4 * kg + (e & 3);
}

// Values (TGROUP layout, channel-separable tokenwise): one word group, a thread per 4 channels.  TEAM: of `threads` threads of a
// workgroup from `first` on, red theirs, all of which come here; rows(x, inv_c) hands over the rows and the channels' parameters.
struct OwnRows {};
template <int DT, int BITS, typename ROWS = OwnRows>
__device__ inline void pack_values(const QPArgs& a, int sub, int unit, int b, float (*red)[kPackThreads / 64][16], int first = 0, int threads = 0, const ROWS& rows = ROWS()) {
  constexpr bool TEAM = !std::is_same<ROWS, OwnRows>::value;
  constexpr int E = 32 / BITS, TBAT = E < 8 ? E : 8, NBAT = E / TBAT, TB = 4 * E;
  constexpr int FPG = 16 / BITS, NG = TBAT / FPG, ESZ = DT == ZC_F32 ? 4 : 2;
  constexpr float QMAX = (float)((1 << BITS) - 1);
  const int n = a.n[sub], blk = unit >> 2, kg = unit & 3;
  const int32_t* idx = a.idx[sub] + (int64_t)b * n;
  const int tid = TEAM ? threadIdx.x - first : threadIdx.x, lane = tid & 63, wave = tid >> 6, nwaves = TEAM ? threads >> 6 : blockDim.x >> 6;
  const bool valid = kPackCpt * tid < a.W;
  const int w = valid ? kPackCpt * tid : 0, h = w / a.D, c = w - h * a.D;
  const char* base = reinterpret_cast<const char*>(a.x) + ((int64_t)b * a.sB + (int64_t)h * a.sH + c) * ESZ;
  auto rel_of = [&](int e) { return value_token<BITS>(blk, kg, e); };

  float x[E][kPackCpt], inv_c[kPackCpt];
  if constexpr (TEAM) {
    rows(x, inv_c);
  } else {
#pragma unroll
    for (int e = 0; e < E; ++e) load4<DT>(base + (int64_t)idx[min(rel_of(e), n - 1)] * a.sL * ESZ, x[e]);
    load4<ZC_F32>(param_row(a, b, sub, 0) + w, inv_c);
  }
  // bookkeeping of the group's tokens by lanes 0 .. E - 1 of the first wave
  const int my_rel = rel_of(lane < E ? lane : 0);
  const bool mine = tid < E && my_rel < n;
  const int64_t o0 = (int64_t)b * a.cap[sub] + a.begin[sub];
  if (mine && a.pos[sub]) (a.pos[sub] + o0)[my_rel] = (int32_t)(idx[my_rel] + a.pos_offset);

  // ranges: (min, -max) of TBAT tokens at a time over the wave, all of the group over the waves
#pragma unroll
  for (int q = 0; q < NBAT; ++q) {
    float mm[TBAT];
#pragma unroll
    for (int t = 0; t < TBAT; ++t) {
      float (&v)[kPackCpt] = x[q * TBAT + t];
#pragma unroll
      for (int i = 0; i < kPackCpt; ++i) v[i] *= inv_c[i];
      mm[t] = swap_min_rows(fminf(fminf(v[0], v[1]), fminf(v[2], v[3])), fminf(fminf(-v[0], -v[1]), fminf(-v[2], -v[3])));
    }
    const float wmin = wave_min_rest<2 * TBAT>(mm);
    if ((lane & 3) == 0) {
      const int vi = value_of_lane<2 * TBAT>(lane);
      red[q][wave][vi < TBAT ? vi : 8 + vi - TBAT] = wmin;
    }
  }
  __syncthreads();
  float si[NBAT], z[NBAT];
#pragma unroll
  for (int q = 0; q < NBAT; ++q) {
    float r = INFINITY;
    for (int v = lane >> 4; v < nwaves; v += 4) r = fminf(r, red[q][v][lane & 15]);
    r = swap_min_rows(r, r);
    r = swap_min_halves(r, r);
    // lanes 0..7 of a row hold the minima, 8..15 the negated maxima: all get both
    const float other = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(r), 0x128, 0xF, 0xF, true));   // row_ror:8
    const float tmin = lane & 8 ? other : r, tmax = -(lane & 8 ? r : other);
    float R = tmax - tmin;
    if (R == 0.f) R = QMAX;                        // max == min: s := 1
    const float y = __builtin_amdgcn_rcpf(R);
    z[q] = -rintf(refined_ratio(tmin, QMAX, R, y));   // tie-exact: a whole row depends on it
    si[q] = QMAX * y;
    if (mine && (lane >> 3) == q) {                // (lane e < E: batch e / 8; with fewer than 8 tokens, batch 0)
      (a.tok_scale[sub] + o0)[my_rel] = R * (1.f / QMAX);
      (a.tok_zero[sub] + o0)[my_rel] = z[q];
    }
  }
  if (!valid) return;                                // (a row is whole heads of 64 or 128 channels: lanes 0..7, read below, stay or go together)
  uint32_t words[kPackCpt] = {};
#pragma unroll
  for (int q = 0; q < NBAT; ++q)
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      float acc[kPackCpt] = {};
#pragma unroll
      for (int f = 0; f < FPG; ++f) {
        const int t = g * FPG + f, e = q * TBAT + t;
        const float st = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(si[q]), t));
        const float zt = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(z[q]), t));
        const float mult = rel_of(e) < n ? (float)(1 << (BITS * f)) : 0.f;
#pragma unroll
        for (int i = 0; i < kPackCpt; ++i) acc[i] = fmaf(__builtin_amdgcn_fmed3f(rintf(x[e][i] * st) + zt, 0.f, QMAX), mult, acc[i]);
      }
#pragma unroll
      for (int i = 0; i < kPackCpt; ++i) words[i] |= (uint32_t)acc[i] << (BITS * (q * TBAT + g * FPG));
    }
  int w1 = TEAM ? tid : threadIdx.x;                              // (the channel again, not held in registers meanwhile)
  asm volatile("" : "+v"(w1));
  w1 *= kPackCpt;
  const int h1 = w1 >> (a.D == 128 ? 7 : 6), c1 = w1 & (a.D - 1);
  const int64_t gblk = a.begin[sub] / TB + blk, nblk = a.cap[sub] / TB;
  uint32_t* dst = reinterpret_cast<uint32_t*>(a.codes[sub]) + ((((int64_t)b * a.H + h1) * nblk + gblk) * 4 + kg) * a.D + c1;
  *reinterpret_cast<uint4*>(dst) = make_uint4(words[0], words[1], words[2], words[3]);
}

constexpr int kPackTokens = 4;         // keys: tokens of a thread

// Keys (ROW layout, channelwise): a thread per 8 channels of kPackTokens tokens.
template <int DT, int BITS>
__device__ inline void pack_keys(const QPArgs& a, int sub, int wg, int b, int first_quad) {
  constexpr int RAW = DT == ZC_F32 ? 2 : 1, ESZ = DT == ZC_F32 ? 4 : 2;
  const int n = a.n[sub];
  const uint32_t i = (uint32_t)wg * blockDim.x + threadIdx.x, quad = i / (uint32_t)a.NV;
  const int t0 = (first_quad + (int)quad) * kPackTokens, w = (int)(i - quad * a.NV) * 8, h = w / a.D, c = w - h * a.D;
  if (t0 >= n) return;
  const int32_t* idx = a.idx[sub] + (int64_t)b * n;
  const char* base = reinterpret_cast<const char*>(a.x) + ((int64_t)b * a.sB + (int64_t)h * a.sH + c) * ESZ;
  int32_t tok[kPackTokens];
#pragma unroll
  for (int t = 0; t < kPackTokens; ++t) tok[t] = idx[min(t0 + t, n - 1)];
  uint4 raw[kPackTokens][RAW];
#pragma unroll
  for (int t = 0; t < kPackTokens; ++t)
#pragma unroll
    for (int r = 0; r < RAW; ++r) raw[t][r] = *reinterpret_cast<const uint4*>(base + (int64_t)tok[t] * a.sL * ESZ + 16 * r);
  float p0[8], p1[8], p2[8];
  load8<ZC_F32>(param_row(a, b, sub, 0), w, p0);
  load8<ZC_F32>(param_row(a, b, sub, 1), w, p1);
  load8<ZC_F32>(param_row(a, b, sub, 2), w, p2);
  if (w == 0 && a.pos[sub]) {
#pragma unroll
    for (int t = 0; t < kPackTokens; ++t)
      if (t0 + t < n) a.pos[sub][(int64_t)b * a.cap[sub] + a.begin[sub] + t0 + t] = (int32_t)(tok[t] + a.pos_offset);
  }
  const int rowb = a.D * BITS / 8;
  uint8_t* dst = a.codes[sub] + (((int64_t)b * a.H + h) * a.cap[sub] + a.begin[sub] + t0) * rowb + c * BITS / 8;
  const int left = min(kPackTokens, n - t0);
#pragma unroll 1
  for (int t = 0; t < left; ++t) {                 // (rolled: the registers move up instead of the code being repeated)
    float v[8];
    widen8<DT>(raw[0], v);
    store_row_codes<DT, BITS>(dst, v, p0, p1, p2);
    dst += rowb;
#pragma unroll
    for (int u = 0; u + 1 < kPackTokens; ++u)
#pragma unroll
      for (int r = 0; r < RAW; ++r) raw[u][r] = raw[u + 1][r];
  }
}

// What a launch of k_pack_kv packs: workgroups of the keys' subsets, then word groups of the values'
// (a count of 0: no such tensor); where it does not start at a subset's first token, from which
// group of kPackTokens tokens or word group on.
struct PackRange { int wgs[4]; int first; };

// grid (sum of r.wgs, B)
template <int DT>
__global__ __launch_bounds__(kPackThreads, 5) void k_pack_kv(QPPair p, PackRange r) {
  __shared__ float red[2][kPackThreads / 64][16];
  const int b = blockIdx.y;
  int wg = blockIdx.x;
  const int nk = r.wgs[0] + r.wgs[1];
  if (wg < nk) {
    const QPArgs& a = p.t[0];
    const int sub = wg >= r.wgs[0] ? 1 : 0;
    if (sub) wg -= r.wgs[0];
    const int bits = a.bits[sub];
    if (bits == 4) pack_keys<DT, 4>(a, sub, wg, b, r.first);
    else if (bits == 2) pack_keys<DT, 2>(a, sub, wg, b, r.first);
    else pack_keys<DT, 8>(a, sub, wg, b, r.first);
  } else {
    const QPArgs& a = p.t[1];
    wg -= nk;
    const int sub = wg >= r.wgs[2] ? 1 : 0;
    if (sub) wg -= r.wgs[2];
    wg += r.first;
    const int bits = a.bits[sub];
    if (bits == 4) pack_values<DT, 4>(a, sub, wg, b, red);
    else if (bits == 2) pack_values<DT, 2>(a, sub, wg, b, red);
    else pack_values<DT, 8>(a, sub, wg, b, red);
  }
}

// ---- short chunks: one launch ------------------------------------------------------------------
// A flushed window, or a short prompt: both launches above are little more than a launch and a few trips to memory each.
// Here a workgroup that needs the statistics of a subset's channels takes them itself, from all of the subset's tokens: up to
// 180 KB out of an L2, which costs less than the second launch and the parameters' way through memory.
//   keys    16 lanes across a row of 128 channels, their rows in registers until the parameters are there
//   values  a team of W / 4 threads per word group, 256 threads or one team a workgroup; its token list comes to LDS in one trip, the rows of
//           its own tokens are requested first, then all of them, 16 bytes a lane, whose largest magnitudes meet in LDS
// Bound by the chain of those trips and, from 100 KB on, by the vector issue of the repeated statistics (16-bit magnitudes are
// compared as integers, two at a time: 1 instruction a value; four teams and 1024 threads a workgroup, which repeat them
// less, took 12.5 us for 64 tokens of 1024 channels).  us per joint call, bf16, as two launches and here: 64 tokens
// of 4 heads of 64 channels 7.9 and 6.5, of 8 heads of 128 8.3 and 6.9, 16 prompts of them 11.5 and 7.5; 100 tokens 8.4 and 7.4, 11.6 and 10.0.
constexpr int kShortTokens = 128;                       // most tokens of a subset
constexpr int kShortLanes = 16, kShortRows = 8;         // keys: lanes across a row, most rows of a thread
struct ShortPlan {
  int key_wgs, value_wgs[2];        // of a subset (0: no such tensor)
  int team, teams;                  // values: threads of a team, teams of a workgroup
  int lanes, rows;                  // values, statistics: lanes across a row, rows at a time
};

template <int DT, int BITS>
__device__ inline void short_keys_codes(const QPArgs& a, int sub, int b, int h, int c, int x, int y, int step, int n,
                                        const uint4 (&raw)[kShortRows][DT == ZC_F32 ? 2 : 1], const float (*prm)[128]) {
  float p0[8], p1[8], p2[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) { p0[i] = prm[0][x * 8 + i]; p1[i] = prm[1][x * 8 + i]; p2[i] = prm[2][x * 8 + i]; }
  const int rowb = a.D * BITS / 8;
  uint8_t* dst = a.codes[sub] + (((int64_t)b * a.H + h) * a.cap[sub] + a.begin[sub] + y) * rowb + c * BITS / 8;
#pragma unroll
  for (int r = 0; r < kShortRows; ++r) {
    if (r * step >= n) break;
    if (r * step + y < n) {
      float v[8];
      widen8<DT>(raw[r], v);
      store_row_codes<DT, BITS>(dst + (int64_t)r * step * rowb, v, p0, p1, p2);
    }
  }
}

template <int DT>
__device__ inline void short_keys(const QPArgs& a, int sub, int grp, int b, float (*red)[2][128], float (*prm)[128]) {
  constexpr int RAW = DT == ZC_F32 ? 2 : 1, ESZ = DT == ZC_F32 ? 4 : 2;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nwaves = blockDim.x >> 6;
  const int x = tid & (kShortLanes - 1), y = tid / kShortLanes, step = blockDim.x / kShortLanes;
  const int n = a.n[sub];
  const int vec = min(grp * kShortLanes + x, a.NV - 1);         // (lanes past the row repeat its last vector)
  const int w = vec * 8, h = w / a.D, c = w % a.D;
  const char* base = reinterpret_cast<const char*>(a.x) + ((int64_t)b * a.sB + (int64_t)h * a.sH + c) * ESZ;
  const int32_t* idx = a.idx[sub] + (int64_t)b * n;
  uint4 raw[kShortRows][RAW];
  float mn[8], mneg[8];                                         // minimum, minimum of -x
#pragma unroll
  for (int i = 0; i < 8; ++i) { mn[i] = INFINITY; mneg[i] = INFINITY; }
  int32_t tok[kShortRows];
#pragma unroll
  for (int r = 0; r < kShortRows; ++r)
    if (r * step < n) tok[r] = idx[min(r * step + y, n - 1)];   // (rows past the end repeat the last one)
#pragma unroll
  for (int r = 0; r < kShortRows; ++r)
    if (r * step < n) {
      const uint4* src = reinterpret_cast<const uint4*>(base + (int64_t)tok[r] * a.sL * ESZ);
#pragma unroll
      for (int q = 0; q < RAW; ++q) raw[r][q] = src[q];
    }
  if (grp == 0 && a.pos[sub] && x == 0) {
#pragma unroll
    for (int r = 0; r < kShortRows; ++r)
      if (r * step + y < n) a.pos[sub][(int64_t)b * a.cap[sub] + a.begin[sub] + r * step + y] = (int32_t)(tok[r] + a.pos_offset);
  }
#pragma unroll
  for (int r = 0; r < kShortRows; ++r)
    if (r * step < n) {
      float v[8];
      widen8<DT>(raw[r], v);
#pragma unroll
      for (int i = 0; i < 8; ++i) { mn[i] = fminf(mn[i], v[i]); mneg[i] = fminf(mneg[i], -v[i]); }
    }
  {                                                             // over the four rows of a wave, as in k_columns
    float u[4];
#pragma unroll
    for (int j = 0; j < 8; ++j) mn[j] = swap_min_halves(mn[j], mneg[j]);
#pragma unroll
    for (int j = 0; j < 4; ++j) u[j] = swap_min_rows(mn[j], mn[j + 4]);
    *reinterpret_cast<float4*>(&red[wave][lane >> 5][(lane & 15) * 8 + 4 * ((lane >> 4) & 1)]) = make_float4(u[0], u[1], u[2], u[3]);
  }
  __syncthreads();
  const int wc = grp * kShortLanes * 8 + tid;
  if (tid < kShortLanes * 8 && wc < a.W) {
    float lo = INFINITY, neg = INFINITY;
    for (int v = 0; v < nwaves; ++v) { lo = fminf(lo, red[v][0][tid]); neg = fminf(neg, red[v][1][tid]); }
    float cs, cz;
    const float3 pr = channel_params(ZC_SCHEME_CHANNEL, n, (float)((1 << a.bits[sub]) - 1), lo, -neg, &cs, &cz);
    const int64_t o = (int64_t)(sub * a.B + b) * a.W + wc;
    a.chan_scale[o] = cs;
    a.chan_zero[o] = cz;
    prm[0][tid] = pr.x; prm[1][tid] = pr.y; prm[2][tid] = pr.z;
  }
  __syncthreads();
  if (grp * kShortLanes + x >= a.NV) return;
  const int bits = a.bits[sub];
  if (bits == 4) short_keys_codes<DT, 4>(a, sub, b, h, c, x, y, step, n, raw, prm);
  else if (bits == 2) short_keys_codes<DT, 2>(a, sub, b, h, c, x, y, step, n, raw, prm);
  else short_keys_codes<DT, 8>(a, sub, b, h, c, x, y, step, n, raw, prm);
}

// The larger magnitude of the 16-bit numbers in each half (bits: a NaN's are above infinity's).
__device__ inline uint32_t larger_magnitudes(uint32_t m, uint32_t x) {
  typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, m), __builtin_bit_cast(u16x2, x & 0x7fff7fffu)));
}

template <int DT, int BITS>
__device__ inline void short_values(const QPArgs& a, int sub, int wg, int b, const ShortPlan& s, uint4* stage, int32_t* sidx,
                                    float (*red)[2][kPackThreads / 64][16]) {
  constexpr int E = 32 / BITS, ESZ = DT == ZC_F32 ? 4 : 2, CPL = 16 / ESZ;      // CPL: channels of a lane in the statistics
  constexpr int BATCH = DT == ZC_F32 ? 8 : 12;        // rows requested at once
  const int n = a.n[sub], tid = threadIdx.x;
  const int32_t* idx = a.idx[sub] + (int64_t)b * n;
  const int64_t row_bytes = a.sL * ESZ;
  const char* xb = reinterpret_cast<const char*>(a.x) + (int64_t)b * a.sB * ESZ;
  const int nwaves = s.team >> 6, team = __builtin_amdgcn_readfirstlane(tid >> 6) / nwaves;
  const int tx = tid - team * s.team, unit = wg * s.teams + team;
  const int w = kPackCpt * tx < a.W ? kPackCpt * tx : 0;
  const char* own_base = xb + ((int64_t)(w / a.D) * a.sH + w % a.D) * ESZ;
  typedef typename std::conditional<DT == ZC_F32, uint4, uint2>::type Row;
  for (int t = tid; t < n; t += blockDim.x) sidx[t] = idx[t];       // (one trip for every look-up below)
  __syncthreads();
  Row own[E];
  if (n > 0) {
#pragma unroll
    for (int e = 0; e < E; ++e) own[e] = *reinterpret_cast<const Row*>(own_base + (int64_t)sidx[min(value_token<BITS>(unit >> 2, unit & 3, e), n - 1)] * row_bytes);
  }
  // statistics: s.rows tokens at a time, a lane per 16 bytes of a row
  const int sy = tid / s.lanes, sw = (tid - sy * s.lanes) * CPL;
  uint4 most = make_uint4(0u, 0u, 0u, 0u);
  float4 lo4 = make_float4(INFINITY, INFINITY, INFINITY, INFINITY), neg4 = lo4;
  if (sy < s.rows) {
    const char* base = xb + ((int64_t)(sw / a.D) * a.sH + sw % a.D) * ESZ;
    for (int t0 = sy; t0 < n; t0 += BATCH * s.rows) {
      uint4 rw[BATCH];
#pragma unroll
      for (int r = 0; r < BATCH; ++r) rw[r] = *reinterpret_cast<const uint4*>(base + (int64_t)sidx[min(t0 + r * s.rows, n - 1)] * row_bytes);
#pragma unroll
      for (int r = 0; r < BATCH; ++r) {
        if constexpr (DT == ZC_F32) {
          const float4 v = __builtin_bit_cast(float4, rw[r]);
          lo4.x = fminf(lo4.x, v.x); lo4.y = fminf(lo4.y, v.y); lo4.z = fminf(lo4.z, v.z); lo4.w = fminf(lo4.w, v.w);
          neg4.x = fminf(neg4.x, -v.x); neg4.y = fminf(neg4.y, -v.y); neg4.z = fminf(neg4.z, -v.z); neg4.w = fminf(neg4.w, -v.w);
        } else {
          most.x = larger_magnitudes(most.x, rw[r].x); most.y = larger_magnitudes(most.y, rw[r].y);
          most.z = larger_magnitudes(most.z, rw[r].z); most.w = larger_magnitudes(most.w, rw[r].w);
        }
      }
    }
    uint4* mine = stage + sy * s.lanes + (sw / CPL);
    if constexpr (DT == ZC_F32) {
      mine[0] = __builtin_bit_cast(uint4, lo4);
      mine[kPackThreads] = __builtin_bit_cast(uint4, neg4);
    } else {
      mine[0] = most;
    }
  }
  __syncthreads();
  float lo[kPackCpt], neg[kPackCpt];
  if constexpr (DT == ZC_F32) {
#pragma unroll
    for (int i = 0; i < kPackCpt; ++i) { lo[i] = INFINITY; neg[i] = INFINITY; }
#pragma unroll 2
    for (int t = 0; t < s.rows; ++t) {
      const float4 l = __builtin_bit_cast(float4, stage[t * s.lanes + w / CPL]), g = __builtin_bit_cast(float4, stage[kPackThreads + t * s.lanes + w / CPL]);
      lo[0] = fminf(lo[0], l.x); lo[1] = fminf(lo[1], l.y); lo[2] = fminf(lo[2], l.z); lo[3] = fminf(lo[3], l.w);
      neg[0] = fminf(neg[0], g.x); neg[1] = fminf(neg[1], g.y); neg[2] = fminf(neg[2], g.z); neg[3] = fminf(neg[3], g.w);
    }
  } else {
    uint2 m = make_uint2(0u, 0u);
#pragma unroll 2
    for (int t = 0; t < s.rows; ++t) {
      const uint2 v = reinterpret_cast<const uint2*>(stage)[(t * s.lanes * CPL + w) / kPackCpt];
      m.x = larger_magnitudes(m.x, v.x); m.y = larger_magnitudes(m.y, v.y);
    }
    const uint32_t mag[kPackCpt] = {m.x & 0xffffu, m.x >> 16, m.y & 0xffffu, m.y >> 16};
    bool nan = false;
#pragma unroll
    for (int i = 0; i < kPackCpt; ++i) {
      neg[i] = -half_bits_to_float<DT>(mag[i]);
      lo[i] = neg[i];
      nan |= mag[i] > (DT == ZC_F16 ? 0x7c00u : 0x7f80u);
    }
    if (nan) {                                       // a NaN is none of the channel's numbers: its statistics again, without it
#pragma unroll
      for (int i = 0; i < kPackCpt; ++i) { lo[i] = INFINITY; neg[i] = INFINITY; }
#pragma unroll 1
      for (int t = 0; t < n; ++t) {
        float v[kPackCpt];
        load4<DT>(own_base + (int64_t)idx[t] * row_bytes, v);
#pragma unroll
        for (int i = 0; i < kPackCpt; ++i) { lo[i] = fminf(lo[i], v[i]); neg[i] = fminf(neg[i], -v[i]); }
      }
    }
  }
  float cs[kPackCpt], inv_c[kPackCpt], cz;
#pragma unroll
  for (int i = 0; i < kPackCpt; ++i) inv_c[i] = channel_params(ZC_SCHEME_CST, n, 0.f, lo[i], -neg[i], &cs[i], &cz).x;
  if (unit == 0 && kPackCpt * tx < a.W) {
    const int64_t o = (int64_t)(sub * a.B + b) * a.W + w;
    typedef float f4a __attribute__((ext_vector_type(4), aligned(4)));         // (the validation does not hold these arrays to 16 bytes)
    *reinterpret_cast<f4a*>(a.chan_scale + o) = f4a{cs[0], cs[1], cs[2], cs[3]};
    *reinterpret_cast<f4a*>(a.chan_zero + o) = f4a{0.f, 0.f, 0.f, 0.f};
  }
  if (n == 0) return;
  const auto rows = [&](float (&x)[E][kPackCpt], float (&inv)[kPackCpt]) {
#pragma unroll
    for (int e = 0; e < E; ++e) load4<DT>(&own[e], x[e]);
#pragma unroll
    for (int i = 0; i < kPackCpt; ++i) inv[i] = inv_c[i];
  };
  pack_values<DT, BITS>(a, sub, unit, b, red[team], team * s.team, s.team, rows);
}

// grid (2 s.key_wgs + s.value_wgs, B); s.team * s.teams threads
template <int DT>
__global__ __launch_bounds__(kPackThreads) void k_short_kv(QPPair p, ShortPlan s) {
  __shared__ __align__(16) uint4 stage[2 * kPackThreads];
  __shared__ float red[4][2][kPackThreads / 64][16];
  __shared__ __align__(16) float prm[3][128];
  __shared__ int32_t sidx[kShortTokens];
  const int b = blockIdx.y;
  int wg = blockIdx.x;
  if (b == 0 && wg == 0 && threadIdx.x < 2) {
    const QPArgs& a = p.t[threadIdx.x];                 // (of one tensor: both are it)
    a.chunk_row[0] = a.begin[0]; a.chunk_row[1] = a.n[0];
    a.chunk_row[2] = a.begin[1]; a.chunk_row[3] = a.n[1];
  }
  if (wg < 2 * s.key_wgs) {
    const int sub = wg >= s.key_wgs ? 1 : 0;
    short_keys<DT>(p.t[0], sub, wg - sub * s.key_wgs, b, reinterpret_cast<float (*)[2][128]>(stage), prm);
  } else {
    const QPArgs& a = p.t[1];
    wg -= 2 * s.key_wgs;
    const int sub = wg >= s.value_wgs[0] ? 1 : 0;
    if (sub) wg -= s.value_wgs[0];
    const int bits = a.bits[sub];
    if (bits == 4) short_values<DT, 4>(a, sub, wg, b, s, stage, sidx, red);
    else if (bits == 2) short_values<DT, 2>(a, sub, wg, b, s, stage, sidx, red);
    else short_values<DT, 8>(a, sub, wg, b, s, stage, sidx, red);
  }
}

// (what k_pack_kv takes does not come here, see pack_route: no instances for channelwise ROW tensors and
// narrow channel-separable TGROUP ones)
template <int DT, int LAYOUT, int MAXT>
static int launch_qp_l(const QPArgs& a, bool tokwise, dim3 grid, dim3 block, hipStream_t st) {
  if (!tokwise) {
    if constexpr (LAYOUT == ZC_LAYOUT_TGROUP && MAXT == 256) {
      hipLaunchKernelGGL((k_quant_pack<DT, LAYOUT, false, false, MAXT>), grid, block, 0, st, a);
      return ZC_OK;
    }
  } else if (a.scheme == ZC_SCHEME_TOKEN) {
    hipLaunchKernelGGL((k_quant_pack<DT, LAYOUT, true, true, MAXT>), grid, block, 0, st, a);
    return ZC_OK;
  } else if constexpr (LAYOUT == ZC_LAYOUT_ROW || MAXT > 256) {
    hipLaunchKernelGGL((k_quant_pack<DT, LAYOUT, true, false, MAXT>), grid, block, 0, st, a);
    return ZC_OK;
  }
  return ZC_ERR_UNSUPPORTED;
}
template <int DT, int MAXT>
static int launch_qp_t(const QPArgs& a, int layout, bool tokwise, dim3 grid, dim3 block, hipStream_t st) {
  if (layout == ZC_LAYOUT_ROW) return launch_qp_l<DT, ZC_LAYOUT_ROW, MAXT>(a, tokwise, grid, block, st);
  return launch_qp_l<DT, ZC_LAYOUT_TGROUP, MAXT>(a, tokwise, grid, block, st);
}
template <int DT>
static int launch_qp(const QPArgs& a, int layout, bool tokwise, dim3 grid, dim3 block, hipStream_t st) {
  if (block.x <= 256) return launch_qp_t<DT, 256>(a, layout, tokwise, grid, block, st);
  if (block.x <= 768) return launch_qp_t<DT, 768>(a, layout, tokwise, grid, block, st);
  return launch_qp_t<DT, 1024>(a, layout, tokwise, grid, block, st);
}

}  // namespace zc

using namespace zc;

// Token ranges per subset of the split column sweep: enough for three workgroups a CU, and at
// least kSplitRows rows a thread.  (n: tokens of the longer subset; a call for two tensors
// cuts less.)
static int64_t col_splits(int64_t B, int64_t NV, int64_t n, int tensors) {
  const int64_t by_chip = 768 / (ceil_div64(NV, kSplitLanes) * 2 * tensors * B), by_rows = n * kSplitLanes / (kSplitThreads * kSplitRows);
  const int64_t s = by_chip < by_rows ? by_chip : by_rows;
  return s < 1 ? 1 : s;
}

// [B, 2, W] parameters, and the minima of the split column sweep.
extern "C" size_t zc_quantize_pack_workspace(int64_t B, int64_t H, int64_t L, int64_t D) {
  if (B <= 0 || H <= 0 || D <= 0 || L < 0) return 0;
  const int64_t W = H * D, split = col_splits(B, W / 8, L, 1);
  return (size_t)align_up64(B * 2 * W * 4 * (int64_t)sizeof(float), 256) + (split > 1 ? (size_t)B * 2 * split * W * sizeof(float2) : 0);
}

// Validation and kernel arguments of one tensor's compression call.
static int qp_prepare(const zc_tensor4* x, const int32_t* salient_idx, int64_t k, const int32_t* regular_idx, int64_t n_reg,
                      int64_t pos_offset, const zc_packed* out, void* ws, size_t ws_bytes, QPArgs& a) {
  int rc = zc_validate_tensor(x);
  if (rc) return rc;
  rc = zc_validate_packed(out, true);
  if (rc) return rc;
  if (k < 0 || n_reg < 0 || k > x->L || n_reg > x->L || k + n_reg > x->L) return ZC_ERR_INVALID_ARG;
  if ((k > 0 && !salient_idx) || (n_reg > 0 && !regular_idx)) return ZC_ERR_INVALID_ARG;
  if (x->B != out->B || x->H != out->H || x->D != out->D) return ZC_ERR_INVALID_ARG;
  const int64_t W = x->H * x->D;
  if (W / 8 > kVPT * 1024) return ZC_ERR_UNSUPPORTED;
  if (x->B > 65535) return ZC_ERR_UNSUPPORTED;
  if (out->n_chunks >= out->max_chunks) return ZC_ERR_CAPACITY;
  const int64_t end_hi = align_up64(out->n_hi + k, ZC_SLOT_ALIGN);
  const int64_t end_lo = align_up64(out->n_lo + n_reg, ZC_SLOT_ALIGN);
  if (end_hi > out->cap_hi || end_lo > out->cap_lo) return ZC_ERR_CAPACITY;
  const size_t need = zc_quantize_pack_workspace(x->B, x->H, k + n_reg, x->D);
  if (!ws || ws_bytes < need || (reinterpret_cast<uintptr_t>(ws) & 15)) return ZC_ERR_WORKSPACE;

  a.x = x->ptr; a.sB = x->sB; a.sH = x->sH; a.sL = x->sL;
  a.B = (int)x->B; a.H = (int)x->H; a.D = (int)x->D; a.W = (int)W; a.NV = (int)(W / 8);
  a.idx[0] = salient_idx; a.idx[1] = regular_idx;
  a.n[0] = (int)k; a.n[1] = (int)n_reg;
  a.begin[0] = (int)out->n_hi; a.begin[1] = (int)out->n_lo;
  a.bits[0] = out->bits_hi; a.bits[1] = out->bits_lo;
  a.cap[0] = out->cap_hi; a.cap[1] = out->cap_lo;
  a.codes[0] = out->codes_hi; a.codes[1] = out->codes_lo;
  a.tok_scale[0] = out->tok_scale_hi; a.tok_zero[0] = out->tok_zero_hi;
  a.tok_scale[1] = out->tok_scale_lo; a.tok_zero[1] = out->tok_zero_lo;
  a.pos[0] = out->pos_hi; a.pos[1] = out->pos_lo;
  const int64_t chunk_off = (int64_t)out->n_chunks * 2 * x->B * W;
  a.chan_scale = out->chan_scale + chunk_off;
  a.chan_zero = out->chan_zero + chunk_off;
  a.params = reinterpret_cast<float*>(ws);
  a.chunk_row = out->chunk_table + 4 * out->n_chunks;
  a.pos_offset = pos_offset;
  a.scheme = out->scheme;
  a.resident = 0;
  // word groups of 32 / bits tokens; a TGROUP block holds 4 of them
  a.units[0] = (int)ceil_div64(k, 4 * (32 / out->bits_hi)) * 4;
  a.units[1] = (int)ceil_div64(n_reg, 4 * (32 / out->bits_lo)) * 4;
  // word groups per workgroup: one while the launch is small (latency), up to a whole
  // block of consecutive slots when there is enough work to fill the chip anyway
  {
    const int64_t total = (int64_t)(a.units[0] + a.units[1]) * x->B;
    int upw = 1;
    while (upw < 4 && total / (2 * upw) >= 1024) upw *= 2;
    a.upw = upw;
    a.wgs[0] = a.units[0] / upw;
    a.wgs[1] = a.units[1] / upw;
  }
  return ZC_OK;
}

// Shape of the column sweep over `tensors` tensors of one call (same sizes and subsets): lanes
// across a row, threads of a workgroup, and which tensors stay resident.
// The widest rows that leave a workgroup per CU; narrower ones where a resident subset only
// then fits the registers.  Keys are resident wherever they fit - except in a call for both
// tensors with too few workgroups to hide the packing behind each other's loads, where one
// packing launch serves both (one prompt of 4096 tokens, 8 heads: 26.1 against 27.5 us; of 16-bit
// tensors also at a workgroup per CU: 4 such prompts 34.9 against 39.2, 16 of 1000 tokens 31.4 and
// 35.5, but 5 of 4096 43.1 and 41.0; 16 of 1000 tokens of 4 heads in fp32 28.3 and 27.6); and
// except for wide 16-bit rows of both that fit in slices of 16 channels only, a quarter of a
// cache line (12000 tokens of 32 heads of 128 channels: 105 against 121 us; of 64: 216 and 279) -
// above 512 channels where that also takes workgroups of 1024 threads (8192 tokens of 8 heads, 8
// prompts: 134 against 146 us; of 16 heads, 2 prompts: 73 and 95; but of 2 heads, 8 prompts, 61 and
// 50, and 4096 tokens of 8 heads, 8 prompts, in workgroups of 512: 69 and 66).
constexpr int64_t kCUs = 256;
struct ColPlan { int threads, split; };
static ColPlan col_plan(QPArgs* a, const zc_packed* const* out, int tensors, int dtype, bool joint_pack) {
  const int64_t n = a[0].n[0] > a[0].n[1] ? a[0].n[0] : a[0].n[1], rows = kColRows(dtype);
  const auto wgs = [&](int vl) { return ceil_div64(a[0].NV, vl) * 2 * a[0].B; };      // of one tensor
  int vl = 16;
  while (vl > 2 && wgs(vl) * tensors < 256) vl /= 2;
  int threads = wgs(vl) * tensors < 256 ? 1024 : 512;
  int v = vl, th = threads;
  while (v > 2 && n > rows * th / v) v /= 2;
  if (n > rows * th / v) th = 1024;
  const bool strips = tensors == 2 && dtype != ZC_F32 && v == 2 && a[0].NV > (th == 1024 ? 64 : 256);
  const bool few_wgs = dtype == ZC_F32 ? wgs(v) < kCUs : wgs(v) <= kCUs;
  const bool fits = n <= rows * th / v && !(joint_pack && few_wgs) && !strips;
  bool any = false;
  for (int t = 0; t < tensors; ++t) {
    const auto near = [&](int sub) { return a[t].H * a[t].cap[sub] * a[t].D * a[t].bits[sub] / 8 < kPartBytes; };
    a[t].resident = fits && out[t]->scheme == ZC_SCHEME_CHANNEL && out[t]->layout == ZC_LAYOUT_ROW && near(0) && near(1);
    any |= a[t].resident != 0;
  }
  for (int t = 0; t < tensors; ++t) a[t].vl = any ? v : vl;
  // Few tokens: workgroups of 256 threads, so that no waves are started for rows that are not there
  // (keys and values of 8 heads in bf16, 16 tokens of 64 prompts: 30.8 -> 22.6 us; 100 tokens of one
  // prompt: 13.0 -> 12.6).
  const auto few = [&](int l) { return n * l <= (wgs(l) * tensors >= 1024 ? 1024 : 512); };
  if (any) return {few(v) ? 256 : th, 1};
  if (few(vl)) return {256, 1};
  // One batch of rows a thread instead of two, where a workgroup has its CU to itself (keys and values of 4096 tokens of 8
  // heads, bf16 15.1 -> 14.8 us, fp32 20.7 -> 19.5; 2400 of 16 heads 15.6 -> 15.1).
  if (threads == 512 && wgs(vl) * tensors <= kCUs && n * vl > kStatBatch * 512 && n * vl <= kStatBatch * 1024) threads = 1024;
  // Few channels over many tokens leave most of the chip idle, each workgroup with a long chain
  // of rows: token ranges and one more launch pay where a thread would have more than 16 rows
  // (8 of fp32), or 32 where the workgroups fill the chip as they are.  131072 tokens of one head of 128
  // channels in bf16: 137 us whole, 55 in ranges; of 8 heads 203 and 130; 12000 tokens of 4 heads
  // in fp32: 29.5 and 23.7, but 3000 tokens of 32 heads (14 rows, 256 workgroups) 30.0 and 32.9.
  const int64_t most = wgs(vl) * tensors >= 256 ? 32 : dtype == ZC_F32 ? 8 : 16;
  if (n * vl > most * threads) {
    const int64_t split = col_splits(a[0].B, a[0].NV, n, tensors);
    if (split > 1) {
      for (int t = 0; t < tensors; ++t) a[t].vl = kSplitLanes;
      return {kSplitThreads, (int)split};
    }
  }
  return {threads, 1};
}

template <int DT>
static void launch_columns(const QPPair& p, int tensors, ColPlan c, hipStream_t st) {
  // (a grid counts the threads of a dimension in 32 bits: the batch has one of its own)
  const dim3 grid((unsigned)(ceil_div64(p.t[0].NV, p.t[0].vl) * c.split * 2 * tensors), (unsigned)p.t[0].B);
  if (c.split > 1) hipLaunchKernelGGL((k_columns<DT, kSplitThreads, true>), grid, dim3(kSplitThreads), 0, st, p, tensors, c.split);
  else if (c.threads == 256) hipLaunchKernelGGL((k_columns<DT, 256>), grid, dim3(256), 0, st, p, tensors, c.split);
  else if (c.threads == 512) hipLaunchKernelGGL((k_columns<DT, 512>), grid, dim3(512), 0, st, p, tensors, c.split);
  else hipLaunchKernelGGL((k_columns<DT, 1024>), grid, dim3(1024), 0, st, p, tensors, c.split);
}
static int qp_launch_columns(QPPair& p, const zc_packed* const* out, int tensors, int dtype, bool joint_pack, hipStream_t st) {
  bool stats = false;                  // (plain tokenwise: no channel statistics)
  for (int t = 0; t < tensors; ++t) stats |= p.t[t].scheme != ZC_SCHEME_TOKEN;
  ColPlan c = {0, 1};
  if (stats) {
    c = col_plan(p.t, out, tensors, dtype, joint_pack);
    if (dtype == ZC_F32) launch_columns<ZC_F32>(p, tensors, c, st);
    else if (dtype == ZC_F16) launch_columns<ZC_F16>(p, tensors, c, st);
    else launch_columns<ZC_BF16>(p, tensors, c, st);
    ZC_LAUNCH_CHECK();
  }
  if (!stats || c.split > 1) {
    hipLaunchKernelGGL(k_column_params, dim3((unsigned)ceil_div64(p.t[0].W, 256), (unsigned)(2 * tensors), (unsigned)p.t[0].B), dim3(256), 0, st, p, c.split);
    ZC_LAUNCH_CHECK();
  }
  return ZC_OK;
}

// Host bookkeeping of an appended chunk.
static void qp_commit(zc_packed* out, int64_t k, int64_t n_reg) {
  int32_t* row = out->chunk_table_host + 4 * out->n_chunks;
  row[0] = (int32_t)out->n_hi; row[1] = (int32_t)k; row[2] = (int32_t)out->n_lo; row[3] = (int32_t)n_reg;
  out->n_hi = align_up64(out->n_hi + k, ZC_SLOT_ALIGN);
  out->n_lo = align_up64(out->n_lo + n_reg, ZC_SLOT_ALIGN);
  out->n_chunks += 1;
}

static int qp_launch_pack(const QPArgs& a, int dtype, int layout, hipStream_t st) {
  if (a.units[0] + a.units[1] == 0) return ZC_OK;
  const bool tokwise = a.scheme != ZC_SCHEME_CHANNEL;
  int TXq = (int)align_up64(ceil_div64(a.NV, kVPT), 64);
  int zchunks = 1;
  if (!tokwise && TXq > 256) { zchunks = (int)ceil_div64(a.NV, 256); TXq = 256; }
  dim3 grid((unsigned)(a.wgs[0] + a.wgs[1]), (unsigned)a.B, (unsigned)zchunks), block(TXq);
  int rc;
  if (dtype == ZC_F32) rc = launch_qp<ZC_F32>(a, layout, tokwise, grid, block, st);
  else if (dtype == ZC_F16) rc = launch_qp<ZC_F16>(a, layout, tokwise, grid, block, st);
  else rc = launch_qp<ZC_BF16>(a, layout, tokwise, grid, block, st);
  if (rc) return rc;
  ZC_LAUNCH_CHECK();
  return ZC_OK;
}

// The kernel that packs a tensor which does not stay resident, whichever place it has in a call:
// k_pack_kv takes keys (channelwise, ROW layout) of any width and values (channel-separable,
// TGROUP layout) whose rows fit a workgroup, k_quant_pack the others.
enum class PackRoute { Keys, Values, General };
static PackRoute pack_route(const QPArgs& a, int layout) {
  if (a.scheme == ZC_SCHEME_CHANNEL && layout == ZC_LAYOUT_ROW) return PackRoute::Keys;
  if (a.scheme == ZC_SCHEME_CST && layout == ZC_LAYOUT_TGROUP && a.W <= kPackCpt * kPackThreads) return PackRoute::Values;
  return PackRoute::General;
}
// Keys in the first place and values in the second share a launch.
static bool pack_joint(const QPPair& p, const zc_packed* const* out, int tensors) {
  return tensors == 2 && pack_route(p.t[0], out[0]->layout) == PackRoute::Keys && pack_route(p.t[1], out[1]->layout) == PackRoute::Values;
}
static int launch_pack_kv(const QPPair& p, bool keys, bool values, int dtype, hipStream_t st) {
  const int threads = values ? (int)align_up64(p.t[1].W / kPackCpt, 64) : 256;
  const auto launch = [&](const PackRange& r) -> int {
    const dim3 grid((unsigned)(r.wgs[0] + r.wgs[1] + r.wgs[2] + r.wgs[3]), (unsigned)p.t[0].B), block(threads);
    if (dtype == ZC_F32) hipLaunchKernelGGL(k_pack_kv<ZC_F32>, grid, block, 0, st, p, r);
    else if (dtype == ZC_F16) hipLaunchKernelGGL(k_pack_kv<ZC_F16>, grid, block, 0, st, p, r);
    else hipLaunchKernelGGL(k_pack_kv<ZC_BF16>, grid, block, 0, st, p, r);
    ZC_LAUNCH_CHECK();
    return ZC_OK;
  };
  int64_t wgs[4] = {0, 0, 0, 0}, total = 0;
  for (int sub = 0; sub < 2; ++sub) {
    if (keys) wgs[sub] = ceil_div64(ceil_div64(p.t[0].n[sub], kPackTokens) * p.t[0].NV, threads);
    if (values) wgs[2 + sub] = p.t[1].units[sub];
  }
  for (int64_t n : wgs) total += n;
  if (total == 0) return ZC_OK;
  const int64_t most = 0xffffffffll / threads;             // (a grid counts the threads of a dimension in 32 bits)
  if (total <= most) return launch({{(int)wgs[0], (int)wgs[1], (int)wgs[2], (int)wgs[3]}, 0});
  // more than that: a subset at a time, in pieces of whole groups of tokens
  const int64_t piece = most / p.t[0].NV * p.t[0].NV;
  for (int seg = 0; seg < 4; ++seg)
    for (int64_t done = 0; done < wgs[seg]; done += piece) {
      PackRange r = {{0, 0, 0, 0}, (int)(seg < 2 ? done * threads / p.t[0].NV : done)};
      r.wgs[seg] = (int)(wgs[seg] - done < piece ? wgs[seg] - done : piece);
      const int rc = launch(r);
      if (rc) return rc;
    }
  return ZC_OK;
}

// Whether a call's tensors are short enough for k_short_kv, and its shape.  Of one prompt the line lies where reading the longer
// subset once a workgroup costs as much as the launch.  us as two launches and as one, bf16: 8 heads of 128
// channels, 70 tokens in it (143 KB) 8.4 and 7.4, 90 (184 KB) 8.5 and 7.9, 105 (215 KB) 8.4 and 8.5; fp32, 12 heads of 64, 70 (215 KB) 8.3 and 8.7, and,
// with 58 rows a thread (178 KB), 8.2 and 8.3: no more than 48.
// Of many prompts it lies in what all workgroups of values read together: the two launches read every byte twice, here it comes out of an L2
// once for each word group of its subset (divided by the teams).  That costs nothing up to some 26 MB of values alone and 36 of
// both tensors; beyond, up to as many readings of a byte as the second launch and its start are worth.  us as two launches and as one, both
// tensors: 8 heads of 128 channels, bf16, 45 tokens in each subset, 16 and 128 prompts (18 and 142 MB, 6 readings) 9.6 and 7.4, 33.8 and 31.7; 90, 16 prompts
// (59 MB, 10) 12.7 and 16.3; 4 heads, fp16, 90 and 22, 64 (26 MB, 3.6) 19.5 and 11.6; fp32, 8 heads, 45 each, 64 (94 MB, 8) 22.4 and 32.3; 15 each, 256 (126 MB, 4) 45.7 and
// 38.2; 11 and 45, 256 (4) 54.3 and 74.0; values alone: 8 heads, bf16, 90 each, 256 prompts (943 MB, 10) 57.4 and 120; 4 heads of 64, 120 and 30, 256 (35 MB, 1.8) 19.1 and 11.9; 8 heads of
// 64, fp32, 60 each, 256 (94 MB, 3) 28.3 and 37.8.  Joint calls of more than 1024 channels gain nothing from half a workgroup a CU on: 16 heads of 128, 30 and 7, 32 prompts 17.1 and 19.1.
// Keys alone are one launch either way (k_columns starts more workgroups, and in fp32 holds more in flight): bf16, 4 heads of 64, 60 tokens, one prompt
// 1.05 times faster here, 120 tokens of 64 prompts (256 workgroups) 1.06 slower, of 256 prompts 1.26 faster; fp32, 30 tokens 1.05 faster, 60 1.13
// slower, 30 of 256 prompts (1024) 1.11 slower.
constexpr int64_t kShortBytes = 180 * 1024, kShortReads = 48;
static bool short_plan(const QPPair& p, const zc_packed* const* out, int tensors, int dtype, ShortPlan& s) {
  const QPArgs& a = p.t[0];
  const PackRoute route = pack_route(a, out[0]->layout);
  if (tensors == 2 ? !pack_joint(p, out, 2) : route == PackRoute::General) return false;
  const bool keys = route == PackRoute::Keys, values = tensors == 2 || !keys;
  const int64_t n = a.n[0] > a.n[1] ? a.n[0] : a.n[1], row_bytes = (int64_t)a.W * (dtype == ZC_F32 ? 4 : 2);
  s.key_wgs = keys ? (int)ceil_div64(a.NV, kShortLanes) : 0;
  if (n > kShortTokens) return false;
  if (values && n * row_bytes > kShortBytes) return false;
  if (!values) {
    const int64_t wgs = 2 * s.key_wgs * (int64_t)a.B;
    if (dtype == ZC_F32 ? n > 32 || wgs > 512 : n > 60 && wgs < (n > 96 ? 384 : n > 72 ? 256 : 128)) return false;
  }
  s.team = values ? (int)align_up64(a.W / kPackCpt, 64) : 256;
  s.teams = s.team <= 64 ? 4 : s.team <= 128 ? 2 : 1;
  s.lanes = (int)(row_bytes / 16);
  s.rows = values ? s.team * s.teams / s.lanes : 0;
  if ((keys && n > kShortRows * (s.team * s.teams / kShortLanes)) || (values && n > kShortReads * s.rows)) return false;
  for (int sub = 0; sub < 2; ++sub) {
    const int wgs = (int)ceil_div64(a.units[sub], s.teams);
    s.value_wgs[sub] = !values ? 0 : wgs > 0 ? wgs : 1;                // (an empty subset's parameters are written too)
  }
  if (values) {
    const int64_t row = row_bytes * a.B, read = row * ((int64_t)s.value_wgs[0] * a.n[0] + (int64_t)s.value_wgs[1] * a.n[1]), all = row * (a.n[0] + a.n[1]);
    const int64_t again = keys ? (dtype == ZC_F32 ? 11 : 22) : 9;      // readings of a byte, in quarters
    if (read > (keys ? 36 : 26) * 1000000 && 4 * read > again * all) return false;
    if (keys && a.W > 1024 && (s.value_wgs[0] + s.value_wgs[1]) * (int64_t)a.B >= 128) return false;
  }
  return true;
}
static int launch_short(const QPPair& p, int dtype, const ShortPlan& s, hipStream_t st) {
  const dim3 grid((unsigned)(2 * s.key_wgs + s.value_wgs[0] + s.value_wgs[1]), (unsigned)p.t[0].B), block((unsigned)(s.team * s.teams));
  if (dtype == ZC_F32) hipLaunchKernelGGL(k_short_kv<ZC_F32>, grid, block, 0, st, p, s);
  else if (dtype == ZC_F16) hipLaunchKernelGGL(k_short_kv<ZC_F16>, grid, block, 0, st, p, s);
  else hipLaunchKernelGGL(k_short_kv<ZC_BF16>, grid, block, 0, st, p, s);
  ZC_LAUNCH_CHECK();
  return ZC_OK;
}

// Codes of what the column sweep has not packed.
static int qp_launch_packs(const QPPair& p, const zc_packed* const* out, int tensors, int dtype, hipStream_t st) {
  if (pack_joint(p, out, tensors)) return launch_pack_kv(p, !p.t[0].resident, true, dtype, st);
  for (int t = 0; t < tensors; ++t) {
    const QPArgs& a = p.t[t];
    if (a.resident) continue;
    const PackRoute route = pack_route(a, out[t]->layout);
    const int rc = route == PackRoute::General ? qp_launch_pack(a, dtype, out[t]->layout, st)
                                               : launch_pack_kv({{a, a}}, route == PackRoute::Keys, route == PackRoute::Values, dtype, st);
    if (rc) return rc;
  }
  return ZC_OK;
}

// Parameters and codes of a call's tensors.
static int qp_launch(QPPair& p, const zc_packed* const* out, int tensors, int dtype, hipStream_t st) {
  if (tensors == 1) p.t[1] = p.t[0];
  ShortPlan s;
  if (short_plan(p, out, tensors, dtype, s)) return launch_short(p, dtype, s, st);
  // statistics and parameters of both and codes of resident keys, then what is not packed yet
  const int rc = qp_launch_columns(p, out, tensors, dtype, tensors == 2 && pack_joint(p, out, 2), st);
  return rc ? rc : qp_launch_packs(p, out, tensors, dtype, st);
}

extern "C" int zc_quantize_pack(const zc_tensor4* x, const int32_t* salient_idx, int64_t k,
                                const int32_t* regular_idx, int64_t n_reg, int64_t pos_offset,
                                zc_packed* out, void* ws, size_t ws_bytes, void* stream) {
  QPPair p;
  QPArgs& a = p.t[0];
  int rc = qp_prepare(x, salient_idx, k, regular_idx, n_reg, pos_offset, out, ws, ws_bytes, a);
  if (rc) return rc;
  hipStream_t st = (hipStream_t)stream;
  const zc_packed* const outs[1] = {out};
  rc = qp_launch(p, outs, 1, x->dtype, st);
  if (rc) return rc;
  qp_commit(out, k, n_reg);
  return ZC_OK;
}

extern "C" size_t zc_quantize_pack_kv_workspace(int64_t B, int64_t H, int64_t L, int64_t D) {
  return 2 * (size_t)align_up64((int64_t)zc_quantize_pack_workspace(B, H, L, D), 256);
}

extern "C" int zc_quantize_pack_kv(const zc_tensor4* xk, const zc_tensor4* xv, const int32_t* salient_idx, int64_t k,
                                   const int32_t* regular_idx, int64_t n_reg, int64_t pos_offset,
                                   zc_packed* outK, zc_packed* outV, void* ws, size_t ws_bytes, void* stream) {
  if (!xk || !xv || !outK || !outV || outK == outV) return ZC_ERR_INVALID_ARG;
  if (xk->dtype != xv->dtype || xk->B != xv->B || xk->H != xv->H || xk->D != xv->D || xk->L != xv->L) return ZC_ERR_INVALID_ARG;
  const size_t half = (size_t)align_up64((int64_t)zc_quantize_pack_workspace(xk->B, xk->H, k + n_reg, xk->D), 256);
  if (!ws || ws_bytes < 2 * half || (reinterpret_cast<uintptr_t>(ws) & 15)) return ZC_ERR_WORKSPACE;
  QPPair p;
  int rc = qp_prepare(xk, salient_idx, k, regular_idx, n_reg, pos_offset, outK, ws, half, p.t[0]);
  if (rc) return rc;
  rc = qp_prepare(xv, salient_idx, k, regular_idx, n_reg, pos_offset, outV, reinterpret_cast<uint8_t*>(ws) + half, half, p.t[1]);
  if (rc) return rc;
  hipStream_t st = (hipStream_t)stream;
  const int dt = xk->dtype;
  const zc_packed* const outs[2] = {outK, outV};
  rc = qp_launch(p, outs, 2, dt, st);
  if (rc) return rc;
  qp_commit(outK, k, n_reg);
  qp_commit(outV, k, n_reg);
  return ZC_OK;
}
