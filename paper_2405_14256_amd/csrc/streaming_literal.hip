// The pieces Algorithm 3 needs when its re-compression branch is taken at its word
// (every 100 steps everything but the newest 100 tokens is compressed again, ranked by the
// attention rows of the window's probe steps):
//   zc_decode_probs      the attention row a of one decode step over the whole cache
//                        (Eq. 4's probabilities), in token order, for the probe steps;
//   zc_rows_saliency     Eq. 8 on such explicit rows: column sums over the rows that see a
//                        token, divided by their number, mean over heads;
//   zc_dequantize_cache  the compressed tokens as they now are (Eq. 5's x_hat), scattered
//                        to their token positions in a full-precision tensor - the input
//                        of the next compression.
// None of them is on the per-step hot path (a probe step is one step in ten, a
// re-compression one in a hundred), but each is bound by memory or latency like the step itself.
#include <type_traits>

#include "zc_common.hpp"

namespace zc {

// ---- zc_decode_probs -----------------------------------------------------------------------
constexpr int kProbSegs = 64;     // segments (chunk x subset, and the tail) one launch takes
constexpr int kProbTile = 16;     // cache slots (or tail tokens) of one matrix-core tile
constexpr int kTailSub = 2;       // `sub` of the tail's segment

struct ProbsSeg {
  int begin, len;           // slots (tail: tokens)
  int first_block;          // this segment's first workgroup
  int chunk, sub;
};
struct ProbsArgs {
  const void* q;
  int64_t q_sB, q_sH;
  int B, Hq, Hkv, G, D;
  const uint8_t* kc[2];
  const float* k_ts[2];
  const float* k_tz[2];
  const int32_t* pos[2];
  const float* k_cs;
  const float* k_cz;
  int k_tok;
  int64_t cap[2];
  int bits[2];
  const void* tail_k;
  int64_t tk_sB, tk_sH, tk_sL;
  int tail_pos0;
  float scale_log2;
  const float* lse;         // [B, Hq] natural log
  float* probs;             // [B, Hq, N]
  int N;
  int tpw, tail_tpw;        // units per wave (of one tile: 1), the tail's tiles per wave
  int n_segs;
  ProbsSeg seg[kProbSegs];
};

typedef float f4 __attribute__((ext_vector_type(4)));
// Four elements of a parameter or position array, which the validation does not hold to 16
// bytes (the instruction is the same, alignment to 4 is what it needs).
typedef float f4a __attribute__((ext_vector_type(4), aligned(4)));
typedef int i4a __attribute__((ext_vector_type(4), aligned(4)));
__device__ inline float4 load4(const float* p) { const f4a t = *reinterpret_cast<const f4a*>(p); return make_float4(t.x, t.y, t.z, t.w); }
__device__ inline int4 load4(const int32_t* p) { const i4a t = *reinterpret_cast<const i4a*>(p); return make_int4(t.x, t.y, t.z, t.w); }
__device__ inline void load8(const float* p, float (&v)[8]) {
  const float4 a = load4(p), b = load4(p + 4);
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
typedef uint32_t u4 __attribute__((ext_vector_type(4)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));

// Bound: vector-instruction issue (the unpacking), below a few thousand tokens latency.
// Logits on the matrix cores: D[slot][column] = sum_c code[slot][c] q'[column][c] with
// v_mfma_f32_16x16x32_f16.  A code enters exactly at every width, less half the range (what cancels
// against the zero points stays out of the accumulators; the sums of q' take that bias off the
// zero points: 8-bit keys with token scales 8.3e-6 -> 1.3e-6 relative error of a probability, 6.7e-6
// on the vector ALUs); q' enters as fp16 value and
// residual (scaled by 2^11), two columns per head, after a power of two per head has brought its
// largest element to [1, 2): 22 bits, whatever the scale of the query.  A lane's quarter row
// (channels kg D / 4 ...) is contiguous in the ROW layout and goes from memory straight to its
// registers.  The tail's few tokens take v_mfma_f32_16x16x4_f32 instead (no rounding of K).
// Tiles go two at a time: what a tile's 16 slots take after the products (the logit, its exponential, the store) only the
// lanes of the value columns need, so a second tile's slots take the residual columns' lanes there, and positions and
// parameters are requested once for both.  Measured, us per call: on the vector ALUs with q' in LDS / with fp32 matrix
// instructions for the packed tokens too / a tile at a time / now:
//   4096 tokens, 8 KV heads of 4 query heads      13.6 /   8.5 /  6.7 /  5.6
//   8000 tokens, the same, batch 8                   - /     - / 22.9 / 17.3
//   2000 tokens, 40 KV heads of 1, batch 16      103.3 / 124.1 / 48.7 / 33.9
constexpr float kProbLo = 2048.f;

// Codes of a quarter row (NK = D / 4 channels) as fp16 operand registers, two codes each: register
// i of word w holds its codes code_slot<BITS>(i) and code_slot<BITS>(i) + (half-word distance).
// 1024 + code is the code under the exponent of 1024; one packed subtraction leaves code - bias.
template <int BITS> constexpr float code_bias() { return (float)(1 << (BITS - 1)); }
template <int BITS, int NK>
__device__ inline void codes_to_half(const uint32_t* w, uint32_t (&r)[NK / 2]) {
  constexpr int E = 32 / BITS;                        // codes per word, E / 2 registers
  constexpr uint32_t M = BITS == 8 ? 0x00ff00ffu : BITS == 4 ? 0x000f000fu : 0x00030003u;
  const h2 off = h2{(_Float16)(1024.f + code_bias<BITS>()), (_Float16)(1024.f + code_bias<BITS>())};
#pragma unroll
  for (int i = 0; i < NK / E; ++i)
#pragma unroll
    for (int j = 0; j < E / 2; ++j) {
      const h2 x = __builtin_bit_cast(h2, ((w[i] >> (BITS * j)) & M) | 0x64006400u) - off;
      r[i * (E / 2) + j] = __builtin_bit_cast(uint32_t, x);
    }
}
// channel (inside the quarter row) of the low (half = 0) or high code of register i
template <int BITS>
__device__ constexpr int channel_of(int i, int half) {
  constexpr int E = 32 / BITS;
  return i / (E / 2) * E + i % (E / 2) + half * (E / 2);
}

// s x in fp16, rounded once: multiplication and conversion are one instruction (v_fma_mixlo_f16,
// from the contraction; the empty assembly keeps two of them from being combined into products
// in fp32 and a packed conversion).  Rounded to fp32 in between, a product that lies next to an
// fp16 midpoint lands on it, and where cache rows are de-quantized there are such: s is R / (2^k - 1) for a 16-bit number R, so
// some levels are short fractions of R.  A channel's extreme that moves by one unit in this
// way can move the zero point it is compressed with next.
__device__ inline uint16_t mul_to_half(float s, float x) {
#pragma clang fp contract(fast)
  uint16_t h = __builtin_bit_cast(uint16_t, (_Float16)(s * x));
  asm("" : "+v"(h));
  return h;
}

// Slots of a segment, TILES tiles at a time; of two, the second one's results are in the odd lanes of a column pair, which the first
// one leaves idle once value and residual are added up.
template <int DT, int D, int BITS, bool TOK, int TILES, bool LOOP>
__device__ inline void probs_segment(const ProbsArgs& a, int b, int hk, int chunk, int sub, int begin, int len, int unit0, int nunits) {
  constexpr int NK = D / 4, KS = D / 32;              // channels per lane and tile; matrix instructions per tile
  constexpr int NW = NK * BITS / 32, ROWB = D * BITS / 8, UNIT = TILES * kProbTile;
  const int lane = threadIdx.x & 63, n = lane & 15, kg = lane >> 4;
  const int g = n >> 1, part = n & 1;                 // head and part (value, residual) of this lane's column
  const bool nvalid = g < a.G;
  const int64_t cap = sub ? a.cap[1] : a.cap[0];
  const uint8_t* kc = (sub ? a.kc[1] : a.kc[0]) + (((int64_t)b * a.Hkv + hk) * cap + begin + n) * ROWB + kg * (ROWB / 4);
  const int slot0 = (TILES == 2 ? kProbTile * part : 0) + 4 * kg;        // of a unit: the four slots whose results this lane has
  const int64_t tok0 = (int64_t)b * cap + begin + slot0;
  const int32_t* pos_src = (sub ? a.pos[1] : a.pos[0]) + tok0;
  const float *ts_src = nullptr, *tz_src = nullptr;
  if constexpr (TOK) { ts_src = (sub ? a.k_ts[1] : a.k_ts[0]) + tok0; tz_src = (sub ? a.k_tz[1] : a.k_tz[0]) + tok0; }

  // a unit's inputs of this lane: the quarter rows of slots n and 16 + n, positions and token parameters of its four slots
  // (slots past the segment's end lie inside the same 64-slot unit of the arena)
  struct In { uint32_t w[TILES][NW]; int4 pos; float4 ts, tz; };
  auto load = [&](int unit, In& in) {
#pragma unroll
    for (int t = 0; t < TILES; ++t) {
      const uint8_t* row = kc + ((int64_t)unit * UNIT + t * kProbTile) * ROWB;
      if constexpr (NW >= 4) {
#pragma unroll
        for (int i = 0; i < NW; i += 4) {
          const uint4 x = *reinterpret_cast<const uint4*>(row + 4 * i);
          in.w[t][i] = x.x; in.w[t][i + 1] = x.y; in.w[t][i + 2] = x.z; in.w[t][i + 3] = x.w;
        }
      } else if constexpr (NW == 2) {
        const uint2 x = *reinterpret_cast<const uint2*>(row);
        in.w[t][0] = x.x; in.w[t][1] = x.y;
      } else {
        in.w[t][0] = *reinterpret_cast<const uint32_t*>(row);
      }
    }
    in.pos = load4(pos_src + unit * UNIT);
    if constexpr (TOK) {
      in.ts = load4(ts_src + unit * UNIT);
      in.tz = load4(tz_src + unit * UNIT);
    }
  };
  In in;
  load(unit0, in);

  // q' = q * channel scale * sm_scale * log2(e) of head g (unused columns: 0), its two channel sums
  const int64_t hq = (int64_t)b * a.Hq + hk * a.G + (nvalid ? g : 0);
  const float lse2 = a.lse[hq] * kLog2e;
  u4 qB[KS];
  float aq = 0.f, bq = 0.f, unscale;
  constexpr float tok_bias = TOK ? code_bias<BITS>() : 0.f, chan_bias = code_bias<BITS>() - tok_bias;   // off the zero points in use, which are integers
  {
    const int64_t qoff = (int64_t)b * a.q_sB + (int64_t)(hk * a.G + (nvalid ? g : 0)) * a.q_sH + kg * NK;
    const int64_t coff = ((int64_t)(chunk * 2 + sub) * a.B + b) * (a.Hkv * D) + hk * D + kg * NK;
    const float scale = nvalid ? a.scale_log2 : 0.f;
    float qp[NK], top = 0.f;
#pragma unroll
    for (int c8 = 0; c8 < NK; c8 += 8) {
      float v[8], cs[8], cz[8];
      load8<DT>(a.q, qoff + c8, v);
      load8(a.k_cs + coff + c8, cs);
      load8(a.k_cz + coff + c8, cz);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float x = v[i] * cs[i] * scale;
        qp[c8 + i] = x;
        top = fmaxf(top, fabsf(x));
        aq += x;
        bq = fmaf(x, cz[i] - chan_bias, bq);
      }
    }
    aq += __shfl_xor(aq, 16); aq += __shfl_xor(aq, 32);
    bq += __shfl_xor(bq, 16); bq += __shfl_xor(bq, 32);
    top = fmaxf(top, __shfl_xor(top, 16));
    top = fmaxf(top, __shfl_xor(top, 32));
    // the power of two that brings the largest element to [1, 2) (clamped: both factors are finite)
    const int e = min(max((int)(__float_as_uint(top) >> 23), 1), 253);
    const float up = __uint_as_float((uint32_t)(254 - e) << 23);
    unscale = __uint_as_float((uint32_t)e << 23);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      uint32_t r[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        uint32_t value = 0, rest = 0;
#pragma unroll
        for (int half = 0; half < 2; ++half) {        // (products with powers of two: each rounded once, to fp16)
          const float x = qp[channel_of<BITS>(4 * ks + i, half)];
          const uint16_t hi = mul_to_half(up, x);
          const float left = fmaf(x, up, -(float)__builtin_bit_cast(_Float16, hi));
          value |= (uint32_t)hi << (16 * half);
          rest |= (uint32_t)mul_to_half(kProbLo, left) << (16 * half);
        }
        r[i] = part ? rest : value;
      }
      qB[ks] = u4{r[0], r[1], r[2], r[3]};
    }
  }
  float* out = a.probs + hq * a.N;
  const bool store = nvalid && (TILES == 2 || part == 0);

  for (int i = 0; i < (LOOP ? a.tpw : 1); ++i) {
    const int unit = unit0 + 4 * i;
    if (unit >= nunits) break;
    uint32_t r[TILES][NK / 2];
#pragma unroll
    for (int t = 0; t < TILES; ++t) codes_to_half<BITS, NK>(in.w[t], r[t]);
    const int pos[4] = {in.pos.x, in.pos.y, in.pos.z, in.pos.w};
    float ts[4], tz[4];
    if constexpr (TOK) {
      ts[0] = in.ts.x; ts[1] = in.ts.y; ts[2] = in.ts.z; ts[3] = in.ts.w;
      tz[0] = in.tz.x; tz[1] = in.tz.y; tz[2] = in.tz.z; tz[3] = in.tz.w;
    }
    if constexpr (LOOP) load(min(unit + 4, nunits - 1), in);      // the next unit's inputs are in flight meanwhile (no branch: it would copy them)
    f4 acc[TILES];
#pragma unroll
    for (int t = 0; t < TILES; ++t) acc[t] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int t = 0; t < TILES; ++t)
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, u4{r[t][4 * ks], r[t][4 * ks + 1], r[t][4 * ks + 2], r[t][4 * ks + 3]}),
                                                        __builtin_bit_cast(h8, qB[ks]), acc[t], 0, 0, 0);
    const float first[4] = {acc[0].x, acc[0].y, acc[0].z, acc[0].w}, second[4] = {acc[TILES - 1].x, acc[TILES - 1].y, acc[TILES - 1].z, acc[TILES - 1].w};
    const auto neighbour = [](float x) { return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xB1, 0xF, 0xF, true)); };
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float near_first = neighbour(first[v]), near_second = neighbour(second[v]);      // (by all lanes, not under the selects)
      const bool odd = TILES == 2 && part;
      const float value = odd ? near_second : first[v], rest = odd ? second[v] : near_first;
      const float dot = fmaf(rest, 1.f / kProbLo, value) * unscale;
      const float logit2 = TOK ? ts[v] * (dot - (tz[v] - tok_bias) * aq - bq) : dot - bq;
      const float p = exp2f(logit2 - lse2);
      if (store && unit * UNIT + slot0 + v < len && pos[v] >= 0 && pos[v] < a.N) out[pos[v]] = p;
    }
  }
}

// the full-precision tail, token tail_pos0 + t at row t
template <int DT, int D>
__device__ inline void probs_tail(const ProbsArgs& a, int b, int hk, int len, int tile0, int ntiles) {
  constexpr int NK = D / 4;
  const int lane = threadIdx.x & 63, n = lane & 15, kg = lane >> 4;
  const bool nvalid = n < a.G;
  const int64_t hq = (int64_t)b * a.Hq + hk * a.G + (nvalid ? n : 0);
  const int64_t qoff = (int64_t)b * a.q_sB + (int64_t)(hk * a.G + (nvalid ? n : 0)) * a.q_sH + kg * NK;
  const float scale = nvalid ? a.scale_log2 : 0.f;
  const float lse2 = a.lse[hq] * kLog2e;
  float* out = a.probs + hq * a.N + a.tail_pos0;
  for (int tile = tile0; tile < ntiles && tile < tile0 + 4 * a.tail_tpw; tile += 4) {
    const int t = min(tile * kProbTile + n, len - 1);
    const int64_t off = (int64_t)b * a.tk_sB + (int64_t)hk * a.tk_sH + (int64_t)t * a.tk_sL + kg * NK;
    f4 acc = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c8 = 0; c8 < NK; c8 += 8) {
      float kv[8], qv[8];
      load8<DT>(a.tail_k, off + c8, kv);
      load8<DT>(a.q, qoff + c8, qv);
#pragma unroll
      for (int i = 0; i < 8; ++i) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(kv[i], qv[i] * scale, acc, 0, 0, 0);
    }
    const float dot[4] = {acc.x, acc.y, acc.z, acc.w};
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int tt = tile * kProbTile + 4 * kg + v;
      if (nvalid && tt < len) out[tt] = exp2f(dot[v] - lse2);       // (the host checks tail_pos0 + tail_len <= N)
    }
  }
}

// grid (workgroups of all segments, Hkv, B); a wave takes a.tpw units of its segment (a.tail_tpw tiles of the tail).  TOK: keys with token parameters.
template <int DT, int D, bool TOK, int TILES, bool LOOP>
__global__ __launch_bounds__(256) void k_decode_probs(ProbsArgs a) {
  const int hk = blockIdx.y, b = blockIdx.z;
  const int wave = threadIdx.x >> 6;
  // the workgroup's segment: the last that starts at or before it (a lane per segment: one by
  // one, the segments of a cache of many chunks would be a chain of as many loads)
  const int lane = threadIdx.x & 63;
  const bool before = lane < a.n_segs && (int)blockIdx.x >= a.seg[lane].first_block;
  const int si = __builtin_popcountll(__builtin_amdgcn_ballot_w64(before)) - 1;
  const int begin = a.seg[si].begin, len = a.seg[si].len, sub = a.seg[si].sub;
  const bool is_tail = sub == kTailSub;
  const int first = ((int)blockIdx.x - a.seg[si].first_block) * 4 * (is_tail ? a.tail_tpw : a.tpw) + wave, count = ceil_div(len, is_tail ? kProbTile : TILES * kProbTile);
  const int bits = is_tail ? 0 : sub ? a.bits[1] : a.bits[0];
  if (first >= count) return;
  if (is_tail) probs_tail<DT, D>(a, b, hk, len, first, count);
  else if (bits == 4) probs_segment<DT, D, 4, TOK, TILES, LOOP>(a, b, hk, a.seg[si].chunk, sub, begin, len, first, count);
  else if (bits == 2) probs_segment<DT, D, 2, TOK, TILES, LOOP>(a, b, hk, a.seg[si].chunk, sub, begin, len, first, count);
  else probs_segment<DT, D, 8, TOK, TILES, LOOP>(a, b, hk, a.seg[si].chunk, sub, begin, len, first, count);
}

// scores[b, i] = mean_h ( sum_{j : row_len[j] > i} rows[j, b, h, i] ) / #{j : row_len[j] > i}
//
// Bound: reading the rows once (4 P B Hq n_out bytes).  A thread per column with the heads and
// rows as its loop - the obvious split - leaves the chip to n_out / 256 workgroups that wait for
// one load after the other: 94 us for 10 rows of 32 heads and 4096 columns (5.2 MB).  Here a
// workgroup takes COLS columns and gives every head a lane group of its own: the head's P rows
// are requested back to back (eight at a time), the per-head sums meet in LDS and are added
// head by head, so the summation order - rows within a head, then heads - and with it every
// score, is the one of that loop.  Where the columns alone fill the chip the loop stays the better
// one (and few heads leave the lane groups without work): 10 rows of 2 heads and 16 x 33000 columns
// 13 against 39 us, of 8 heads 37 against 47; of 32 heads and 16 x 4000 columns 36 against 17.
constexpr int kRowThreads = 1024;
constexpr int kRowHeads = 64;      // heads whose sums LDS holds at once

// The sum over a head's rows (column i of them starts at src), a batch of rows requested before any is added.
__device__ inline float rows_sum(const float* __restrict__ src, const int32_t* __restrict__ row_len, int P, int64_t row_pitch, int i) {
  float col = 0.f;
  int j = 0;
  auto rows_of = [&](auto n_c) {
    constexpr int N = decltype(n_c)::value;
    float v[N];
#pragma unroll
    for (int jj = 0; jj < N; ++jj) v[jj] = src[(int64_t)(j + jj) * row_pitch];
#pragma unroll
    for (int jj = 0; jj < N; ++jj)
      if (row_len[j + jj] > i) col += v[jj];
    j += N;
  };
  while (j + 8 <= P) rows_of(std::integral_constant<int, 8>{});
  if (P & 4) rows_of(std::integral_constant<int, 4>{});
  if (P & 2) rows_of(std::integral_constant<int, 2>{});
  if (P & 1) rows_of(std::integral_constant<int, 1>{});
  return col;
}

__device__ inline float rows_score(float total, const int32_t* __restrict__ row_len, int P, int Hq, int i, int normalize) {
  int cnt = 0;
  for (int j = 0; j < P; ++j) cnt += row_len[j] > i ? 1 : 0;
  float s = total / (float)Hq;
  if (normalize) s = cnt > 0 ? s / (float)cnt : 0.f;
  return s;
}

// A thread per column, for calls that fill the chip with columns.  FOURS: four rows or more.
template <bool FOURS>
__global__ __launch_bounds__(256) void k_rows_saliency_columns(const float* __restrict__ rows, const int32_t* __restrict__ row_len,
                                                               int P, int Hq, int64_t row_stride, int n_out, int normalize,
                                                               float* __restrict__ scores) {
  const int i = blockIdx.x * 256 + threadIdx.x, b = blockIdx.y, B = gridDim.y;
  if (i >= n_out) return;
  const int64_t row_pitch = (int64_t)B * Hq * row_stride;
  const float* src = rows + (int64_t)b * Hq * row_stride + i;
  float total = 0.f;
  for (int h = 0; h < Hq; ++h, src += row_stride) {
    // (pointers that advance, and the rows past the fours one by one: the address arithmetic of
    // rows_sum would be most of a short call)
    const float* p = src;
    float col = 0.f;
    int j = 0;
    if constexpr (FOURS) {
      for (; j + 4 <= P; j += 4) {
        float v[4];
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) { v[jj] = *p; p += row_pitch; }
#pragma unroll
        for (int jj = 0; jj < 4; ++jj)
          if (row_len[j + jj] > i) col += v[jj];
      }
    }
    for (; j < P; ++j, p += row_pitch)
      if (row_len[j] > i) col += *p;
    total += col;
  }
  scores[(int64_t)b * n_out + i] = rows_score(total, row_len, P, Hq, i, normalize);
}

template <int COLS>
__global__ __launch_bounds__(kRowThreads) void k_rows_saliency(const float* __restrict__ rows, const int32_t* __restrict__ row_len,
                                                               int P, int Hq, int64_t row_stride, int n_out, int normalize,
                                                               float* __restrict__ scores) {
  constexpr int NG = kRowThreads / COLS;
  __shared__ float part[kRowHeads][COLS];
  const int cx = threadIdx.x % COLS, g = threadIdx.x / COLS;
  const int b = blockIdx.y, B = gridDim.y;
  const int64_t col0 = ((int64_t)blockIdx.z * gridDim.x + blockIdx.x) * COLS;
  if (col0 >= n_out) return;
  const int i = (int)min(col0 + cx, (int64_t)0x7fffffff);
  const int ic = min(i, n_out - 1);                  // (columns past the end repeat the last one and are not stored)
  const int64_t row_pitch = (int64_t)B * Hq * row_stride;
  float total = 0.f;
  for (int h0 = 0; h0 < Hq; h0 += kRowHeads) {
    const int hn = min(kRowHeads, Hq - h0);
    for (int h = g; h < hn; h += NG)
      part[h][cx] = rows_sum(rows + ((int64_t)b * Hq + h0 + h) * row_stride + ic, row_len, P, row_pitch, i);
    __syncthreads();
    if (g == 0)
      for (int h = 0; h < hn; ++h) total += part[h][cx];
    if (h0 + kRowHeads < Hq) __syncthreads();        // (the sums have been read before they are overwritten)
  }
  if (g == 0 && i < n_out) scores[(int64_t)b * n_out + i] = rows_score(total, row_len, P, Hq, i, normalize);
}

// ---- zc_dequantize_cache -------------------------------------------------------------------
constexpr int kDqSegs = 8;         // segments (a chunk's subsets, in pieces where they are huge) one launch takes
constexpr int kDqThreads = 256;
constexpr int64_t kDqBlocks = (1ll << 32) / kDqThreads - 1;     // most workgroups of a launch: its threads are counted in 32 bits

struct DequantSeg {
  int begin, len;        // slots
  int first_block;       // this segment's first workgroup
  int chunk, sub;
};
struct DequantArgs {
  const uint8_t* codes[2];
  const float* tok_scale[2];
  const float* tok_zero[2];
  const int32_t* pos[2];
  const float* chan_scale;   // [max_chunks, 2, B, W]
  const float* chan_zero;
  int B, H, D, W, layout, tokwise;
  int bits[2];
  int64_t cap[2];
  void* out;
  int64_t o_sB, o_sH, o_sL;
  int out_L;
  int n_segs;
  DequantSeg seg[kDqSegs];
};

// Vectors of a ROW launch from which a thread takes four slots (us with one and four: 2^18 of bf16 4.0 and
// 4.3, 3/8 of 2^20 4.5 and 4.7, 2^19 5.25 and 5.05, 3/4 6.8 and 5.8, 2^20 7.9 and 6.6; fp16 5.5 and 5.45, 7.0
// and 6.2, 8.2 and 7.1 from 2^19 on; fp32, bound by its stores: 8 prompts of 4096 tokens of a head of 128 channels
// (2^19) 7.25 and 7.65, 32 of 200 of 8 heads 9.5 and 9.9, 4 of 4096 of 4 heads (2^20) 10.9 and 11.0, one of 5000 of
// 17 heads (1.3 x 2^20) 12.9 and 12.7, of 8000 of 16 heads (2^21) 16.7 and 16.2).
static constexpr int64_t four_slots_from(int dtype) { return dtype == ZC_F32 ? 5 << 18 : 1 << 19; }

// Eight consecutive elements rounded to DT and stored (16-byte aligned).
template <int DT>
__device__ inline void store8(void* base, int64_t off, const float (&v)[8]) {
  if constexpr (DT == ZC_F32) {
    float4* p = reinterpret_cast<float4*>(reinterpret_cast<float*>(base) + off);
    p[0] = make_float4(v[0], v[1], v[2], v[3]);
    p[1] = make_float4(v[4], v[5], v[6], v[7]);
  } else {
    // (two to an instruction, rounding to nearest even: 8000 tokens of two prompts re-compressed
    // in bf16 91.6 -> 88.0 us against rounding by integer arithmetic)
    static_assert(DT == ZC_BF16, "fp16 elements are rounded where they are multiplied");
    uint32_t h[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      typedef float f2 __attribute__((ext_vector_type(2)));
      typedef __bf16 b2 __attribute__((ext_vector_type(2)));
      h[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f2{v[2 * i], v[2 * i + 1]}), b2));
    }
    *reinterpret_cast<uint4*>(reinterpret_cast<uint16_t*>(base) + off) = make_uint4(h[0], h[1], h[2], h[3]);
  }
}

// Bound: writing out (2 or 4 bytes per element; the codes are a quarter of that at most).  A
// thread expands whole packed words and stores rows 16 bytes (32 for fp32) at a time - one
// element per thread and a launch per segment took 8.6 us for each of the two subsets of 4096
// tokens with 8 heads of 128 channels:
//   ROW     a thread per 8 channels of a slot (1 to 2 words), or of four consecutive slots where that
//           still fills the chip: the channel parameters are 64 bytes a thread, four times what it
//           stores per slot (4 x 4096 tokens of 40 heads of 128 channels, fp16: 45.9 -> 32.7 us; 2 x 32768
//           of 8 heads, bf16: 44.6 -> 25.9; but one prompt of 1000 of them 3.4 -> 4.0);
//   TGROUP  a thread per 8 channels and field group of a word group (the same bit field range of 8
//           words: the codes of 4 consecutive slots), one store per slot; a thread per whole word
//           group (8 to 16 stores) left half the chip without one.
// Consecutive threads take consecutive channels of a row.
// The two subsets of a chunk share one launch: workgroup ranges per segment travel in the arguments.
// Chunks go one after the other: where two hold the same position, the later one's row stays.
template <int DT, int BITS, int RS>
__device__ inline void dequantize_segment(const DequantArgs& a, const DequantSeg sg, int unit, int b) {
  constexpr int E = 32 / BITS, TB = 4 * E;
  constexpr uint32_t CM = (1u << BITS) - 1u;
  const int sub = sg.sub;
  const int VPR = a.D / 8;                          // channel vectors of a head's row
  const int64_t cap = a.cap[sub];
  const int64_t chan0 = ((int64_t)(sg.chunk * 2 + sub) * a.B + b) * a.W;
  const int vec = unit & (VPR - 1), rest = unit / VPR;    // rest: (head, slot) or (head, field group)
  const bool row_layout = a.layout == ZC_LAYOUT_ROW;
  const int per_head = row_layout ? ceil_div(sg.len, RS) : ceil_div(sg.len, TB) * E;
  const int h = rest / per_head, r = rest % per_head;
  if (h >= a.H) return;
  const int c = vec * 8;
  const int64_t bh = (int64_t)b * a.H + h;
  float cs[8], cz[8];
  load8(a.chan_scale + chan0 + h * a.D + c, cs);
  load8(a.chan_zero + chan0 + h * a.D + c, cz);
  const int64_t obase = (int64_t)b * a.o_sB + (int64_t)h * a.o_sH + c;
  auto expand = [&](int position, float ts, float tz, auto code_of) {
    if (position < 0 || position >= a.out_L) return;
    const int64_t off = obase + (int64_t)position * a.o_sL;
    if constexpr (DT == ZC_F16) {
      uint32_t h[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) h[i] = mul_to_half(cs[i] * ts, (float)code_of(i) - tz - cz[i]);
      *reinterpret_cast<uint4*>(reinterpret_cast<uint16_t*>(a.out) + off) =
          make_uint4(h[0] | h[1] << 16, h[2] | h[3] << 16, h[4] | h[5] << 16, h[6] | h[7] << 16);
    } else {
      float v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = cs[i] * ts * ((float)code_of(i) - tz - cz[i]);
      store8<DT>(a.out, off, v);
    }
  };
  if (row_layout && RS == 1) {
    const int64_t slot = (int64_t)sg.begin + r, ti = (int64_t)b * cap + slot;
    const uint8_t* src = a.codes[sub] + (bh * cap + slot) * (a.D * BITS / 8) + c * BITS / 8;
    uint32_t w[2] = {0u, 0u};
    if constexpr (BITS == 8) { const uint2 t = *reinterpret_cast<const uint2*>(src); w[0] = t.x; w[1] = t.y; }
    else if constexpr (BITS == 4) w[0] = *reinterpret_cast<const uint32_t*>(src);
    else w[0] = *reinterpret_cast<const uint16_t*>(src);
    float ts = 1.f, tz = 0.f;
    if (a.tokwise) { ts = a.tok_scale[sub][ti]; tz = a.tok_zero[sub][ti]; }
    expand(a.pos[sub][ti], ts, tz, [&](int i) { return (w[i / E] >> (BITS * (i % E))) & CM; });
  } else if (row_layout) {
    constexpr int NW = BITS == 8 ? 2 : 1;
    const int rel = r * RS, n = min(RS, sg.len - rel);
    const int64_t slot = (int64_t)sg.begin + rel, ti = (int64_t)b * cap + slot;
    const int rowb = a.D * BITS / 8;
    const uint8_t* src = a.codes[sub] + (bh * cap + slot) * rowb + c * BITS / 8;
    uint32_t w[RS][NW];
    int pos[RS];
    float ts[RS], tz[RS];
#pragma unroll
    for (int e = 0; e < RS; ++e) {           // (a slot past the end repeats the last one and is not stored)
      const int at = min(e, n - 1);
      if constexpr (BITS == 8) { const uint2 t = *reinterpret_cast<const uint2*>(src + at * rowb); w[e][0] = t.x; w[e][1] = t.y; }
      else if constexpr (BITS == 4) w[e][0] = *reinterpret_cast<const uint32_t*>(src + at * rowb);
      else w[e][0] = *reinterpret_cast<const uint16_t*>(src + at * rowb);
      pos[e] = a.pos[sub][ti + at];
      ts[e] = 1.f; tz[e] = 0.f;
      if (a.tokwise) { ts[e] = a.tok_scale[sub][ti + at]; tz[e] = a.tok_zero[sub][ti + at]; }
    }
#pragma unroll
    for (int e = 0; e < RS; ++e)
      if (e < n) expand(pos[e], ts[e], tz[e], [&](int i) { return (w[e][i / E] >> (BITS * (i % E))) & CM; });
  } else {
    // field group jf of word group kg of block blk: slots rel .. rel + 3 (inside the block, so inside the arena)
    const int jf = r % (E / 4), kg = (r / (E / 4)) & 3, blk = r / E;
    const int tile = BITS == 2 ? ((jf & 1) * 2 + (jf >> 1)) : jf;
    const int rel = blk * TB + 16 * tile + 4 * kg;
    if (rel >= sg.len) return;
    const uint32_t* src = reinterpret_cast<const uint32_t*>(a.codes[sub]) + ((bh * (cap / TB) + sg.begin / TB + blk) * 4 + kg) * a.D + c;
    const uint4 lo = reinterpret_cast<const uint4*>(src)[0], hi = reinterpret_cast<const uint4*>(src)[1];
    uint32_t w[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    const int64_t ti = (int64_t)b * cap + sg.begin + rel;
    const int4 pos4 = load4(a.pos[sub] + ti);
    float4 ts4 = make_float4(1.f, 1.f, 1.f, 1.f), tz4 = make_float4(0.f, 0.f, 0.f, 0.f);
    if (a.tokwise) {
      ts4 = load4(a.tok_scale[sub] + ti);
      tz4 = load4(a.tok_zero[sub] + ti);
    }
    const int pos[4] = {pos4.x, pos4.y, pos4.z, pos4.w};
    const float ts[4] = {ts4.x, ts4.y, ts4.z, ts4.w}, tz[4] = {tz4.x, tz4.y, tz4.z, tz4.w};
#pragma unroll
    for (int i = 0; i < 8; ++i) w[i] >>= 4 * BITS * jf;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (rel + e < sg.len) expand(pos[e], ts[e], tz[e], [&](int i) { return (w[i] >> (BITS * e)) & CM; });
  }
}

// grid (workgroups of all segments, B)
template <int DT, int RS>
__global__ __launch_bounds__(kDqThreads) void k_dequantize_cache(DequantArgs a) {
  int si = 0;
  while (si + 1 < a.n_segs && (int)blockIdx.x >= a.seg[si + 1].first_block) ++si;
  const DequantSeg sg = a.seg[si];
  const int unit = ((int)blockIdx.x - sg.first_block) * kDqThreads + threadIdx.x;
  const int bits = a.bits[sg.sub];
  if (bits == 4) dequantize_segment<DT, 4, RS>(a, sg, unit, blockIdx.y);
  else if (bits == 2) dequantize_segment<DT, 2, RS>(a, sg, unit, blockIdx.y);
  else dequantize_segment<DT, 8, RS>(a, sg, unit, blockIdx.y);
}

}  // namespace zc

using namespace zc;

// Workgroups a head in the grid: a multiple of eight, or four, gives every XCD the same segments of all heads - the long ones, or
// the tail's - and one workgroup more without work deals them out; where workgroups are few it only costs (4 a head, 520 to 1500 workgroups: 1.11
// times faster, up to 520 0.99; multiples of eight, from 1500 on 1.03, up to 1500 0.99).
static int64_t probs_grid(int64_t blocks, int64_t heads) {
  const int64_t n = blocks * heads;
  return blocks + ((blocks == 4 && n > 520) || (blocks % 8 == 0 && n > 1500) ? 1 : 0);
}
// Tiles of the packed segments: one at a time, one a wave, while no CU gets a second workgroup, or two at most where pairs would give it two as
// well (latency); else two at a time (a unit), `tpw` units a wave.  One tile's time over one unit's, 2500 drawn calls: up to 256 workgroups 0.95 to 0.99, 257
// to 512 and more than 256 by units 0.95 to 0.98, but up to 256 by units 1.13 to 1.16 (16 heads of 1383, 368 and 192 workgroups, 5.5 and 4.65 us), 513 to 768 1.06 to 1.09.
struct ProbsShape { bool pairs; int tpw; };
// What units a wave cost: the start of a wave (the query operand; a unit is 0.3 of it for 128 channels and 0.4 for 64, in fp32 it is 1.2)
// and its units, times what the workgroups of the fullest CU take: three (128 channels) or four go at a time, a lone one at 0.55 of that, and of
// further ones the last count half, as they start when others end.  Grids that give XCDs the same segments pay 8 %, more than six units, whose ends
// are coarse, 6 %.  Of 2500 drawn calls timed in all ten shapes the one of least cost is 0.7 % slower than the best in the geometric mean; all are 1.20 times faster than by a tile at
// a time with up to eight a wave.  us, one tile and 1, 2, 3, 4, 6, 9 units a wave:
// 9 x 8 heads of 22847 tokens, bits 8 and 4, fp16 105, 69, 52, 46, 43, 57 (2.3 rounds of 4), 43; 13 x 40 of 1552 54, 37, 32, 28, 26, 32, 25; 5 x 40 of 347
// 10.3, 8.9, 10.0 (4 workgroups a head), 7.8, 7.8; 2 x 8 of 1383 5.5, 4.65, 5.9, 6.6, 7.0.
static double probs_cost(int64_t blocks, int64_t heads, int64_t units, const zc_tensor4* q) {
  const int64_t grid = probs_grid(blocks, heads), wgs = grid * heads;
  const double places = q->D == 128 ? 3.0 : 4.0, x = (double)wgs / 256.0, n = (double)ceil_div64(wgs, 256);
  const double f = n <= 1.0 ? 0.55 : n <= places ? 0.35 + 0.65 * n / places : 0.5 * (x + n) / places > 1.0 ? 0.5 * (x + n) / places : 1.0;
  return f * ((q->dtype == ZC_F32 ? 1.2 : 1.0) + (q->D == 128 ? 0.3 : 0.4) * (double)units) * (grid % 8 == 0 || grid == 4 ? 1.08 : 1.0) * (units > 6 ? 1.06 : 1.0);
}
static ProbsShape probs_shape(const zc_packed* Kp, int64_t heads, int64_t tail_wgs, const zc_tensor4* q) {
  constexpr int kLong = 64;
  int64_t longs[kLong], one = tail_wgs, rest = tail_wgs, longest = 0;      // workgroups by single tiles; the tail's and those of segments of up to four units
  int n_longs = 0;
  for (int ci = 0; ci < Kp->n_chunks; ++ci)
    for (int sb = 0; sb < 2; ++sb) {
      const int64_t len = Kp->chunk_table_host[4 * ci + 2 * sb + 1], units = ceil_div64(len, 2 * kProbTile);
      if (len <= 0) continue;
      one += ceil_div64(len, 4 * kProbTile);
      if (units > longest) longest = units;
      if (units <= 4) ++rest;
      else if (n_longs < kLong) longs[n_longs++] = units;
      else longs[kLong - 1] += units;                        // (a price, not the grid)
    }
  ProbsShape best = {true, 1};
  double least = 0.0;
  for (int tpw = 1; tpw <= 9; ++tpw) {
    int64_t blocks = rest;
    for (int i = 0; i < n_longs; ++i) blocks += ceil_div64(longs[i], 4 * tpw);
    if (tpw == 1 && one * heads <= (probs_grid(blocks, heads) * heads > 256 ? 512 : 256)) return {false, 1};
    const double cost = probs_cost(blocks, heads, tpw, q);
    if (tpw == 1 || cost < least) { least = cost; best.tpw = tpw; }
    if (blocks * heads <= 256 || 4 * tpw >= longest) break;    // (more a wave leaves no fewer to wait for)
  }
  return best;
}

extern "C" int zc_decode_probs(const zc_tensor4* q, const zc_packed* Kp, const zc_tensor4* tail_k, int64_t tail_len,
                               int64_t tail_pos0, float sm_scale, const float* lse, float* probs_out, int64_t N,
                               void* stream) {
  int rc = zc_validate_tensor(q);
  if (rc) return rc;
  if (q->L != 1) return ZC_ERR_INVALID_ARG;
  rc = zc_validate_packed(Kp, false);
  if (rc) return rc;
  if (Kp->layout != ZC_LAYOUT_ROW || Kp->B != q->B || Kp->D != q->D) return ZC_ERR_INVALID_ARG;
  if (q->H % Kp->H != 0 || q->H / Kp->H > ZC_MAX_GROUP) return ZC_ERR_UNSUPPORTED;
  if (!lse || !probs_out || (reinterpret_cast<uintptr_t>(lse) & 3) || (reinterpret_cast<uintptr_t>(probs_out) & 3)) return ZC_ERR_INVALID_ARG;
  if (tail_len < 0 || tail_pos0 < 0 || N < 1 || N > 0x7fffffff || tail_pos0 + tail_len > N) return ZC_ERR_INVALID_ARG;
  if ((Kp->cap_hi > 0 && !Kp->pos_hi) || (Kp->cap_lo > 0 && !Kp->pos_lo)) return ZC_ERR_INVALID_ARG;   // token order needs the positions
  if (tail_len > 0) {
    rc = zc_validate_tensor(tail_k);
    if (rc) return rc;
    if (tail_k->dtype != q->dtype || tail_k->B != q->B || tail_k->H != Kp->H || tail_k->D != q->D || tail_k->L < tail_len)
      return ZC_ERR_INVALID_ARG;
  }
  if (q->B > 65535 || Kp->H > 65535) return ZC_ERR_UNSUPPORTED;
  int64_t tiles = ceil_div64(tail_len, kProbTile);
  for (int ci = 0; ci < Kp->n_chunks; ++ci)
    for (int sb = 0; sb < 2; ++sb) tiles += ceil_div64(Kp->chunk_table_host[4 * ci + 2 * sb + 1], kProbTile);
  if (tiles > 0x7fffffff) return ZC_ERR_UNSUPPORTED;
  if (tiles == 0) return ZC_OK;

  ProbsArgs a;
  a.q = q->ptr; a.q_sB = q->sB; a.q_sH = q->sH;
  a.B = (int)q->B; a.Hq = (int)q->H; a.Hkv = (int)Kp->H; a.G = a.Hq / a.Hkv; a.D = (int)q->D;
  a.kc[0] = Kp->codes_hi; a.kc[1] = Kp->codes_lo;
  a.k_ts[0] = Kp->tok_scale_hi; a.k_ts[1] = Kp->tok_scale_lo;
  a.k_tz[0] = Kp->tok_zero_hi; a.k_tz[1] = Kp->tok_zero_lo;
  a.pos[0] = Kp->pos_hi; a.pos[1] = Kp->pos_lo;
  a.k_cs = Kp->chan_scale; a.k_cz = Kp->chan_zero; a.k_tok = Kp->scheme != ZC_SCHEME_CHANNEL;
  a.cap[0] = Kp->cap_hi; a.cap[1] = Kp->cap_lo;
  a.bits[0] = Kp->bits_hi; a.bits[1] = Kp->bits_lo;
  a.tail_k = tail_len ? tail_k->ptr : nullptr;
  a.tk_sB = tail_len ? tail_k->sB : 0; a.tk_sH = tail_len ? tail_k->sH : 0; a.tk_sL = tail_len ? tail_k->sL : 0;
  a.tail_pos0 = (int)tail_pos0;
  a.scale_log2 = (sm_scale == 0.f ? 1.0f / sqrtf((float)q->D) : sm_scale) * kLog2e;
  a.lse = lse; a.probs = probs_out; a.N = (int)N;
  // The tail's tiles go one at a time, up to eight a wave (16 x 40 heads of 70 tokens and 78, one and three a wave 45.6 and 32.0 us, with its
  // decode); those of the packed segments one or two at a time, as many a wave as costs least.
  const int64_t heads = (int64_t)a.Hkv * a.B, all = tiles * heads, tail_tiles = ceil_div64(tail_len, kProbTile);
  a.tail_tpw = (int)(all < 2 * 2048 ? 1 : all >= 8 * 2048 ? 8 : all / 2048);
  const ProbsShape shape = probs_shape(Kp, heads, ceil_div64(tail_tiles, 4 * a.tail_tpw), q);
  const int unit = shape.pairs ? 2 * kProbTile : kProbTile;
  a.tpw = shape.tpw;
  hipStream_t st = (hipStream_t)stream;
  int64_t blocks = 0;
  a.n_segs = 0;
  auto flush = [&]() -> int {
    if (a.n_segs == 0) return ZC_OK;
    const dim3 grid((unsigned)probs_grid(blocks, heads), (unsigned)a.Hkv, (unsigned)a.B);
    const auto launch = [&](auto tile, auto pair, auto pairs) { hipLaunchKernelGGL(unit == kProbTile ? tile : a.tpw == 1 ? pair : pairs, grid, dim3(256), 0, st, a); };
#define ZC_PRD(DT, D, TOK) launch(k_decode_probs<DT, D, TOK, 1, false>, k_decode_probs<DT, D, TOK, 2, false>, k_decode_probs<DT, D, TOK, 2, true>)
#define ZC_PR(DT)                                      \
  do {                                                 \
    if (a.k_tok && q->D == 128) ZC_PRD(DT, 128, true); \
    else if (a.k_tok) ZC_PRD(DT, 64, true);            \
    else if (q->D == 128) ZC_PRD(DT, 128, false);      \
    else ZC_PRD(DT, 64, false);                        \
  } while (0)
    if (q->dtype == ZC_F32) ZC_PR(ZC_F32);
    else if (q->dtype == ZC_F16) ZC_PR(ZC_F16);
    else ZC_PR(ZC_BF16);
#undef ZC_PR
#undef ZC_PRD
    ZC_LAUNCH_CHECK();
    a.n_segs = 0;
    blocks = 0;
    return ZC_OK;
  };
  auto add = [&](int begin, int64_t len, int chunk, int sub) -> int {
    if (len == 0) return ZC_OK;
    if (a.n_segs == kProbSegs) {
      const int rcf = flush();
      if (rcf) return rcf;
    }
    a.seg[a.n_segs++] = {begin, (int)len, (int)blocks, chunk, sub};
    blocks += sub == kTailSub ? ceil_div64(ceil_div64(len, kProbTile), 4 * a.tail_tpw) : ceil_div64(ceil_div64(len, unit), 4 * a.tpw);
    return ZC_OK;
  };
  for (int ci = 0; ci < Kp->n_chunks; ++ci)
    for (int sb = 0; sb < 2; ++sb) {
      rc = add(Kp->chunk_table_host[4 * ci + 2 * sb], Kp->chunk_table_host[4 * ci + 2 * sb + 1], ci, sb);
      if (rc) return rc;
    }
  rc = add(0, tail_len, 0, kTailSub);
  if (rc) return rc;
  return flush();
}

extern "C" int zc_rows_saliency(const float* rows, const int32_t* row_len, int32_t P, int64_t B, int64_t Hq,
                                int64_t row_stride, int64_t n_out, int32_t normalize, float* scores, void* stream) {
  if (!rows || !row_len || !scores || P < 1 || B < 1 || B > 65535 || Hq < 1 || n_out < 0 || n_out > row_stride ||
      row_stride > 0x7fffffff)
    return ZC_ERR_INVALID_ARG;
  if ((reinterpret_cast<uintptr_t>(rows) & 3) || (reinterpret_cast<uintptr_t>(scores) & 3) || (reinterpret_cast<uintptr_t>(row_len) & 3))
    return ZC_ERR_INVALID_ARG;
  if (n_out == 0) return ZC_OK;
  hipStream_t st = (hipStream_t)stream;
  // a thread per column (the line by measurement: 64 workgroups of 256 columns per head, up to 16
  // heads; with up to three rows, whose loop is short, 9 per head, and always up to four heads)
  const int64_t by_column = ceil_div64(n_out, 256) * B;
  if (P < 4 ? by_column >= 9 * Hq || Hq <= 4 : by_column >= 64 * Hq && Hq <= 16) {
    hipLaunchKernelGGL((P < 4 ? k_rows_saliency_columns<false> : k_rows_saliency_columns<true>), dim3((unsigned)ceil_div64(n_out, 256), (unsigned)B),
                       dim3(256), 0, st, rows, row_len, (int)P, (int)Hq, row_stride, (int)n_out, normalize ? 1 : 0, scores);
    ZC_LAUNCH_CHECK();
    return ZC_OK;
  }
  // 32 columns (whole 128-byte lines) a workgroup while 64 would leave compute units without one
  const bool narrow = ceil_div64(n_out, 64) * B < 256;
  const int64_t tiles = ceil_div64(n_out, narrow ? 32 : 64);
  const int64_t per_z = tiles < (1 << 21) ? tiles : 1 << 21;        // (a grid counts the threads of a dimension in 32 bits)
  const dim3 grid((unsigned)per_z, (unsigned)B, (unsigned)ceil_div64(tiles, per_z));
  if (narrow)
    hipLaunchKernelGGL(k_rows_saliency<32>, grid, dim3(kRowThreads), 0, st, rows, row_len, (int)P, (int)Hq, row_stride, (int)n_out,
                       normalize ? 1 : 0, scores);
  else
    hipLaunchKernelGGL(k_rows_saliency<64>, grid, dim3(kRowThreads), 0, st, rows, row_len, (int)P, (int)Hq, row_stride, (int)n_out,
                       normalize ? 1 : 0, scores);
  ZC_LAUNCH_CHECK();
  return ZC_OK;
}

extern "C" int zc_dequantize_cache(const zc_packed* p, const zc_tensor4* out, void* stream) {
  int rc = zc_validate_packed(p, false);
  if (rc) return rc;
  rc = zc_validate_tensor(out);
  if (rc) return rc;
  if (out->B != p->B || out->H != p->H || out->D != p->D) return ZC_ERR_INVALID_ARG;
  if ((p->cap_hi > 0 && !p->pos_hi) || (p->cap_lo > 0 && !p->pos_lo)) return ZC_ERR_INVALID_ARG;
  if (p->B > 65535 || out->L > 0x7fffffff) return ZC_ERR_UNSUPPORTED;
  const int64_t W = p->H * p->D;
  hipStream_t st = (hipStream_t)stream;
  DequantArgs a;
  a.codes[0] = p->codes_hi; a.codes[1] = p->codes_lo;
  a.tok_scale[0] = p->tok_scale_hi; a.tok_scale[1] = p->tok_scale_lo;
  a.tok_zero[0] = p->tok_zero_hi; a.tok_zero[1] = p->tok_zero_lo;
  a.pos[0] = p->pos_hi; a.pos[1] = p->pos_lo;
  a.chan_scale = p->chan_scale; a.chan_zero = p->chan_zero;
  a.B = (int)p->B; a.H = (int)p->H; a.D = (int)p->D; a.W = (int)W;
  a.layout = p->layout;
  a.tokwise = p->scheme != ZC_SCHEME_CHANNEL;
  a.bits[0] = p->bits_hi; a.bits[1] = p->bits_lo;
  a.cap[0] = p->cap_hi; a.cap[1] = p->cap_lo;
  a.out = out->ptr; a.o_sB = out->sB; a.o_sH = out->sH; a.o_sL = out->sL; a.out_L = (int)out->L;
  int64_t blocks = 0, row_slots = 1;
  a.n_segs = 0;
  auto flush = [&]() -> int {
    if (a.n_segs == 0) return ZC_OK;
    const dim3 grid((unsigned)blocks, (unsigned)p->B);
    const auto launch = [&](auto one, auto four) { hipLaunchKernelGGL(row_slots == 4 ? four : one, grid, dim3(kDqThreads), 0, st, a); };
    if (out->dtype == ZC_F32) launch(k_dequantize_cache<ZC_F32, 1>, k_dequantize_cache<ZC_F32, 4>);
    else if (out->dtype == ZC_F16) launch(k_dequantize_cache<ZC_F16, 1>, k_dequantize_cache<ZC_F16, 4>);
    else launch(k_dequantize_cache<ZC_BF16, 1>, k_dequantize_cache<ZC_BF16, 4>);
    ZC_LAUNCH_CHECK();
    a.n_segs = 0;
    blocks = 0;
    return ZC_OK;
  };
  // (a segment enters as pieces of whole blocks that keep a thread's index below 2^30)
  const int64_t vpr = p->D / 8;
  int64_t most = (1ll << 30) / (p->H * vpr) / ZC_SLOT_ALIGN * ZC_SLOT_ALIGN;
  if (most < ZC_SLOT_ALIGN) most = ZC_SLOT_ALIGN;
  for (int chunk = 0; chunk < p->n_chunks; ++chunk) {
    rc = flush();                // (the chunk before this one)
    if (rc) return rc;
    const int32_t* row = p->chunk_table_host + 4 * chunk;
    row_slots = p->layout == ZC_LAYOUT_ROW && ((int64_t)row[1] + row[3]) * p->H * vpr * p->B >= four_slots_from(out->dtype) ? 4 : 1;
    for (int which = 0; which < 2; ++which) {
      for (int64_t done = 0, len = row[2 * which + 1]; done < len; done += most) {
        const int64_t part = len - done < most ? len - done : most;
        // a unit is 8 channels of a slot (ROW) or of 4 slots (TGROUP: 32 / bits such groups per block of 4 * 32 / bits slots)
        const int64_t per_head = p->layout == ZC_LAYOUT_ROW ? ceil_div64(part, row_slots) : ceil_div64(part, 4 * (32 / a.bits[which])) * (32 / a.bits[which]);
        const int64_t n = ceil_div64(per_head * p->H * vpr, kDqThreads);
        if (a.n_segs == kDqSegs || blocks + n > kDqBlocks) {
          rc = flush();
          if (rc) return rc;
        }
        a.seg[a.n_segs++] = {(int)(row[2 * which] + done), (int)part, (int)blocks, chunk, which};
        blocks += n;
      }
    }
  }
  return flush();
}
