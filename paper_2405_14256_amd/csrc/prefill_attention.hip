// zc_prefill_attention: the attention output of every prompt token at once and the
// log-normaliser of every row (Algorithm 2's attention line: Eq. 2 applied to V, with
// the causal mask).  The log-normalisers of the probe rows are what Eq. 9 needs to
// turn a logit into a probability, so zc_probe_saliency given them (lse_ext) runs its
// column sweep only.
//
// A wave owns 32 query rows of a (batch, query head); long row blocks are launched first.
//   logits  D[key][query]     = sum_c K[key][c] Q[query][c]        (A = K tile, B = Q rows in registers)
//   output  D[channel][query] = sum_key Vt[channel][key] P[query][key]   (A = V tile transposed, B = P)
// Both results put a query in a lane (column r = lane & 31): the running reference, the
// sum and the rescaling of a row are lane-local (one exchange between the two
// half-waves, which hold different keys of the same query), and the probabilities a
// lane has just computed are, converted in place, exactly the B operand of the
// second product - the order of the keys inside a matrix instruction's k index is
// free as long as both operands use the same one.
#include <type_traits>

#include "mfma_tiles.hpp"

namespace zc {

struct PrefillArgs {
  const void *q, *k, *v;
  void* o;
  int64_t q_sB, q_sH, q_sL, k_sB, k_sH, k_sL, v_sB, v_sH, v_sL, o_sB, o_sH, o_sL;
  int B, Hq, Hkv, G, L;
  float scale_log2;
  float* lse;   // [B, Hq, L] natural log, or null
  int group;    // query heads an XCD works on at a time (prefill_block)
  const int32_t* probe_pos;    // rows whose normalisers go to lse_probe too, or null
  int P;
  float* lse_probe;            // [B, Hq, P]
};

constexpr int kPfKeys = 64;    // keys per tile
constexpr int kMostKeys = 128; // of any kernel's tiles: so many rows past the end of k and v the 32-bit offsets must not wrap
typedef float v4f __attribute__((ext_vector_type(4)));

template <int DT>
__device__ inline uint32_t pack_pair(float lo, float hi) {
  typedef float f2 __attribute__((ext_vector_type(2)));
  if constexpr (DT == ZC_F16) {
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{lo, hi}, h2));
  } else {
    typedef __bf16 b2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{lo, hi}, b2));
  }
}

// Workgroup -> (batch, query head, first row).  Row blocks go from the longest to the
// shortest, and inside one length over the heads of a group, so that the last workgroups to
// start are short ones (a head after the other, the last head's long blocks start when the
// chip is already draining).  Where the heads divide over the 8 XCDs every XCD keeps its own
// heads, in groups just large enough for two rounds of its slots: the workgroups in flight
// then read few K and V heads through its L2.
__device__ inline void prefill_block(const PrefillArgs& a, int rows, int* b, int* hq, int* q0) {
  const int nqb = ceil_div(a.L, rows), heads = a.B * a.Hq;
  int id = blockIdx.x, head, qb;
  if (nqb == 1) {                      // (short prompts: a division costs as much as their products)
    qb = 0;
    head = heads & 7 ? id : (id & 7) * (heads >> 3) + (id >> 3);
  } else if (heads & 7) {
    qb = id / heads;
    head = id % heads;
  } else {
    const int hpx = heads >> 3, rank = id >> 3;
    const int g = rank / (a.group * nqb), rem = rank % (a.group * nqb);
    const int size = min(a.group, hpx - g * a.group);
    qb = rem / size;
    head = (id & 7) * hpx + g * a.group + rem % size;
  }
  *q0 = (nqb - 1 - qb) * rows;
  if (a.B == 1) {
    *b = 0;
    *hq = head;
  } else {
    *b = head / a.Hq;
    *hq = head % a.Hq;
  }
}

// The normalisers of a workgroup's rows, in LDS (rows q0 .. q0 + ROWS - 1 of one head), to the
// probes at these rows; a probe at no row gets 0 from the block of row 0.  Every workgroup
// looks at all probes, in any order and with repetitions, two a thread at most: beyond that a
// launch of its own (k_gather_lse) is cheaper.  (8 heads of 64 channels, 256 rows, 26 probes, fp32,
// with the saliency that follows: 20.0 us with the launch, 18.4 without; 32 heads of 1000 rows of 128
// channels, 100 probes, bf16: 34.4 and 32.4; 2 x 32 heads of 3001 rows, 300 probes: 193.8 and 192.4.)
constexpr int kProbesAThread = 2;
template <int ROWS, int THREADS>
__device__ inline void probe_normalisers(const PrefillArgs& a, int64_t head, int q0, const float* slse) {
#pragma unroll
  for (int u = 0; u < kProbesAThread; ++u) {
    const int i = threadIdx.x + u * THREADS;
    if (i < a.P) {
      const int pos = a.probe_pos[i], row = pos - q0;
      if (row >= 0 && row < ROWS && pos < a.L) a.lse_probe[head * a.P + i] = slse[row];
      else if (q0 == 0 && (pos < 0 || pos >= a.L)) a.lse_probe[head * a.P + i] = 0.f;
    }
  }
}

// Where a row's reference starts: below every logit, but finite, so that a wave whose logits are all -inf so far has weights of
// 2^(-inf) = 0 and not of 2^(-inf + inf), and a wave without keys joins with a factor for its zeros that is a number.
constexpr float kLowest = -3.40282347e38f;

// Chunk slot permutation of a V tile row: the transposing load reads 64 bytes of four
// consecutive keys per half-wave (32 bytes per 16 lanes); these land in different banks.
template <int D>
__device__ inline int v_swizzle(int key) {
  return D == 128 ? 4 * (key & 3) ^ (key & 2) : 2 * (key & 2) ^ 2 * (key & 1);
}

// ---- fp32 ---------------------------------------------------------------------------
// One workgroup per 32 query rows; its NW waves share the keys, a wave every NW-th block of 32,
// each with a reference, sum and output of its own that are joined in LDS at the end.  Both
// operands go straight from memory to registers: a lane's V words are 32 consecutive channels
// of a key, which is the transposed operand as it stands (one fp32 word per k index).
// Bound by the fp32 matrix instructions, a sixteenth of the 16-bit rate, and in small calls by
// the chain of a row block's key blocks, which the split shortens: 8 heads of 64 channels, 256
// rows: 22.8 -> 11 us; 1024 rows: 76 -> 27 us; 32 heads of 128 channels, 4096 rows: 1114 ->
// 1053 us (against 128 rows a workgroup with 64-key tiles in LDS, V transposed on the way).
// Requesting the next K block under the second product costs a wave per SIMD: 26 % slower there.
template <int D, int NW>
__global__ __launch_bounds__(64 * NW, 1) void k_prefill_attention32(PrefillArgs a) {
  using T = Tile<ZC_F32, D>;
  constexpr int CT = D / 32;
  constexpr int OROW = D + 4;                    // floats of a row in the joining stage
  __shared__ __align__(16) float so[32 * OROW];
  __shared__ float sm[NW][32], sl[NW][32];

  int hq, b, q0;
  prefill_block(a, 32, &b, &hq, &q0);
  const int hk = hq / a.G;
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, kh = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint8_t* qb = reinterpret_cast<const uint8_t*>(a.q) + ((int64_t)b * a.q_sB + (int64_t)hq * a.q_sH) * 4;
  const uint8_t* kb = reinterpret_cast<const uint8_t*>(a.k) + ((int64_t)b * a.k_sB + (int64_t)hk * a.k_sH) * 4;
  const uint8_t* vb = reinterpret_cast<const uint8_t*>(a.v) + ((int64_t)b * a.v_sB + (int64_t)hk * a.v_sH) * 4;
  const uint32_t q_rowb = (uint32_t)(a.q_sL * 4), k_rowb = (uint32_t)(a.k_sL * 4), v_rowb = (uint32_t)(a.v_sL * 4);
  const auto rs_q = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(qb), 0, (uint32_t)(a.L - 1) * q_rowb + T::ROWB, kBufFlags);
  const auto rs_k = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(kb), 0, (uint32_t)(a.L - 1) * k_rowb + T::ROWB, kBufFlags);
  const auto rs_v = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(vb), 0, (uint32_t)(a.L - 1) * v_rowb + T::ROWB, kBufFlags);
  const int qpos = q0 + r;

  // (rows past the end, of any tensor, arrive as zeros)
  u32x4 qf[T::NKC];
  {
    const int voff = qpos < a.L ? (int)((uint32_t)qpos * q_rowb) + kh * 16 : kOutOfRange;
#pragma unroll
    for (int kc = 0; kc < T::NKC; ++kc) qf[kc] = __builtin_amdgcn_raw_buffer_load_b128(rs_q, voff + kc * 32, 0, 0);
  }
  v16f oacc[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) oacc[ct] = v16f{};
  float m = kLowest, l = 0.f;       // running maximum (log2 units) and this half-wave's share of the sum

  const int nblk = q0 / 32 + 1;                  // blocks of 32 keys the rows see: the last is the diagonal
  for (int blk = w; blk < nblk; blk += NW) {
    const int key0 = blk * 32;
    const int koff = (int)((uint32_t)(key0 + r) * k_rowb) + kh * 16;
    u32x4 kf[T::NKC];
#pragma unroll
    for (int kc = 0; kc < T::NKC; ++kc) kf[kc] = __builtin_amdgcn_raw_buffer_load_b128(rs_k, koff + kc * 32, 0, 0);
    float vf[CT][16];                            // [channel tile][accumulator of the logits]: key acc_row(v, kh), channel 32 ct + r
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int voff = (int)((uint32_t)(key0 + acc_row(v, kh)) * v_rowb) + r * 4;
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) vf[ct][v] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_v, voff + ct * 128, 0, 0));
    }
    v16f s = {};
#pragma unroll
    for (int kc = 0; kc < T::NKC; ++kc) mma_chunk<ZC_F32>(s, kf[kc], qf[kc]);
    if (blk == nblk - 1) {
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (acc_row(v, kh) > r) s[v] = -INFINITY;
    }
    // (the maximum is taken over the raw products - the scale is positive - and the scale
    // enters with the subtraction of the reference: one fused multiply-add per logit)
    float tmax = s[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) tmax = fmaxf(tmax, s[v]);
    tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
    const float m_new = fmaxf(m, tmax * a.scale_log2);
    if (__builtin_amdgcn_ballot_w64(m_new > m)) {
      const float alpha = __builtin_amdgcn_exp2f(m - m_new);
      l *= alpha;
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[ct][i] *= alpha;
      m = m_new;
    }
    float psum = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      s[v] = __builtin_amdgcn_exp2f(fmaf(s[v], a.scale_log2, -m));
      psum += s[v];
    }
    l += psum;
#pragma unroll
    for (int v = 0; v < 16; ++v)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) oacc[ct] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[ct][v], s[v], oacc[ct], 0, 0, 0);
  }

  if constexpr (NW == 1) {            // nothing to join: lane = row, accumulator v of tile ct = channel 32 ct + acc_row(v, kh)
    const float l_tot = l + __shfl_xor(l, 32);
    if (qpos < a.L) {
      const float inv = 1.f / l_tot;
      float* orow = reinterpret_cast<float*>(a.o) + (int64_t)b * a.o_sB + (int64_t)hq * a.o_sH + (int64_t)qpos * a.o_sL;
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int v4 = 0; v4 < 4; ++v4)
          *reinterpret_cast<float4*>(orow + 32 * ct + acc_row(4 * v4, kh)) =
              make_float4(oacc[ct][4 * v4] * inv, oacc[ct][4 * v4 + 1] * inv, oacc[ct][4 * v4 + 2] * inv, oacc[ct][4 * v4 + 3] * inv);
    }
    const float lse = (m + log2f(l_tot)) * kLn2;
    const int64_t head = (int64_t)b * a.Hq + hq;
    if (a.lse && kh == 0 && qpos < a.L) a.lse[head * a.L + qpos] = lse;
    if (a.probe_pos) {
      if (kh == 0) sl[0][r] = lse;
      __syncthreads();
      probe_normalisers<32, 64>(a, head, q0, sl[0]);
    }
    return;
  }
  // ---- join the waves: a common reference and sum, then the outputs one wave after the other ----
  // (a wave without keys has m = kLowest, l = 0 and zeros; wave 0 always has the block of key 0)
  const float l_wave = l + __shfl_xor(l, 32);
  if (kh == 0) { sm[w][r] = m; sl[w][r] = l_wave; }
  __syncthreads();
  float M = sm[0][r];
#pragma unroll
  for (int v = 1; v < NW; ++v) M = fmaxf(M, sm[v][r]);
  float l_tot = 0.f;
#pragma unroll
  for (int v = 0; v < NW; ++v) l_tot += sl[v][r] * __builtin_amdgcn_exp2f(sm[v][r] - M);
  const float mine = __builtin_amdgcn_exp2f(m - M) / l_tot;
  const int used = min(NW, nblk);
  for (int v = used - 1; v >= 0; --v) {
    if (w == v) {
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int v4 = 0; v4 < 4; ++v4) {
          float4* p = reinterpret_cast<float4*>(&so[r * OROW + 32 * ct + acc_row(4 * v4, kh)]);       // four consecutive channels
          float4 o = make_float4(oacc[ct][4 * v4] * mine, oacc[ct][4 * v4 + 1] * mine, oacc[ct][4 * v4 + 2] * mine, oacc[ct][4 * v4 + 3] * mine);
          if (v < used - 1) { const float4 t = *p; o.x += t.x; o.y += t.y; o.z += t.z; o.w += t.w; }
          *p = o;
        }
    }
    __syncthreads();
  }
  for (int i = tid; i < 32 * (D / 4); i += 64 * NW) {
    const int row = i / (D / 4), c = (i % (D / 4)) * 4;
    if (q0 + row < a.L)
      *reinterpret_cast<float4*>(reinterpret_cast<float*>(a.o) + (int64_t)b * a.o_sB + (int64_t)hq * a.o_sH + (int64_t)(q0 + row) * a.o_sL + c) =
          *reinterpret_cast<const float4*>(&so[row * OROW + c]);
  }
  const float lse = (M + log2f(l_tot)) * kLn2;
  const int64_t head = (int64_t)b * a.Hq + hq;
  if (a.lse && w == 0 && kh == 0 && qpos < a.L) a.lse[head * a.L + qpos] = lse;
  if (a.probe_pos) {
    if (w == 0 && kh == 0) sl[0][r] = lse;       // (the sums were read in front of the barriers above)
    __syncthreads();
    probe_normalisers<32, 64 * NW>(a, head, q0, sl[0]);
  }
}

// The same for calls that leave most of the chip idle: 16 rows a workgroup, in 16 x 16 matrix instructions (the
// same rate), eight waves, and their outputs joined at once from a place of their own each.  Bound by the chain of a
// wave's trip to memory, its 32 cycles for every 1024 products and the join: 8 heads of 64 channels, 256 rows 11.0 -> 7.9 us,
// 64 rows 6.9 -> 5.2; of 128 channels 16.8 -> 12.2 and 9.5 -> 6.7.
// Operand layouts of the 16 x 16 x 4 instruction: lane (g = lane / 16, i = lane % 16) holds element [i][k = g] of an
// operand and elements [4 g + v][i] of the result; the order of a product's k index is free.
template <int D>
__global__ __launch_bounds__(512, 1) void k_prefill_attention32_few(PrefillArgs a) {
  constexpr int NW = 8, NKC = D / 16, CT = D / 16;
  constexpr int OROW = D + 4;                    // floats of a row in the joining stage
  __shared__ __align__(16) float so[NW][16 * OROW];
  __shared__ float sm[NW][16], sl[NW][16];

  int hq, b, q0;
  prefill_block(a, 16, &b, &hq, &q0);
  const int hk = hq / a.G;
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint8_t* qb = reinterpret_cast<const uint8_t*>(a.q) + ((int64_t)b * a.q_sB + (int64_t)hq * a.q_sH) * 4;
  const uint8_t* kb = reinterpret_cast<const uint8_t*>(a.k) + ((int64_t)b * a.k_sB + (int64_t)hk * a.k_sH) * 4;
  const uint8_t* vb = reinterpret_cast<const uint8_t*>(a.v) + ((int64_t)b * a.v_sB + (int64_t)hk * a.v_sH) * 4;
  const uint32_t q_rowb = (uint32_t)(a.q_sL * 4), k_rowb = (uint32_t)(a.k_sL * 4), v_rowb = (uint32_t)(a.v_sL * 4);
  const auto rs_q = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(qb), 0, (uint32_t)(a.L - 1) * q_rowb + D * 4, kBufFlags);
  const auto rs_k = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(kb), 0, (uint32_t)(a.L - 1) * k_rowb + D * 4, kBufFlags);
  const auto rs_v = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(vb), 0, (uint32_t)(a.L - 1) * v_rowb + D * 4, kBufFlags);
  const int qpos = q0 + r;

  // (rows past the end, of any tensor, arrive as zeros)
  u32x4 qf[NKC];
  {
    const int voff = qpos < a.L ? (int)((uint32_t)qpos * q_rowb) + g * 16 : kOutOfRange;
#pragma unroll
    for (int kc = 0; kc < NKC; ++kc) qf[kc] = __builtin_amdgcn_raw_buffer_load_b128(rs_q, voff + kc * 64, 0, 0);
  }
  v4f oacc[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) oacc[ct] = v4f{};
  float m = kLowest, l = 0.f;       // running maximum (log2 units) and this lane group's share of the sum

  const int nblk = q0 / 32 + 1;                  // blocks of 32 keys the rows see: the last holds the diagonal
  for (int blk = w; blk < nblk; blk += NW) {
    const int key0 = blk * 32;
    u32x4 kf[2][NKC];
    float vf[2][4][CT];                          // [key tile][accumulator of the logits]: key 16 t + 4 g + v, channel 16 ct + r
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int koff = (int)((uint32_t)(key0 + 16 * t + r) * k_rowb) + g * 16;
#pragma unroll
      for (int kc = 0; kc < NKC; ++kc) kf[t][kc] = __builtin_amdgcn_raw_buffer_load_b128(rs_k, koff + kc * 64, 0, 0);
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int voff = (int)((uint32_t)(key0 + 16 * t + 4 * g + v) * v_rowb) + r * 4;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) vf[t][v][ct] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_v, voff + ct * 64, 0, 0));
      }
    v4f s[2] = {v4f{}, v4f{}};
#pragma unroll
    for (int kc = 0; kc < NKC; ++kc) {
      // (the elements one by one on purpose, see mma_chunk)
#pragma unroll
      for (int t = 0; t < 2; ++t) s[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(kf[t][kc].x), __uint_as_float(qf[kc].x), s[t], 0, 0, 0);
#pragma unroll
      for (int t = 0; t < 2; ++t) s[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(kf[t][kc].y), __uint_as_float(qf[kc].y), s[t], 0, 0, 0);
#pragma unroll
      for (int t = 0; t < 2; ++t) s[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(kf[t][kc].z), __uint_as_float(qf[kc].z), s[t], 0, 0, 0);
#pragma unroll
      for (int t = 0; t < 2; ++t) s[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(kf[t][kc].w), __uint_as_float(qf[kc].w), s[t], 0, 0, 0);
    }
    if (blk == nblk - 1) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (key0 + 16 * t + 4 * g + v > qpos) s[t][v] = -INFINITY;
    }
    // (as in k_prefill_attention32: the maximum over the raw products, the scale with the subtraction)
    float tmax = fmaxf(fmaxf(fmaxf(s[0][0], s[0][1]), fmaxf(s[0][2], s[0][3])), fmaxf(fmaxf(s[1][0], s[1][1]), fmaxf(s[1][2], s[1][3])));
    tmax = fmaxf(tmax, __shfl_xor(tmax, 16));
    tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
    const float m_new = fmaxf(m, tmax * a.scale_log2);
    if (__builtin_amdgcn_ballot_w64(m_new > m)) {
      const float alpha = __builtin_amdgcn_exp2f(m - m_new);
      l *= alpha;
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int i = 0; i < 4; ++i) oacc[ct][i] *= alpha;
      m = m_new;
    }
    float psum = 0.f;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        s[t][v] = __builtin_amdgcn_exp2f(fmaf(s[t][v], a.scale_log2, -m));
        psum += s[t][v];
      }
    l += psum;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) oacc[ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[t][v][ct], s[t][v], oacc[ct], 0, 0, 0);
  }

  // ---- join the waves: a common reference and sum, then the outputs of all of them at once ----
  // (a wave without keys has m = kLowest, l = 0 and zeros; wave 0 always has the block of key 0)
  float l_wave = l + __shfl_xor(l, 16);
  l_wave += __shfl_xor(l_wave, 32);
  if (g == 0) { sm[w][r] = m; sl[w][r] = l_wave; }
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) *reinterpret_cast<v4f*>(&so[w][r * OROW + 16 * ct + 4 * g]) = oacc[ct];      // four consecutive channels
  __syncthreads();
  const int used = min(NW, nblk);
  for (int i = tid; i < 16 * (D / 4); i += 64 * NW) {
    const int row = i / (D / 4), c = (i % (D / 4)) * 4;
    float pm[NW], M = kLowest, total = 0.f;
#pragma unroll
    for (int v = 0; v < NW; ++v) { pm[v] = sm[v][row]; M = fmaxf(M, pm[v]); }
#pragma unroll
    for (int v = 0; v < NW; ++v) {
      pm[v] = __builtin_amdgcn_exp2f(pm[v] - M);
      total = fmaf(sl[v][row], pm[v], total);
    }
    v4f o = v4f{};
#pragma unroll
    for (int v = 0; v < NW; ++v)
      if (v < used) o += *reinterpret_cast<const v4f*>(&so[v][row * OROW + c]) * (pm[v] / total);
    const int64_t head = (int64_t)b * a.Hq + hq;
    if (q0 + row < a.L) {
      *reinterpret_cast<v4f*>(reinterpret_cast<float*>(a.o) + (int64_t)b * a.o_sB + (int64_t)hq * a.o_sH + (int64_t)(q0 + row) * a.o_sL + c) = o;
      if (c == 0 && a.lse) a.lse[head * a.L + q0 + row] = (M + log2f(total)) * kLn2;
    }
  }
  if (a.probe_pos) {
    __syncthreads();                             // (every wave has read the sums)
    if (tid < 16) {
      float M = kLowest, total = 0.f;
#pragma unroll
      for (int v = 0; v < NW; ++v) M = fmaxf(M, sm[v][tid]);
#pragma unroll
      for (int v = 0; v < NW; ++v) total = fmaf(sl[v][tid], __builtin_amdgcn_exp2f(sm[v][tid] - M), total);
      so[0][tid] = (M + log2f(total)) * kLn2;
    }
    __syncthreads();
    probe_normalisers<16, 64 * NW>(a, (int64_t)b * a.Hq + hq, q0, so[0]);
  }
}

// ---- 16-bit types -------------------------------------------------------------------
// One workgroup per 32 * NW query rows, a wave per 32 of them, two waves on a SIMD; 64-key
// tiles of K and V stream through LDS for all of them.  Keys go by halves of a 64-key tile, and a wave's diagonal falls on exactly one half, so no
// wave multiplies a half it cannot see.  Both tiles come global -> LDS directly; the V
// operand is read with the transposing LDS load, in row-major tiles as they arrived.
//
// Bound by the matrix cores and the power they draw: a half is 16 matrix instructions of 32
// cycles (d = 128) and about 300 cycles of vector instructions, so the two have to run at the
// same time.  The logits of half h + 1 are multiplied while the exponentials of half h are
// taken, and the operands of each product are requested one phase before.  32 heads of 32768
// rows, bf16: 8.80 -> 7.74 ms (1.14 PFLOP/s; a large library product reaches 1.21); 2 x 32
// heads of 3001 rows, fp16: 220 -> 171 us; 16 heads of 4096 rows of 64 channels: 89 -> 60 us.
// Scheduling barriers between the slices of the first product, or a raised wave priority
// around the second, cost 3 to 5 %.
//
// The running maximum of a half is taken beside the second product of the half before.  (A
// reference that moves only when a sum leaves its range spares most of that and of the
// rescaling, 3 %, but a row's largest weight is then rounded like the others instead of being
// 1: the distance to 64-bit results grows by 17 %.)
template <int DT, int D, int NW>
__global__ __launch_bounds__(64 * NW, 2) void k_prefill_attention16(PrefillArgs a) {
  using T = Tile<DT, D>;
  constexpr int TILE_B = kPfKeys * T::ROWB;
  constexpr int NI = kPfKeys / T::RPI / NW;      // transfers per wave, tile and tensor
  constexpr int CT = D / 32;                     // 32-channel tiles of the output
  constexpr int EPS = 16 / T::NKC;               // logits per slice
  constexpr int VS = T::NKC / 4;                 // the slice that requests the first V operand
  static_assert(NI >= 1, "a wave moves whole transfers");
  __shared__ __align__(1024) uint8_t Ks[2][TILE_B];
  __shared__ __align__(1024) uint8_t Vs[2][TILE_B];
  typedef short s16x4 __attribute__((ext_vector_type(4)));

  int hq, b, q0;
  prefill_block(a, 32 * NW, &b, &hq, &q0);
  const int hk = hq / a.G;
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, kh = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint8_t* qb = reinterpret_cast<const uint8_t*>(a.q) + ((int64_t)b * a.q_sB + (int64_t)hq * a.q_sH) * 2;
  const uint8_t* kb = reinterpret_cast<const uint8_t*>(a.k) + ((int64_t)b * a.k_sB + (int64_t)hk * a.k_sH) * 2;
  const uint8_t* vb = reinterpret_cast<const uint8_t*>(a.v) + ((int64_t)b * a.v_sB + (int64_t)hk * a.v_sH) * 2;
  const uint32_t q_rowb = (uint32_t)(a.q_sL * 2), k_rowb = (uint32_t)(a.k_sL * 2), v_rowb = (uint32_t)(a.v_sL * 2);
  const auto rs_q = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(qb), 0, (uint32_t)(a.L - 1) * q_rowb + T::ROWB, kBufFlags);
  const auto rs_k = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(kb), 0, (uint32_t)(a.L - 1) * k_rowb + T::ROWB, kBufFlags);
  const auto rs_v = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(vb), 0, (uint32_t)(a.L - 1) * v_rowb + T::ROWB, kBufFlags);

  const int ntiles = (min(q0 + 32 * NW, a.L) - 1) / kPfKeys + 1;     // key tiles the workgroup can see
  const int wq0 = q0 + 32 * w;                                        // first row of this wave
  const int qpos = wq0 + r;                                           // this lane's row
  const int nh = wq0 < a.L ? wq0 / 32 + 1 : 0;                        // halves this wave can see: the last is its diagonal

  const uint32_t ks_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)&Ks[0][0];
  const uint32_t vs_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)&Vs[0][0];
  int kvoff[NI], vvoff[NI];
#pragma unroll
  for (int jj = 0; jj < NI; ++jj) {
    const int row = (w + NW * jj) * T::RPI + lane / T::CPR;
    kvoff[jj] = (int)(row * k_rowb) + (((lane % T::CPR) ^ T::swz(row)) << 4);
    vvoff[jj] = (int)(row * v_rowb) + (((lane % T::CPR) ^ v_swizzle<D>(row)) << 4);
  }
  // (the tile's offset is part of the per-lane offset, which the range check sees: rows
  // past the end arrive as zeros)
  auto k_issue = [&](int t) {
    const int toff = (int)((uint32_t)t * kPfKeys * k_rowb);
#pragma unroll
    for (int jj = 0; jj < NI; ++jj) dma16<0>(ks_lds + (t & 1) * TILE_B + (w + NW * jj) * 1024, rs_k, kvoff[jj] + toff, 0);
  };
  auto v_issue = [&](int t) {
    const int toff = (int)((uint32_t)t * kPfKeys * v_rowb);
#pragma unroll
    for (int jj = 0; jj < NI; ++jj) dma16<0>(vs_lds + (t & 1) * TILE_B + (w + NW * jj) * 1024, rs_v, vvoff[jj] + toff, 0);
  };

  k_issue(0);
  v_issue(0);
  if (ntiles > 1) k_issue(1);
  // this wave's query rows, straight into operand registers (rows past the end: zeros)
  u32x4 qf[T::NKC];
  {
    const int voff = qpos < a.L ? (int)((uint32_t)qpos * q_rowb) + kh * 16 : kOutOfRange;
#pragma unroll
    for (int kc = 0; kc < T::NKC; ++kc) qf[kc] = __builtin_amdgcn_raw_buffer_load_b128(rs_q, voff + kc * 32, 0, 0);
  }

  // ---- operands from LDS -----------------------------------------------------------------
  struct KFrag { u32x4 x[T::NKC]; };
  // (LDS addresses: one register per lane and chunk pattern, tile and half in the offset of
  // the instruction; the empty assembly keeps the compiler from holding a register for each)
  typedef __attribute__((address_space(3))) const uint8_t* lds_ptr;
  uint32_t kaddr = ks_lds + T::slot(r, kh);           // chunk 2 kc + kh sits at kaddr ^ (32 kc)
  asm volatile("" : "+v"(kaddr));
  auto k_read = [&](int half, KFrag& f) {
#pragma unroll
    for (int kc = 0; kc < T::NKC; ++kc)
      f.x[kc] = *(__attribute__((address_space(3))) const u32x4*)((lds_ptr)(uintptr_t)(kaddr ^ (32 * kc)) + half * 32 * T::ROWB);
  };
  // The transposing load: in every 16 lanes, lanes 4 i .. 4 i + 3 name the 16 channels of key
  // i, and lane c receives channel c of the four keys.  A lane's 8 k-indices of operand chunk
  // s are the keys its logit accumulators 8 s .. 8 s + 7 stand for: 16 s + 4 kh + {0 .. 3} and
  // 16 s + 8 + 4 kh + {0 .. 3}.
  const int vkey = 4 * kh + ((lane & 15) >> 2);
  const int vsub = ((lane >> 4) & 1) * 2 + ((lane & 3) >> 1);         // 16-byte chunk inside a 32-channel tile
  uint32_t vaddr[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    vaddr[ct] = vs_lds + vkey * T::ROWB + (((4 * ct + vsub) ^ v_swizzle<D>(vkey)) << 4) + (lane & 1) * 8;
    asm volatile("" : "+v"(vaddr[ct]));
  }
  auto v_read = [&](int half, int s, int ct, u32x4& f) {
    // (the swizzle depends on the key's lowest two bits only)
    const lds_ptr base = (lds_ptr)(uintptr_t)vaddr[ct] + (half * 32 + 16 * s) * T::ROWB;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)base);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(base + 8 * T::ROWB));
    const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
    f.x = l2.x; f.y = l2.y; f.z = h2.x; f.w = h2.y;
  };

  v16f oacc[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct)
#pragma unroll
    for (int i = 0; i < 16; ++i) oacc[ct][i] = 0.f;
  float m = kLowest, l = 0.f;       // the row's running maximum (log2 units) and this half-wave's share of the sum
  KFrag kf;
  v16f s0, s1;

  wait_all_loads();
  __syncthreads();
  k_read(0, kf);
  s0 = v16f{};
#pragma unroll
  for (int kc = 0; kc < T::NKC; ++kc) mma_chunk<DT>(s0, kf.x[kc], qf[kc]);
  k_read(1, kf);
  kaddr += TILE_B;                                   // the K operands of a step are read one tile ahead

  // Largest logit (log2 units) of a half in either half-wave.  (The maximum is taken over the raw
  // products - the scale is positive - and the scale enters the weights with the subtraction of
  // the reference: one fused multiply-add per logit.)
  auto half_max = [&](const v16f& sc) {
    float t = sc[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) t = fmaxf(t, sc[v]);
    const auto both = __builtin_amdgcn_permlane32_swap(__float_as_uint(t), __float_as_uint(t), false, false);
    return fmaxf(__uint_as_float(both[0]), __uint_as_float(both[1])) * a.scale_log2;
  };
  float tmax = half_max(s0);                         // of the half whose weights are taken next

  // One half: weights of the logits sc, output += V^T P; unless it is the wave's LAST, the logits
  // of the half after it (operands in kf) meanwhile, their maximum, and the request of the
  // operands of the half after that.
  auto step = [&](auto last_c, int half, v16f& sc, v16f& sn) {
    constexpr bool LAST = decltype(last_c)::value;
    u32x4 vf[2][CT];
    if constexpr (LAST) {
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (acc_row(v, kh) > r) sc[v] = -INFINITY;
      tmax = half_max(sc);
    }
    const float m_new = fmaxf(m, tmax);
    if (__builtin_amdgcn_ballot_w64(m_new > m)) {
      // (0 either way; without the select the schedule differs: 2 x 32 heads, 3001 rows 178.1 -> 177.2 us, but 11 x 32 over 4, 157 rows, with probes 16.6 -> 17.3)
      const float alpha = (m == kLowest) ? 0.f : __builtin_amdgcn_exp2f(m - m_new);
      l *= alpha;
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[ct][i] *= alpha;
      m = m_new;
    }
    uint32_t pw[8];                                  // the weights, two to a word
    float psum = 0.f;
    const float nm = -m;
    if constexpr (!LAST) sn = v16f{};
#pragma unroll
    for (int kc = 0; kc < T::NKC; ++kc) {
      if constexpr (!LAST) mma_chunk<DT>(sn, kf.x[kc], qf[kc]);
      if (kc >= VS && kc < VS + CT) v_read(half, 0, kc - VS, vf[0][kc - VS]);     // (into registers kf has left)
#pragma unroll
      for (int e = kc * EPS; e < (kc + 1) * EPS; e += 2) {
        const float p0 = __builtin_amdgcn_exp2f(fmaf(sc[e], a.scale_log2, nm));
        const float p1 = __builtin_amdgcn_exp2f(fmaf(sc[e + 1], a.scale_log2, nm));
        psum += p0;
        psum += p1;
        pw[e >> 1] = pack_pair<DT>(p0, p1);
      }
    }
    l += psum;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) v_read(half, 1, ct, vf[1][ct]);
    if constexpr (!LAST) k_read(half, kf);
    u32x4 pb[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) { pb[s].x = pw[4 * s]; pb[s].y = pw[4 * s + 1]; pb[s].z = pw[4 * s + 2]; pb[s].w = pw[4 * s + 3]; }
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) mma_chunk<DT>(oacc[ct], vf[s][ct], pb[s]);
    if constexpr (!LAST) tmax = half_max(sn);        // (beside the second product, which leaves the vector units idle)
  };
  // Tile t's barrier: K(t + 1) and V(t) are complete in LDS, and nobody still reads K(t)
  // (its second half was requested before) or V(t - 1), whose buffers are filled next.
  auto top = [&](int t) {
    wait_all_loads();
    __syncthreads();
    if (t + 1 < ntiles) v_issue(t + 1);
    if (t + 2 < ntiles) k_issue(t + 2);
  };
  int turn = TILE_B;
  auto next_buffers = [&]() {                        // tile t + 1: V from the other buffer, K (of t + 2) too
    kaddr -= turn;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) vaddr[ct] += turn;
    turn = -turn;
  };
  const int t_full = nh > 0 ? (nh - 1) / 2 : 0;      // tiles both of whose halves lie before the wave's diagonal
  int t = 0;
  for (; t < t_full; ++t) {
    top(t);
    step(std::false_type{}, 0, s0, s1);
    step(std::false_type{}, 1, s1, s0);
    next_buffers();
  }
  if (nh > 0) {                                      // the tile of the diagonal (t < ntiles: the wave has rows)
    top(t++);
    if (nh & 1) {
      step(std::true_type{}, 0, s0, s1);
    } else {
      step(std::false_type{}, 0, s0, s1);
      step(std::true_type{}, 1, s1, s0);
    }
  }
  for (; t < ntiles; ++t) top(t);                    // the other waves' tiles: their transfers and barriers

  // ---- normalise and store: lane = row, accumulator v of tile ct = channel 32 ct + acc_row(v, kh) ----
  const float l_tot = l + __shfl_xor(l, 32);
  if (qpos < a.L) {
    const float inv = 1.f / l_tot;
    uint8_t* orow = reinterpret_cast<uint8_t*>(a.o) + ((int64_t)b * a.o_sB + (int64_t)hq * a.o_sH + (int64_t)qpos * a.o_sL) * 2;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int v4 = 0; v4 < 4; ++v4) {
        const int c = 32 * ct + acc_row(4 * v4, kh);        // four consecutive channels
        *reinterpret_cast<uint2*>(orow + c * 2) =
            make_uint2(pack_pair<DT>(oacc[ct][4 * v4] * inv, oacc[ct][4 * v4 + 1] * inv), pack_pair<DT>(oacc[ct][4 * v4 + 2] * inv, oacc[ct][4 * v4 + 3] * inv));
      }
  }
  const float lse = (m + log2f(l_tot)) * kLn2;
  const int64_t head = (int64_t)b * a.Hq + hq;
  if (a.lse && kh == 0 && qpos < a.L) a.lse[head * a.L + qpos] = lse;
  if (a.probe_pos) {
    float* slse = reinterpret_cast<float*>(&Ks[0][0]);
    __syncthreads();                               // (every wave is done with its tiles)
    if (kh == 0) slse[32 * w + r] = lse;
    __syncthreads();
    probe_normalisers<32 * NW, 64 * NW>(a, head, q0, slse);
  }
}

// The same for calls that leave much of the chip idle: KS of a workgroup's four waves share 32 rows, each with every KS-th
// 32 keys, a reference, a sum and an output of its own, joined in LDS at the end; a tile is 32 KS keys, of which a wave takes
// one step.  Bound by the chain of a row block's steps, which a wave alone on its SIMD takes 0.6 us for (128 channels), and by the
// start and the join.  us, one wave a row and here: 16 heads over 4 of 64 channels, 1000 rows 16.2 -> 9.1 (four), 2000 28.0 ->
// 19.4 (two); 8 of 64, 700 rows 11.7 -> 7.3; 32 over 8 of 128, 120 rows 7.0 -> 5.9, 300 9.7 -> 8.6, 1000 23.7 -> 19.5; 16 of 128, 2000 rows
// 39.5 -> 30.9; but 2000 rows of 32 heads of 128, a full chip, 49.1 -> 51.0.
template <int DT, int D, int KS>
__global__ __launch_bounds__(256, KS == 4 && D == 128 ? 1 : 2) void k_prefill_attention16_keys(PrefillArgs a) {
  using T = Tile<DT, D>;
  constexpr int NW = 4, ROWS = 32 * NW / KS, KEYS = 32 * KS;
  static_assert(KEYS <= kMostKeys && kPfKeys <= kMostKeys, "the entry's check of the offsets");
  constexpr int TILE_B = KEYS * T::ROWB;
  constexpr int NI = KEYS / T::RPI / NW;      // transfers per wave, tile and tensor
  constexpr int CT = D / 32;                     // 32-channel tiles of the output
  constexpr int EPS = 16 / T::NKC;               // logits per slice
  constexpr int VS = T::NKC / 4;                 // the slice that requests the first V operand
  static_assert(NI >= 1, "a wave moves whole transfers");
  __shared__ __align__(1024) uint8_t tiles[4 * TILE_B];                // K, K, V, V; then the waves' outputs
  __shared__ float sum[NW][2][64];
  __shared__ float slse[ROWS];
  typedef short s16x4 __attribute__((ext_vector_type(4)));

  int hq, b, q0;
  prefill_block(a, ROWS, &b, &hq, &q0);
  const int hk = hq / a.G;
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, kh = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint8_t* qb = reinterpret_cast<const uint8_t*>(a.q) + ((int64_t)b * a.q_sB + (int64_t)hq * a.q_sH) * 2;
  const uint8_t* kb = reinterpret_cast<const uint8_t*>(a.k) + ((int64_t)b * a.k_sB + (int64_t)hk * a.k_sH) * 2;
  const uint8_t* vb = reinterpret_cast<const uint8_t*>(a.v) + ((int64_t)b * a.v_sB + (int64_t)hk * a.v_sH) * 2;
  const uint32_t q_rowb = (uint32_t)(a.q_sL * 2), k_rowb = (uint32_t)(a.k_sL * 2), v_rowb = (uint32_t)(a.v_sL * 2);
  const auto rs_q = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(qb), 0, (uint32_t)(a.L - 1) * q_rowb + T::ROWB, kBufFlags);
  const auto rs_k = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(kb), 0, (uint32_t)(a.L - 1) * k_rowb + T::ROWB, kBufFlags);
  const auto rs_v = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(vb), 0, (uint32_t)(a.L - 1) * v_rowb + T::ROWB, kBufFlags);

  const int kg = w % KS;                                              // this wave's 32 keys of every tile
  const int ntiles = (min(q0 + ROWS, a.L) - 1) / KEYS + 1;            // key tiles the workgroup can see
  const int wq0 = q0 + 32 * (w / KS);                                 // first row of this wave
  const int qpos = wq0 + r;                                           // this lane's row
  const int nh = wq0 < a.L ? wq0 / 32 + 1 : 0;                        // blocks of 32 keys its rows can see: the last is the diagonal
  const int nt = (nh + KS - 1 - kg) / KS;                             // tiles of which its keys are among them
  const bool diagonal = (nh - 1) % KS == kg;                          // the last of them is the diagonal

  const uint32_t ks_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)&tiles[0];
  const uint32_t vs_lds = ks_lds + 2 * TILE_B;
  int kvoff[NI], vvoff[NI];
#pragma unroll
  for (int jj = 0; jj < NI; ++jj) {
    const int row = (w + NW * jj) * T::RPI + lane / T::CPR;
    kvoff[jj] = (int)(row * k_rowb) + (((lane % T::CPR) ^ T::swz(row)) << 4);
    vvoff[jj] = (int)(row * v_rowb) + (((lane % T::CPR) ^ v_swizzle<D>(row)) << 4);
  }
  // (the tile's offset is part of the per-lane offset, which the range check sees: rows
  // past the end arrive as zeros)
  auto k_issue = [&](int t) {
    const int toff = (int)((uint32_t)t * KEYS * k_rowb);
#pragma unroll
    for (int jj = 0; jj < NI; ++jj) dma16<0>(ks_lds + (t & 1) * TILE_B + (w + NW * jj) * 1024, rs_k, kvoff[jj] + toff, 0);
  };
  auto v_issue = [&](int t) {
    const int toff = (int)((uint32_t)t * KEYS * v_rowb);
#pragma unroll
    for (int jj = 0; jj < NI; ++jj) dma16<0>(vs_lds + (t & 1) * TILE_B + (w + NW * jj) * 1024, rs_v, vvoff[jj] + toff, 0);
  };

  k_issue(0);
  v_issue(0);
  if (ntiles > 1) k_issue(1);
  // this wave's query rows, straight into operand registers (rows past the end: zeros)
  u32x4 qf[T::NKC];
  {
    const int voff = qpos < a.L ? (int)((uint32_t)qpos * q_rowb) + kh * 16 : kOutOfRange;
#pragma unroll
    for (int kc = 0; kc < T::NKC; ++kc) qf[kc] = __builtin_amdgcn_raw_buffer_load_b128(rs_q, voff + kc * 32, 0, 0);
  }

  // ---- operands from LDS -----------------------------------------------------------------
  struct KFrag { u32x4 x[T::NKC]; };
  // (LDS addresses: one register per lane and chunk pattern, tile and half in the offset of
  // the instruction; the empty assembly keeps the compiler from holding a register for each)
  typedef __attribute__((address_space(3))) const uint8_t* lds_ptr;
  uint32_t kaddr = ks_lds + T::slot(r, kh);           // chunk 2 kc + kh sits at kaddr ^ (32 kc)
  asm volatile("" : "+v"(kaddr));
  auto k_read = [&](KFrag& f) {
#pragma unroll
    for (int kc = 0; kc < T::NKC; ++kc) f.x[kc] = *(__attribute__((address_space(3))) const u32x4*)((lds_ptr)(uintptr_t)(kaddr ^ (32 * kc)));
  };
  // The transposing load: in every 16 lanes, lanes 4 i .. 4 i + 3 name the 16 channels of key
  // i, and lane c receives channel c of the four keys.  A lane's 8 k-indices of operand chunk
  // s are the keys its logit accumulators 8 s .. 8 s + 7 stand for: 16 s + 4 kh + {0 .. 3} and
  // 16 s + 8 + 4 kh + {0 .. 3}.
  const int vkey = 4 * kh + ((lane & 15) >> 2);
  const int vsub = ((lane >> 4) & 1) * 2 + ((lane & 3) >> 1);         // 16-byte chunk inside a 32-channel tile
  uint32_t vaddr[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    vaddr[ct] = vs_lds + vkey * T::ROWB + (((4 * ct + vsub) ^ v_swizzle<D>(vkey)) << 4) + (lane & 1) * 8;
    asm volatile("" : "+v"(vaddr[ct]));
  }
  auto v_read = [&](int s, int ct, u32x4& f) {
    // (the swizzle depends on the key's lowest two bits only)
    const lds_ptr base = (lds_ptr)(uintptr_t)vaddr[ct] + 16 * s * T::ROWB;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)base);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(base + 8 * T::ROWB));
    const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
    f.x = l2.x; f.y = l2.y; f.z = h2.x; f.w = h2.y;
  };

  v16f oacc[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct)
#pragma unroll
    for (int i = 0; i < 16; ++i) oacc[ct][i] = 0.f;
  float m = kLowest, l = 0.f;       // the row's running maximum (log2 units) and this half-wave's share of the sum
  KFrag kf;
  v16f s0, s1;

  kaddr += kg * 32 * T::ROWB;                        // (every address: of this wave's keys)
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) vaddr[ct] += kg * 32 * T::ROWB;
  wait_all_loads();
  __syncthreads();
  k_read(kf);
  s0 = v16f{};
#pragma unroll
  for (int kc = 0; kc < T::NKC; ++kc) mma_chunk<DT>(s0, kf.x[kc], qf[kc]);
  kaddr += TILE_B;                                   // the K operands of a step are those of the next tile

  // Largest logit (log2 units) of a half in either half-wave.  (The maximum is taken over the raw
  // products - the scale is positive - and the scale enters the weights with the subtraction of
  // the reference: one fused multiply-add per logit.)
  auto half_max = [&](const v16f& sc) {
    float t = sc[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) t = fmaxf(t, sc[v]);
    const auto both = __builtin_amdgcn_permlane32_swap(__float_as_uint(t), __float_as_uint(t), false, false);
    return fmaxf(__uint_as_float(both[0]), __uint_as_float(both[1])) * a.scale_log2;
  };
  float tmax = half_max(s0);                         // of the half whose weights are taken next

  // One step: weights of the logits sc, output += V^T P; unless it is the wave's LAST, the logits of its keys of the next tile
  // meanwhile, and their maximum.
  auto step = [&](auto last_c, v16f& sc, v16f& sn) {
    constexpr bool LAST = decltype(last_c)::value;
    u32x4 vf[2][CT];
    if constexpr (LAST) {
      if (diagonal) {
#pragma unroll
        for (int v = 0; v < 16; ++v)
          if (acc_row(v, kh) > r) sc[v] = -INFINITY;
        tmax = half_max(sc);
      }
    } else {
      k_read(kf);
    }
    const float m_new = fmaxf(m, tmax);
    if (__builtin_amdgcn_ballot_w64(m_new > m)) {
      const float alpha = __builtin_amdgcn_exp2f(m - m_new);
      l *= alpha;
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[ct][i] *= alpha;
      m = m_new;
    }
    uint32_t pw[8];                                  // the weights, two to a word
    float psum = 0.f;
    const float nm = -m;
    if constexpr (!LAST) sn = v16f{};
#pragma unroll
    for (int kc = 0; kc < T::NKC; ++kc) {
      if constexpr (!LAST) mma_chunk<DT>(sn, kf.x[kc], qf[kc]);
      if (kc >= VS && kc < VS + CT) v_read(0, kc - VS, vf[0][kc - VS]);     // (into registers kf has left)
#pragma unroll
      for (int e = kc * EPS; e < (kc + 1) * EPS; e += 2) {
        const float p0 = __builtin_amdgcn_exp2f(fmaf(sc[e], a.scale_log2, nm));
        const float p1 = __builtin_amdgcn_exp2f(fmaf(sc[e + 1], a.scale_log2, nm));
        psum += p0;
        psum += p1;
        pw[e >> 1] = pack_pair<DT>(p0, p1);
      }
    }
    l += psum;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) v_read(1, ct, vf[1][ct]);
    u32x4 pb[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) { pb[s].x = pw[4 * s]; pb[s].y = pw[4 * s + 1]; pb[s].z = pw[4 * s + 2]; pb[s].w = pw[4 * s + 3]; }
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) mma_chunk<DT>(oacc[ct], vf[s][ct], pb[s]);
    if constexpr (!LAST) tmax = half_max(sn);        // (beside the second product, which leaves the vector units idle)
  };
  // Tile t's barrier: K(t + 1) and V(t) are complete in LDS, and nobody still reads K(t) or V(t - 1), whose buffers are filled next.
  auto top = [&](int t) {
    wait_all_loads();
    __syncthreads();
    if (t + 1 < ntiles) v_issue(t + 1);
    if (t + 2 < ntiles) k_issue(t + 2);
  };
  int turn = TILE_B;
  auto next_buffers = [&]() {                        // tile t + 1: V from the other buffer, K (of t + 2) too
    kaddr -= turn;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) vaddr[ct] += turn;
    turn = -turn;
  };
  int t = 0;
  for (; t + 2 < nt; t += 2) {
    top(t);
    step(std::false_type{}, s0, s1);
    next_buffers();
    top(t + 1);
    step(std::false_type{}, s1, s0);
    next_buffers();
  }
  if (t + 1 < nt) {
    top(t++);
    step(std::false_type{}, s0, s1);
    next_buffers();
    s0 = s1;
  }
  if (nt > 0) {
    top(t++);
    step(std::true_type{}, s0, s1);
  }
  for (; t < ntiles; ++t) top(t);                    // the other waves' tiles: their transfers and barriers

  // ---- join the waves of a row: all outputs to LDS, each wave finishes an equal part of the channels ----
  // (a wave without keys has m = kLowest, l = 0 and zeros; the first wave has key 0)
  constexpr int PART = CT * 4 / KS;                  // groups of four channels of a lane
  float4* stage = reinterpret_cast<float4*>(tiles);
  const float l_wave = l + __shfl_xor(l, 32);
  __syncthreads();                                   // (every wave is done with its tiles)
#pragma unroll
  for (int ct = 0; ct < CT; ++ct)
#pragma unroll
    for (int v4 = 0; v4 < 4; ++v4)
      stage[((w * CT + ct) * 4 + v4) * 64 + lane] = make_float4(oacc[ct][4 * v4], oacc[ct][4 * v4 + 1], oacc[ct][4 * v4 + 2], oacc[ct][4 * v4 + 3]);
  sum[w][0][lane] = m;
  sum[w][1][lane] = l_wave;
  __syncthreads();
  const int w0 = w - kg;                             // the row's waves: w0 .. w0 + KS - 1
  float M = kLowest, l_tot = 0.f, f[KS];
#pragma unroll
  for (int v = 0; v < KS; ++v) { f[v] = sum[w0 + v][0][lane]; M = fmaxf(M, f[v]); }
#pragma unroll
  for (int v = 0; v < KS; ++v) {
    f[v] = __builtin_amdgcn_exp2f(f[v] - M);
    l_tot = fmaf(sum[w0 + v][1][lane], f[v], l_tot);
  }
  if (qpos < a.L) {
    const float inv = 1.f / l_tot;
    uint8_t* orow = reinterpret_cast<uint8_t*>(a.o) + ((int64_t)b * a.o_sB + (int64_t)hq * a.o_sH + (int64_t)qpos * a.o_sL) * 2;
#pragma unroll
    for (int u = 0; u < PART; ++u) {
      const int part = kg * PART + u;                // group part % 4 of channel tile part / 4
      float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int v = 0; v < KS; ++v) {
        const float4 p = stage[((w0 + v) * CT * 4 + part) * 64 + lane];
        o.x = fmaf(p.x, f[v], o.x); o.y = fmaf(p.y, f[v], o.y); o.z = fmaf(p.z, f[v], o.z); o.w = fmaf(p.w, f[v], o.w);
      }
      const int c = 32 * (part >> 2) + 8 * (part & 3) + 4 * kh;                // (acc_row: four consecutive channels)
      *reinterpret_cast<uint2*>(orow + c * 2) = make_uint2(pack_pair<DT>(o.x * inv, o.y * inv), pack_pair<DT>(o.z * inv, o.w * inv));
    }
  }
  const float lse = (M + log2f(l_tot)) * kLn2;
  const int64_t head = (int64_t)b * a.Hq + hq;
  if (a.lse && kg == 0 && kh == 0 && qpos < a.L) a.lse[head * a.L + qpos] = lse;
  if (a.probe_pos) {
    if (kg == 0 && kh == 0) slse[wq0 - q0 + r] = lse;
    __syncthreads();
    probe_normalisers<ROWS, 64 * NW>(a, head, q0, slse);
  }
}

// lse_probe[b, h, p] = lse[b, h, probe_pos[p]]
__global__ void k_gather_lse(const float* __restrict__ lse, const int32_t* __restrict__ probe_pos, float* __restrict__ out,
                             int64_t heads, int L, int P) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= heads * P) return;
  const int64_t h = i / P;
  const int p = (int)(i % P);
  const int pos = probe_pos[p];
  out[i] = (pos >= 0 && pos < L) ? lse[h * L + pos] : 0.f;
}

// Whether the attention kernel's workgroups of `threads` threads bring the probes' normalisers themselves.
static void probes_in_kernel(PrefillArgs& a, int threads) {
  if (a.P > kProbesAThread * threads) a.probe_pos = nullptr;
}

// Query heads an XCD works on at a time: whole KV heads, at least two rounds of its slots, and
// groups of one size (a small last group would start its long blocks when the chip drains).
static int head_group(const PrefillArgs& a, int nqb, int slots) {
  const int hpx = (a.B * a.Hq) >> 3, least = a.G * ceil_div(2 * slots, nqb * a.G);
  const int groups = hpx / least;
  return groups > 1 ? a.G * ceil_div(hpx, groups * a.G) : hpx > 0 ? hpx : 1;
}

// Waves that share a row's keys in a 16-bit call: 1, 2 or 4, by what each way costs in us: a workgroup's start, then the steps of the
// longest row block or a SIMD's share of all steps, and what further workgroups a CU add.  Fitted to 400 calls of 1 to 640
// heads and 64 to 9000 rows, timed all three ways (rms 4 to 8 %; calls below 4000 heads x row blocks of 32); one wave unless another way is 8 % cheaper by
// that: all 400 are within 2 % of one wave or faster, 1.18 times in the geometric mean (1.19 with the best way each).  Beyond 2000
// heads x row blocks a full chip gains nothing (448 heads of 64, 130 rows, one and two waves 10.8 and 11.1 us; 1024 heads of 128 channels, 160 rows 44.9 and 48.5; 4096 of 192 206 and 225).  Up to 64 rows there is
// one step to share and a start that costs more (8 heads of 128, 64 rows 5.1 and 5.7 us; 640 of 64 rows 12.5 and 13.8; 512 of 64 channels, 32 rows 4.2
// and 4.8), except where registers decide: of 64 channels a CU has three workgroups of two waves a row and two of one (640 heads, 48 rows 7.0
// and 6.1 us; 1024 8.0 and 8.4; 4096 27.4 and 24.7).
static int key_split(int64_t heads, int64_t L, int D) {
  struct Way { double start, step, share, more; int split, places; double second; };
  const Way ways[2][3] = {{{3.45, 0.40, 0.356, 3.27, 1, 1, 0.0}, {3.90, 0.455, 0.362, 1.52, 2, 1, 0.0}, {4.06, 0.525, 0.451, 1.58, 4, 1, 0.0}},
                          {{4.98, 0.58, 0.560, 5.90, 1, 1, 0.0}, {4.80, 0.755, 0.638, 3.13, 2, 1, 0.4}, {5.16, 0.833, 1.100, 3.70, 4, 0, 0.0}}};
  const int64_t blocks = ceil_div64(L, 32);
  if (blocks <= 2) return D == 64 && 9 * ceil_div64(heads, 768) < 8 * ceil_div64(heads, 512) ? 2 : 1;
  if (heads * blocks > 2000) return 1;
  const double all = (double)heads * (double)blocks * (double)(blocks + 1) / 2048.0;     // steps of a SIMD
  int best = 1;
  double least = 0.0;
  for (const Way& w : ways[D == 128]) {
    const int64_t n = heads * ceil_div64(blocks, 4 / w.split);
    // (one workgroup a CU: whole rounds; two: about as they come, of 128 channels and two waves a row the first of them costs
    // more: 96 heads, 175 rows, 288 workgroups, one and two waves 7.95 and 8.8 us)
    double further = w.places ? (double)n / 256.0 - 1.0 : (double)(ceil_div64(n, 256) - 1);
    if (n > 256 && further < w.second * (double)n / 256.0) further = w.second * (double)n / 256.0;
    const double chain = w.step * (double)ceil_div64(blocks, w.split), shared = w.share * all;
    const double t = w.start + (chain > shared ? chain : shared) + (further > 0.0 ? w.more * further : 0.0);
    if (w.split == 1) least = 0.92 * t;
    else if (t < least) { least = t; best = w.split; }
  }
  return best;
}

template <int DT, int D>
static int launch_prefill(PrefillArgs& a, hipStream_t st) {
  const int64_t heads = (int64_t)a.B * a.Hq;
  const auto blocks = [&](int rows, int slots, int threads) {          // slots: workgroups an XCD holds at a time
    const int nqb = ceil_div(a.L, rows);
    probes_in_kernel(a, threads);
    a.group = head_group(a, nqb, slots);
    return dim3((unsigned)(nqb * heads));
  };
  if constexpr (DT == ZC_F32) {
    // The keys of a row block are split while that evens out the chip: a SIMD's share of all
    // blocks is heads (n + 1) / 2048 times the n of the longest row block.  One wave or two, at
    // 2.1: 88 / 94 and 335 / 331 us, at 2.0: 579 / 549; two or four, at 1.6: 232 / 261, at 1.1: 264 / 237.
    const int64_t share = heads * (ceil_div(a.L, 32) + 1);
    // 16 rows a workgroup of eight waves while all of them run at once (two a CU for 64 channels, one for 128), of long rows
    // also in two rounds: of 64 channels for few heads only, as workgroups of 32 rows need one round there and are about as many as fit.
    // us, four waves of 32 rows and this: 8 heads of 64 channels, 256 rows (128 workgroups) 11.0
    // and 7.9; 16 x 8 heads, 64 rows (512) 7.1 and 6.8, 100 rows (896) 9.7 and 11.8; 8 heads, 2047 rows (1024) 60.8 and 53.9; 14 heads, 1168 rows
    // (1022) 39.5 and 37.7; 16 heads, 974 rows (976) 34.0 and 32.9, 1022 rows (1024) 34.4 and 36.2; 20 heads, 602 rows (760) 23.1 and 22.4;
    // 24 heads, 557 rows (840) 22.5 and 22.8, 637 rows (960) 24.6 and 25.7; 32 heads, 512 rows (1024) 20.9 and 25.2;
    // 128 channels: 32 heads, 100 rows (224) 11.1 and 7.5; 4 x 16 heads, 100 rows (448) 11.4 and 12.3; 16 heads, 512 rows (512) 27.7 and
    // 25.0; 8 heads, 1023 rows (512) 47.5 and 34.8; 12 heads, 1500 rows (1128) 86.9 and 98.4.
    const int64_t few = heads * ceil_div(a.L, 16), places = D == 64 ? 512 : 256;
    const bool two_rounds = few <= 2 * places && a.L >= 512 && (D == 128 || heads <= 14 || (heads <= 20 && few <= 1000));
    if (few <= places || two_rounds) hipLaunchKernelGGL(k_prefill_attention32_few<D>, blocks(16, 32, 512), dim3(512), 0, st, a);
    else if (share >= 4300) hipLaunchKernelGGL((k_prefill_attention32<D, 1>), blocks(32, 256, 64), dim3(64), 0, st, a);
    else if (share >= 3100) hipLaunchKernelGGL((k_prefill_attention32<D, 2>), blocks(32, 128, 128), dim3(128), 0, st, a);
    else hipLaunchKernelGGL((k_prefill_attention32<D, 4>), blocks(32, 64, 256), dim3(256), 0, st, a);
  } else {
    // Four waves per workgroup, 128 rows: twice the workgroups to even the lengths out.  Eight read a
    // K and V tile once for 256 rows, which only shows over long rows of 128 channels (32 heads
    // of 32768 rows, bf16 7738 against 7796 us, fp16 8204 against 8303; of 16384 rows 1992 / 1997 and
    // 2112 / 2127; but of 8192 rows 543 / 528, of 4096 rows at batch 2 289 / 276, 16 heads of 12000
    // rows of 64 channels 376 / 346).
    if constexpr (D == 128) {
      if (a.L >= 16384 && ceil_div(a.L, 256) * heads >= 512) {
        hipLaunchKernelGGL((k_prefill_attention16<DT, D, 8>), blocks(256, 32, 512), dim3(512), 0, st, a);
        ZC_LAUNCH_CHECK();
        return ZC_OK;
      }
    }
    const int split = key_split(heads, a.L, D);
    if (split == 4) hipLaunchKernelGGL((k_prefill_attention16_keys<DT, D, 4>), blocks(32, D == 128 ? 32 : 64, 256), dim3(256), 0, st, a);
    else if (split == 2) hipLaunchKernelGGL((k_prefill_attention16_keys<DT, D, 2>), blocks(64, 64, 256), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((k_prefill_attention16<DT, D, 4>), blocks(128, 64, 256), dim3(256), 0, st, a);
  }
  ZC_LAUNCH_CHECK();
  return ZC_OK;
}

}  // namespace zc

using namespace zc;

extern "C" int zc_prefill_attention(const zc_tensor4* q, const zc_tensor4* k, const zc_tensor4* v, float sm_scale,
                                    const zc_tensor4* out, float* lse,
                                    const int32_t* probe_pos, int32_t P, float* lse_probe, void* stream) {
  int rc = zc_validate_tensor(q);
  if (rc) return rc;
  rc = zc_validate_tensor(k);
  if (rc) return rc;
  rc = zc_validate_tensor(v);
  if (rc) return rc;
  rc = zc_validate_tensor(out);
  if (rc) return rc;
  if (q->dtype != k->dtype || q->dtype != v->dtype || q->dtype != out->dtype) return ZC_ERR_INVALID_ARG;
  if (q->D != k->D || q->D != v->D || q->D != out->D) return ZC_ERR_INVALID_ARG;
  if (q->B != k->B || q->B != v->B || q->B != out->B || k->H != v->H || q->H != out->H) return ZC_ERR_INVALID_ARG;
  if (q->L < 1 || q->L != k->L || q->L != v->L || q->L != out->L) return ZC_ERR_INVALID_ARG;
  if (q->H % k->H != 0) return ZC_ERR_INVALID_ARG;
  if (lse && (reinterpret_cast<uintptr_t>(lse) & 3)) return ZC_ERR_INVALID_ARG;
  if (P < 0 || (P > 0 && (!probe_pos || !lse_probe || !lse))) return ZC_ERR_INVALID_ARG;
  if (q->B > 65535 || q->H > 65535 || q->L > 0x7fffffff - 256) return ZC_ERR_UNSUPPORTED;
  {
    // one (batch, head) slab of every tensor is addressed with 32-bit byte offsets; a tile of k_prefill_attention16_keys may
    // reach up to 127 rows past the end of k and v, and "nothing" is requested at 0xFFFFF000
    const int64_t eb = q->dtype == ZC_F32 ? 4 : 2;
    if (q->L * q->sL * eb >= 0xFFFFF000ll || (k->L + kMostKeys) * k->sL * eb >= 0xFFFFF000ll ||
        (v->L + kMostKeys) * v->sL * eb >= 0xFFFFF000ll)
      return ZC_ERR_UNSUPPORTED;
  }
  const int64_t grid = ceil_div64(q->L, 32) * q->H * q->B;         // (the smallest row blocks but for those of 16 rows, at most 1024)
  if (grid > 0x7fffffff) return ZC_ERR_UNSUPPORTED;

  PrefillArgs a;
  a.q = q->ptr; a.k = k->ptr; a.v = v->ptr; a.o = out->ptr;
  a.q_sB = q->sB; a.q_sH = q->sH; a.q_sL = q->sL;
  a.k_sB = k->sB; a.k_sH = k->sH; a.k_sL = k->sL;
  a.v_sB = v->sB; a.v_sH = v->sH; a.v_sL = v->sL;
  a.o_sB = out->sB; a.o_sH = out->sH; a.o_sL = out->sL;
  a.B = (int)q->B; a.Hq = (int)q->H; a.Hkv = (int)k->H; a.G = a.Hq / a.Hkv; a.L = (int)q->L;
  a.scale_log2 = (sm_scale == 0.f ? 1.0f / sqrtf((float)q->D) : sm_scale) * kLog2e;
  a.lse = lse;
  a.probe_pos = P > 0 ? probe_pos : nullptr;
  a.P = (int)P;
  a.lse_probe = lse_probe;
  hipStream_t st = (hipStream_t)stream;
#define ZC_PF(DT) (q->D == 128 ? launch_prefill<DT, 128>(a, st) : launch_prefill<DT, 64>(a, st))
  if (q->dtype == ZC_F32) rc = ZC_PF(ZC_F32);
  else if (q->dtype == ZC_F16) rc = ZC_PF(ZC_F16);
  else rc = ZC_PF(ZC_BF16);
#undef ZC_PF
  if (rc) return rc;
  if (P > 0 && !a.probe_pos) {
    const int64_t heads = q->B * q->H, n = heads * P;
    hipLaunchKernelGGL(k_gather_lse, dim3((unsigned)ceil_div64(n, 256)), dim3(256), 0, st, lse, probe_pos, lse_probe, heads, a.L, (int)P);
    ZC_LAUNCH_CHECK();
  }
  return ZC_OK;
}
