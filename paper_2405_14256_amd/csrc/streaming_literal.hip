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
#include "zc_common.hpp"

namespace zc {

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
  const int32_t* chunk_table;
  int n_chunks;
  int n_seg_tiles;          // 64-slot tiles of all packed segments together
  const void* tail_k;
  int64_t tk_sB, tk_sH, tk_sL;
  int tail_len, tail_pos0;
  float scale_log2;
  const float* lse;         // [B, Hq] natural log
  float* probs;             // [B, Hq, N]
  int N;
};

constexpr int kProbSlots = 64;    // cache slots (or tail tokens) per workgroup

// grid (tiles, Hkv, B), 256 threads: thread (t, kq) = (slot of the tile, quarter of its row)
template <int DT, int D>
__global__ __launch_bounds__(256) void k_decode_probs(ProbsArgs a) {
  __shared__ float qp[ZC_MAX_GROUP][D];
  __shared__ float aq[ZC_MAX_GROUP], bq[ZC_MAX_GROUP];
  const int tile = blockIdx.x, hk = blockIdx.y, b = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int G = a.G;
  const int t = tid >> 2, kq = tid & 3;

  // which segment (chunk, subset) this tile belongs to: walk the chunk table
  int ci = -1, sub = 0, begin = 0, len = 0, first = 0;
  bool is_tail = tile >= a.n_seg_tiles;
  if (!is_tail) {
    int cursor = 0;
    for (int c = 0; c < a.n_chunks && ci < 0; ++c)
      for (int s = 0; s < 2; ++s) {
        const int l = a.chunk_table[4 * c + 2 * s + 1];
        const int nt = ceil_div(l, kProbSlots);
        if (tile < cursor + nt) { ci = c; sub = s; begin = a.chunk_table[4 * c + 2 * s]; len = l; first = (tile - cursor) * kProbSlots; break; }
        cursor += nt;
      }
    if (ci < 0) return;                 // (the host's tile count and the device table disagree: nothing to do)
  } else {
    first = (tile - a.n_seg_tiles) * kProbSlots;
    len = a.tail_len;
  }
  const int ntok = min(kProbSlots, len - first);

  // q' = q * channel scale * sm_scale * log2(e), and its two channel sums
  const int64_t chan_off = is_tail ? 0 : ((int64_t)(ci * 2 + sub) * a.B + b) * (a.Hkv * D) + hk * D;
  for (int i = tid; i < G * D; i += 256) {
    const int g = i / D, c = i % D;
    const float qv = load1<DT>(a.q, (int64_t)b * a.q_sB + (int64_t)(hk * G + g) * a.q_sH + c);
    qp[g][c] = qv * (is_tail ? 1.f : a.k_cs[chan_off + c]) * a.scale_log2;
  }
  __syncthreads();
  for (int g = wave; g < G; g += 4) {
    float sa = 0.f, sb = 0.f;
    for (int c = lane; c < D; c += 64) { sa += qp[g][c]; sb += qp[g][c] * (is_tail ? 0.f : a.k_cz[chan_off + c]); }
    sa = wave_sum(sa); sb = wave_sum(sb);
    if (lane == 0) { aq[g] = sa; bq[g] = sb; }
  }
  __syncthreads();

  float dot[ZC_MAX_GROUP];
#pragma unroll
  for (int g = 0; g < ZC_MAX_GROUP; ++g) dot[g] = 0.f;
  int position = -1;
  float ts = 1.f, tz = 0.f;
  if (t < ntok) {
    if (!is_tail) {
      const int bits = a.bits[sub];
      const int E = 32 / bits;
      const uint32_t cmask = (1u << bits) - 1u;
      const int row_bytes = D * bits / 8, q_bytes = row_bytes / 4;
      const int64_t slot = (int64_t)begin + first + t;
      const uint8_t* row = a.kc[sub] + (((int64_t)b * a.Hkv + hk) * a.cap[sub] + slot) * row_bytes + kq * q_bytes;
      const int nwords = q_bytes / 4;
      for (int wi = 0; wi < nwords; ++wi) {
        const uint32_t wv = reinterpret_cast<const uint32_t*>(row)[wi];
        for (int e = 0; e < E; ++e) {
          const float code = (float)((wv >> (bits * e)) & cmask);
          const int c = kq * (D / 4) + wi * E + e;
#pragma unroll
          for (int g = 0; g < ZC_MAX_GROUP; ++g)
            if (g < G) dot[g] = fmaf(qp[g][c], code, dot[g]);
        }
      }
      position = a.pos[sub][(int64_t)b * a.cap[sub] + slot];
      if (a.k_tok) {
        ts = a.k_ts[sub][(int64_t)b * a.cap[sub] + slot];
        tz = a.k_tz[sub][(int64_t)b * a.cap[sub] + slot];
      }
    } else {
      const int64_t off = (int64_t)b * a.tk_sB + (int64_t)hk * a.tk_sH + (int64_t)(first + t) * a.tk_sL + kq * (D / 4);
      for (int c8 = 0; c8 < D / 4; c8 += 8) {
        float kv[8];
        load8<DT>(a.tail_k, off + c8, kv);
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
          for (int g = 0; g < ZC_MAX_GROUP; ++g)
            if (g < G) dot[g] = fmaf(qp[g][kq * (D / 4) + c8 + i], kv[i], dot[g]);
      }
      position = a.tail_pos0 + first + t;
    }
  }
#pragma unroll
  for (int g = 0; g < ZC_MAX_GROUP; ++g) {
    if (g < G) {
      dot[g] += __shfl_xor(dot[g], 1);
      dot[g] += __shfl_xor(dot[g], 2);
    }
  }
  if (t < ntok && kq == 0 && position >= 0 && position < a.N) {
#pragma unroll
    for (int g = 0; g < ZC_MAX_GROUP; ++g) {
      if (g < G) {
        const int64_t hq = (int64_t)b * a.Hq + hk * G + g;
        const float logit2 = ts * (dot[g] - tz * aq[g] - bq[g]);
        a.probs[hq * a.N + position] = exp2f(logit2 - a.lse[hq] * kLog2e);
      }
    }
  }
}

// scores[b, i] = mean_h ( sum_{j : row_len[j] > i} rows[j, b, h, i] ) / #{j : row_len[j] > i}
//
// Bound: reading the rows once (4 P B Hq n_out bytes).  A thread per column with the heads and
// rows as its loop - the obvious split - leaves the chip to n_out / 256 workgroups that wait for
// one load after the other: 94 us for 10 rows of 32 heads and 4096 columns (5.2 MB).  Here a
// workgroup takes COLS columns and gives every head a lane group of its own: the head's P rows
// are requested back to back (kRowBatch at a time), the per-head sums meet in LDS and are added
// head by head, so the summation order - rows within a head, then heads - and with it every
// score, is the one of that loop.
constexpr int kRowThreads = 1024;
constexpr int kRowHeads = 64;      // heads whose sums LDS holds at once
constexpr int kRowBatch = 8;       // rows of a head requested at once

template <int COLS>
__global__ __launch_bounds__(kRowThreads) void k_rows_saliency(const float* __restrict__ rows, const int32_t* __restrict__ row_len,
                                                               int P, int Hq, int64_t row_stride, int n_out, int normalize,
                                                               float* __restrict__ scores) {
  constexpr int NG = kRowThreads / COLS;
  __shared__ float part[kRowHeads][COLS];
  const int cx = threadIdx.x % COLS, g = threadIdx.x / COLS;
  const int b = blockIdx.y, B = gridDim.y;
  const int i = blockIdx.x * COLS + cx;
  const int ic = min(i, n_out - 1);                  // (columns past the end repeat the last one and are not stored)
  const int64_t row_pitch = (int64_t)B * Hq * row_stride;
  float total = 0.f;
  for (int h0 = 0; h0 < Hq; h0 += kRowHeads) {
    const int hn = min(kRowHeads, Hq - h0);
    for (int h = g; h < hn; h += NG) {
      const float* src = rows + ((int64_t)b * Hq + h0 + h) * row_stride + ic;
      float col = 0.f;
      for (int j0 = 0; j0 < P; j0 += kRowBatch) {
        float v[kRowBatch];
#pragma unroll
        for (int jj = 0; jj < kRowBatch; ++jj) v[jj] = src[(int64_t)min(j0 + jj, P - 1) * row_pitch];
#pragma unroll
        for (int jj = 0; jj < kRowBatch; ++jj)
          if (j0 + jj < P && row_len[j0 + jj] > i) col += v[jj];
      }
      part[h][cx] = col;
    }
    __syncthreads();
    if (g == 0)
      for (int h = 0; h < hn; ++h) total += part[h][cx];
    if (h0 + kRowHeads < Hq) __syncthreads();        // (the sums have been read before they are overwritten)
  }
  if (g == 0 && i < n_out) {
    int cnt = 0;
    for (int j = 0; j < P; ++j) cnt += row_len[j] > i ? 1 : 0;
    float s = total / (float)Hq;
    if (normalize) s = cnt > 0 ? s / (float)cnt : 0.f;
    scores[(int64_t)b * n_out + i] = s;
  }
}

// ---- zc_dequantize_cache -------------------------------------------------------------------
constexpr int kDqSegs = 24;        // segments (chunk x subset) one launch takes
constexpr int kDqThreads = 256;

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

// Eight consecutive elements rounded to DT and stored (16-byte aligned).
template <int DT>
__device__ inline void store8(void* base, int64_t off, const float (&v)[8]) {
  if constexpr (DT == ZC_F32) {
    float4* p = reinterpret_cast<float4*>(reinterpret_cast<float*>(base) + off);
    p[0] = make_float4(v[0], v[1], v[2], v[3]);
    p[1] = make_float4(v[4], v[5], v[6], v[7]);
  } else {
    uint16_t h[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) store1<DT>(h, i, v[i]);
    *reinterpret_cast<uint4*>(reinterpret_cast<uint16_t*>(base) + off) =
        make_uint4(h[0] | (uint32_t)h[1] << 16, h[2] | (uint32_t)h[3] << 16, h[4] | (uint32_t)h[5] << 16, h[6] | (uint32_t)h[7] << 16);
  }
}

// Bound: writing out (2 or 4 bytes per element; the codes are a quarter of that at most).  A
// thread expands whole packed words and stores rows 16 bytes (32 for fp32) at a time - one
// element per thread and a launch per segment took 8.6 us for each of the two subsets of 4096
// tokens with 8 heads of 128 channels:
//   ROW     a thread per 8 channels of a slot (1 to 2 words);
//   TGROUP  a thread per 8 channels and field group of a word group (the same bit field range of 8
//           words: the codes of 4 consecutive slots), one store per slot; a thread per whole word
//           group (8 to 16 stores) left half the chip without one.
// Consecutive threads take consecutive channels of a row.
// All segments (chunk x subset) share one launch: workgroup ranges per segment travel in the arguments.
template <int DT, int BITS>
__device__ inline void dequantize_segment(const DequantArgs& a, const DequantSeg sg, int unit, int b) {
  constexpr int E = 32 / BITS, TB = 4 * E;
  constexpr uint32_t CM = (1u << BITS) - 1u;
  const int sub = sg.sub;
  const int VPR = a.D / 8;                          // channel vectors of a head's row
  const int64_t cap = a.cap[sub];
  const int64_t chan0 = ((int64_t)(sg.chunk * 2 + sub) * a.B + b) * a.W;
  const int vec = unit & (VPR - 1), rest = unit / VPR;    // rest: (head, slot) or (head, field group)
  const bool row_layout = a.layout == ZC_LAYOUT_ROW;
  const int per_head = row_layout ? sg.len : ceil_div(sg.len, TB) * E;
  const int h = rest / per_head, r = rest % per_head;
  if (h >= a.H) return;
  const int c = vec * 8;
  const int64_t bh = (int64_t)b * a.H + h;
  float cs[8], cz[8];
  load8<ZC_F32>(a.chan_scale, chan0 + h * a.D + c, cs);
  load8<ZC_F32>(a.chan_zero, chan0 + h * a.D + c, cz);
  const int64_t obase = (int64_t)b * a.o_sB + (int64_t)h * a.o_sH + c;
  auto expand = [&](int position, float ts, float tz, auto code_of) {
    if (position < 0 || position >= a.out_L) return;
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = cs[i] * ts * ((float)code_of(i) - tz - cz[i]);
    store8<DT>(a.out, obase + (int64_t)position * a.o_sL, v);
  };
  if (row_layout) {
    const int64_t slot = (int64_t)sg.begin + r, ti = (int64_t)b * cap + slot;
    const uint8_t* src = a.codes[sub] + (bh * cap + slot) * (a.D * BITS / 8) + c * BITS / 8;
    uint32_t w[2] = {0u, 0u};
    if constexpr (BITS == 8) { const uint2 t = *reinterpret_cast<const uint2*>(src); w[0] = t.x; w[1] = t.y; }
    else if constexpr (BITS == 4) w[0] = *reinterpret_cast<const uint32_t*>(src);
    else w[0] = *reinterpret_cast<const uint16_t*>(src);
    float ts = 1.f, tz = 0.f;
    if (a.tokwise) { ts = a.tok_scale[sub][ti]; tz = a.tok_zero[sub][ti]; }
    expand(a.pos[sub][ti], ts, tz, [&](int i) { return (w[i / E] >> (BITS * (i % E))) & CM; });
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
    const int4 pos4 = *reinterpret_cast<const int4*>(a.pos[sub] + ti);
    float4 ts4 = make_float4(1.f, 1.f, 1.f, 1.f), tz4 = make_float4(0.f, 0.f, 0.f, 0.f);
    if (a.tokwise) {
      ts4 = *reinterpret_cast<const float4*>(a.tok_scale[sub] + ti);
      tz4 = *reinterpret_cast<const float4*>(a.tok_zero[sub] + ti);
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
template <int DT>
__global__ __launch_bounds__(kDqThreads) void k_dequantize_cache(DequantArgs a) {
  int si = 0;
  while (si + 1 < a.n_segs && (int)blockIdx.x >= a.seg[si + 1].first_block) ++si;
  const DequantSeg sg = a.seg[si];
  const int unit = ((int)blockIdx.x - sg.first_block) * kDqThreads + threadIdx.x;
  const int bits = a.bits[sg.sub];
  if (bits == 4) dequantize_segment<DT, 4>(a, sg, unit, blockIdx.y);
  else if (bits == 2) dequantize_segment<DT, 2>(a, sg, unit, blockIdx.y);
  else dequantize_segment<DT, 8>(a, sg, unit, blockIdx.y);
}

}  // namespace zc

using namespace zc;

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
  int64_t seg_tiles = 0;
  for (int ci = 0; ci < Kp->n_chunks; ++ci)
    for (int s = 0; s < 2; ++s) seg_tiles += ceil_div64(Kp->chunk_table_host[4 * ci + 2 * s + 1], kProbSlots);
  const int64_t tiles = seg_tiles + ceil_div64(tail_len, kProbSlots);
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
  a.chunk_table = Kp->chunk_table; a.n_chunks = Kp->n_chunks;
  a.n_seg_tiles = (int)seg_tiles;
  a.tail_k = tail_len ? tail_k->ptr : nullptr;
  a.tk_sB = tail_len ? tail_k->sB : 0; a.tk_sH = tail_len ? tail_k->sH : 0; a.tk_sL = tail_len ? tail_k->sL : 0;
  a.tail_len = (int)tail_len; a.tail_pos0 = (int)tail_pos0;
  a.scale_log2 = (sm_scale == 0.f ? 1.0f / sqrtf((float)q->D) : sm_scale) * kLog2e;
  a.lse = lse; a.probs = probs_out; a.N = (int)N;
  dim3 grid((unsigned)tiles, (unsigned)a.Hkv, (unsigned)a.B);
  hipStream_t st = (hipStream_t)stream;
#define ZC_PR(DT)                                                                        \
  do {                                                                                   \
    if (q->D == 128) hipLaunchKernelGGL((k_decode_probs<DT, 128>), grid, dim3(256), 0, st, a); \
    else hipLaunchKernelGGL((k_decode_probs<DT, 64>), grid, dim3(256), 0, st, a);          \
  } while (0)
  if (q->dtype == ZC_F32) ZC_PR(ZC_F32);
  else if (q->dtype == ZC_F16) ZC_PR(ZC_F16);
  else ZC_PR(ZC_BF16);
#undef ZC_PR
  ZC_LAUNCH_CHECK();
  return ZC_OK;
}

extern "C" int zc_rows_saliency(const float* rows, const int32_t* row_len, int32_t P, int64_t B, int64_t Hq,
                                int64_t row_stride, int64_t n_out, int32_t normalize, float* scores, void* stream) {
  if (!rows || !row_len || !scores || P < 1 || B < 1 || B > 65535 || Hq < 1 || n_out < 0 || n_out > row_stride ||
      row_stride > 0x7fffffff)
    return ZC_ERR_INVALID_ARG;
  if ((reinterpret_cast<uintptr_t>(rows) & 3) || (reinterpret_cast<uintptr_t>(scores) & 3) || (reinterpret_cast<uintptr_t>(row_len) & 3))
    return ZC_ERR_INVALID_ARG;
  if (n_out == 0) return ZC_OK;
  // 32 columns (whole 128-byte lines) a workgroup while 64 would leave compute units without one
  const bool narrow = ceil_div64(n_out, 64) * B < 256;
  const dim3 grid((unsigned)ceil_div64(n_out, narrow ? 32 : 64), (unsigned)B);
  hipStream_t st = (hipStream_t)stream;
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
  int64_t blocks = 0;
  a.n_segs = 0;
  auto flush = [&]() -> int {
    if (a.n_segs == 0) return ZC_OK;
    const dim3 grid((unsigned)blocks, (unsigned)p->B);
    if (out->dtype == ZC_F32) hipLaunchKernelGGL(k_dequantize_cache<ZC_F32>, grid, dim3(kDqThreads), 0, st, a);
    else if (out->dtype == ZC_F16) hipLaunchKernelGGL(k_dequantize_cache<ZC_F16>, grid, dim3(kDqThreads), 0, st, a);
    else hipLaunchKernelGGL(k_dequantize_cache<ZC_BF16>, grid, dim3(kDqThreads), 0, st, a);
    ZC_LAUNCH_CHECK();
    a.n_segs = 0;
    blocks = 0;
    return ZC_OK;
  };
  // (a segment enters as pieces of whole blocks that keep a thread's index below 2^30)
  const int64_t vpr = p->D / 8;
  int64_t most = (1ll << 30) / (p->H * vpr) / ZC_SLOT_ALIGN * ZC_SLOT_ALIGN;
  if (most < ZC_SLOT_ALIGN) most = ZC_SLOT_ALIGN;
  for (int chunk = 0; chunk < p->n_chunks; ++chunk)
    for (int which = 0; which < 2; ++which) {
      const int32_t* row = p->chunk_table_host + 4 * chunk;
      for (int64_t done = 0, len = row[2 * which + 1]; done < len; done += most) {
        const int64_t part = len - done < most ? len - done : most;
        // a unit is 8 channels of a slot (ROW) or of 4 slots (TGROUP: 32 / bits such groups per block of 4 * 32 / bits slots)
        const int64_t per_head = p->layout == ZC_LAYOUT_ROW ? part : ceil_div64(part, 4 * (32 / a.bits[which])) * (32 / a.bits[which]);
        const int64_t n = ceil_div64(per_head * p->H * vpr, kDqThreads);
        if (a.n_segs == kDqSegs || blocks + n > 0x7fffffff) {
          rc = flush();
          if (rc) return rc;
        }
        a.seg[a.n_segs++] = {(int)(row[2 * which] + done), (int)part, (int)blocks, chunk, which};
        blocks += n;
      }
    }
  return flush();
}
