// zc_decode_attention: single-query attention over the packed mixed-precision
// cache plus the full-precision tail (Eq. 4; the attention line of
// Algorithm 3), de-quantizing on the fly.
//
// This file is the entry point: validation, the split of the work over workgroups and
// waves, and the library's own scratch; the kernel (every code width) is in
// decode_mfma_kernel.hpp.
//
// No value is ever de-quantized element by element.  With
//   x_hat[t,c] = cs[c] * ts[t] * (code[t,c] - tz[t] - cz[c])
// the logit is   ts[t] * ( sum_c q'[c] code[t,c] - tz[t] * sum_c q'[c] - sum_c q'[c] cz[c] ),
// q'[c] = q[c] * cs[c] * sm_scale * log2(e), and the output is
//   o[c] = cs[c] * ( sum_t w[t] code[t,c] - sum_t w[t] tz[t] - cz[c] * sum_t w[t] ),  w[t] = p[t] * ts[t],
// accumulated per chunk and subset (each has its own channel parameters).
#include <atomic>

#include "decode_args.hpp"

namespace zc {

static int split_cap(int64_t B, int64_t Hq) {
  int64_t s = 2048 / (B * Hq);
  if (s < 1) s = 1;
  if (s > kMaxSplits) s = kMaxSplits;
  return (int)s;
}

}  // namespace zc

using namespace zc;

extern "C" size_t zc_decode_attention_workspace(int64_t B, int64_t Hq, int64_t D) {
  if (B <= 0 || Hq <= 0 || D <= 0) return 0;
  return (size_t)B * Hq * (split_cap(B, Hq) + kTailSplits) * (D + 2) * sizeof(float);
}

// ---- the library's own scratch buffer, for callers that cannot allocate -----------------
// zc_decode_attention_static keeps the partial (m, Z, o) of the split-K workgroups in
// this array instead of a caller's workspace.  Every GPU the library runs on holds its
// own copy at its own address; the name below is only a host-side handle, the address
// on the current device comes from hipGetSymbolAddress, once per device.
static __device__ __align__(256) unsigned char scratch[ZC_STATIC_SCRATCH_BYTES];

static int static_scratch_of_current_device(void** ptr) {
  constexpr int kMaxDevices = 64;
  static std::atomic<void*> of_device[kMaxDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return ZC_ERR_HIP;
  void* p = of_device[dev].load(std::memory_order_acquire);
  if (!p) {
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return ZC_ERR_HIP;
    of_device[dev].store(p, std::memory_order_release);
  }
  *ptr = p;
  return ZC_OK;
}

static int decode_entry(const zc_tensor4* q, const zc_packed* Kp, const zc_packed* Vp,
                        const zc_tensor4* tail_k, const zc_tensor4* tail_v, int64_t tail_len,
                        float sm_scale, void* out, float* lse_out,
                        void* ws, size_t ws_bytes, bool static_ws, void* stream) {
  int rc = zc_validate_tensor(q);
  if (rc) return rc;
  if (q->L != 1) return ZC_ERR_INVALID_ARG;
  rc = zc_validate_packed(Kp, false);
  if (rc) return rc;
  rc = zc_validate_packed(Vp, false);
  if (rc) return rc;
  if (Kp->layout != ZC_LAYOUT_ROW || Vp->layout != ZC_LAYOUT_TGROUP) return ZC_ERR_INVALID_ARG;
  if (Kp->B != q->B || Vp->B != q->B || Kp->H != Vp->H || Kp->D != q->D || Vp->D != q->D) return ZC_ERR_INVALID_ARG;
  if (Kp->bits_hi != Vp->bits_hi || Kp->bits_lo != Vp->bits_lo) return ZC_ERR_INVALID_ARG;
  if (Kp->cap_hi != Vp->cap_hi || Kp->cap_lo != Vp->cap_lo || Kp->n_chunks != Vp->n_chunks) return ZC_ERR_INVALID_ARG;
  if (q->H % Kp->H != 0 || q->H / Kp->H > ZC_MAX_GROUP) return ZC_ERR_UNSUPPORTED;
  if (!out || (reinterpret_cast<uintptr_t>(out) & 15)) return ZC_ERR_INVALID_ARG;
  if (tail_len < 0) return ZC_ERR_INVALID_ARG;
  if (tail_len > 0) {
    rc = zc_validate_tensor(tail_k);
    if (rc) return rc;
    rc = zc_validate_tensor(tail_v);
    if (rc) return rc;
    if (tail_k->dtype != q->dtype || tail_v->dtype != q->dtype) return ZC_ERR_INVALID_ARG;
    if (tail_k->B != q->B || tail_v->B != q->B || tail_k->H != Kp->H || tail_v->H != Kp->H ||
        tail_k->D != q->D || tail_v->D != q->D || tail_k->L < tail_len || tail_v->L < tail_len)
      return ZC_ERR_INVALID_ARG;
    // the matrix-core kernel addresses the tail rows of one (batch, KV head) with 32-bit byte offsets
    const int64_t eb = q->dtype == ZC_F32 ? 4 : 2;
    if (tail_len * tail_k->sL * eb >= 0xFFFFF000ll || tail_len * tail_v->sL * eb >= 0xFFFFF000ll) return ZC_ERR_UNSUPPORTED;
  }
  if (q->B > 65535 || Kp->H > 65535) return ZC_ERR_UNSUPPORTED;
  // the matrix-core kernel addresses one (batch, KV head) part of an arena with 32-bit offsets,
  // and requests "nothing" by pointing every lane at offset 0xFFFFF000, which must lie past the end
  constexpr int64_t kPartLimit = 0xFFFFF000ll;
  if (Kp->cap_hi * (q->D * Kp->bits_hi / 8) >= kPartLimit || Kp->cap_lo * (q->D * Kp->bits_lo / 8) >= kPartLimit ||
      Kp->cap_hi * 4 >= kPartLimit || Kp->cap_lo * 4 >= kPartLimit)
    return ZC_ERR_UNSUPPORTED;
  const size_t need = zc_decode_attention_workspace(q->B, q->H, q->D);
  if (static_ws) {
    if (need > (size_t)ZC_STATIC_SCRATCH_BYTES) return ZC_ERR_STATIC_LIMIT;
    rc = static_scratch_of_current_device(&ws);
    if (rc) return rc;
  } else if (!ws || ws_bytes < need || (reinterpret_cast<uintptr_t>(ws) & 15)) {
    return ZC_ERR_WORKSPACE;
  }

  // the chunk tables must agree; the packed cache's cost line: half-blocks of 32 slots (8-bit
  // codes: of 16), and kSegCost per segment
  const int hs_hi = Kp->bits_hi == 8 ? 16 : 32, hs_lo = Kp->bits_lo == 8 ? 16 : 32;
  int64_t units = 0;
  for (int ci = 0; ci < Kp->n_chunks; ++ci) {
    const int32_t* rk = Kp->chunk_table_host + 4 * ci;
    const int32_t* rv = Vp->chunk_table_host + 4 * ci;
    for (int i = 0; i < 4; ++i)
      if (rk[i] != rv[i]) return ZC_ERR_INVALID_ARG;
    const int64_t nh = ceil_div64(rk[1], hs_hi), nl = ceil_div64(rk[3], hs_lo);
    units += nh + nl + (nh > 0 ? kSegCost : 0) + (nl > 0 ? kSegCost : 0);
  }
  if (units > 0x7fffffff) return ZC_ERR_UNSUPPORTED;

  DecArgs a;
  a.q = q->ptr; a.q_sB = q->sB; a.q_sH = q->sH;
  a.B = (int)q->B; a.Hq = (int)q->H; a.Hkv = (int)Kp->H; a.G = a.Hq / a.Hkv; a.D = (int)q->D;
  a.kc[0] = Kp->codes_hi; a.kc[1] = Kp->codes_lo;
  a.k_ts[0] = Kp->tok_scale_hi; a.k_ts[1] = Kp->tok_scale_lo;
  a.k_tz[0] = Kp->tok_zero_hi; a.k_tz[1] = Kp->tok_zero_lo;
  a.k_cs = Kp->chan_scale; a.k_cz = Kp->chan_zero; a.k_tok = Kp->scheme != ZC_SCHEME_CHANNEL;
  a.vc[0] = reinterpret_cast<const uint32_t*>(Vp->codes_hi);
  a.vc[1] = reinterpret_cast<const uint32_t*>(Vp->codes_lo);
  a.v_ts[0] = Vp->tok_scale_hi; a.v_ts[1] = Vp->tok_scale_lo;
  a.v_tz[0] = Vp->tok_zero_hi; a.v_tz[1] = Vp->tok_zero_lo;
  a.v_cs = Vp->chan_scale; a.v_cz = Vp->chan_zero; a.v_tok = Vp->scheme != ZC_SCHEME_CHANNEL;
  a.cap[0] = Kp->cap_hi; a.cap[1] = Kp->cap_lo;
  a.bits[0] = Kp->bits_hi; a.bits[1] = Kp->bits_lo;
  a.chunk_table = Kp->chunk_table; a.n_chunks = Kp->n_chunks;
  a.chunks_inline = Kp->n_chunks <= kInlineChunks;
  for (int i = 0; i < 4 * kInlineChunks; ++i) a.chunk_rows[i] = (a.chunks_inline && i < 4 * Kp->n_chunks) ? Kp->chunk_table_host[i] : 0;
  a.tail_k = tail_len ? tail_k->ptr : nullptr;
  a.tail_v = tail_len ? tail_v->ptr : nullptr;
  a.tk_sB = tail_len ? tail_k->sB : 0; a.tk_sH = tail_len ? tail_k->sH : 0; a.tk_sL = tail_len ? tail_k->sL : 0;
  a.tv_sB = tail_len ? tail_v->sB : 0; a.tv_sH = tail_len ? tail_v->sH : 0; a.tv_sL = tail_len ? tail_v->sL : 0;
  a.tail_len = (int)tail_len;
  a.scale_log2 = (sm_scale == 0.f ? 1.0f / sqrtf((float)q->D) : sm_scale) * kLog2e;
  {
    // compute units of the current device (asked once per process and device id)
    static int cu_of_device[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return ZC_ERR_HIP;
    int ncu = (dev >= 0 && dev < 64) ? cu_of_device[dev] : 0;
    if (ncu == 0) {
      if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || ncu <= 0) ncu = 256;
      if (dev >= 0 && dev < 64) cu_of_device[dev] = ncu;
    }
    a.n_cu = ncu;
  }
  int S = split_cap(q->B, q->H);
  a.n_pw = 0; a.n_tw = 0; a.tw_full = 0; a.tw_rem = 0; a.tail_alone = 0;
  a.pw_q = a.pw_r = a.tu_q = a.tu_r = 0;
  {
    const int64_t heads = q->B * Kp->H;
    const int64_t tail_units = ceil_div64(tail_len, kTailUnit), tail_cost = tail_units > 0 ? 2 * tail_units + kSegCost : 0;
    // Packed cache.  About eight cost units per workgroup is the finest useful split;
    // the reduce kernel reads at most 32 partials per head.
    int64_t want = ceil_div64(units, 8);
    if (want > 32) want = 32;
    if (want > S) want = S;
    if (heads * want <= a.n_cu) {
      S = (int)want;                 // one workgroup per CU at most: only latency counts
    } else {
      // The launch runs in rounds of two workgroups per CU; a workgroup costs a fixed
      // part (start-up, operand, merge: about 48 units' worth, measured) plus its units.
      int64_t best = 0, best_cost = 0;
      for (int64_t c = 1; c <= want; ++c) {
        const int64_t cost = ceil_div64(heads * c, 2 * (int64_t)a.n_cu) * (48 + ceil_div64(units, c));
        if (best == 0 || cost < best_cost) { best = c; best_cost = cost; }
      }
      S = (int)best;
      // One workgroup per CU instead of two: a wave alone on its SIMD issues faster, and half the partials to reduce are
      // worth two units (a workgroup that is alone with its head writes the result itself: the launch that reduces is
      // worth twelve); but a unit takes it kLone / 32 of what one takes each of two (the last row: alone with its head), and `one`
      // may leave CUs idle.  us per call with 57 tokens of tail, two and one: 64 heads of 128 channels at 4 and 2 bits,
      // 14 units each 10.7 and 10.1, 20 units 11.0 and 10.8, 28 (takes two) 12.2 and 12.7; 16 heads of 64, 12 units 8.3 and 7.7, 20
      // (two) 8.9 and 8.8, 32 (two) 9.7 and 10.0; 32 heads of 128 at 8 and 4 bits, 36 units 17.9 and 15.5, 110 (two) 30.0 and 30.2; of
      // 64, 14 units 9.2 and 8.7, 50 (two) 13.8 and 14.7; 86 heads of 64, where one leaves a third of the CUs idle, 24 units (two)
      // 10.0 and 10.4; 12 heads of 64, where two are on half the CUs only, 44 units 14.2 and 13.2.
      constexpr int64_t kLone[3][3] = {{21, 20, 19}, {19, 17, 16}, {23, 22, 20}};      // 64 channels, 128; none, one or both code widths 8 bits
      const int64_t one = a.n_cu / heads, gain = one == 1 ? 12 : 2;
      const int64_t lone = kLone[one == 1 ? 2 : q->D == 128][(Kp->bits_hi == 8) + (Kp->bits_lo == 8)];
      if (one > 0 && one < best && lone * ceil_div64(units + tail_cost, one) <= 32 * (gain + ceil_div64(units + tail_cost, best))) S = (int)one;
    }
    // Tail: waves of its own.  One unit (16 tokens) per wave while the launch stays
    // below one workgroup per CU; else a share of the waves in proportion to its cost
    // (about two half-blocks' worth per unit, plus a start).
    int64_t n_tw = 0;
    bool extra_waves = false;
    if (tail_units > 0) {
      if (units == 0 || heads * (S + ceil_div64(tail_units, 4)) <= a.n_cu) {
        n_tw = tail_units;
        extra_waves = true;
      } else {
        n_tw = (4 * S * tail_cost + (units + tail_cost) / 2) / (units + tail_cost);
        if (n_tw < 1) n_tw = 1;
        if (n_tw > 4 * S - 1) n_tw = 4 * S - 1;
      }
      if (n_tw > tail_units) n_tw = tail_units;
      if (n_tw > 4 * kTailSplits) n_tw = 4 * kTailSplits;
    }
    if (units == 0) S = 0;
    a.tail_alone = 0;
    int64_t WG = S;
    if (extra_waves) {
      if (units > 0 && heads * (S + n_tw) <= a.n_cu && S + n_tw <= 32 && S + n_tw <= split_cap(q->B, q->H) + kTailSplits) {
        a.tail_alone = 1;            // plenty of idle CUs: a workgroup per tail unit, nothing else in it
        WG = S + n_tw;
      } else {
        WG = ceil_div64(4 * (int64_t)S + n_tw, 4);
      }
    }
    if (WG > 32) WG = 32;
    if (WG < 1) WG = 1;              // empty cache: one workgroup writes the zeros
    if (units == 0) n_tw = 4 * WG;   // every wave is a tail wave (those past the last unit idle)
    a.n_tw = (int)n_tw;
    a.n_pw = a.tail_alone ? (int)(4 * S) : (int)(4 * WG - n_tw);
    a.tw_full = (int)(n_tw / WG);
    a.tw_rem = (int)(n_tw % WG);
    a.pw_q = a.n_pw > 0 ? (int)(units / a.n_pw) : 0;
    a.pw_r = a.n_pw > 0 ? (int)(units % a.n_pw) : 0;
    a.tu_q = a.n_tw > 0 ? (int)(tail_units / a.n_tw) : 0;
    a.tu_r = a.n_tw > 0 ? (int)(tail_units % a.n_tw) : 0;
    S = (int)WG;
  }
  a.S = S;
  const int64_t nq = q->B * q->H;
  float* wsf = reinterpret_cast<float*>(ws);
  a.part_m = wsf;
  a.part_z = wsf + nq * S;
  a.part_o = wsf + 2 * nq * S;
  a.out = out;
  a.lse_out = lse_out;

  hipStream_t st = (hipStream_t)stream;
  return launch_decode_mfma(a, q->dtype, st);
}

extern "C" int zc_decode_attention(const zc_tensor4* q, const zc_packed* Kp, const zc_packed* Vp,
                                   const zc_tensor4* tail_k, const zc_tensor4* tail_v, int64_t tail_len,
                                   float sm_scale, void* out, float* lse_out,
                                   void* ws, size_t ws_bytes, void* stream) {
  return decode_entry(q, Kp, Vp, tail_k, tail_v, tail_len, sm_scale, out, lse_out, ws, ws_bytes, false, stream);
}

extern "C" int zc_decode_attention_static(const zc_tensor4* q, const zc_packed* Kp, const zc_packed* Vp,
                                          const zc_tensor4* tail_k, const zc_tensor4* tail_v, int64_t tail_len,
                                          float sm_scale, void* out, float* lse_out, void* stream) {
  return decode_entry(q, Kp, Vp, tail_k, tail_v, tail_len, sm_scale, out, lse_out, nullptr, 0, true, stream);
}
