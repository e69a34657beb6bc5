// zc_select_salient: exact top-k split of the token scores (Algorithm 2,
// "Split(., p~, r%)").  One workgroup per batch row (of few long rows up to
// eight, which share the writing: select_sliced): an MSB-first radix select
// on the order-preserving uint32 image of the scores finds the k-th largest
// key and how many tokens equal to it are taken (lowest indices first); one
// ordered compaction pass then writes both index lists in ascending order.
// Rows of up to 16384 tokens are kept in registers (k_select_small), of up to
// 34816, and many rows of more than 4096, in LDS (k_select_cached); longer rows
// are re-read from memory by every pass (k_select_stream).
#include <type_traits>

#include "zc_common.hpp"

namespace zc {

constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / 64;

constexpr int kSelMaxCached = 34816;     // keys of one row that fit the LDS of a CU next to the small arrays
// The digit histogram is kept in kSelRep copies, a lane adding to copy (lane mod kSelRep); the
// copies are 257 words apart, so they sit in different LDS banks.  Scores of one prompt share
// their exponent bits: with a single histogram all 64 lanes of a wave add to the same few
// words and the adds serialize (a pass over 32 k keys took 13 us that way).
constexpr int kSelRep = 16;
constexpr int kSelRepStride = 257;

// Which bin of a digit histogram holds the `need`-th largest key: threads 0..255 own a bin
// each (hist[tid] filled by its owner), suffix sums from the largest digit down; the owner of
// the one bin with (keys above) < need <= (keys above) + (keys in it) publishes the digit,
// what is still to take inside it and how many keys it holds.  Called by all threads; two barriers inside.
__device__ inline void pick_bin(const int* hist, int* wave_tot, int need, int tid, int* s_bin, int* s_need, int* s_cnt) {
  const int lane_ = tid & 63, wv = tid >> 6;
  int suf = 0;
  if (tid < 256) {
    suf = hist[tid];                               // becomes the sum of bins >= tid inside the wave
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_down(suf, o);
      if (lane_ + o < 64) suf += t;
    }
    if (lane_ == 0) wave_tot[wv] = suf;
  }
  __syncthreads();
  if (tid < 256) {
    for (int w2 = wv + 1; w2 < 4; ++w2) suf += wave_tot[w2];
    const int above = suf - hist[tid];             // keys in bins > tid
    if (above < need && suf >= need) {             // exactly one bin satisfies this
      *s_bin = tid;
      *s_need = need - above;
      *s_cnt = hist[tid];
    }
  }
  __syncthreads();
}

constexpr int kSelCand = 1024;                 // candidates one wave finishes the search on
// Few rows leave most CUs idle while one of them writes a row's lists, 64 entries a store to a few lines each: kSelSlices
// workgroups then repeat the search for the k-th key, which costs no time, and write an eighth of the lists each (a quarter of up to 4096
// tokens).  Rows of more than 2048 tokens, while a CU has one such workgroup at most.  us per launch, one workgroup a row and
// eight, one row and 32 rows, k = 0.4 L: 2500 tokens 5.3 / 5.65 and 5.1 / 5.3; 4096 5.5 / 5.9 and 5.2 / 5.5; 8192 7.2 / 7.7 and 6.5 / 6.8; 16384 12.7 /
// 13.2 and 10.7 / 11.1; 21108 18.0 / 18.6 and 15.5 / 15.9; 32768 20.7 / 21.4 and 16.5 / 17.1 (15.9 / 16.6 with four loads requested at once).
constexpr int kSelSlices = 8;
static bool select_sliced(int64_t B) { return B * kSelSlices <= 256; }
constexpr int kSelPieces = 136;                // of 256 tokens: kSelMaxCached
constexpr int kSelBufFlags = 0x00020000;       // buffer descriptor: raw 32-bit data, no swizzle
constexpr int kSelDropped = (int)0xFFFFF000u;  // a store offset past the end of every output: the store is dropped

// The row's keys live in LDS, four to a 16-byte word (the row padded to a multiple of 256 with
// key 0, which lies below the key of every number: -inf maps to 0x007fffff).
//   1. load: scores -> keys -> LDS, and the smallest and largest key of the row.  Their common
//      leading bits are decided already: the radix passes start at the first bit in which two
//      keys of the row differ (scores of one prompt share sign and most exponent bits - a pass
//      over those bits would put every key into one or two bins).
//   2. radix passes of eight bits by the whole workgroup, until the chosen bin holds at most
//      kSelCand keys (normally after the first) or no bit is left.
//   3. one sweep in which every wave counts, in its run of consecutive tokens, the keys above
//      the chosen bin and collects those inside it (the candidates).
//   4. wave 0 alone finishes the radix select on the candidates - no barriers - and adds, per
//      run, how many candidates lie above the k-th key and how many equal it.
//   5. ordered compaction: a lane owns four consecutive tokens, a wave its run; the index lists
//      are written through buffer descriptors, a store that does not apply (the other list's,
//      a pad's) being pointed past the end of its buffer, where it is dropped.
// VEC: the row starts on a 16-byte boundary (16-byte loads of the scores).
// SLICED: gridDim.y workgroups share a row: each finds the k-th key for itself (one CU's chain of steps either way) and
// compacts pieces of 256 tokens of its own, whose counts are kept per piece.
template <bool VEC, bool SLICED>
__global__ __launch_bounds__(kSelThreads) void k_select_cached(
    const float* __restrict__ scores, int L, int k, int32_t* __restrict__ salient,
    int32_t* __restrict__ regular, uint8_t* __restrict__ mask) {
  extern __shared__ uint4 skeys4[];       // the row's keys
  __shared__ __align__(16) int hist[256];
  __shared__ __align__(16) int hrep[kSelRep * kSelRepStride];   // histogram copies; then the candidates
  __shared__ int s_bin, s_need, s_cnt, s_ncand;
  __shared__ uint32_t s_thr;
  __shared__ int s_wave_gt[kSelWaves], s_wave_eq[kSelWaves];
  __shared__ uint32_t s_wave_min[kSelWaves], s_wave_max[kSelWaves];
  __shared__ int s_piece[SLICED ? kSelPieces : 1];             // low half: keys above the k-th, high half: equal to it
  static_assert(kSelCand * 2 <= kSelRep * kSelRepStride && kSelWaves * 256 <= kSelRep * kSelRepStride,
                "the candidates and the compaction stages reuse the histogram copies");

  const int b = blockIdx.x;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float* sc = scores + (int64_t)b * L;
  const int n4 = ((L + 255) & ~255) >> 2;            // 16-byte words of keys, pads included

  // ---- 1. load ----------------------------------------------------------------
  for (int i = tid; i < kSelRep * kSelRepStride; i += kSelThreads) hrep[i] = 0;
  if (tid == 0) s_ncand = 0;
  uint32_t kmin = 0xffffffffu, kmax = 0u;
  int c0 = tid;
  if constexpr (VEC) {                               // four words requested at once (one workgroup a row, 32768 tokens 21.5 -> 20.6 us)
    for (; c0 + 3 * kSelThreads < L >> 2; c0 += 4 * kSelThreads) {
      float4 t[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) t[u] = reinterpret_cast<const float4*>(sc)[c0 + u * kSelThreads];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint4 kk = make_uint4(float_key(t[u].x), float_key(t[u].y), float_key(t[u].z), float_key(t[u].w));
        kmin = min(min(kmin, min(kk.x, kk.y)), min(kk.z, kk.w));
        kmax = max(max(kmax, max(kk.x, kk.y)), max(kk.z, kk.w));
        skeys4[c0 + u * kSelThreads] = kk;
      }
    }
  }
  for (int c = c0; c < n4; c += kSelThreads) {
    const int i = 4 * c;
    uint32_t kk[4] = {0u, 0u, 0u, 0u};
    if (i + 3 < L) {
      float f[4];
      if constexpr (VEC) {
        const float4 t = reinterpret_cast<const float4*>(sc)[c];
        f[0] = t.x; f[1] = t.y; f[2] = t.z; f[3] = t.w;
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) f[u] = sc[i + u];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        kk[u] = float_key(f[u]);
        kmin = min(kmin, kk[u]); kmax = max(kmax, kk[u]);
      }
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (i + u < L) {
          kk[u] = float_key(sc[i + u]);
          kmin = min(kmin, kk[u]); kmax = max(kmax, kk[u]);
        }
    }
    skeys4[c] = make_uint4(kk[0], kk[1], kk[2], kk[3]);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    kmin = min(kmin, (uint32_t)__shfl_xor((int)kmin, o));
    kmax = max(kmax, (uint32_t)__shfl_xor((int)kmax, o));
  }
  if (lane == 0) { s_wave_min[wave] = kmin; s_wave_max[wave] = kmax; }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kSelWaves; ++w) { kmin = min(kmin, s_wave_min[w]); kmax = max(kmax, s_wave_max[w]); }
  // (values every lane holds alike are moved to scalar registers, here and below: what is
  // computed from them then costs no vector instruction)
  kmin = __builtin_amdgcn_readfirstlane(kmin);
  kmax = __builtin_amdgcn_readfirstlane(kmax);

  // ---- 2. radix passes by the whole workgroup ----------------------------------------
  const uint32_t diff = kmin ^ kmax;
  int lo = diff ? 32 - __clz(diff) : 0;              // the low `lo` bits are undecided
  uint32_t prefix = lo >= 32 ? 0u : ((kmax >> lo) << lo);
  int need = k;          // how many still to take among keys matching the prefix
  if (k > 0 && k < L) {
    bool first = true;
    while (lo > 0) {
      const int top = lo;
      lo = top > 8 ? top - 8 : 0;
      const uint32_t hi_mask = top >= 32 ? 0u : (0xffffffffu << top);
      const uint32_t dmask = (1u << (top - lo)) - 1u;
      if (!first) {
        for (int i = tid; i < kSelRep * kSelRepStride; i += kSelThreads) hrep[i] = 0;
        __syncthreads();
      }
      first = false;
      int* mine = &hrep[(tid & (kSelRep - 1)) * kSelRepStride];
      for (int c = tid; c < n4; c += kSelThreads) {
        const uint4 kk = skeys4[c];
        // (a pad matches only an all-zero prefix and then falls into bin 0, below every key)
        if ((kk.x & hi_mask) == prefix) atomicAdd(&mine[(kk.x >> lo) & dmask], 1);
        if ((kk.y & hi_mask) == prefix) atomicAdd(&mine[(kk.y >> lo) & dmask], 1);
        if ((kk.z & hi_mask) == prefix) atomicAdd(&mine[(kk.z >> lo) & dmask], 1);
        if ((kk.w & hi_mask) == prefix) atomicAdd(&mine[(kk.w >> lo) & dmask], 1);
      }
      __syncthreads();
      if (tid < 256) {
        int h = 0;
#pragma unroll
        for (int r = 0; r < kSelRep; ++r) h += hrep[r * kSelRepStride + tid];
        hist[tid] = h;                               // (read back by this thread only)
      }
      pick_bin(hist, s_wave_gt, need, tid, &s_bin, &s_need, &s_cnt);
      prefix |= (uint32_t)__builtin_amdgcn_readfirstlane(s_bin) << lo;
      need = __builtin_amdgcn_readfirstlane(s_need);
      const int in_bin = __builtin_amdgcn_readfirstlane(s_cnt);       // (pads included when the bin is the lowest of all)
      __syncthreads();
      if (in_bin <= kSelCand) break;
    }
  }
  // Tokens with key > thr_gt are salient; of those equal to thr_eq, the first `need` by index.
  // k == 0 takes none, k == L takes all (every key of a number lies above 0).
  uint32_t thr_gt = prefix, thr_eq = prefix;
  if (k >= L) { thr_gt = 0u; thr_eq = 0xffffffffu; need = 0; lo = 0; }
  if (k <= 0) { thr_gt = 0xffffffffu; thr_eq = 0xffffffffu; need = 0; lo = 0; }

  // ---- 3. per run: keys above the chosen bin, keys inside it ----------------------------
  const int seg = (((L + kSelWaves - 1) / kSelWaves) + 255) & ~255;   // tokens per wave, whole pieces
  const int i0 = min(wave * seg, L), i1 = min(i0 + seg, L);
  const bool collect = lo > 0;                      // bits left: the keys inside the bin are candidates
  uint2* cand = reinterpret_cast<uint2*>(hrep);     // (key, run)
  {
    const uint32_t pg = thr_gt >> lo, pe = thr_eq >> lo;
    int cnt = 0;                                    // low half: keys above, high half: keys equal (no bits left)
    if constexpr (SLICED) { if (tid < kSelPieces) s_piece[tid] = 0; }      // (a wave's own are written after this barrier)
    if constexpr (SLICED) __syncthreads();
    auto piece = [&](auto whole_c, int base) {
      constexpr bool WHOLE = decltype(whole_c)::value;              // no pad in this piece
      const uint4 kk = skeys4[(base >> 2) + lane];
      const int i = base + 4 * lane;
      const uint32_t k4[4] = {kk.x, kk.y, kk.z, kk.w};
      bool in[4];
      int nin = 0;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t t = k4[u] >> lo;
        cnt += t > pg ? 1 : 0;                       // (a pad is never above: its key is 0)
        in[u] = WHOLE ? t == pe : (t == pe && i + u < i1);
        nin += in[u] ? 1 : 0;
      }
      if (!collect) cnt += nin << 16;
      else if (__ballot(nin != 0)) {                 // wave-uniform; rare: a bin holds a small part of the row
        const int incl = wave_inclusive_sum(nin);
        int at = 0;
        if (lane == 63) at = atomicAdd(&s_ncand, incl);
        at = __builtin_amdgcn_readlane(at, 63) + incl - nin;
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (in[u]) cand[at++] = make_uint2(k4[u], SLICED ? (uint32_t)base >> 8 : (uint32_t)wave);
      }
      if constexpr (SLICED) {
        const int all = wave_inclusive_sum(cnt);
        if (lane == 63) s_piece[base >> 8] = all;
        cnt = 0;
      }
    };
    for (int base = i0; base < i1; base += 256) {
      if (base + 256 <= i1) piece(std::true_type{}, base);
      else piece(std::false_type{}, base);
    }
    // (a wave's run has at most 34816 / 16 rounded up to 256 = 2304 tokens: the halves cannot carry)
    if constexpr (!SLICED) {
      cnt = __builtin_amdgcn_readlane(wave_inclusive_sum(cnt), 63);
      if (lane == 0) { s_wave_gt[wave] = cnt & 0xffff; s_wave_eq[wave] = cnt >> 16; }
    }
  }
  __syncthreads();

  // ---- 4. wave 0 finishes the search on the candidates --------------------------------------
  if (collect) {
    if (wave == 0) {
      const int n = __builtin_amdgcn_readfirstlane(s_ncand);          // <= kSelCand: the chosen bin's count bounds it
      const int nq = (n + 63) >> 6;
      // the candidates in registers, 16 a lane at most; an unused place holds a key that differs
      // from the prefix in the decided bits and so never matches below
      uint32_t ck[kSelCand / 64];
#pragma unroll
      for (int q = 0; q < kSelCand / 64; ++q) {
        ck[q] = ~prefix;
        if (q < nq && q * 64 + lane < n) ck[q] = cand[q * 64 + lane].x;
      }
      int top = lo, nd = need;
      uint32_t pre = prefix;
      while (top > 0) {
        const int lo2 = top > 8 ? top - 8 : 0;
        const uint32_t dm = (1u << (top - lo2)) - 1u;
        reinterpret_cast<int4*>(hist)[lane] = make_int4(0, 0, 0, 0);
#pragma unroll
        for (int q = 0; q < kSelCand / 64; ++q)
          if (q < nq && (ck[q] >> top) == (pre >> top)) atomicAdd(&hist[(ck[q] >> lo2) & dm], 1);
        // (LDS serves a wave's requests in order; the compiler must not move the read up)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const int4 h = reinterpret_cast<const int4*>(hist)[lane];      // bins 4 lane .. 4 lane + 3
        const int incl = wave_inclusive_sum(h.x + h.y + h.z + h.w);
        const int a3 = __builtin_amdgcn_readlane(incl, 63) - incl;    // candidates in bins above this lane's
        const int a2 = a3 + h.w, a1 = a2 + h.z, a0 = a1 + h.y;
        int d = -1, rest = 0;
        if (a3 < nd && nd <= a3 + h.w) { d = 3; rest = nd - a3; }
        else if (a2 < nd && nd <= a2 + h.z) { d = 2; rest = nd - a2; }
        else if (a1 < nd && nd <= a1 + h.y) { d = 1; rest = nd - a1; }
        else if (a0 < nd && nd <= a0 + h.x) { d = 0; rest = nd - a0; }
        const int owner = __builtin_ctzll(__ballot(d >= 0));          // exactly one lane owns the bin
        const int bin = __builtin_amdgcn_readlane(4 * lane + d, owner);
        nd = __builtin_amdgcn_readlane(rest, owner);
        pre |= (uint32_t)bin << lo2;
        top = lo2;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      }
      for (int j = lane; j < n; j += 64) {
        const uint2 c = cand[j];
        if constexpr (SLICED) {
          if (c.x >= pre) atomicAdd(&s_piece[c.y], c.x > pre ? 1 : 0x10000);
        } else if (c.x > pre) atomicAdd(&s_wave_gt[c.y], 1);
        else if (c.x == pre) atomicAdd(&s_wave_eq[c.y], 1);
      }
      if (lane == 0) { s_thr = pre; s_need = nd; }
    }
    __syncthreads();
    thr_gt = thr_eq = __builtin_amdgcn_readfirstlane(s_thr);
    need = __builtin_amdgcn_readfirstlane(s_need);
  }

  // ---- 5. ordered compaction -------------------------------------------------------
  int run_gt = 0, run_eq = 0;
  if constexpr (!SLICED)
    for (int w = 0; w < wave; ++w) { run_gt += s_wave_gt[w]; run_eq += s_wave_eq[w]; }
  run_gt = __builtin_amdgcn_readfirstlane(run_gt);
  run_eq = __builtin_amdgcn_readfirstlane(run_eq);
  const auto rs_sal = __builtin_amdgcn_make_buffer_rsrc(salient + (int64_t)b * k, 0, (uint32_t)k * 4u, kSelBufFlags);
  const auto rs_reg = __builtin_amdgcn_make_buffer_rsrc(regular + (int64_t)b * (L - k), 0, (uint32_t)(L - k) * 4u, kSelBufFlags);
  uint8_t* mk = mask ? mask + (int64_t)b * L : nullptr;
  const bool mk_words = (reinterpret_cast<uintptr_t>(mk) & 3) == 0;
  // A lane classifies four consecutive tokens, but consecutive lanes must write consecutive
  // list entries (a store instruction costs what the number of memory lines it touches costs):
  // the tokens of a piece go to a 256-word stage of the wave in list order - the salient ones,
  // then the others - and leave it 64 consecutive words at a time.
  int32_t* stage = hrep + wave * 256;               // (the candidates are no longer needed)
  const int first = SLICED ? 256 * (int)(blockIdx.y * kSelWaves + wave) : i0, end = SLICED ? L : i1;
  const int stride = SLICED ? 256 * kSelWaves * (int)gridDim.y : 256;
  for (int base = first; base < end; base += stride) {
    if constexpr (SLICED) {                          // what the pieces before this one hold (halves of 16 bits: no more than 34816 tokens)
      uint32_t before = 0u;
#pragma unroll
      for (int u = 0; u < (kSelPieces + 63) / 64; ++u) before += 64 * u + lane < base >> 8 ? (uint32_t)s_piece[min(64 * u + lane, kSelPieces - 1)] : 0u;
      before = (uint32_t)__builtin_amdgcn_readlane(wave_inclusive_sum((int)before), 63);
      run_gt = (int)(before & 0xffffu);
      run_eq = (int)(before >> 16);
    }
    const uint4 kk = skeys4[(base >> 2) + lane];
    const int i = base + 4 * lane;
    const uint32_t k4[4] = {kk.x, kk.y, kk.z, kk.w};
    bool gt[4], eq[4];                               // (a pad is neither: thr_eq is the key of a number, or ~0)
    int mine = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      gt[u] = k4[u] > thr_gt;
      eq[u] = k4[u] == thr_eq;
      mine += (gt[u] ? 1 : 0) + (eq[u] ? 0x10000 : 0);
    }
    const int incl = wave_inclusive_sum(mine);
    const int total = __builtin_amdgcn_readlane(incl, 63);
    const int sal0 = run_gt + min(run_eq, need);                      // salient tokens before this piece
    const int nsal = run_gt + (total & 0xffff) + min(run_eq + (total >> 16), need) - sal0;   // ... inside it
    int eq_before = run_eq + ((incl - mine) >> 16);
    int p = run_gt + ((incl - mine) & 0xffff) + min(eq_before, need) - sal0;   // salient before this token, inside the piece
    uint32_t mbytes = 0u;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      // (no token of the piece equals the k-th key, nearly always: then salient means above it)
      const bool is_sal = gt[u] || (eq[u] && eq_before < need);
      stage[is_sal ? p : nsal + (4 * lane + u - p)] = i + u;
      mbytes |= (is_sal ? 1u : 0u) << (8 * u);
      p += is_sal ? 1 : 0;
      eq_before += eq[u] ? 1 : 0;
    }
    if (mk) {
      if (mk_words && base + 256 <= L) *reinterpret_cast<uint32_t*>(mk + i) = mbytes;
      else {
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (i + u < L) mk[i + u] = (uint8_t)((mbytes >> (8 * u)) & 1u);
      }
    }
    // (LDS serves a wave's requests in order; the compiler must keep the order too)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // An entry past the end of its list is dropped by the buffer's range check: a pad (token
    // >= L, "regular", only at the end of the row) lands at an index >= L - k.
    const int reg0 = base - sal0 - nsal;              // list index of the piece's first regular token, minus nsal
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int j = 64 * u + lane;
      const uint32_t tok = (uint32_t)stage[j];
      if (64 * u < nsal)                             // wave-uniform: some of these 64 are salient
        __builtin_amdgcn_raw_buffer_store_b32(tok, rs_sal, j < nsal ? 4 * (sal0 + j) : kSelDropped, 0, 0);
      if (64 * u + 64 > nsal)                        // ... some are not
        __builtin_amdgcn_raw_buffer_store_b32(tok, rs_reg, j < nsal ? kSelDropped : 4 * (reg0 + j), 0, 0);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    run_gt += total & 0xffff;
    run_eq += total >> 16;
  }
}

// ---- rows of up to kSelSmallMax tokens: keys in registers ------------------------------------
// Nothing here is bound by memory or arithmetic: a row is one workgroup's chain of barriers, LDS
// round trips and instruction fetches (code is cold at every launch, about half a microsecond a
// KB).  So the kernel is short (1.8 KB for 256 tokens, 5 for 4096, of which rows without many keys
// in one digit execute 3.7) and a workgroup no larger
// than its row: up to four keys a thread (8 and 16 where 1024 threads need them) in coalesced
// loads (a wave's run is 64 KPT consecutive tokens, lane l holds tokens 64 u + l of it), digits
// that give a thread two bins, so that one pass usually leaves few enough candidates for a
// bisection with ballots, and the positions in both lists from ballots, stored as they are.
// us per launch, k_select_cached -> here, k = 0.4 L: 100 tokens 6.7 -> 3.3; 1000: 6.9 -> 4.0; 2048:
// 7.4 -> 4.5; 4096: 8.5 -> 5.6; 8192: 10.4 -> 7.4; 16384: 14.3 -> 12.5; with nine tenths of the scores
// equal 4096: 9.3 -> 5.1; 16384: 16.2 -> 11.6.  At 32768 tokens 32 keys a thread are 20 KB of code: 21.9
// against 20.3, so the longer rows stay there.  So do rows of more than 4096 tokens once there are
// more of them than the chip runs at a time and the threads are not full: of more than 8192 from 257
// rows on, while two workgroups of k_select_cached share a CU's LDS (512 rows of 9000: 17.6 against
// 21.9, of 15600: 24.8 and 28.5, but of 15900: 34.2 and 29.1; 256 rows of 12000: 14.3 and 12.6); of fewer
// from 769 on (4096 of 6000: 89 and 97; 1024: 26.1 and 27.1; 768 of 5000: 21.2 and 20.0).

constexpr int kSelSmallMax = 16384;            // 16 keys a thread, 1024 threads
constexpr int kSelPairMax = 15616;             // tokens of which k_select_cached fits a CU twice
static bool select_small(int64_t B, int64_t L) {
  if (L <= 4096) return true;
  return L <= kSelSmallMax && !(L <= kSelPairMax && B > (L > 8192 ? 256 : 768));
}
constexpr int kKthMax = 256;                   // candidates of the bisection, at most
constexpr int kSharedDigits = 7;               // lanes of 64 that may share a digit with the lane before them

// The need-th largest of a wave's keys, N a lane, that agree in every bit at and above `lo` with
// `prefix`; unused places hold 0 (below every probed threshold).  Returns the key; `need` becomes
// how many keys equal to it are taken.  Every lane of the wave gets the same answer.
template <int N>
__device__ inline uint32_t kth_of_wave(const uint32_t (&c)[N], uint32_t prefix, int lo, int& need) {
  uint32_t t = prefix;
  auto count_ge = [&](uint32_t v) {
    int n = 0;
#pragma unroll
    for (int u = 0; u < N; ++u) n += __builtin_popcountll(__builtin_amdgcn_ballot_w64(c[u] >= v));
    return n;
  };
#pragma unroll 1
  for (int bit = lo - 1; bit >= 0; --bit) {
    const uint32_t probe = t | (1u << bit);
    if (count_ge(probe) >= need) t = probe;
  }
  if (t != 0xffffffffu) need -= count_ge(t + 1u);
  return t;
}

__device__ inline uint32_t wave_or(uint32_t x) {        // OR over the wave (the steps of wave_inclusive_sum)
  int v = (int)x;
  v |= __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true);
  v |= __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true);
  v |= __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true);
  v |= __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true);
  v |= __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);
  v |= __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);
  return (uint32_t)__builtin_amdgcn_readlane(v, 63);
}

__device__ inline int lanes_below(uint64_t mask) {      // set bits below this lane
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
}

// One more in hist[digit] for every key of a wave that matches the prefix.  Adds of a wave to one
// word go one after the other, and a row may hold one value thousands of times (columns that no
// probe sees) or many keys that share a digit.  SHARED: where lanes next to each other share one
// (looked for in their first keys only), the wave's keys of that digit are counted by ballots and
// added at once.  Nine tenths of equal scores, together with skipping the bits that all candidates
// share: 4096 tokens 14.0 -> 5.1 us, 16384 46.4 -> 11.6; the look costs 0.1 us (4096 tokens 5.5 -> 5.6).
template <bool SHARED, int KPT>
__device__ inline void count_digits(int* hist, const uint32_t (&key)[KPT], int lane, uint32_t prefix, uint32_t above, int lo, uint32_t dmask) {
  const int mine = (int)((key[0] >> lo) & dmask);
  uint64_t shared = 0;
  if constexpr (SHARED) {
    const uint64_t in = __builtin_amdgcn_ballot_w64((key[0] & above) == prefix);
    const int left = __builtin_amdgcn_update_dpp(-1, mine, 0x111, 0xF, 0xF, false);            // row_shr:1
    shared = __builtin_amdgcn_ballot_w64(left == mine) & in & in << 1;
  }
  if (__builtin_expect(__builtin_popcountll(shared) <= kSharedDigits, 1)) {
#pragma unroll
    for (int u = 0; u < KPT; ++u)
      if ((key[u] & above) == prefix) atomicAdd(&hist[(key[u] >> lo) & dmask], 1);
    return;
  }
  // (the two digits found first: of others there are few each)
  const int one = __builtin_amdgcn_readlane(mine, __builtin_ctzll(shared));
  shared &= ~__builtin_amdgcn_ballot_w64(mine == one);
  const int two = shared ? __builtin_amdgcn_readlane(mine, __builtin_ctzll(shared)) : -2;
  int n1 = 0, n2 = 0;
#pragma unroll
  for (int u = 0; u < KPT; ++u) {
    const int d = (key[u] & above) == prefix ? (int)((key[u] >> lo) & dmask) : -1;
    n1 += __builtin_popcountll(__builtin_amdgcn_ballot_w64(d == one));
    n2 += __builtin_popcountll(__builtin_amdgcn_ballot_w64(d == two));
    if (d >= 0 && d != one && d != two) atomicAdd(&hist[d], 1);
  }
  if (lane == 0) {
    atomicAdd(&hist[one], n1);
    if (two >= 0) atomicAdd(&hist[two], n2);
  }
}

// One wave (THREADS == 64): no LDS, no barrier, the bisection over all keys.  SLICES workgroups (grid.y) share a row: each finds
// the k-th key for itself and stores KPT / SLICES keys a thread.
template <int THREADS, int KPT, int SLICES>
__global__ __launch_bounds__(THREADS) void k_select_small(
    const float* __restrict__ scores, int L, int k, int32_t* __restrict__ salient,
    int32_t* __restrict__ regular, uint8_t* __restrict__ mask) {
  constexpr bool ONE_WAVE = THREADS == 64;
  constexpr bool MANY = THREADS > 256;           // (in four waves the adds are few: that code would cost more than they do)
  constexpr int NWAVE = THREADS / 64, RUN = 64 * KPT;
  constexpr int BINS = 2 * THREADS, DIGIT = __builtin_ctz(BINS);    // two bins a thread
  __shared__ __align__(16) int hist[ONE_WAVE ? 1 : BINS];
  __shared__ uint32_t cand[ONE_WAVE ? 1 : kKthMax];
  __shared__ int s_wave[NWAVE], s_bin, s_need, s_cnt, s_ncand;
  __shared__ uint32_t s_diff[NWAVE], s_same[NWAVE];

  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int wave = ONE_WAVE ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6);
  const float* sc = scores + (int64_t)b * L;
  const int i0 = wave * RUN + lane;
  uint32_t key[KPT], diff = 0u;
  const uint32_t key0 = float_key(sc[0]);
#pragma unroll
  for (int u = 0; u < KPT; ++u) key[u] = float_key(sc[min(i0 + 64 * u, L - 1)]);
#pragma unroll
  for (int u = 0; u < KPT; ++u) diff |= key[u] ^ key0;           // (a repeated last token adds nothing)
#pragma unroll
  for (int u = 0; u < KPT; ++u)
    if (i0 + 64 * u >= L) key[u] = 0u;

  // Tokens with key > thr are salient; of those equal to it, the first `need` by index.
  uint32_t thr;
  int need = k;
  if (k <= 0) { thr = 0xffffffffu; need = 0; }
  else if (k >= L) { thr = 0u; need = L; }                     // (every valid token is above or equal)
  else {
    // the bits in which two keys of the row differ
    diff = wave_or(diff);
    if constexpr (!ONE_WAVE) {
      if (lane == 0) s_diff[wave] = diff;
      reinterpret_cast<int2*>(hist)[tid] = make_int2(0, 0);
      if (tid == 0) s_ncand = 0;
      __syncthreads();
      diff = wave_or(s_diff[lane & (NWAVE - 1)]);
    }
    int lo = diff ? 32 - __clz(diff) : 0;                      // the low `lo` bits are undecided
    thr = lo >= 32 ? 0u : __builtin_amdgcn_readfirstlane(key0) & (0xffffffffu << lo);
    if constexpr (ONE_WAVE) {
      thr = kth_of_wave(key, thr, lo, need);
    } else {
      int in_bin = L;
#pragma unroll 1
      for (bool first = true; lo > 0 && in_bin > kKthMax; first = false) {
        if (MANY && __builtin_expect(!first, 0)) {
          // Many keys in one digit: equal ones, or close ones beside one far away.  The bits that all of
          // them share are decided.
          uint32_t ones = 0u, zeros = 0u;
          const uint32_t above = 0xffffffffu << lo;            // (lo < 32 after a pass)
#pragma unroll
          for (int u = 0; u < KPT; ++u)
            if ((key[u] & above) == thr) { ones |= key[u]; zeros |= ~key[u]; }
          ones = wave_or(ones);
          zeros = wave_or(zeros);
          if (lane == 0) { s_diff[wave] = ones; s_same[wave] = zeros; }
          __syncthreads();
          ones = wave_or(s_diff[lane & (NWAVE - 1)]);
          zeros = wave_or(s_same[lane & (NWAVE - 1)]);
          const uint32_t differ = ones & zeros & ~above;
          lo = differ ? 32 - __clz(differ) : 0;
          thr = ones & (0xffffffffu << lo);
          if (lo == 0) break;
        }
        const int top = lo;
        lo = max(top - DIGIT, 0);
        // (a pad's key of 0 lies below every number's; it matches a prefix of zeros and adds to digit 0)
        count_digits<MANY>(hist, key, lane, thr, top >= 32 ? 0u : 0xffffffffu << top, lo, (1u << (top - lo)) - 1u);
        __syncthreads();
        // keys above each bin: thread t owns bins BINS - 1 - 2 t and the one below it
        const int2 h = reinterpret_cast<const int2*>(hist)[BINS / 2 - 1 - tid];
        const int incl = wave_inclusive_sum(h.x + h.y);
        if (lane == 63) s_wave[wave] = incl;
        __syncthreads();
        // (cleared for the next pass, which the next barrier separates from it)
        reinterpret_cast<int2*>(hist)[BINS / 2 - 1 - tid] = make_int2(0, 0);
        int before = lane < wave ? s_wave[lane] : 0;
        before = __builtin_amdgcn_readlane(wave_inclusive_sum(before), 63);
        const int a0 = before + incl - h.x - h.y, a1 = a0 + h.y;      // keys above the upper bin, above the lower
        if (a0 < need && need <= a1 + h.x) {                   // exactly one thread
          const bool upper = need <= a1;
          s_bin = BINS - 1 - 2 * tid - (upper ? 0 : 1);
          s_need = need - (upper ? a0 : a1);
          s_cnt = upper ? h.y : h.x;
        }
        __syncthreads();
        thr |= (uint32_t)__builtin_amdgcn_readfirstlane(s_bin) << lo;
        need = __builtin_amdgcn_readfirstlane(s_need);
        in_bin = __builtin_amdgcn_readfirstlane(s_cnt);
      }
      if (lo > 0) {                                            // the keys of the bin: candidates of the bisection
#pragma unroll
        for (int u = 0; u < KPT; ++u)
          if ((key[u] & 0xffffffffu << lo) == thr) cand[atomicAdd(&s_ncand, 1)] = key[u];
        __syncthreads();
        // (by every wave for itself: no barrier)
        if (in_bin <= 64) {
          const uint32_t c[1] = {lane < in_bin ? cand[lane] : 0u};
          thr = kth_of_wave(c, thr, lo, need);
        } else {
          uint32_t c[kKthMax / 64];
#pragma unroll
          for (int u = 0; u < kKthMax / 64; ++u) c[u] = 64 * u + lane < in_bin ? cand[64 * u + lane] : 0u;
          thr = kth_of_wave(c, thr, lo, need);
        }
      }
    }
  }

  // ---- positions in both lists --------------------------------------------------------------
  uint64_t gt[KPT], eq[KPT];
  int ngt = 0, neq = 0;
  asm volatile("" : "+s"(L));                                  // (or the comparisons with it are kept from the start on)
#pragma unroll
  for (int u = 0; u < KPT; ++u) {
    const bool valid = i0 + 64 * u < L;
    gt[u] = __builtin_amdgcn_ballot_w64(valid && key[u] > thr);
    eq[u] = __builtin_amdgcn_ballot_w64(valid && key[u] == thr);
    ngt += __builtin_popcountll(gt[u]);
    neq += __builtin_popcountll(eq[u]);
  }
  int run_gt = 0, run_eq = 0;                                  // salient candidates before this wave's run
  if constexpr (!ONE_WAVE) {
    if (lane == 0) s_wave[wave] = (int)((uint32_t)ngt | (uint32_t)neq << 16);
    __syncthreads();
    const int before = __builtin_amdgcn_readlane(wave_inclusive_sum(lane < wave ? s_wave[lane] : 0), 63);
    run_gt = before & 0xffff;
    run_eq = (uint32_t)before >> 16;
  }
  int32_t* sal = salient + (int64_t)b * k;
  int32_t* reg = regular + (int64_t)b * (L - k);
#pragma unroll
  for (int u = 0; u < KPT; ++u) {
    const int i = i0 + 64 * u;
    const int eq_before = run_eq + lanes_below(eq[u]);
    const bool is_sal = (gt[u] >> lane & 1) || ((eq[u] >> lane & 1) && eq_before < need);
    const int p = run_gt + lanes_below(gt[u]) + min(eq_before, need);
    if (i < L && (SLICES == 1 || u / (KPT / SLICES) == (int)blockIdx.y)) {
      int32_t* dst = is_sal ? sal + p : reg + (i - p);
      *dst = i;
      if (mask) mask[(int64_t)b * L + i] = is_sal ? 1 : 0;
    }
    run_gt += __builtin_popcountll(gt[u]);
    run_eq += __builtin_popcountll(eq[u]);
  }
}

// Rows too long for LDS: every pass reads the scores from memory.
__global__ __launch_bounds__(kSelThreads) void k_select_stream(
    const float* __restrict__ scores, int L, int k, int32_t* __restrict__ salient,
    int32_t* __restrict__ regular, uint8_t* __restrict__ mask) {
  __shared__ int hist[256];
  __shared__ int hrep[kSelRep * kSelRepStride];
  __shared__ int s_bin, s_need, s_cnt;
  __shared__ int s_wave_gt[kSelWaves], s_wave_eq[kSelWaves];

  const int b = blockIdx.x;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const float* sc = scores + (int64_t)b * L;
  int32_t* sal = salient + (int64_t)b * k;
  int32_t* reg = regular + (int64_t)b * (L - k);
  uint8_t* mk = mask ? mask + (int64_t)b * L : nullptr;
  const int seg = ((L + kSelWaves - 1) / kSelWaves + 63) & ~63;      // keys per wave, a multiple of 64
  const int i0 = min(wave * seg, L), i1 = min(i0 + seg, L);
  auto key_at = [&](int i) -> uint32_t { return float_key(sc[i]); };

  // ---- radix select of the k-th largest key ---------------------------------
  uint32_t prefix = 0;   // key bits decided so far (high bits)
  int need = k;          // how many still to take among keys matching the prefix
  if (k > 0 && k < L) {
    for (int pass = 0; pass < 4; ++pass) {
      const int shift = 24 - 8 * pass;
      const uint32_t hi_mask = pass == 0 ? 0u : (0xffffffffu << (shift + 8));
      for (int i = tid; i < kSelRep * kSelRepStride; i += kSelThreads) hrep[i] = 0;
      __syncthreads();
      int* mine = &hrep[(tid & (kSelRep - 1)) * kSelRepStride];
      for (int i = tid; i < L; i += 4 * kSelThreads) {      // four keys requested before the first add
        uint32_t k4[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) k4[u] = i + u * kSelThreads < L ? key_at(i + u * kSelThreads) : 0u;
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (i + u * kSelThreads < L && (k4[u] & hi_mask) == prefix) atomicAdd(&mine[(k4[u] >> shift) & 0xff], 1);
      }
      __syncthreads();
      if (tid < 256) {
        int h = 0;
#pragma unroll
        for (int r = 0; r < kSelRep; ++r) h += hrep[r * kSelRepStride + tid];
        hist[tid] = h;                               // (read back by this thread only)
      }
      pick_bin(hist, s_wave_gt, need, tid, &s_bin, &s_need, &s_cnt);
      prefix |= (uint32_t)s_bin << shift;
      need = s_need;
      __syncthreads();
    }
  }
  // Tokens with key > prefix are salient; of those equal to it, the first
  // `need` by index.  k == 0 takes none, k == L takes all.
  const bool take_all = (k >= L);
  const bool take_none = (k <= 0);

  // Ordered compaction without a barrier per step: every wave first counts the salient
  // candidates of its run (> and == the k-th key), the waves exchange the counts once, then
  // every wave writes its run in order from its own base offsets.
  auto classify = [&](int i, uint32_t key, bool& gt, bool& eq) {
    gt = false; eq = false;
    if (i < i1) {
      if (take_all) gt = true;
      else if (!take_none) { gt = key > prefix; eq = key == prefix; }
    }
  };
  int cnt_gt = 0, cnt_eq = 0;
  for (int base = i0; base < i1; base += 64) {
    bool gt, eq;
    const int i = base + lane;
    classify(i, (i < i1 && !take_all && !take_none) ? key_at(i) : 0u, gt, eq);
    cnt_gt += __popcll(__ballot(gt));
    cnt_eq += __popcll(__ballot(eq));
  }
  if (lane == 0) { s_wave_gt[wave] = cnt_gt; s_wave_eq[wave] = cnt_eq; }
  __syncthreads();
  int run_gt = 0, run_eq = 0;
  for (int w = 0; w < wave; ++w) { run_gt += s_wave_gt[w]; run_eq += s_wave_eq[w]; }
  const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  auto emit = [&](int i, uint32_t key) {
    bool gt, eq;
    classify(i, key, gt, eq);
    const uint64_t bgt = __ballot(gt), beq = __ballot(eq);
    const int gt_before = run_gt + __popcll(bgt & below);
    const int eq_before = run_eq + __popcll(beq & below);
    if (i < i1) {
      const bool is_sal = gt || (eq && eq_before < need);
      const int sal_before = gt_before + min(eq_before, need);
      if (is_sal) sal[sal_before] = i;
      else reg[i - sal_before] = i;
      if (mk) mk[i] = is_sal ? 1 : 0;
    }
    run_gt += __popcll(bgt);
    run_eq += __popcll(beq);
  };
  for (int base = i0; base < i1; base += 64) {
    const int i = base + lane;
    emit(i, (i < i1 && !take_all && !take_none) ? key_at(i) : 0u);
  }
}

}  // namespace zc

extern "C" size_t zc_select_salient_workspace(int64_t, int64_t) { return 0; }

extern "C" int zc_select_salient(const float* scores, int64_t B, int64_t L, int64_t k,
                                 int32_t* salient_idx, int32_t* regular_idx, uint8_t* mask,
                                 void* ws, size_t ws_bytes, void* stream) {
  (void)ws; (void)ws_bytes;
  if (B < 0 || L < 0 || k < 0 || k > L || L > 0x7fffffff || B > 65535 * 32) return ZC_ERR_INVALID_ARG;
  if (B == 0 || L == 0) return ZC_OK;
  if (!scores || (k > 0 && !salient_idx) || (k < L && !regular_idx)) return ZC_ERR_INVALID_ARG;
  if ((reinterpret_cast<uintptr_t>(scores) & 3) || (reinterpret_cast<uintptr_t>(salient_idx) & 3) ||
      (reinterpret_cast<uintptr_t>(regular_idx) & 3))
    return ZC_ERR_INVALID_ARG;
  if (zc::select_small(B, L)) {
    const auto launch = [&](auto kernel, unsigned threads, unsigned slices = 1) {
      hipLaunchKernelGGL(kernel, dim3((unsigned)B, slices), dim3(threads), 0, (hipStream_t)stream, scores, (int)L, (int)k, salient_idx, regular_idx, mask);
    };
    const bool sliced = zc::select_sliced(B);
    if (L <= 64 * 4) launch(zc::k_select_small<64, 4, 1>, 64);
    else if (L <= 256 * 4) launch(zc::k_select_small<256, 4, 1>, 256);
    else if (L <= 512 * 4) launch(zc::k_select_small<512, 4, 1>, 512);
    else if (L <= 1024 * 4 && sliced) launch(zc::k_select_small<1024, 4, 4>, 1024, 4);
    else if (L <= 1024 * 4) launch(zc::k_select_small<1024, 4, 1>, 1024);
    else if (L <= 1024 * 8 && sliced) launch(zc::k_select_small<1024, 8, 8>, 1024, 8);
    else if (L <= 1024 * 8) launch(zc::k_select_small<1024, 8, 1>, 1024);
    else if (sliced) launch(zc::k_select_small<1024, 16, 8>, 1024, 8);
    else launch(zc::k_select_small<1024, 16, 1>, 1024);
  } else if (L <= zc::kSelMaxCached) {
    const size_t lds = (size_t)((L + 255) & ~(int64_t)255) * sizeof(uint32_t);
    // rows start on 16-byte boundaries when the array does and L is a multiple of four (or B is 1)
    const bool vec = (reinterpret_cast<uintptr_t>(scores) & 15) == 0 && (B == 1 || (L & 3) == 0);
    const bool sliced = zc::select_sliced(B);
    const auto kernel = vec ? (sliced ? &zc::k_select_cached<true, true> : &zc::k_select_cached<true, false>)
                            : (sliced ? &zc::k_select_cached<false, true> : &zc::k_select_cached<false, false>);
    if (lds > 32 * 1024) {
      // a launch above the default dynamic-LDS limit needs the attribute raised (idempotent)
      if (hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)(zc::kSelMaxCached * sizeof(uint32_t))) != hipSuccess)
        return ZC_ERR_HIP;
    }
    hipLaunchKernelGGL(kernel, dim3((unsigned)B, sliced ? zc::kSelSlices : 1), dim3(zc::kSelThreads), lds,
                       (hipStream_t)stream, scores, (int)L, (int)k, salient_idx, regular_idx, mask);
  } else {
    hipLaunchKernelGGL(zc::k_select_stream, dim3((unsigned)B), dim3(zc::kSelThreads), 0,
                       (hipStream_t)stream, scores, (int)L, (int)k, salient_idx, regular_idx, mask);
  }
  ZC_LAUNCH_CHECK();
  return ZC_OK;
}
