// zc_probe_saliency: normalized attention score of every key token from a
// probe subset of query rows (Eq. 9 substituted into Eq. 8).
//
// The probe rows of A = Softmax(Q_probe K^T / sqrt(d)) are never stored.  Two
// matrix-core sweeps recompute the logits instead:
//   k_probe_lse     one workgroup per 128 probe rows and column range (the row blocks of a
//                   head share its workgroups by the columns they can see): the probe rows
//                   sit in registers as matrix operands, 64-column K tiles stream through
//                   LDS (global -> LDS transfers, the next tile's in flight), logits come
//                   out of the MFMA as D[column][row] so that every lane owns one probe row
//                   and keeps its running (reference, sum) in two registers; writes the
//                   pair per row and column range (sweep 2 joins the ranges of few probes,
//                   k_probe_lse_merge those of others).
//   k_probe_colsum  one workgroup per 128 key columns: K fragments stay in
//                   registers, 64-row probe tiles stream through LDS with their
//                   positions and log-sum-exps, logits come out as D[row][column] so
//                   that every lane owns one column and sums exp(logit - lse) over
//                   the rows in registers; divides by the number of probes that can
//                   see the column.
//   k_probe_mean    mean over query heads.
// Causality: rows are sorted by position, so a column tile starts at the first
// probe that can see it and a row tile stops at its last row's position.
// Inputs in fp16 / bf16 use the 32x32x16 MFMA, fp32 inputs the 32x32x2 fp32 MFMA
// (no rounding of the operands); accumulation and softmax are fp32.
// Both sweeps are bound by instruction issue: a wave's 32 x 64 logits take 16 matrix
// instructions and 32 triples (fma, exponential, add) a lane, which barely overlap, 0.6 us of
// a SIMD at the clock the chip holds, however many waves it has.  Small prompts are bound by
// how the work falls on the CUs and by the waves' start: 32 heads of 128 channels over 8, 4096
// tokens, 410 probe rows, bf16: 58.3 -> 44.1 us with operands brought in as whole rows, four
// workgroups a CU and row blocks sharing workgroups by the columns they see (sweep 1 26 -> 24 us,
// sweep 2 31.6 -> 19); 16384 tokens 390 -> 380.  Then 43.3 -> 38.5 by keeping the waves of a full chip at the
// same number of tiles to go (priority_by_tiles: 42.8 -> 39.6 in sweeps that a launch still joined), a mix of row
// blocks on every CU, 32 rows a wave for a last block of at most 64, what the probes are looked up by in LDS
// from one trip to memory, and sweep 2 joining the pairs of sweep 1; 16 x 40 heads, 4096 tokens: 645 -> 614;
// 8 heads of 64 channels, 700 tokens: 13.7 -> 12.1; 16 x 16 heads of 128, 500 tokens, fp32: 78.7 -> 61.7.
#include "mfma_tiles.hpp"

namespace zc {

constexpr int kProbeParts = 8;       // column ranges of a block of probe rows the workspace is sized for
constexpr int kMaxProbeParts = 12;   // most (what else they need is borrowed from the per-head scores, which come later)

constexpr int kProbeTable = 512;     // most probes whose positions, rows and log-sum-exps a workgroup keeps in LDS

struct ProbeArgs {
  const void* q;
  const void* k;
  int64_t q_sB, q_sH, q_sL, k_sB, k_sH, k_sL;
  int B, Hq, Hkv, G, Lk, Lq, P;
  const int32_t* probe_rows;
  const int32_t* probe_pos;
  float scale_log2;
  const float* lse_in;   // natural log, [B, Hq, P]; null: use lse2
  float* lse2;           // [B, Hq, P] log-sum-exp in log2 units: sweep 1's result
  float2* lse_part;      // (reference in log2 units, sum) of the column ranges: [B, Hq, max_parts, P], not joined [B, Hq, P, max_parts]
  int max_parts;         // not joined: even (a row's pairs are read two at a time)
  int join;              // 1: sweep 2 joins a row's pairs itself (lse2 is not written); 0: k_probe_lse_merge does
  int head_wgs;          // workgroups of a head in sweep 1 (one per row block: no column ranges)
  float* per_head;       // [B, Hq, Lk]
  // the waves of sweep 1 / sweep 2 are kept at about the same number of tiles to go from so many tiles / probe rows before
  // their ends on (0: not at all)
  int even1, even2;
  int whole1;            // sweep 1: whole tiles go past the general case
  int group;             // sweep 2: query heads whose columns an XCD takes from the first on together (0: a head after the other)
  int few_cols;          // few probe rows, sweep 2 and the mean in one launch: of so many times 16 columns a workgroup (0: not)
  int few_blocks;        // of so many blocks of 16 probe rows a wave
  int normalize;         // 1: divide a column's sum by the number of probes that see it (Eq. 8); 0: Eq. 7
};

// A copy the compiler knows nothing of: what is computed from it is computed where it is used, not
// kept in a register across a loop.
__device__ inline int opaque(int x) { asm volatile("" : "+v"(x)); return x; }

// N 32x32 results of one row of operands in LDS (row: the address of its chunk kh; chunk
// 2 kc + kh sits at slot (2 kc + kh) ^ swz, one exclusive or away: on the address itself, so the
// tiles start at a multiple of a row's size, kTileAlign) and N in registers.  An
// operand is requested two steps ahead: left to itself the compiler, short of registers, waits
// for each in front of the instructions that use it.
constexpr int kTileAlign = 512;                // the longest row
template <int DT, int N, int NKC>
__device__ inline void products(v16f (&acc)[2], uint32_t row, const u32x4 (&f)[2][NKC]) {
  using lds_u32x4 = __attribute__((address_space(3))) const u32x4;
  constexpr int kDsRead = 0x100, kMfma = 0x8, MPC = DT == ZC_F32 ? 4 * N : N;     // matrix instructions of a step
  row = (uint32_t)opaque((int)row);              // (or the addresses of two instances are formed in front of both)
#pragma unroll
  for (int n = 0; n < N; ++n)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[n][i] = 0.f;
  u32x4 a[2];
  a[0] = *reinterpret_cast<lds_u32x4*>(row);
  a[1] = *reinterpret_cast<lds_u32x4*>(row ^ 32);
  __builtin_amdgcn_sched_group_barrier(kDsRead, 2, 0);
#pragma unroll
  for (int kc = 0; kc < NKC; ++kc) {
    const u32x4 af = a[kc & 1];
#pragma unroll
    for (int n = 0; n < N; ++n) mma_chunk<DT>(acc[n], af, f[n][kc]);
    __builtin_amdgcn_sched_group_barrier(kMfma, MPC, 0);
    if (kc + 2 < NKC) {
      a[kc & 1] = *reinterpret_cast<lds_u32x4*>(row ^ ((kc + 2) << 5));
      __builtin_amdgcn_sched_group_barrier(kDsRead, 1, 0);
    }
  }
}

// The (reference, sum) pairs of a probe row's column ranges, and the log-sum-exp of all of them.
struct RowPairs {
  float2 v[kMaxProbeParts];
  __device__ void load(const ProbeArgs& a, int64_t head, int row) {
    const float2* src = a.lse_part + head * a.max_parts * a.P + row;
#pragma unroll
    for (int sp = 0; sp < kMaxProbeParts; ++sp)
      if (sp < a.max_parts) v[sp] = src[(int64_t)sp * a.P];
  }
  __device__ void load_row(const float2* src, int max_parts) {       // side by side, 16 bytes aligned
#pragma unroll
    for (int sp = 0; sp < kMaxProbeParts; sp += 2) {
      const float4 two = reinterpret_cast<const float4*>(src)[min(sp, max_parts - 2) / 2];
      v[sp] = make_float2(two.x, two.y);
      v[sp + 1] = make_float2(two.z, two.w);
    }
  }
  __device__ float joined(int max_parts) {
    float M = -INFINITY;
#pragma unroll
    for (int sp = 0; sp < kMaxProbeParts; ++sp) {
      if (sp >= kProbeParts && sp >= max_parts) v[sp] = make_float2(-INFINITY, 0.f);
      M = fmaxf(M, v[sp].x);
    }
    // (a range without a reference: 0 times 2^-inf)
    const float base = M > -INFINITY ? M : 0.f;
    float Z = 0.f;
#pragma unroll
    for (int sp = 0; sp < kMaxProbeParts; ++sp) Z = fmaf(v[sp].y, __builtin_amdgcn_exp2f(v[sp].x - base), Z);
    return M + log2f(Z);
  }
};

// Waves with more tiles to go first: of equal waves a SIMD serves the oldest, so that the youngest is left with
// most of its tiles when the others have ended, alone and waiting for each (32 heads, 4096 tokens, 410 probes:
// the median wave of sweep 1 ended at 14.7 us, the last at 23.1).  Where all workgroups run at once: of several
// rounds the ends should be spread, so that the starts of the next are (even_waves).
constexpr int kEvenTiles = 5;                  // with so many to go a wave leaves the highest priority
__device__ inline void priority_by_tiles(int left) {
  if (left > kEvenTiles) __builtin_amdgcn_s_setprio(3);
  else if (left >= 4) __builtin_amdgcn_s_setprio(2);
  else if (left >= 2) __builtin_amdgcn_s_setprio(1);
  else __builtin_amdgcn_s_setprio(0);
}

constexpr int kLseRows = 128;                  // probe rows per workgroup of sweep 1
constexpr int kLseCols = 64;                   // columns per K tile of sweep 1
constexpr int kBlockCols = 128;                // columns of a workgroup of sweep 2
static_assert(kLseCols <= kBlockCols, "the entry's check of the offsets past the end of k");

// The row blocks of a head share its a.head_wgs workgroups in proportion to the column tiles their
// rows can see (a block near the end of a prompt sees ten times those of one near its start; a
// last block of at most 64 rows counts half: its waves multiply 32 rows each), each at least
// one and at most a.max_parts.  Lane i of a wave holds block i.
struct LseShare { int block, part, parts, tiles; };      // block < 0: a workgroup without work
__device__ inline LseShare lse_share(const ProbeArgs& a, int nrb, int j) {
  LseShare s;
  const auto tiles_of = [&](int block) { return min(a.probe_pos[min(a.P, (block + 1) * kLseRows) - 1], a.Lk - 1) / kLseCols + 1; };
  if (nrb == 1 || a.head_wgs == nrb) {                   // nothing to share
    s.block = nrb == 1 ? 0 : j;
    s.part = j - s.block;
    s.parts = nrb == 1 ? a.head_wgs : 1;
    s.tiles = __builtin_amdgcn_readfirstlane(tiles_of(s.block));
    return s;
  }
  if (nrb > 64) {                                        // (more than 8192 probe rows: even ranges)
    s.parts = min(a.head_wgs / nrb, a.max_parts);
    s.block = j / s.parts; s.part = j % s.parts;
    if (s.block >= nrb) s.block = -1;
    else s.tiles = tiles_of(s.block);
    return s;
  }
  const int i = threadIdx.x & 63, tiles = i < nrb ? tiles_of(i) : 0;
  const int weight = a.P - i * kLseRows <= kLseRows / 2 ? (tiles + 1) / 2 : tiles;
  // One each, what is left by the cumulated tiles (the last block's: all of them, whatever the rounding).
  // Cut to whole numbers with a quarter added: without it two blocks that see 31 and 32 columns share
  // four workgroups as one and three (16 x 32 heads over 8 of 128 channels, the last 200 of 2000 rows, fp32:
  // 1585 us, 1110 with two each), with a half one more goes too early where shares grow (2 x 900 rows,
  // all of them probes, bf16: 43.5 and 45.8).  The best of 64 tried shares cost 0.4 us more than it gave.
  const int upto = wave_inclusive_sum(weight), from = upto - weight, total = __builtin_amdgcn_readlane(upto, 63);
  const float rate = (float)(a.head_wgs - nrb) / (float)total;
  const auto shared_by = [&](int t) { return t == total ? a.head_wgs - nrb : min((int)fmaf((float)t, rate, 0.25f), a.head_wgs - nrb); };
  const int share = i < nrb ? min(1 + max(shared_by(upto) - shared_by(from), 0), a.max_parts) : 0;
  const int end = wave_inclusive_sum(share);
  const uint64_t past = __builtin_amdgcn_ballot_w64(j < end);   // the blocks that end behind workgroup j
  s.block = past ? __builtin_ctzll(past) : -1;
  if (s.block < 0) return s;
  s.parts = __builtin_amdgcn_readlane(share, s.block);
  s.part = j - (__builtin_amdgcn_readlane(end, s.block) - s.parts);
  s.tiles = __builtin_amdgcn_readlane(tiles, s.block);
  return s;
}

// Four workgroups to a CU (128 registers, 35 KB of LDS) for rows of up to 256 bytes.  WHOLE: tiles that every row of a wave sees go
// past the general case (whole_tiles).
template <int DT, int D, bool WHOLE>
__global__ __launch_bounds__(256, (DT == ZC_F32 && D == 128) ? 2 : 4) void k_probe_lse(ProbeArgs a) {
  using T = Tile<DT, D>;
  constexpr int TILE_B = kLseCols * T::ROWB;
  constexpr int NI = kLseCols / T::RPI / 4;     // transfers per wave and K tile
  __shared__ __align__(kTileAlign) uint8_t Ks[2][TILE_B];
  static_assert(__alignof__(Ks) % T::ROWB == 0 && TILE_B % T::ROWB == 0, "products forms addresses by exclusive or");
  __shared__ int spos[kLseRows];
  __shared__ float sm[2][kLseRows], sz[2][kLseRows];

  // logical order: workgroup of a head fastest, then query head, then batch
  const int nrb = ceil_div(a.P, kLseRows);
  int j = xcd_contiguous(blockIdx.x, gridDim.x);
  // An XCD deals its workgroups to 32 CUs in turn, so that a CU of a full chip would hold the same ranges of
  // four heads, all of them near the end of the prompt or all of few rows: from one round of 32 to the next
  // the heads begin a quarter further on.
  const int head = j / a.head_wgs, turn = gridDim.x >= 768 && gridDim.x <= 1024 ? (head * a.head_wgs >> 5) * (min(a.head_wgs, 32) >> 2) : 0;
  const LseShare share = lse_share(a, nrb, (j + turn) % a.head_wgs);
  if (share.block < 0) return;
  j = head;
  const int rb0 = share.block * kLseRows;
  const int hq = j % a.Hq, b = j / a.Hq, hk = hq / a.G;
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, kh = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rh = w >> 1, ch = w & 1;            // this wave: rows row0 .. + 63, columns ch * 32 .. + 31 of a tile
  const uint8_t* qb = reinterpret_cast<const uint8_t*>(a.q) + ((int64_t)b * a.q_sB + (int64_t)hq * a.q_sH) * T::EB;
  const uint8_t* kb = reinterpret_cast<const uint8_t*>(a.k) + ((int64_t)b * a.k_sB + (int64_t)hk * a.k_sH) * T::EB;
  const uint32_t k_rowb = (uint32_t)(a.k_sL * T::EB), q_rowb = (uint32_t)(a.q_sL * T::EB);
  const auto rs_k = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(kb), 0, (uint32_t)(a.Lk - 1) * k_rowb + T::ROWB, kBufFlags);
  const auto rs_q = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(qb), 0, (uint32_t)(a.Lq - 1) * q_rowb + T::ROWB, kBufFlags);

  const int nvalid = min(kLseRows, a.P - rb0);
  const bool two = nvalid > kLseRows / 2;       // (of a block of at most 64 rows 32 a wave)
  const int row0 = rh * (two ? 64 : 32);
  // this workgroup's share of the column tiles
  const int per = ceil_div(share.tiles, share.parts);
  const int t_begin = share.part * per, t_end = min(t_begin + per, share.tiles);

  // A K tile goes global -> LDS directly, every wave a quarter of its transfers;
  // the per-lane part of the addresses is fixed, the tile adds a scalar.
  const uint32_t ks_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)&Ks[0][0];
  // (where the swizzle repeats from one of a wave's transfers to the next, so does the rest)
  constexpr bool SAME = 4 * T::RPI / T::RP256 % T::SW == 0;
  int kvoff[SAME ? 1 : NI];
#pragma unroll
  for (int jj = 0; jj < (SAME ? 1 : NI); ++jj) {
    const int row = (w + 4 * jj) * T::RPI + lane / T::CPR;
    kvoff[jj] = (int)(row * k_rowb) + (((lane % T::CPR) ^ T::swz(row)) << 4);
  }
  // (the tile's offset goes into the per-lane offset, which is what the range check
  // sees: rows past the end of K then arrive as zeros)
  auto issue = [&](int t, int buf) {
    const int toff = (int)((uint32_t)t * kLseCols * k_rowb);
#pragma unroll
    for (int jj = 0; jj < NI; ++jj) dma16<0>(ks_lds + buf * TILE_B + (w + 4 * jj) * 1024, rs_k, SAME ? kvoff[0] + (toff + (int)(4 * jj * T::RPI * k_rowb)) : kvoff[SAME ? 0 : jj] + toff, 0);
  };
  // The probe rows of this block come through the two tile buffers into operand registers: whole
  // rows to a transfer (read straight into operand layout, 32 bytes of every cache line at a
  // time, they took 6 us of a 27 us launch).
  int last[2];                                   // last column a lane's row sees, less the lane's first in a tile (< 0: none)
  {
    int row[2 * NI];
    const auto rs_row = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(a.probe_rows ? a.probe_rows : a.probe_pos), 0, (uint32_t)a.P * 4u, kBufFlags);
    const int i0 = w * T::RPI + lane / T::CPR;
#pragma unroll
    for (int jj = 0; jj < 2 * NI; ++jj) row[jj] = (int)__builtin_amdgcn_raw_buffer_load_b32(rs_row, (rb0 + i0) * 4 + 16 * jj * T::RPI, 0, 0);
    const int my_pos = a.probe_pos[min(rb0 + (tid & (kLseRows - 1)), a.P - 1)];
#pragma unroll
    for (int jj = 0; jj < 2 * NI; ++jj) {
      const int off = opaque((int)((uint32_t)row[jj] * q_rowb) + (((lane % T::CPR) ^ T::swz(SAME ? i0 : i0 + 4 * jj * T::RPI)) << 4));
      dma16<0>(ks_lds + (w + 4 * jj) * 1024, rs_q, i0 + 4 * jj * T::RPI < nvalid ? off : kOutOfRange, 0);
    }
    if (tid < kLseRows) spos[tid] = tid < nvalid ? my_pos : -1;
  }
  wait_all_loads();
  __syncthreads();
  using lds_u32x4 = __attribute__((address_space(3))) const u32x4;
  u32x4 qf[2][T::NKC];
  // (a row past the last probe has logits of 0 and starts with a reference: without one its terms of
  // a whole tile would be infinite and the wave would evaluate every such tile twice: 32 heads over 8
  // of 128 channels, 16384 tokens, 40 probes, bf16: 63.9 -> 55.2 us, 64 probes 54.4)
  float m[2];
#pragma unroll
  for (int rb = 0; rb < 2; ++rb) {
    const int i = row0 + rb * 32 + r;
    m[rb] = spos[i] < 0 ? 0.f : -INFINITY;
    last[rb] = spos[i] < 0 ? -1 : spos[i] - 4 * kh;
#pragma unroll
    for (int kc = 0; kc < T::NKC; ++kc) qf[rb][kc] = *reinterpret_cast<lds_u32x4*>((ks_lds + T::slot(row0 + r, kh) ^ (kc << 5)) + rb * 32 * T::ROWB);
  }
  __syncthreads();
  if (t_begin < t_end) issue(t_begin, 0);
  // rows are sorted by position: a block's first row bounds what is fully visible,
  // its last real row what is visible at all
  // (scalars: read from LDS they would each hold a register)
  const auto pos_at = [&](int i) { return __builtin_amdgcn_readfirstlane(spos[i]); };
  // the same per 32-row block: its first row's position (-1: no row) and its last real row's
  int pfirst[2], plast[2];
#pragma unroll
  for (int rb = 0; rb < 2; ++rb) {
    const int base = row0 + rb * 32;
    pfirst[rb] = pos_at(base);
    plast[rb] = base < nvalid && (two || rb == 0) ? pos_at(min(base + 31, nvalid - 1)) : -1;
  }
  const int pos_last = max(plast[0], plast[1]);
  const bool both = plast[1] >= 0;
  bool ready = false;                            // no row without a reference
  float z[2] = {0.f, 0.f};
  const uint32_t abase = ks_lds + T::slot(ch * 32 + r, kh);

  if (a.even1) priority_by_tiles(t_end - t_begin);
  for (int t = t_begin; t < t_end; ++t) {
    const int cur = (t - t_begin) & 1;
    wait_all_loads();    // this wave's transfers of tile t have landed ...
    __syncthreads();     // ... and everyone's; nobody still reads the other buffer
    if (t + 1 < t_end) issue(t + 1, cur ^ 1);
    if (t_end - t <= a.even1) priority_by_tiles(t_end - t);
    if (t * kLseCols > pos_last) continue;       // nothing of this tile is visible to the wave's rows
    v16f acc[2];
    if (both) products<DT, 2>(acc, abase + cur * TILE_B, qf);
    else products<DT, 1>(acc, abase + cur * TILE_B, qf);
    __builtin_amdgcn_sched_barrier(0);           // (here and below: what follows would be moved up, into registers there are not)
    const int colb = t * kLseCols + ch * 32;     // this wave's 32 columns of the tile
    // Every row has its reference and sees every column: nothing but the terms (what the general case asks of every block
    // was 22 of a wave-tile's 151 vector instructions: all rows of 32 heads of 128 channels, 32768 tokens, 3276 probes,
    // both sweeps 1271 -> 1216 us).
    if (WHOLE && ready && colb + 31 <= pfirst[0]) {
      float sum[2] = {0.f, 0.f};
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) {
        if (rb == 1 && !both) break;
        sum[rb] = __builtin_amdgcn_exp2f(fmaf(acc[rb][0], a.scale_log2, -m[rb]));
#pragma unroll
        for (int v = 1; v < 16; ++v) {
          sum[rb] += __builtin_amdgcn_exp2f(fmaf(acc[rb][v], a.scale_log2, -m[rb]));
          if (v % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (__builtin_amdgcn_ballot_w64(!(sum[0] + sum[1] < 0x1p60f)) == 0) {
        z[0] += sum[0];
        z[1] += sum[1];
        continue;
      }
    }
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
      if (colb > plast[rb]) continue;            // none of them visible to this block's rows
      // The reference point m of a row only has to keep exp2 in range, not to be the maximum: it
      // is taken from the first columns the row sees and moved only when a tile's sum shows that
      // some logit lies 2^60 above it (the log-sum-exp m + log2(z) does not depend on the choice).
      const bool whole = colb + 31 <= pfirst[rb];            // every row of the block sees every column
      const int vis = last[rb] - colb;                       // of its columns (acc_row(v, 0)) a lane sees those up to vis
      bool set = __builtin_amdgcn_ballot_w64(m[rb] == -INFINITY && vis >= 0) != 0;
      float base = m[rb];                                    // what the logits are taken relative to
#pragma unroll 1
      for (int pass = 0; pass < 2; ++pass) {
        if (set) {
          const int seen = opaque(vis);                      // (or the compiler takes this maximum, and below the comparisons, every time)
          float tmax = -INFINITY;
#pragma unroll
          for (int v = 0; v < 16; ++v) tmax = fmaxf(tmax, acc_row(v, 0) <= seen ? acc[rb][v] : -INFINITY);
          // (no visible column: as it was, whatever a negative scale makes of -inf; with one the reference is the smallest
          // visible logit, which serves as well.  Scaling every term instead takes 12 more registers.)
          const float m_new = seen >= 0 ? fmaxf(m[rb], tmax * a.scale_log2) : m[rb];
          if (m_new > -INFINITY) z[rb] *= __builtin_amdgcn_exp2f(m[rb] - m_new);
          m[rb] = m_new;
          base = m_new > -INFINITY ? m_new : 0.f;            // (every visible logit -inf so far: their terms are 0, not exp2(-inf + inf))
        }
        float sum = 0.f;
        if (whole) {
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            sum += __builtin_amdgcn_exp2f(fmaf(acc[rb][v], a.scale_log2, -base));
            if (v % 4 == 3) __builtin_amdgcn_sched_barrier(0);
          }
        } else {
          const int seen = opaque(vis);
          const float ref = __int_as_float(opaque(__float_as_int(base)));     // (or it joins the two loops, and holds all 16 terms)
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const float e = __builtin_amdgcn_exp2f(fmaf(acc[rb][v], a.scale_log2, -ref));
            sum += acc_row(v, 0) <= seen ? e : 0.f;
            if (v % 4 == 3) __builtin_amdgcn_sched_barrier(0);
          }
        }
        if (set || __builtin_amdgcn_ballot_w64(!(sum < 0x1p60f)) == 0) {
          z[rb] += sum;
          break;
        }
        set = true;
      }
    }
    if (WHOLE && !ready) ready = __builtin_amdgcn_ballot_w64(m[0] == -INFINITY || (both && m[1] == -INFINITY)) == 0;
  }
  // merge the two half-waves, then the two column halves
  const int t1 = opaque(tid), r1 = t1 & 31;
#pragma unroll
  for (int rb = 0; rb < 2; ++rb) {
    const auto mh = __builtin_amdgcn_permlane32_swap(__float_as_uint(m[rb]), __float_as_uint(m[rb]), false, false);
    const auto zh = __builtin_amdgcn_permlane32_swap(__float_as_uint(z[rb]), __float_as_uint(z[rb]), false, false);
    const float m0 = __uint_as_float(mh[0]), m1 = __uint_as_float(mh[1]), M = fmaxf(m0, m1);
    float Z = 0.f;
    if (M > -INFINITY) Z = __uint_as_float(zh[0]) * exp2f(m0 - M) + __uint_as_float(zh[1]) * exp2f(m1 - M);
    if ((t1 & 32) == 0 && (two || rb == 0)) { sm[ch][row0 + rb * 32 + r1] = M; sz[ch][row0 + rb * 32 + r1] = Z; }
  }
  __syncthreads();
  if (t1 < kLseRows && rb0 + t1 < a.P) {
    const float M = fmaxf(sm[0][t1], sm[1][t1]);
    float Z = 0.f;
    if (M > -INFINITY) Z = sz[0][t1] * exp2f(sm[0][t1] - M) + sz[1][t1] * exp2f(sm[1][t1] - M);
    const int64_t row = ((int64_t)b * a.Hq + hq) * a.P + rb0 + t1;
    if (a.head_wgs == nrb) {
      a.lse2[row] = M + log2f(Z);
    } else {
      const int per_row = a.join ? 1 : a.max_parts, per_part = a.join ? a.P : 1;
      float2* dst = a.lse_part + ((int64_t)b * a.Hq + hq) * a.max_parts * a.P + (int64_t)(rb0 + t1) * per_row;
      dst[(int64_t)share.part * per_part] = make_float2(M, Z);
      if (share.part == share.parts - 1)                 // the ranges this block does not have
        for (int p = share.parts; p < a.max_parts; ++p) dst[(int64_t)p * per_part] = make_float2(-INFINITY, 0.f);
    }
  }
}

// Merges the (reference, sum) pairs of a probe row's column ranges, a thread per row.  Bound by its launch and one trip to
// memory: rows of all heads share workgroups, and a row's pairs lie side by side (a workgroup of 64 rows per head and
// [max_parts, P], as sweep 2 reads them: 2.6 -> 3.0 us of calls of up to 32 probes, 160 heads, 18 probes 14.5 -> 15.3 us a call).
__global__ __launch_bounds__(256) void k_probe_lse_merge(const float2* __restrict__ part, float* __restrict__ lse2, int64_t rows, int max_parts) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= rows) return;
  RowPairs v;
  v.load_row(part + i * max_parts, max_parts);
  lse2[i] = v.joined(max_parts);
}

// Four workgroups to a CU (128 registers, 38.5 KB of LDS) for rows of up to 256 bytes, so that four
// independent waves a SIMD overlap matrix and vector work and 1024 workgroups start at once.
// An instance each for up to kProbeTable probes, for such whose pairs it joins, and for more: as branches of one
// kernel they were 10.8 KB of cold code instead of 6.8 to 8.8, and a lone wave paid their scalar tests in every tile.  us given
// normalisers, one kernel and three: 32 heads of 128 channels, 4096 tokens, 64 probes 9.6 and 9.0, 410 18.0 and 16.9; all rows of a
// head of 64 channels as probes, 8192 rows 104 and 94, 8 heads of 2048 30.6 and 28.3 (tiles behind the first open one are no longer
// asked for their first position either).
enum class Probes { Few, FewJoined, Many };
template <int DT, int D, Probes PROBES>
__global__ __launch_bounds__(256, (DT == ZC_F32 && D == 128) ? 1 : 4) void k_probe_colsum(ProbeArgs a) {
  using T = Tile<DT, D>;
  constexpr int QT = 64;                        // probe rows per tile
  static_assert(kBlockCols == 2 * QT, "a block's columns come through the two tile buffers");
  constexpr int TILE_B = QT * T::ROWB;
  constexpr int NI = QT / T::RPI / 4;           // transfers per wave and tile
  __shared__ __align__(kTileAlign) uint8_t Qs[2][TILE_B];
  static_assert(__alignof__(Qs) % T::ROWB == 0 && TILE_B % T::ROWB == 0, "products forms addresses by exclusive or");
  // positions (-1: no probe), offsets of their rows in q and log-sum-exps (log2 units) of the probes from pstart on: entry j at
  // j modulo the table
  __shared__ __align__(16) int spos[kProbeTable];
  __shared__ __align__(16) int srow[kProbeTable];
  __shared__ __align__(16) float slse[kProbeTable];
  float (*scol)[128] = reinterpret_cast<float (*)[128]>(&Qs[0][0]);     // (in the place of the tiles, at the end)
  __shared__ int bins[128];                     // probes at each of this workgroup's columns
  __shared__ __align__(16) int before[4];       // probes in front of them, by wave
  static_assert(T::ROWB > 256 || (sizeof(Qs) + sizeof(spos) + sizeof(srow) + sizeof(slse) + sizeof(bins) + sizeof(before) + 2047) / 2048 * 8 <= 160, "four workgroups to a CU");

  // Logical order: the first columns, which the most probes see, of all heads of a group, then the next ones: the
  // last workgroups to start are the shortest, and a CU's workgroups, 32 apart in an XCD's range, see few
  // rows and many.  Where the heads divide over the 8 XCDs every XCD has its own, in groups of two rounds of
  // its places, so that the workgroups in flight read few heads' rows through its L2.  Otherwise head after
  // head, every other one backwards.  us given normalisers, head after head and so: 2 x 32 heads, 3001 tokens
  // 23.4 and 22.7; 24 heads, 9000 tokens 52.4 and 47.1; 32 heads, 32768 tokens 665 and 632; 16 x 16 heads of 64,
  // 2000 tokens 30.9 and 27.9; 32 heads, 4096 tokens 18.7 and 18.0, fp32 111 and 98; up to a
  // workgroup a CU the divisions only cost time (16 x 8 heads of 64, 400 tokens 7.1 and 7.3), and of up to 64
  // probes in 16 bits every workgroup has as much to do (32 heads, 8192 tokens 12.8 and 13.2; in fp32 the matrix cores do less
  // where 32 rows see the columns: 16 x 16 heads, 500 tokens, both sweeps 62.7 and 61.2).
  const int nct = ceil_div(a.Lk, kBlockCols);
  int j, ct;
  if (a.group) {
    const int hpx = (a.B * a.Hq) >> 3, rank = blockIdx.x >> 3, g = rank / (a.group * nct), rem = rank - g * (a.group * nct);
    const int size = min(a.group, hpx - g * a.group);
    ct = rem / size;
    j = (blockIdx.x & 7) * hpx + g * a.group + rem - ct * size;
  } else {
    j = xcd_contiguous(blockIdx.x, gridDim.x);
    ct = j % nct; j /= nct;
    if ((j % a.Hq) & 1) ct = nct - 1 - ct;
  }
  const int hq = j % a.Hq, b = j / a.Hq, hk = hq / a.G;
  const int col0 = ct * kBlockCols;
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, kh = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rbw = w >> 1, cbp = w & 1;
  const uint8_t* qb = reinterpret_cast<const uint8_t*>(a.q) + ((int64_t)b * a.q_sB + (int64_t)hq * a.q_sH) * T::EB;
  const uint8_t* kb = reinterpret_cast<const uint8_t*>(a.k) + ((int64_t)b * a.k_sB + (int64_t)hk * a.k_sH) * T::EB;
  const int64_t lrow = ((int64_t)b * a.Hq + hq) * a.P;
  const uint32_t k_rowb = (uint32_t)(a.k_sL * T::EB), q_rowb = (uint32_t)(a.q_sL * T::EB);
  const auto rs_k = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(kb), 0, (uint32_t)(a.Lk - 1) * k_rowb + T::ROWB, kBufFlags);
  const auto rs_q = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(qb), 0, (uint32_t)(a.Lq - 1) * q_rowb + T::ROWB, kBufFlags);
  const auto rs_pos = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(a.probe_pos), 0, (uint32_t)a.P * 4u, kBufFlags);
  const auto rs_row = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(a.probe_rows ? a.probe_rows : a.probe_pos), 0, (uint32_t)a.P * 4u, kBufFlags);
  const float* lse_src = (a.lse_in ? a.lse_in : a.lse2) + lrow;
  const auto rs_lse = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(lse_src), 0, (uint32_t)a.P * 4u, kBufFlags);

  // One pass over the probe positions: how many lie in front of these columns (the first probe
  // that sees them, as positions ascend) and how many at each of them.
  // Meanwhile the K columns come through the two tile buffers (whole rows to a transfer, as in
  // sweep 1; columns past the end: zeros).
  const uint32_t qs_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)&Qs[0][0];
  constexpr bool table = PROBES != Probes::Many, join = PROBES == Probes::FewJoined;
  constexpr int NT = kProbeTable / 256;
  int tpos[NT], trow[NT];
  float tlse[NT];
  if (tid < 128) bins[tid] = 0;
  {
    constexpr bool SAME = 4 * T::RPI / T::RP256 % T::SW == 0;      // (the swizzle repeats from one of a wave's transfers to the next)
    const int i0 = w * T::RPI + lane / T::CPR;
    int off = (int)((uint32_t)(col0 + i0) * k_rowb);
#pragma unroll
    for (int jj = 0; jj < 2 * NI; ++jj) {
      dma16<0>(qs_lds + (w + 4 * jj) * 1024, rs_k, off + (((lane % T::CPR) ^ T::swz(SAME ? i0 : i0 + 4 * jj * T::RPI)) << 4), 0);
      off += (int)(4 * T::RPI * k_rowb);
    }
    int n = 0;
    const auto count = [&](bool real, int pos) {
      n += real && pos < col0 ? 1 : 0;
      if (real && (uint32_t)(pos - col0) < 128u) atomicAdd(&bins[pos - col0], 1);
    };
    if constexpr (table) {
      // few probes: all that is to be looked up of them comes with the positions
      RowPairs pairs[NT];
#pragma unroll
      for (int u = 0; u < NT; ++u)
        if (u * 256 < a.P) {
          const int i = u * 256 + tid;
          tpos[u] = (int)__builtin_amdgcn_raw_buffer_load_b32(rs_pos, i * 4, 0, 0);
          trow[u] = (int)__builtin_amdgcn_raw_buffer_load_b32(rs_row, i * 4, 0, 0);
          if constexpr (join) pairs[u].load(a, (int64_t)b * a.Hq + hq, min(i, a.P - 1));
          else tlse[u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_lse, i * 4, 0, 0));
        }
      __syncthreads();                           // (the bins are empty)
#pragma unroll
      for (int u = 0; u < NT; ++u)
        if (u * 256 < a.P) {
          count(u * 256 + tid < a.P, tpos[u]);
          if constexpr (join) {                  // (but of probes that all lie in front of these columns)
            if (__builtin_amdgcn_ballot_w64(u * 256 + tid < a.P && tpos[u] >= col0)) tlse[u] = pairs[u].joined(a.max_parts);
          }
          if (!join && a.lse_in) tlse[u] *= kLog2e;      // an external log-sum-exp is in natural units
        }
    } else {
      __syncthreads();
      for (int i0 = tid; i0 < a.P; i0 += 4 * 256) {
        int pos[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) pos[u] = (int)__builtin_amdgcn_raw_buffer_load_b32(rs_pos, (i0 + u * 256) * 4, 0, 0);
#pragma unroll
        for (int u = 0; u < 4; ++u) count(i0 + u * 256 < a.P, pos[u]);
      }
    }
    n = wave_inclusive_sum(n);
    if (lane == 63) before[w] = n;
  }
  wait_all_loads();
  __syncthreads();
  using lds_u32x4 = __attribute__((address_space(3))) const u32x4;
  u32x4 kf[2][T::NKC];
#pragma unroll
  for (int cb = 0; cb < 2; ++cb)
#pragma unroll
    for (int kc = 0; kc < T::NKC; ++kc) kf[cb][kc] = *reinterpret_cast<lds_u32x4*>((qs_lds + T::slot(cbp * 64 + r, kh) ^ (kc << 5)) + cb * 32 * T::ROWB);
  const int pstart = __builtin_amdgcn_readfirstlane(before[0] + before[1] + before[2] + before[3]);
  float colsum[2] = {0.f, 0.f};

  // What a tile of 64 probe rows is looked up by: all of it is in LDS where the probes are few; otherwise one half of
  // the table is filled under the first tile of the other, every wave a quarter of it.  (Past the
  // last probe: row 0 of q, which a position of -1 masks.)  The tile itself goes global -> LDS directly one
  // ahead, every wave a quarter of its transfers.
  const uint32_t spos_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) int*)&spos[0];
  const uint32_t srow_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) int*)&srow[0];
  const uint32_t slse_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) float*)&slse[0];
  constexpr int kHalf = kProbeTable / 2;
  static_assert(kHalf == 256 && kHalf == 4 * QT, "an entry a thread; four tiles");
  auto fetch = [&](int entry) {                  // entries entry .. + kHalf - 1, this wave's 64 of them
    const int voff = (pstart + entry + opaque(tid)) * 4;
    const uint32_t to = ((entry & kHalf) + w * 64) * 4;
    dma4(spos_lds + to, rs_pos, voff, 0);
    dma4(srow_lds + to, rs_row, voff, 0);
    dma4(slse_lds + to, rs_lse, voff, 0);
  };
  const auto fetched = [&](int entry) {          // when this wave's have landed
    const int e = (entry & kHalf) + opaque(tid);
    srow[e] = (int)((uint32_t)srow[e] * q_rowb);
    if (a.lse_in) slse[e] *= kLog2e;             // an external log-sum-exp is in natural units
    if (pstart + entry + opaque(tid) >= a.P) spos[e] = -1;
  };
  auto issue = [&](int at, int buf) {
    int from[NI];                                // (read together: the transfers keep their order)
#pragma unroll
    for (int jj = 0; jj < NI; ++jj) from[jj] = srow[at + (w + 4 * jj) * T::RPI + lane / T::CPR];
#pragma unroll
    for (int jj = 0; jj < NI; ++jj) {
      const int row = (w + 4 * jj) * T::RPI + lane / T::CPR;
      dma16<0>(qs_lds + buf * TILE_B + (w + 4 * jj) * 1024, rs_q, opaque(from[jj]) + (((lane % T::CPR) ^ T::swz(row)) << 4), 0);
    }
  };
  if (pstart < a.P) {
    if constexpr (table) {
#pragma unroll
      for (int u = 0; u < NT; ++u) {
        const int at = u * 256 + tid - pstart;
        if (u * 256 + tid < a.P && at >= 0) { spos[at] = tpos[u]; srow[at] = (int)((uint32_t)trow[u] * q_rowb); slse[at] = tlse[u]; }
      }
      const int at = a.P - pstart + tid;         // (to the end of the last tile)
      if (tid < QT && at < kProbeTable) { spos[at] = -1; srow[at] = 0; slse[at] = 0.f; }
    } else {
      fetch(0);
      fetch(kHalf);
      wait_all_loads();
      fetched(0);
      fetched(kHalf);
    }
    __syncthreads();
    issue(0, 0);
  }
  const uint32_t abase = qs_lds + T::slot(rbw * 32 + r, kh);
  const int wcol0 = col0 + cbp * 64;             // this wave's columns: wcol0 .. + 63; of a tile, its rows rbw * 32 .. + 31
  const int pend = a.P - rbw * 32;

  const int even_from = a.even2 ? a.P - a.even2 : 0x7fffffff;
  if (a.even2) priority_by_tiles((a.P - pstart + QT - 1) / QT);
  int at = 0, cur = 0;
  int refill = pstart + kHalf;                   // the first tile of a half: the other one is free; the second: it is full
  bool open = false;                             // (positions ascend: what is visible stays visible)
  for (int pr = pstart; pr < a.P; pr += QT) {
    wait_all_loads();    // this wave's transfers of the tile have landed ...
    __syncthreads();     // ... and everyone's; nobody still reads the other buffer
    if constexpr (!table) {
      if (__builtin_expect(pr == refill, 0)) {
        const int entry = pr - pstart;
        if (entry & QT) { fetched(entry - QT + kHalf); refill += kHalf - QT; }
        else { fetch(entry + kHalf); refill += QT; }
      }
    }
    const int next = (at + QT) & (kProbeTable - 1);
    if (__builtin_expect(pr + QT < a.P, 1)) issue(next, cur ^ 1);
    if (__builtin_expect(pr >= even_from, 0)) priority_by_tiles((a.P - pr + QT - 1) / QT);
    if (__builtin_expect(pr < pend, 1)) {        // (no probe in the wave's rows of a last tile)
      v16f acc[2];
      products<DT, 2>(acc, abase + cur * TILE_B, kf);
      __builtin_amdgcn_sched_barrier(0);         // (what follows would be moved up, into registers there are not)
      const float4* rl4 = reinterpret_cast<const float4*>(&slse[at + rbw * 32 + 4 * kh]);     // rows 8 g + 4 kh ..
      // 32 real rows whose first position is past the wave's last column need no mask
      if (!open) open = wcol0 + 63 <= __builtin_amdgcn_readfirstlane(spos[at + rbw * 32]);
      if (open && pr + 32 <= pend) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const float4 t = rl4[2 * g];
          const float rl[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
          for (int cb = 0; cb < 2; ++cb)
#pragma unroll
            for (int v = 0; v < 4; ++v) colsum[cb] += __builtin_amdgcn_exp2f(fmaf(acc[cb][4 * g + v], a.scale_log2, -rl[v]));
        }
      } else {
        const int4* ps4 = reinterpret_cast<const int4*>(&spos[at + rbw * 32 + 4 * kh]);
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const float4 t = rl4[2 * g];
          const int4 s = ps4[2 * g];
          const float rl[4] = {t.x, t.y, t.z, t.w};
          const int ps[4] = {s.x, s.y, s.z, s.w};
#pragma unroll
          for (int cb = 0; cb < 2; ++cb) {
            const int col = wcol0 + cb * 32 + r;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              const float e = __builtin_amdgcn_exp2f(fmaf(acc[cb][4 * g + v], a.scale_log2, -rl[v]));
              colsum[cb] += col <= ps[v] ? e : 0.f;
            }
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    at = next;
    cur ^= 1;
  }
  wait_all_loads();                              // (a fetch behind the last probe: nothing may land in LDS that is another workgroup's)
  __syncthreads();
  const int t1 = opaque(tid), l1 = t1 & 63;
#pragma unroll
  for (int cb = 0; cb < 2; ++cb) {
    const auto halves = __builtin_amdgcn_permlane32_swap(__float_as_uint(colsum[cb]), __float_as_uint(colsum[cb]), false, false);
    colsum[cb] = __uint_as_float(halves[0]) + __uint_as_float(halves[1]);
    if (l1 < 32) scol[rbw][(cbp * 2 + cb) * 32 + l1] = colsum[cb];
  }
  __syncthreads();
  if (t1 < 128) {
    // probes at a column of this workgroup before this thread's: a scan over two waves
    const int own = bins[t1];
    int lower = pstart + wave_inclusive_sum(own) - own;
    if (w == 1) lower += __builtin_amdgcn_readlane(wave_inclusive_sum(bins[l1]), 63);
    const int col = col0 + t1, cnt = a.P - lower;
    const float total = scol[0][t1] + scol[1][t1];
    if (col < a.Lk) a.per_head[((int64_t)b * a.Hq + hq) * a.Lk + col] = !a.normalize ? total : (cnt > 0 ? total / (float)cnt : 0.f);
  }
}

// Mean over the query heads: block (64 columns, 4 head groups); every group
// sums its heads in order, the four partial sums are then added in order.
__global__ __launch_bounds__(256) void k_probe_mean(const float* __restrict__ per_head, float* __restrict__ scores, int Hq, int Lk) {
  __shared__ float part[4][64];
  const int b = blockIdx.y;
  const int cx = threadIdx.x, gy = threadIdx.y;
  const int i = blockIdx.x * 64 + cx;
  const int per = (Hq + 3) / 4;
  float s = 0.f;
  if (i < Lk) {
    const int h1 = min(Hq, (gy + 1) * per);
    for (int h = gy * per; h < h1; h += 8) {           // (eight heads requested at once, added in order)
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = per_head[((int64_t)b * Hq + min(h + u, h1 - 1)) * Lk + i];
#pragma unroll
      for (int u = 0; u < 8; ++u) s += h + u < h1 ? v[u] : 0.f;
    }
  }
  part[gy][cx] = s;
  __syncthreads();
  if (gy == 0 && i < Lk) scores[(int64_t)b * Lk + i] = (((part[0][cx] + part[1][cx]) + part[2][cx]) + part[3][cx]) / (float)Hq;
}

// ---- few probe rows ----------------------------------------------------------------------
// Sweep 2 and the mean over heads in one launch: a workgroup owns 16 NC columns of a batch element for all heads, a wave a
// run of blocks of 16 probe rows, head after head; rows and columns go straight from memory to operand registers (each is
// used once, and bringing them to LDS in whole lines was no faster: a CU gets about 37 KB a us from beyond its L2 either
// way).  Bound by that and by the chain of the two trips, so 16 columns where the workgroups find a CU each; 32, which read the
// probe rows half as often, where they do not.  us, two launches and this (32 columns and 32 rows a wave before): 8 heads of 64
// channels, bf16, 100 tokens, 10 rows 5.8 and 3.7 (4.5); 256 tokens, 26 rows, fp32 7.8 and 6.4 (7.3); 16 heads of 128, 100 tokens, fp32 10.0 and
// 8.9; 8 x 32 heads over 8, 1000 tokens, 10 rows, bf16 13.0 and 10.0 (10.8); 16 of them, fp32 92 and 38.
__device__ inline int lower_bound_pos(const int32_t* pos, int n, int key) {
  int lo = 0, hi = n;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (pos[mid] < key) lo = mid + 1; else hi = mid;
  }
  return lo;
}

constexpr int kFewRows = 32;          // most probe rows
constexpr int kFewTable = 4096;       // most log-sum-exps of a batch element (heads x rows)
// Whether a wave of 32 columns takes two blocks of a head together (for long fp32 rows there are no registers).
constexpr bool few_both(int64_t P, bool fp32, int64_t D) { return P > 16 && !(fp32 && D == 128); }
typedef float v4f __attribute__((ext_vector_type(4)));
// 16 x 16 result over one 16-byte chunk a lane (lane: row or column lane % 16, k chunk lane / 16).
template <int DT>
__device__ inline void mma16(v4f& acc, u32x4 a, u32x4 b) {
  if constexpr (DT == ZC_BF16) {
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
  } else if constexpr (DT == ZC_F16) {
    acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), acc, 0, 0, 0);
  } else {
    // (the elements one by one on purpose, see mma_chunk)
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(b.x), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(b.y), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(b.z), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(b.w), acc, 0, 0, 0);
  }
}

// BOTH: a wave takes the two blocks of a head together.  PER_HEAD: the heads' own sums too, beside the same sum over all, which
// scores do not depend on.
template <int DT, int D, int NC, bool BOTH, bool PER_HEAD>
__global__ __launch_bounds__(1024) void k_probe_few(ProbeArgs a, float* __restrict__ scores) {
  using T = Tile<DT, D>;
  constexpr int NK = T::ROWB / 64;                   // 16-byte chunks of a lane in a row
  constexpr bool AHEAD = !BOTH && NK * (NC + 2) <= 24;        // the next block's rows are requested in front of a block's products
  __shared__ float slse[kFewTable];
  __shared__ int spos[kFewRows], srow[kFewRows];
  __shared__ float part[16][16 * NC];
  __shared__ float second[PER_HEAD ? 16 : 1][16 * NC];          // of a head whose first block is the wave before's
  const int b = blockIdx.y, col0 = blockIdx.x * 16 * NC;
  const int tid = threadIdx.x, lane = tid & 63, i = lane & 15, g = lane >> 4, nw = blockDim.x >> 6;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t k_rowb = (uint32_t)(a.k_sL * T::EB), q_rowb = (uint32_t)(a.q_sL * T::EB);
  // consecutive blocks of 16 probe rows, head after head, to a wave: one load of K serves those that share it
  const int rt = (a.P + 15) >> 4, u0 = w * a.few_blocks, u1 = min(u0 + a.few_blocks, a.Hq * rt);
  u32x4 kf[NC][NK], qf[AHEAD || BOTH ? 2 : 1][NK];
  auto load_k = [&](int h) {
    const uint8_t* kb = reinterpret_cast<const uint8_t*>(a.k) + ((int64_t)b * a.k_sB + (int64_t)(h / a.G) * a.k_sH) * T::EB;
    const auto rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(kb), 0, (uint32_t)(a.Lk - 1) * k_rowb + T::ROWB, kBufFlags);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int col = col0 + 16 * c + i;             // (columns past the end: zeros)
      const int off = col < a.Lk ? (int)((uint32_t)col * k_rowb) + g * 16 : kOutOfRange;
#pragma unroll
      for (int kc = 0; kc < NK; ++kc) kf[c][kc] = __builtin_amdgcn_raw_buffer_load_b128(rs, off + kc * 64, 0, 0);
    }
  };
  auto load_q = [&](int u, u32x4 (&f)[NK]) {
    const int h = rt == 1 ? u : u >> 1, p = (rt == 1 ? 0 : (u & 1) * 16) + i;
    const uint8_t* qb = reinterpret_cast<const uint8_t*>(a.q) + ((int64_t)b * a.q_sB + (int64_t)h * a.q_sH) * T::EB;
    const auto rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(qb), 0, (uint32_t)(a.Lq - 1) * q_rowb + T::ROWB, kBufFlags);
    const int off = p < a.P ? (int)((uint32_t)srow[p] * q_rowb) + g * 16 : kOutOfRange;
#pragma unroll
    for (int kc = 0; kc < NK; ++kc) f[kc] = __builtin_amdgcn_raw_buffer_load_b128(rs, off + kc * 64, 0, 0);
  };
  if (u0 < u1) load_k(rt == 1 ? u0 : u0 >> 1);       // (needs nothing of the probes)
  const int ntab = a.Hq * a.P;
  const float* lse_src = (a.lse_in ? a.lse_in : a.lse2) + (int64_t)b * ntab;
  const float unit = a.lse_in ? kLog2e : 1.f;        // an external log-sum-exp is in natural units
  if (tid < a.P) {
    const int pos = a.probe_pos[tid];
    spos[tid] = pos;
    srow[tid] = a.probe_rows ? a.probe_rows[tid] : pos;
  }
  for (int t = tid; t < ntab; t += blockDim.x) slse[t] = lse_src[t] * unit;
  __syncthreads();
  float sum[NC], head[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) sum[c] = head[c] = 0.f;
  const int head_col = col0 + 16 * (g % NC) + i;     // per-head scores: the column that a lane of the first NC blocks stores
  // (looked up at every store where a register more would spill, 32 columns of 128 fp32 channels: 8 x 32 heads over 8, 1000 tokens, 10 rows 23.1 -> 21.5 us)
  constexpr bool TIGHT = NK * (NC + 1) >= 24;
  const auto seen = [&]() { return a.normalize ? a.P - lower_bound_pos(spos, a.P, head_col) : 1; };
  const int seen_once = PER_HEAD && !TIGHT ? seen() : 0;
  auto store_head = [&](int h, const float (&total)[NC]) {
    const int seen_by = TIGHT ? seen() : seen_once;
    const float t = total[g % NC == NC - 1 ? NC - 1 : 0];
    if (g < NC && head_col < a.Lk) a.per_head[((int64_t)b * a.Hq + h) * a.Lk + head_col] = seen_by > 0 ? t / (float)seen_by : 0.f;
  };
  auto over_rows = [](float x) {
    x += __shfl_xor(x, 16);
    return x + __shfl_xor(x, 32);
  };
  auto block = [&](int u, const u32x4 (&f)[NK]) {
    const int h = rt == 1 ? u : u >> 1, p0 = (rt == 1 ? 0 : (u & 1) * 16) + 4 * g;
    v4f acc[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[c] = v4f{};
#pragma unroll
    for (int kc = 0; kc < NK; ++kc)                  // (the columns' chains of products side by side)
#pragma unroll
      for (int c = 0; c < NC; ++c) mma16<DT>(acc[c], f[kc], kf[c][kc]);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int col = col0 + 16 * c + i;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int p = p0 + v, pc = min(p, a.P - 1);
        const float e = __builtin_amdgcn_exp2f(fmaf(acc[c][v], a.scale_log2, -slse[h * a.P + pc])), seen = (p < a.P && col <= spos[pc]) ? e : 0.f;
        sum[c] += seen;
        if constexpr (PER_HEAD) head[c] += seen;
      }
    }
    if constexpr (PER_HEAD) {
      if (rt == 1 || (u & 1)) {                      // a head's last block
        float total[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          total[c] = over_rows(head[c]);
          head[c] = 0.f;
          if (rt == 2 && u == u0 && g == 0) second[w][16 * c + i] = total[c];
        }
        if (rt == 1 || u > u0) store_head(h, total);
      }
    }
  };
  if constexpr (BOTH) {
    for (int u = u0; u < u1; u += 2) {
      load_q(u, qf[0]);
      load_q(u + 1, qf[1]);
      block(u, qf[0]);
      block(u + 1, qf[1]);
      if (u + 2 < u1 && (u + 2) % (2 * a.G) == 0) load_k((u + 2) >> 1);
    }
  } else {
    if (u0 < u1) load_q(u0, qf[0]);
    for (int u = u0; u < u1; ++u) {
      if constexpr (AHEAD) { if (u + 1 < u1) load_q(u + 1, qf[1]); }
      block(u, qf[0]);
      if (u + 1 < u1) {
        if ((u + 1) % (a.G * rt) == 0) load_k(rt == 1 ? u + 1 : (u + 1) >> 1);
        if constexpr (AHEAD) {
#pragma unroll
          for (int kc = 0; kc < NK; ++kc) qf[0][kc] = qf[1][kc];
        } else {
          load_q(u + 1, qf[0]);
        }
      }
    }
  }
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    sum[c] = over_rows(sum[c]);
    if (g == 0) part[w][16 * c + i] = sum[c];
  }
  __syncthreads();
  if constexpr (PER_HEAD) {
    if (rt == 2 && (u1 & 1) && u0 < u1) {            // this wave ends with a head's first block (an even number in all: there is a wave after it)
      float total[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) total[c] = over_rows(head[c]) + second[w + 1][16 * c + i];
      store_head(u1 >> 1, total);
    }
  }
  if (tid < 16 * NC && col0 + tid < a.Lk) {
    float total = 0.f;
    for (int v = 0; v < nw; ++v) total += part[v][tid];
    const int cnt = a.P - lower_bound_pos(spos, a.P, col0 + tid);
    if (a.normalize) total = cnt > 0 ? total / (float)cnt : 0.f;
    scores[(int64_t)b * a.Lk + col0 + tid] = total / (float)a.Hq;
  }
}

template <int DT, int D>
static int launch_probe(const ProbeArgs& a, bool need_lse, float* scores, hipStream_t st) {
  if (need_lse) {
    const dim3 grid1((unsigned)((int64_t)a.head_wgs * a.Hq * a.B));
    if (a.whole1) hipLaunchKernelGGL((k_probe_lse<DT, D, true>), grid1, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((k_probe_lse<DT, D, false>), grid1, dim3(256), 0, st, a);
    ZC_LAUNCH_CHECK();
    if (a.head_wgs > ceil_div(a.P, kLseRows) && !a.join) {
      const int64_t rows = (int64_t)a.B * a.Hq * a.P;
      hipLaunchKernelGGL(k_probe_lse_merge, dim3((unsigned)ceil_div64(rows, 256)), dim3(256), 0, st, a.lse_part, a.lse2, rows, a.max_parts);
      ZC_LAUNCH_CHECK();
    }
  }
  if (a.few_cols) {
    const dim3 grid((unsigned)ceil_div(a.Lk, 16 * a.few_cols), (unsigned)a.B), block(64 * ceil_div(a.Hq * ceil_div(a.P, 16), a.few_blocks));
    constexpr bool both = few_both(kFewRows, DT == ZC_F32, D);
    const auto launch = [&](auto plain, auto per_head) { hipLaunchKernelGGL(a.per_head ? per_head : plain, grid, block, 0, st, a, scores); };
    if (a.few_cols == 1) launch(k_probe_few<DT, D, 1, false, false>, k_probe_few<DT, D, 1, false, true>);
    else if (few_both(a.P, DT == ZC_F32, D)) launch(k_probe_few<DT, D, 2, both, false>, k_probe_few<DT, D, 2, both, true>);
    else launch(k_probe_few<DT, D, 2, false, false>, k_probe_few<DT, D, 2, false, true>);
    ZC_LAUNCH_CHECK();
    return ZC_OK;
  }
  const dim3 grid2((unsigned)((int64_t)ceil_div(a.Lk, 128) * a.Hq * a.B));
  if (a.P > kProbeTable) hipLaunchKernelGGL((k_probe_colsum<DT, D, Probes::Many>), grid2, dim3(256), 0, st, a);
  else if (a.join) hipLaunchKernelGGL((k_probe_colsum<DT, D, Probes::FewJoined>), grid2, dim3(256), 0, st, a);
  else hipLaunchKernelGGL((k_probe_colsum<DT, D, Probes::Few>), grid2, dim3(256), 0, st, a);
  ZC_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_probe_mean, dim3(ceil_div(a.Lk, 64), a.B), dim3(64, 4), 0, st, a.per_head, scores, a.Hq, a.Lk);
  ZC_LAUNCH_CHECK();
  return ZC_OK;
}

}  // namespace zc

using namespace zc;

// Workgroups of a head in sweep 1, which its row blocks share (k_probe_lse): enough to fill the
// chip once (four fit a CU); and, however many blocks there are, four to a block on average
// where the columns give each at least 16 tiles, so that the last workgroups to finish are short.
static int64_t probe_head_wgs(int64_t B, int64_t Hq, int64_t P, int64_t Lk, int max_parts, bool fp32) {
  const int64_t heads = B * Hq, nrb = ceil_div64(P, kLseRows), tiles = ceil_div64(Lk, kLseCols);
  // A second range of a single block is a launch more, to merge them: none for prompts of up to four tiles
  // (fp32, where a tile takes twice as long: from 128 heads on), and above 384 heads none to fill the chip.
  // 24 x 8 heads of 64 channels, 130 tokens, 13 probes, one range and three, bf16: 10.0 and 12.7 us, fp32: 15.8
  // and 18.8 (4 x 8 heads, the last 13: 18.0 and 15.6); 64 x 8 heads, 300 tokens, 30 probes, one and two: 22.7
  // and 25.2; 16 x 32 heads over 8 of 128, 500 tokens, 50 probes: 26.7 and 28.6.
  if (nrb == 1 && tiles <= 4 && (!fp32 || heads >= 128)) return 1;
  const int64_t fill = nrb == 1 && heads > 384 ? 1 : 1024 / heads;
  const int64_t even = tiles / 16 < 4 ? tiles / 16 : 4;
  int64_t n = fill > even * nrb ? fill : even * nrb;
  if (n > nrb * max_parts) n = nrb * max_parts;
  if (fp32) {
    // Bound by the matrix cores of the CUs with one workgroup more than others: whole rounds of two a CU, or
    // of one, unless that takes more than a third of the ranges away.  16 heads over 4 of 128 channels, 5000 tokens,
    // 500 probes, 768 and 512 workgroups: 163 and 137 us; 8 heads over 2, 9000 and 900: 250 and 215; 4 heads, 20000
    // and 1000, 384 and 256: 327 and 303; but 36 x 8 heads, 700 tokens, 70 probes, 864 and 288: 138 and 157.
    const int64_t unit = n * heads >= 512 ? 512 : 256, whole = n * heads / unit * unit / heads;
    if (3 * whole >= 2 * n) n = whole;
  }
  if (nrb > 64) n = n / nrb * nrb;
  if (n < nrb) n = nrb;
  // A single block: no more ranges than whole tiles make.  The ranges without one cost their start and
  // a place on a CU, which in fp32, bound by the matrix cores of the CUs that got two, is half the
  // time: 32 heads over 8 of 128 channels, 1000 tokens, 64 probes: 34.4 us with 12 ranges, 26.7 with 8.
  if (nrb == 1) n = ceil_div64(tiles, ceil_div64(tiles, n));
  return n;
}
// Whether a sweep's waves are kept at about the same number of tiles to go: where a CU holds several of its
// workgroups, all of them at once, of at least four tiles each.  us, without and with: 32 heads of 128 channels, 4096
// tokens, 410 probes (1024 workgroups), sweep 2: 19.7 and 18.5; 12 heads of 64, 5000 tokens (480): 13.2 and 12.8; but
// 24 heads, 9000 tokens, fp32 (1704 on 512 places): 344 and 374; 4 x 16 heads of 64, 900 tokens, two tiles: 8.50
// and 8.61.  Sweep 1, whose workgroups all have as many tiles, from three a CU on: 4 heads, 20000 tokens, 1000
// probes (384): 32.2 and 34.0.
static bool even_waves(int64_t wgs, double tiles, const zc_tensor4* q) {
  const int64_t places = q->dtype == ZC_F32 && q->D == 128 ? 512 : 1024;
  return wgs > 256 && wgs <= places && tiles >= 4.0;
}
// Whether sweep 1 has the way past the general case for whole tiles.  Where workgroups run once it is mostly more cold code: the
// rows are spread over the columns, and the start and the tiles seen in part are what a wave does.  us, general case alone and both: 24 heads over 8 of
// 128 channels, 228 tokens, 22 probes 12.9 and 13.4; 40 heads, 2715 and 272 30.7 and 31.3; 24 over 8, 6000 and 600 (1008 workgroups) 52.5 and 53.7; 8
// heads of 64, 3300 and 330 (384) 19.3 and 19.8; 16 x 40 heads, 1500 and 150 (1280) 133.5 and 136.6; 16 x 24 of 128, fp32, 2000 and 200 710.5 and 711.8.  It pays in more
// rounds of rows that see 32 tiles and more, and of a few heads' long row blocks on a chip that is not full: 12 x 32 over 8, 2400 and 240 (1536) 140.2 and
// 135.9; 40 heads, 9276 and 928 (1280) 178.5 and 167.3; 32 over 8, 32768 and 3276 1278 and 1225; 8 of 64, 4300 and 430 21.1 and 21.6, 5600 and 560 26.8 and 25.9, 7000 and
// 700 30.2 and 28.2; 12 of 64, 4300 24.45 and 24.5, 5000 26.8 and 26.3; 32 over 8, fp32, 2500 and 250 100.2 and 100.7, 4096 and 410 221.7 and 220.9, 6000 and 600 425.5 and 418.9.
static bool whole_tiles(int64_t wgs, int64_t head_wgs, int64_t nrb, int64_t tiles, const zc_tensor4* q) {
  if (q->dtype == ZC_F32) return nrb >= 4 && wgs > (q->D == 128 ? 512 : 1024);
  return wgs > 1024 ? tiles >= 32 : nrb >= 4 && wgs <= 960 && 10 * nrb * tiles >= 44 * head_wgs;
}
// Whether few probe rows are served by one launch (k_probe_few), with how many times 16 columns a workgroup and blocks of 16 rows a
// wave, by what the ways cost in us.  One launch: the trips of its start, those of a wave's further blocks, and, a round of
// a workgroup per CU, the bytes each reads (K once a wave), of which a CU gets 37 KB a us, all of them together in several
// rounds 22 (fp32) and 28.  Two: workgroups of a head's 128 columns, of which
// fp32 has one a CU and 16-bit types four.  us, two launches and one, measured and as priced: bf16, 8 heads of 64 channels, 100 tokens, 10
// rows 5.8 / 3.7 and 5.9 / 3.7; 16 heads over 4, 300 tokens, 30 rows 5.9 / 5.6 and 5.9 / 5.7; 32 heads over 8 of 128 channels, 100 tokens
// 6.2 / 7.4 and 6.2 / 7.9; 16 x 32 over 8, 1000 tokens 22.5 / 18.4 (32 columns) and 21.9 / 18.9; fp32, 12 heads of 64,
// 256 tokens, 26 rows 7.9 / 7.5 and 8.1 / 7.8; 16 of 128, 100 tokens 10.0 / 8.9 and 10 / 8.5; 24 over 8, 64 tokens, 7 rows 9.9 / 10.3 and 10 / 10.2.
// Where sweep 1 leaves ranges, the two launches join them on the way and the one needs a launch for that first, 1.8 us more
// (`ranges`; both sweeps, two and one: 2 x 16 heads over 4 of 64, 281 tokens, 28 rows, fp16 10.8 and 11.9; 2 x 16 of 128, 120 and 12, fp32 17.3 and 18.3;
// 4 x 16 over 4 of 64, 167 and 16, fp32 13.8 and 14.1; but 3 x 12 of 64, 105 and 10, fp32 14.1 and 12.7).
struct FewPlan { int cols, blocks; };
static FewPlan probe_few(int64_t B, int64_t Hq, int64_t Hkv, int64_t Lk, int64_t P, int64_t D, bool fp32, bool ranges) {
  FewPlan plan = {0, 0};
  if (P > kFewRows || Hq * P > kFewTable) return plan;
  const int64_t row_bytes = D * (fp32 ? 4 : 2), rt = ceil_div64(P, 16);
  const double wgs = (double)(ceil_div64(Lk, 128) * Hq * B) / 256.0;
  double best, further;
  if (fp32) {
    best = (D == 64 ? 7.9 : 10.0) + (wgs > 1.0 ? (D == 64 ? 2.4 : 5.3) * (wgs - 1.0) : 0.0);
    further = D == 64 ? 1.5 : 2.3;
  } else {
    best = (D == 64 ? 5.8 : 6.1) + 0.5 * (wgs < 4.0 ? wgs : 4.0) + (wgs > 4.0 ? (D == 64 ? 0.85 : 1.15) * (wgs - 4.0) : 0.0);
    further = D == 64 ? 0.2 : 1.1;
  }
  for (int64_t nc = 1; nc <= 2; ++nc)
    for (int64_t share = nc == 2 && few_both(P, fp32, D) ? rt : 1; share <= (nc == 2 && !few_both(P, fp32, D) ? 1 : rt); ++share) {
      const int64_t blocks = ceil_div64(Hq * rt, 16 * share) * share, waves = ceil_div64(Hq * rt, blocks), segments = Hkv > waves ? Hkv : waves;
      const int64_t n = B * ceil_div64(Lk, 16 * nc), rounds = ceil_div64(n, 256);
      const double rate = rounds == 1 ? 37.0 : fp32 ? 22.0 : 28.0;
      const double t = (ranges ? 4.8 : 3.0) + further * (double)(blocks - 1) + (double)(rounds * (segments * 16 * nc + Hq * P) * row_bytes) / (1e3 * rate);
      if (t < best) { best = t; plan = {(int)nc, (int)blocks}; }
    }
  return plan;
}
static size_t lse_bytes(int64_t B, int64_t Hq, int64_t P) { return (size_t)align_up64(B * Hq * P * (kProbeParts * (int64_t)sizeof(float2) + 4), 256); }

// What a call needs at least; and what it takes on top for the pairs of the column ranges to lie beside the per-head
// scores, so that sweep 2 can join them while it writes these: where the probes are few and its workgroups one round
// (of several rounds each reads the pairs again: 16 x 40 heads of 128 channels, 4096 tokens, 410 probes: 352 us
// and a launch of 8.4, joined 398; 32 heads: 19.2 and 4.6, joined 21.4).  Nothing for up to 64 probes, whose
// ranges are then at most the kProbeParts there is room for: where that makes them of two tiles instead of one it is
// still the better way (fp32, 64 probes of 640 tokens, us per call with a launch of its own over 10 ranges and joined:
// 32 heads of 128 channels 23.4 and 20.8, 4 x 16 of 64 22.9 and 20.6; only 4 heads lose, 700 tokens: 20.6 and 20.9).
static size_t probe_least_bytes(int64_t B, int64_t Hq, int64_t Lk, int64_t P) { return lse_bytes(B, Hq, P) + (size_t)B * Hq * Lk * 4; }
constexpr int64_t kJoinWgs = 1024;
static size_t join_bytes(int64_t B, int64_t Hq, int64_t P) {
  const int64_t heads = B * Hq < kJoinWgs ? B * Hq : kJoinWgs, rows = P < kProbeTable ? P : kProbeTable;
  return P <= kLseRows / 2 ? 0 : (size_t)align_up64(heads * rows * (kMaxProbeParts - kProbeParts) * (int64_t)sizeof(float2), 256);
}
static bool probe_join(int64_t B, int64_t Hq, int64_t Lk, int64_t P) {
  return P <= kProbeTable && ceil_div64(Lk, 128) * Hq * B <= kJoinWgs;
}

extern "C" size_t zc_probe_saliency_workspace(int64_t B, int64_t Hq, int64_t Lk, int64_t P) {
  if (B <= 0 || Hq <= 0 || Lk <= 0 || P <= 0) return 0;
  return probe_least_bytes(B, Hq, Lk, P) + join_bytes(B, Hq, P);
}

static int probe_scores(const zc_tensor4* q, const zc_tensor4* k,
                        const int32_t* probe_rows, const int32_t* probe_pos, int32_t P,
                        float sm_scale, const float* lse_ext,
                        float* scores, float* scores_per_head,
                        void* ws, size_t ws_bytes, void* stream, bool normalize) {
  int rc = zc_validate_tensor(q);
  if (rc) return rc;
  rc = zc_validate_tensor(k);
  if (rc) return rc;
  if (q->dtype != k->dtype || q->D != k->D || q->B != k->B) return ZC_ERR_INVALID_ARG;
  if (q->H % k->H != 0) return ZC_ERR_INVALID_ARG;
  if (P < 1 || !probe_pos || !scores || k->L < 1 || q->L < 1) return ZC_ERR_INVALID_ARG;
  if (q->B > 65535 || q->H > 65535 || k->L > 0x7fffffff - 256) return ZC_ERR_UNSUPPORTED;
  if ((reinterpret_cast<uintptr_t>(probe_pos) & 3) || (reinterpret_cast<uintptr_t>(scores) & 3)) return ZC_ERR_INVALID_ARG;
  {
    // the kernels address one (batch, head) slab of q and of k with 32-bit byte offsets,
    // and request "nothing" at offset 0xFFFFF000, which must lie past the end of a slab
    const int64_t eb = q->dtype == ZC_F32 ? 4 : 2;
    // (sweep 2 asks for whole blocks of kBlockCols columns, up to 127 rows past the end of k, sweep 1 for whole tiles of 64: those
    // offsets must not wrap either)
    if (q->L * q->sL * eb >= 0xFFFFF000ll || (k->L + kBlockCols) * k->sL * eb >= 0xFFFFF000ll || (int64_t)P * 4 >= 0xFFFFF000ll) return ZC_ERR_UNSUPPORTED;
  }
  const size_t need = probe_least_bytes(q->B, q->H, k->L, P), extra = join_bytes(q->B, q->H, P);
  if (!ws || ws_bytes < need || (reinterpret_cast<uintptr_t>(ws) & 15)) return ZC_ERR_WORKSPACE;

  ProbeArgs a;
  a.q = q->ptr; a.k = k->ptr;
  a.q_sB = q->sB; a.q_sH = q->sH; a.q_sL = q->sL;
  a.k_sB = k->sB; a.k_sH = k->sH; a.k_sL = k->sL;
  a.B = (int)q->B; a.Hq = (int)q->H; a.Hkv = (int)k->H; a.G = a.Hq / a.Hkv; a.Lk = (int)k->L; a.Lq = (int)q->L; a.P = P;
  a.probe_rows = probe_rows; a.probe_pos = probe_pos;
  a.scale_log2 = (sm_scale == 0.f ? 1.0f / sqrtf((float)q->D) : sm_scale) * kLog2e;
  a.lse_in = lse_ext;
  a.join = !lse_ext && probe_join(q->B, q->H, k->L, P) && ws_bytes >= need + extra;
  const bool ranges = a.join && probe_head_wgs(q->B, q->H, P, k->L, extra > 0 ? kMaxProbeParts : kProbeParts, q->dtype == ZC_F32) > ceil_div64(P, kLseRows);
  const FewPlan few = probe_few(q->B, q->H, k->H, k->L, P, q->D, q->dtype == ZC_F32, ranges);
  a.few_cols = few.cols;
  a.few_blocks = few.blocks;
  if (a.few_cols) a.join = 0;
  float* ws_ph = reinterpret_cast<float*>(reinterpret_cast<uint8_t*>(ws) + lse_bytes(q->B, q->H, P) + (a.join ? extra : 0));
  // [log-sum-exps][column ranges' pairs, up to the end of the workspace: the per-head scores, at
  // their place in it, are written when the pairs have been read]; joined by sweep 2 [pairs][per-head scores]
  const int64_t rows = q->B * q->H * P, lse2_bytes = align_up64(rows * 4, 16), fit = ((int64_t)need - lse2_bytes) / (rows * (int64_t)sizeof(float2));
  a.lse2 = reinterpret_cast<float*>(ws);
  a.lse_part = reinterpret_cast<float2*>(reinterpret_cast<uint8_t*>(ws) + (a.join ? 0 : lse2_bytes));
  a.max_parts = (int)(a.join ? (extra > 0 ? kMaxProbeParts : kProbeParts) : (fit < kMaxProbeParts ? fit : kMaxProbeParts) & ~1);
  const int64_t head_wgs = probe_head_wgs(q->B, q->H, P, k->L, a.max_parts, q->dtype == ZC_F32);
  a.head_wgs = (int)head_wgs;
  if (head_wgs <= ceil_div64(P, kLseRows)) a.join = 0;     // (one range a row block: its log-sum-exps are in lse2)
  if (head_wgs * q->H * q->B > 0x7fffffff || (int64_t)ceil_div64(k->L, 128) * q->H * q->B > 0x7fffffff)
    return ZC_ERR_UNSUPPORTED;
  const int64_t wgs1 = head_wgs * q->H * q->B, wgs2 = ceil_div64(k->L, 128) * q->H * q->B;
  a.even1 = wgs1 >= 768 && even_waves(wgs1, (double)(ceil_div64(P, kLseRows) * ceil_div64(k->L, kLseCols)) / (double)head_wgs, q) ? kEvenTiles : 0;
  a.whole1 = whole_tiles(wgs1, head_wgs, ceil_div64(P, kLseRows), ceil_div64(k->L, kLseCols), q) ? 1 : 0;
  a.even2 = even_waves(wgs2, P / 64.0, q) ? kEvenTiles * 64 : 0;
  {
    const int64_t nct = ceil_div64(k->L, 128), heads = q->B * q->H, hpx = heads / 8, least = ceil_div64(256, nct), groups = hpx / least;
    a.group = heads % 8 == 0 && wgs2 > 256 && (P > 64 || q->dtype == ZC_F32) ? (int)(groups > 1 ? ceil_div64(hpx, groups) : hpx) : 0;
  }
  a.normalize = normalize ? 1 : 0;
  a.per_head = scores_per_head || a.few_cols ? scores_per_head : ws_ph;       // (few rows: only where the caller asks for them)

  hipStream_t st = (hipStream_t)stream;
  const bool need_lse = lse_ext == nullptr;
#define ZC_PROBE(DT) (q->D == 128 ? launch_probe<DT, 128>(a, need_lse, scores, st) : launch_probe<DT, 64>(a, need_lse, scores, st))
  if (q->dtype == ZC_F32) return ZC_PROBE(ZC_F32);
  if (q->dtype == ZC_F16) return ZC_PROBE(ZC_F16);
  return ZC_PROBE(ZC_BF16);
#undef ZC_PROBE
}

extern "C" int zc_probe_saliency(const zc_tensor4* q, const zc_tensor4* k,
                                 const int32_t* probe_rows, const int32_t* probe_pos, int32_t P,
                                 float sm_scale, const float* lse_ext,
                                 float* scores, float* scores_per_head,
                                 void* ws, size_t ws_bytes, void* stream) {
  return probe_scores(q, k, probe_rows, probe_pos, P, sm_scale, lse_ext, scores, scores_per_head, ws, ws_bytes, stream, true);
}

extern "C" int zc_probe_accumulated(const zc_tensor4* q, const zc_tensor4* k,
                                    const int32_t* probe_rows, const int32_t* probe_pos, int32_t P,
                                    float sm_scale, const float* lse_ext,
                                    float* scores, float* scores_per_head,
                                    void* ws, size_t ws_bytes, void* stream) {
  return probe_scores(q, k, probe_rows, probe_pos, P, sm_scale, lse_ext, scores, scores_per_head, ws, ws_bytes, stream, false);
}
