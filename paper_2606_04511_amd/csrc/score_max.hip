// score_max.hip -- the Forecast prefill score contraction on 32x32x16 MFMA (Sec. 4.1, Eq. 4):
// each row's largest candidate score (a measurement of the contraction alone), and the block
// scores of the row-wise selection path (at the end of this file).
//
// The score contraction on its own: every
// candidate block of every query row is scored and each row's scores are reduced on chip to
// their maximum, so that one float per row leaves the kernel.  It isolates the dense contraction
// that the fused select kernel performs before its per-row top-k, on the (64, 64) key grid.
//
// Work unit: the rows of one (batch, group) whose positions fall in one 64-token block (at most
// 64 rows, all with the candidate range [n_init, blk - n_local]).  A workgroup of four
// wavefronts owns one unit.  Each wavefront holds the unit's F rows as the B operand of
// v_mfma_f32_32x32x16_bf16 (two N-tiles of 32 rows, 64 VGPRs) and takes every fourth M-tile of
// 32 candidates, reading the K~ rows of its next M-tile (L2-resident) while the current one is
// multiplied.  The dot product's dimension order is free: lane half h of k-step 4 u + i holds
// dimensions 64 u + 32 h + 8 i .. + 7 of both operands, so a lane reads 64 contiguous bytes of a
// row per u.  Candidates past the range load the last candidate again (a repeated score leaves
// a maximum unchanged) and rows past the unit load its last row (their maximum is not written),
// so every load is unconditional and in bounds.  An accumulator lane holds 16 scores of one
// query column (lane % 32); the two lane halves and the four wavefronts are merged at the end.
//
// Units run from the most candidates to the fewest.  Consecutive workgroups take consecutive
// (batch, group) pairs, and workgroups are dealt to the 8 XCDs in turn, so with a pair count that
// is a multiple of 8 every workgroup of one group lands on one XCD and its K~ stays in that L2.
#include <math.h>

#include <algorithm>

#include "device_util.hpp"
#include "launch.hpp"

namespace sparda {

namespace {

constexpr int kSmThreads = 256;
constexpr int kSmWaves = kSmThreads / kWave;
constexpr int kRowU4 = kHeadDim * 2 / 16;  // 16-byte pieces per 128-dim bf16 row

typedef float f32x16 __attribute__((ext_vector_type(16)));

// The 8 k-step fragments (8 bf16 each) of one row for lane half h.
__device__ __forceinline__ void load_frags(const uint4* row, int h, uint4 (&x)[8]) {
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int i = 0; i < 4; ++i) x[4 * u + i] = row[8 * u + 4 * h + i];
}

// One M-tile of 32 candidates against both N-tiles; folds the scores into the running maxima.
__device__ __forceinline__ void score_tile(const uint4 (&a)[8], const uint4 (&fb)[2][8], float& run0, float& run1) {
  f32x16 c0, c1;
#pragma unroll
  for (int e = 0; e < 16; ++e) c0[e] = c1[e] = 0.f;
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const bf16x8 av = as_bf16x8(a[s]);
    c0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, as_bf16x8(fb[0][s]), c0, 0, 0, 0);
    c1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, as_bf16x8(fb[1][s]), c1, 0, 0, 0);
  }
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    run0 = fmaxf(run0, c0[e]);
    run1 = fmaxf(run1, c1[e]);
  }
}

__global__ __launch_bounds__(kSmThreads) void score_rowmax_kernel(ScoreMaxArgs a) {
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform: scalar loop control
  const int n = lane & 31, h = lane >> 5;
  const int grp = blockIdx.x % a.n_groups;                       // (batch, group) pair
  const int unit = a.n_units - 1 - (int)(blockIdx.x / a.n_groups);  // most candidates first
  const int blk = a.blk0 + unit;
  const int64_t p_lo = max((int64_t)blk * kBlock, a.q_pos0);
  const int64_t p_hi = min((int64_t)blk * kBlock + kBlock, a.q_pos0 + a.n_q);
  const int nr = (int)(p_hi - p_lo);  // 1..64 rows
  const int64_t row0 = (int64_t)grp * a.n_q + (p_lo - a.q_pos0);
  const int c_hi = blk - a.n_local;
  const int n_cand = c_hi >= a.n_init ? c_hi - a.n_init + 1 : 0;
  if (n_cand == 0) {
    if ((int)threadIdx.x < nr) a.row_max[row0 + threadIdx.x] = -INFINITY;
    return;
  }
  __shared__ float part[kSmWaves][64];

  // B operand: the unit's F rows 32 nt + n (clamped to the last row).
  uint4 fb[2][8];
#pragma unroll
  for (int nt = 0; nt < 2; ++nt) {
    const int r = min(32 * nt + n, nr - 1);
    load_frags(reinterpret_cast<const uint4*>(a.f) + (row0 + r) * kRowU4, h, fb[nt]);
  }

  const uint4* kc = reinterpret_cast<const uint4*>(a.kc) + ((int64_t)grp * a.nc_cap + a.n_init) * kRowU4;
  const int n_mt = (n_cand + 31) / 32;
  float run0 = -INFINITY, run1 = -INFINITY;
  if (w < n_mt) {
    // Two register buffers in turn: the M-tile after the current one is requested before the
    // current one is multiplied (past the end the last M-tile is requested again), so the wait
    // before the products covers only the current tile's loads.
    uint4 ab[2][8];
    auto arow = [&](int mt) { return kc + (int64_t)min(32 * min(mt, n_mt - 1) + n, n_cand - 1) * kRowU4; };
    load_frags(arow(w), h, ab[0]);
    for (int mt = w; mt < n_mt; mt += 2 * kSmWaves) {
      load_frags(arow(mt + kSmWaves), h, ab[1]);
      __builtin_amdgcn_sched_barrier(0);  // keep the request ahead of the products
      score_tile(ab[0], fb, run0, run1);
      load_frags(arow(mt + 2 * kSmWaves), h, ab[0]);
      __builtin_amdgcn_sched_barrier(0);
      if (mt + kSmWaves < n_mt) score_tile(ab[1], fb, run0, run1);
    }
  }
  // Lanes n and n + 32 hold the two row halves of column n.
  run0 = fmaxf(run0, __shfl_xor(run0, 32));
  run1 = fmaxf(run1, __shfl_xor(run1, 32));
  if (h == 0) {
    part[w][n] = run0;
    part[w][32 + n] = run1;
  }
  __syncthreads();
  if ((int)threadIdx.x < nr) {
    const int t = threadIdx.x;
    a.row_max[row0 + t] = fmaxf(fmaxf(part[0][t], part[1][t]), fmaxf(part[2][t], part[3][t]));
  }
}

// ---- the persistent form: the group's K~ in LDS --------------------------------------------
//
// When every row of the call has at most kSlMaxCand candidates, one 512-thread workgroup per CU
// stages its group's candidate keys in LDS once (272-byte row pitch: the 16 rows a quarter
// wavefront reads start 4 banks apart, so a 16-byte read is conflict-free) and its eight
// wavefronts take whole units from an LDS counter.  A wavefront requests the next unit's F rows
// before it multiplies the current unit, whose A fragments come from LDS.  A group's units are
// dealt to its workgroups in a serpentine over descending candidate counts, so each workgroup's
// list is balanced and sorted most-expensive first.

constexpr int kSlThreads = 512;
constexpr int kSlWaves = kSlThreads / kWave;
constexpr int kSlMaxCand = 512;
constexpr int kSlPitchU4 = kRowU4 + 1;  // 16-byte pieces per staged row (272 B)

__device__ __forceinline__ void load_lds_frags(const uint4* row, int h, uint4 (&x)[8]) {
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int i = 0; i < 4; ++i) x[4 * u + i] = row[8 * u + 4 * h + i];
}

struct SlUnit {
  int blk, nr, n_cand;
  int64_t row0;
};

// The i-th unit of workgroup slot s of p slots (serpentine over descending block index), or
// blk < 0 past the end.
__device__ __forceinline__ SlUnit sl_unit(const ScoreMaxArgs& a, int grp, int s, int p, int i) {
  SlUnit u;
  const int g = i * p + ((i & 1) ? p - 1 - s : s);
  if (g >= a.n_units) {
    u.blk = -1;
    u.nr = u.n_cand = 0;
    u.row0 = 0;
    return u;
  }
  u.blk = a.blk0 + a.n_units - 1 - g;
  const int64_t p_lo = max((int64_t)u.blk * kBlock, a.q_pos0);
  const int64_t p_hi = min((int64_t)u.blk * kBlock + kBlock, a.q_pos0 + a.n_q);
  u.nr = (int)(p_hi - p_lo);
  u.row0 = (int64_t)grp * a.n_q + (p_lo - a.q_pos0);
  const int c_hi = u.blk - a.n_local;
  u.n_cand = c_hi >= a.n_init ? c_hi - a.n_init + 1 : 0;
  return u;
}

__device__ __forceinline__ void load_unit_f(const ScoreMaxArgs& a, const SlUnit& u, int n, int h,
                                            uint4 (&fb)[2][8]) {
  const int nr = max(u.nr, 1);
#pragma unroll
  for (int nt = 0; nt < 2; ++nt) {
    const int r = min(32 * nt + n, nr - 1);
    load_frags(reinterpret_cast<const uint4*>(a.f) + (u.row0 + r) * kRowU4, h, fb[nt]);
  }
}

// Scores one unit against the staged keys and writes its rows' maxima.
__device__ __forceinline__ void sl_score_unit(const ScoreMaxArgs& a, const SlUnit& u, const uint4* kst,
                                              const uint4 (&fb)[2][8], int n, int h) {
  float run0 = -INFINITY, run1 = -INFINITY;
  const int n_mt = (u.n_cand + 31) / 32;
  // A fragments one M-tile ahead, in two register sets (reads past the end repeat the last tile)
  auto arow = [&](int mt) { return kst + min(32 * min(mt, n_mt - 1) + n, u.n_cand - 1) * kSlPitchU4; };
  uint4 a0[8], a1[8];
  load_lds_frags(arow(0), h, a0);
  for (int mt = 0; mt < n_mt; mt += 2) {
    load_lds_frags(arow(mt + 1), h, a1);
    __builtin_amdgcn_sched_barrier(0);
    score_tile(a0, fb, run0, run1);
    load_lds_frags(arow(mt + 2), h, a0);
    __builtin_amdgcn_sched_barrier(0);
    if (mt + 1 < n_mt) score_tile(a1, fb, run0, run1);
  }
  run0 = fmaxf(run0, __shfl_xor(run0, 32));
  run1 = fmaxf(run1, __shfl_xor(run1, 32));
  if (h == 0) {
    if (n < u.nr) a.row_max[u.row0 + n] = run0;
    if (32 + n < u.nr) a.row_max[u.row0 + 32 + n] = run1;
  }
}

__global__ __launch_bounds__(kSlThreads) void score_rowmax_lds_kernel(ScoreMaxArgs a, int slots) {
  __shared__ uint4 kst[kSlMaxCand * kSlPitchU4];  // [c_max][kSlPitchU4] used
  __shared__ int next_unit;
  const int lane = threadIdx.x & 63;
  const int n = lane & 31, h = lane >> 5;
  const int grp = blockIdx.x % a.n_groups;
  const int slot = blockIdx.x / a.n_groups;
  if (threadIdx.x == 0) next_unit = kSlWaves;
  // the largest candidate count of the call: the last row's
  const int c_hi = (int)((a.q_pos0 + a.n_q - 1) / kBlock) - a.n_local;
  const int c_max = c_hi >= a.n_init ? c_hi - a.n_init + 1 : 0;
  const uint4* kc = reinterpret_cast<const uint4*>(a.kc) + ((int64_t)grp * a.nc_cap + a.n_init) * kRowU4;
  if (c_max > 0) {
    // Every load in flight before the first LDS store.  Pieces past the staged rows are clamped
    // to the last piece: loaded and stored again with the same value (no branch for the
    // compiler to sink a load into).
    constexpr int kIt = kSlMaxCand * kRowU4 / kSlThreads / 2;  // two rounds of 8 pieces
    const int n_pc = c_max * kRowU4;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      uint4 t[kIt];
#pragma unroll
      for (int k = 0; k < kIt; ++k)
        t[k] = kc[min((int)threadIdx.x + (half * kIt + k) * kSlThreads, n_pc - 1)];
#pragma unroll
      for (int k = 0; k < kIt; ++k) {
        const int q = min((int)threadIdx.x + (half * kIt + k) * kSlThreads, n_pc - 1);
        kst[(q / kRowU4) * kSlPitchU4 + q % kRowU4] = t[k];
      }
    }
  }

  // Each wavefront starts with unit w of the slot's list; later units come from the counter.
  // Even wavefronts request their first F rows before the staging barrier and odd ones after
  // it, so that the two wavefronts of a SIMD do not wait for one burst together: the first can
  // multiply while the second one's rows arrive.
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  SlUnit cur = sl_unit(a, grp, slot, slots, w);
  uint4 fb[2][8], fn[2][8];
  const bool first_early = (w & 1) == 0;
  if (first_early && cur.blk >= 0 && cur.n_cand > 0) load_unit_f(a, cur, n, h, fb);
  __syncthreads();
  if (!first_early && cur.blk >= 0 && cur.n_cand > 0) load_unit_f(a, cur, n, h, fb);

  while (cur.blk >= 0) {
    int j = 0;
    if (lane == 0) j = atomicAdd(&next_unit, 1);
    j = __builtin_amdgcn_readfirstlane(j);
    const SlUnit nxt = sl_unit(a, grp, slot, slots, j);
    // The next unit's F rows are requested before this unit's products (past the end, this
    // unit's rows again: in bounds and never used).
    load_unit_f(a, nxt.blk >= 0 && nxt.n_cand > 0 ? nxt : cur, n, h, fn);
    __builtin_amdgcn_sched_barrier(0);
    if (cur.n_cand == 0) {
      if (lane < cur.nr) a.row_max[cur.row0 + lane] = -INFINITY;
    } else {
      sl_score_unit(a, cur, kst, fb, n, h);
    }
    cur = nxt;
    if (cur.blk < 0) break;
    // the same with the buffers' roles exchanged
    if (lane == 0) j = atomicAdd(&next_unit, 1);
    j = __builtin_amdgcn_readfirstlane(j);
    const SlUnit nx2 = sl_unit(a, grp, slot, slots, j);
    load_unit_f(a, nx2.blk >= 0 && nx2.n_cand > 0 ? nx2 : cur, n, h, fb);
    __builtin_amdgcn_sched_barrier(0);
    if (cur.n_cand == 0) {
      if (lane < cur.nr) a.row_max[cur.row0 + lane] = -INFINITY;
    } else {
      sl_score_unit(a, cur, kst, fn, n, h);
    }
    cur = nx2;
  }
}

// ---- block scores of many rows, for the row-wise selection path ------------------------------
//
// Multi-row calls whose rows have more than kSelTileMaxCand candidates keep every candidate's score in
// the workspace (row stride ws_stride, the first candidate at slot 0) for the row-wise top-k.  A unit
// is 64 consecutive rows of one (batch, group), the A operand of two 32-row M-tiles, owned by one
// wavefront; B = 32 keys, so a row's scores of consecutive candidates lie in consecutive lanes and
// leave in 128-byte stores.  On the (32, 16) grid lane n of tile u holds window u of block n: the
// max-pool over a block's five windows (u = -1, the last window of the block before, to 3) is an
// elementwise maximum over five tiles, and only block scores leave the chip.
//
// A workgroup's four wavefronts take four units over one chunk of candidates, staged 128 windows at a
// time in two LDS slots straight from memory: group n of a slot holds the four rows that lane n reads
// (windows 4 n .. 4 n + 3 of the stage, or on the one-key-per-block grid keys n, 32 + n, 64 + n, 96 + n),
// 1040 bytes apart so that the 32 lanes of a read touch every bank once.
//
// What bounds it: the matrix cores (five tiles of 16 products per 32 blocks and 64 rows) and the
// stores.  4096 rows of 8 groups at 128K on the (32, 16) grid: 100-115 us (0.27 GB of block scores, 84
// GFLOP issued); window scores with keys along the accumulator, read from L2 row by row and stored 16
// bytes per row, took 386 us and left four times the bytes for the top-k to pool.
constexpr int kBsGroup = 1040;              // bytes from one group of four staged rows to the next
constexpr int kBsSlot = 33 * kBsGroup;      // group -1 (the block before the stage's first), then 0 .. 31
constexpr int kBsUnits = 4;                 // units (wavefronts) per workgroup

struct BlockScoreArgs {
  SelectArgs s;
  int32_t n_wg;                             // workgroups per (batch, group) and chunk
  int32_t n_chunks, chunk_stages;
};

template <bool kBlocks>  // one key per block, or the (32, 16) grid
__global__ __launch_bounds__(64 * kBsUnits, 2) void block_score_kernel(BlockScoreArgs b) {
  constexpr int kPerStage = kBlocks ? 128 : 32;  // candidates
  __shared__ __align__(16) char slots[2 * kBsSlot];
  const SelectArgs& a = b.s;
  const int lane = threadIdx.x & 63, n = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n_groups = a.batch * a.n_kv_heads;
  const int grp = blockIdx.x % n_groups, x = blockIdx.x / n_groups;
  const int chunk = x % b.n_chunks, wg = b.n_wg - 1 - x / b.n_chunks;  // latest rows (most candidates) first
  // the workgroup's last row has the most candidates and sees the most windows
  const int64_t p_wg = a.q_pos0 + min((wg + 1) * 64 * kBsUnits, a.n_q) - 1;
  const RowGeom g_wg = row_geom(p_wg, a.n_init, a.n_local, a.k_total);
  if (g_wg.n_take >= g_wg.n_cand) return;  // then every row takes all its candidates
  const int c_lo = chunk * b.chunk_stages * kPerStage;
  const int c_hi = min(c_lo + b.chunk_stages * kPerStage, g_wg.n_cand);
  if (c_lo >= c_hi) return;
  int32_t w_min, w_max;  // the windows of its candidates: nothing past them is read
  row_windows(g_wg, a.grid, p_wg, &w_min, &w_max);
  // this wavefront's unit
  const int r0 = (wg * kBsUnits + wave) * 64, nr = min(64, a.n_q - r0);
  const bool live = nr > 0;
  const int64_t p0 = a.q_pos0 + r0;
  const int n_cand = live ? row_geom(p0 + nr - 1, a.n_init, a.n_local, a.k_total).n_cand : 0;
  const int vis0 = grid_win_vis(a.grid, p0);

  bf16x8 fa[2][8];
#pragma unroll
  for (int mt = 0; mt < 2; ++mt) {
    const uint16_t* src = a.f + ((int64_t)grp * a.n_q + (live ? r0 + min(32 * mt + n, nr - 1) : 0)) * kHeadDim + 32 * h;
#pragma unroll
    for (int s = 0; s < 8; ++s) fa[mt][s] = as_bf16x8(ld16(src + 64 * (s >> 2) + 8 * (s & 3)));
  }
  const uint16_t* keys = a.kc + (int64_t)grp * a.nc_cap * kHeadDim;
  const uint32_t slots_at = __builtin_amdgcn_readfirstlane(lds_address(slots));
  const int r4 = lane >> 4;
  // window of row r4 of group i in the stage whose first candidate is c0
  auto stage = [&](int c0, uint32_t slot) {
    auto bring = [&](int i) {
      const int w = kBlocks ? g_wg.cand_lo + c0 + 32 * r4 + i : 4 * (g_wg.cand_lo + c0 + i) + r4;
      const int key = min(max(w, 0), w_max);
      lds_load16(keys, (uint32_t)key * (kHeadDim * 2) + 16 * (lane & 15), slot + (i + 1) * kBsGroup);
    };
#pragma unroll
    for (int i = 0; i < 8; ++i) bring(8 * wave + i);
    if (!kBlocks && wave == 0) bring(-1);
  };
  const int n_stage = (c_hi - c_lo + kPerStage - 1) / kPerStage;
  stage(c_lo, slots_at);
  float* const out = a.ws + ((int64_t)grp * a.n_q + r0) * a.ws_stride;
  for (int st = 0; st < n_stage; ++st) {
    lds_loads_landed();  // this wavefront's part of the slot is here and its reads of the other returned
    __syncthreads();
    const char* now = slots + (st & 1) * kBsSlot;
    const int c0 = c_lo + st * kPerStage;
    if (st + 1 < n_stage) stage(c0 + kPerStage, slots_at + ((st + 1) & 1) * kBsSlot);
    if (!live || c0 >= n_cand) continue;
    auto tile = [&](int group, int row, f32x16& c0_, f32x16& c1_) {
      const char* src = now + (n + 1 + group) * kBsGroup + row * 256 + 64 * h;
      bf16x8 k[8];
#pragma unroll
      for (int s = 0; s < 8; ++s) k[s] = as_bf16x8(*reinterpret_cast<const uint4*>(src + 128 * (s >> 2) + 16 * (s & 3)));
#pragma unroll
      for (int e = 0; e < 16; ++e) c0_[e] = c1_[e] = 0.f;
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        c0_ = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[0][s], k[s], c0_, 0, 0, 0);
        c1_ = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[1][s], k[s], c1_, 0, 0, 0);
      }
    };
    // accumulator element e of lane (n, h) is row 8 (e / 4) + 4 h + e % 4 of the M-tile, key n
    auto store = [&](int c, const f32x16& s0, const f32x16& s1) {
      if (c + n >= n_cand) return;
      int64_t stride = a.ws_stride;
      __asm__ __volatile__("" : "+s"(stride));  // row addresses here: held across the loop they would spill
      float* d = out + (int64_t)(4 * h) * stride + c + n;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int r = 8 * (e >> 2) + (e & 3);
        if (r + 4 * h < nr) d[r * stride] = s0[e];
        if (32 + r + 4 * h < nr) d[(32 + r) * stride] = s1[e];
      }
    };
    if (kBlocks) {
#pragma unroll 1
      for (int t = 0; t < 4 && c0 + 32 * t < n_cand; ++t) {
        f32x16 s0, s1;
        tile(0, t, s0, s1);
        store(c0 + 32 * t, s0, s1);
      }
    } else {
      const int blk = g_wg.cand_lo + c0 + n;  // the lane's block
      f32x16 s0, s1;
      tile(-1, 3, s0, s1);
      if (blk == 0) {  // no window before block 0
#pragma unroll
        for (int e = 0; e < 16; ++e) s0[e] = s1[e] = -INFINITY;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        f32x16 t0, t1;
        tile(0, u, t0, t1);
        if (4 * (g_wg.cand_lo + c0 + 31) + u > vis0) {  // windows that some row does not see whole
          // the last token of the lane's window, from the position of the lane half's first row
          int tail = 16 * (4 * blk + u) + 31 - (int)p0 - 4 * h;
          __asm__ __volatile__("" : "+v"(tail));  // the comparisons here: held across the loop they would spill
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            const int r = 8 * (e >> 2) + (e & 3);
            if (tail > r) t0[e] = -INFINITY;
            if (tail > 32 + r) t1[e] = -INFINITY;
          }
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          s0[e] = fmaxf(s0[e], t0[e]);
          s1[e] = fmaxf(s1[e], t1[e]);
        }
      }
      store(c0, s0, s1);
    }
  }
}

}  // namespace

hipError_t launch_score_rowmax(const ScoreMaxArgs& a, hipStream_t stream) {
  const int c_hi = (int)((a.q_pos0 + a.n_q - 1) / kBlock) - a.n_local;
  const int c_max = c_hi >= a.n_init ? c_hi - a.n_init + 1 : 0;
  // Persistent form whenever the keys fit: about one workgroup per CU and at least one unit per
  // wavefront.  Workgroup b serves group b % n_groups, so with 8 | n_groups a group's workgroups
  // share an XCD.
  if (c_max <= kSlMaxCand) {
    const int slots = std::max(1, std::min(a.n_units / kSlWaves, 256 / a.n_groups));
    hipLaunchKernelGGL(score_rowmax_lds_kernel, dim3((unsigned)(slots * a.n_groups)), dim3(kSlThreads), 0, stream,
                       a, slots);
    return hipGetLastError();
  }
  const int64_t wgs = (int64_t)a.n_units * a.n_groups;
  hipLaunchKernelGGL(score_rowmax_kernel, dim3((unsigned)wgs), dim3(kSmThreads), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_block_scores(const SelectArgs& a, hipStream_t stream) {
  BlockScoreArgs b;
  b.s = a;
  const int n_groups = a.batch * a.n_kv_heads;
  const bool blocks = grid_is_blocks(a.grid);
  const RowGeom g = row_geom(a.q_pos0 + a.n_q - 1, a.n_init, a.n_local, a.k_total);
  const int stages = (g.n_cand + (blocks ? 127 : 31)) / (blocks ? 128 : 32);
  b.n_wg = (a.n_q + 64 * kBsUnits - 1) / (64 * kBsUnits);
  // Chunks of candidates so that about four workgroups per CU are in flight, at least four stages each; where
  // those would not even be one per CU, shorter ones up to two per CU.  Measured with four and with at least
  // one stage (us, 34 500 to 131 072 tokens): one key per block, 70 rows of 8 groups 18-24 and 9-10, 1000 of
  // 8 25-30 and 16-20, 4096 of 8 23-51 and 25-55; (32, 16) grid 15-17 and 8-11, 22-30 and 21-39, 34-110 and
  // 40-112.
  const int64_t base = (int64_t)n_groups * b.n_wg;
  int64_t chunks = std::max<int64_t>(1, std::min<int64_t>((1024 + base - 1) / base, (stages + 3) / 4));
  if (base * chunks < 256) chunks = std::max(chunks, std::min<int64_t>(512 / base, stages));
  b.chunk_stages = (int)((stages + chunks - 1) / chunks);
  b.n_chunks = (stages + b.chunk_stages - 1) / b.chunk_stages;
  const dim3 grid((unsigned)((int64_t)n_groups * b.n_wg * b.n_chunks)), block(64 * kBsUnits);
  if (blocks)
    hipLaunchKernelGGL(block_score_kernel<true>, grid, block, 0, stream, b);
  else
    hipLaunchKernelGGL(block_score_kernel<false>, grid, block, 0, stream, b);
  return hipGetLastError();
}

}  // namespace sparda
