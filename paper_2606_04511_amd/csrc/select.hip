// select.hip -- Forecast scoring and top-k block selection (paper Sec. 4.1, Eq. 4, with the
// attended-set union of Eq. 1).
//
// Per query row at position p: forced = initial blocks U local window, candidates = the complete
// blocks in between, window scores F_row . K~_i (one Forecast head per GQA group, no softmax, no
// scale, float32 accumulation), block score s_j = the max over the windows that overlap block j
// and are complete at p (the identity for the one-key-per-block grid); the k_total - |forced|
// best candidates by (score desc, index asc) join the forced blocks; the row's set is written in
// ascending block order, -1 padded.
//
// Two paths:
//  * row-wise (decode, n_q == 1, and long multi-row cases): a bandwidth-bound GEMV kernel writes
//    the candidate scores of each row to a float32 scratch row (from 16 rows on, MFMA units write
//    pooled block scores, score_max.hip); a second kernel runs one wavefront per row that finds the
//    exact k-th key by counts over keys in registers (up to 4096 candidates) or an 8-bit-digit radix
//    select over a wave-private LDS histogram, and emits the chosen indices in ascending order.
//  * fused decode (one row per (batch, group), <= 16384 candidates, and multi-row calls of few rows):
//    one workgroup per row keeps the row's scores in LDS and runs the block-wide top-k there
//    (select_block.hpp).
//  * fused tile (multi-row prefill with <= 512 candidates per 64-row tile): select_prefill.hip.
#include "device_util.hpp"
#include "launch.hpp"
#include "select_block.hpp"

namespace sparda {

// ---- row-wise path ----------------------------------------------------------------------

// grid.x = row * n_chunks + chunk; a chunk is 256 windows (64 per wavefront).  Lane l reads dims
// 8*(l%16)..+7 of window 4 i + l/16: each wavefront load is 1 KiB contiguous of K~.  Window
// first + x of the row goes to scratch slot x.  kOnce (one row per (batch, group)): no other row
// reads the keys, so they are streamed past the caches (decode step of 64 rows at 128K: 77.6 to
// 74.9 us); rows of one group share them through L2 and load them the ordinary way.
template <bool kOnce>
__global__ __launch_bounds__(256) void rowwise_score_kernel(SelectArgs a, int n_chunks) {
  const int64_t row = blockIdx.x / n_chunks;
  const int chunk = (int)(blockIdx.x % n_chunks);
  const int r = (int)(row % a.n_q);
  const int64_t bm = row / a.n_q;
  const int64_t p = a.q_pos0 + r;
  const RowGeom g = row_geom(p, a.n_init, a.n_local, a.k_total);
  if (g.n_take >= g.n_cand) return;
  int32_t wf, wl;
  row_windows(g, a.grid, p, &wf, &wl);
  const int nw = wl - wf + 1;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int c = lane & 15, rs = lane >> 4;
  const int first = chunk * 256 + wave * 64;
  if (first >= nw) return;
  const uint4 fw = ld16(a.f + row * kHeadDim + c * 8);
  const float f0 = bf16lo(fw.x), f1 = bf16hi(fw.x), f2 = bf16lo(fw.y), f3 = bf16hi(fw.y);
  const float f4 = bf16lo(fw.z), f5 = bf16hi(fw.z), f6 = bf16lo(fw.w), f7 = bf16hi(fw.w);
  const uint16_t* kbase = a.kc + (bm * a.nc_cap + wf) * kHeadDim + c * 8;
  uint4 kw[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int idx = min(first + 4 * i + rs, nw - 1);  // past the last window: a repeat, never stored
    kw[i] = ld16_hint<kOnce>(kbase + (int64_t)idx * kHeadDim);
  }
  float* out = a.ws + row * a.ws_stride;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    float d = f0 * bf16lo(kw[i].x);
    d = fmaf(f1, bf16hi(kw[i].x), d);
    d = fmaf(f2, bf16lo(kw[i].y), d);
    d = fmaf(f3, bf16hi(kw[i].y), d);
    d = fmaf(f4, bf16lo(kw[i].z), d);
    d = fmaf(f5, bf16hi(kw[i].z), d);
    d = fmaf(f6, bf16lo(kw[i].w), d);
    d = fmaf(f7, bf16hi(kw[i].w), d);
    d = row16_sum(d);
    const int idx = first + 4 * i + rs;
    if (c == 0 && idx < nw) out[idx] = d;
  }
}

static hipError_t launch_rowwise_scores(const SelectArgs& a, int64_t rows, int n_chunks, hipStream_t stream) {
  const dim3 grid((unsigned)(rows * n_chunks)), block(256);
  if (a.n_q == 1)
    hipLaunchKernelGGL(rowwise_score_kernel<true>, grid, block, 0, stream, a, n_chunks);
  else
    hipLaunchKernelGGL(rowwise_score_kernel<false>, grid, block, 0, stream, a, n_chunks);
  return hipGetLastError();
}

// Rows with at most this many candidates keep their block keys in registers (row_topk_kernel); longer
// rows run the radix passes over the workspace (rowwise_topk_kernel).
constexpr int kRowTopkMax = 4096;

// kPooled: the row's block scores are in the workspace, candidate 0 at slot 0 (block_score_kernel, or any
// scores on the one-key-per-block grid); otherwise its window scores on the (32, 16) grid, window wf at
// slot 0.
template <bool kPooled>
__device__ __forceinline__ float candidate_score(const SelectArgs& a, const float* sc, int cand_lo, int i, int32_t wf,
                                                 int32_t wvis) {
  return kPooled ? sc[i] : pooled_score(sc, a.grid, cand_lo + i, wf, wvis);
}

// One wavefront per row: forced blocks, padding, count, and the radix top-k over the scratch row.
template <bool kPooled>
__global__ __launch_bounds__(256) void rowwise_topk_kernel(SelectArgs a, int64_t n_rows) {
  __shared__ __align__(16) uint32_t hist[4][256];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + wave;
  if (row >= n_rows) return;
  const int64_t p = a.q_pos0 + (int)(row % a.n_q);
  const RowGeom g = row_geom(p, a.n_init, a.n_local, a.k_total);
  int16_t* out = a.sel + row * a.k_total;
  emit_forced(out, g, a.k_total, lane);
  if (lane == 0) a.cnt[row] = (int16_t)(g.n_forced + g.n_take);
  const float* sc = a.ws + row * a.ws_stride;
  int32_t wf, wl;
  row_windows(g, a.grid, p, &wf, &wl);
  const int32_t wvis = grid_win_vis(a.grid, p);
  wave_topk_emit([&](int i) { return score_key(candidate_score<kPooled>(a, sc, g.cand_lo, i, wf, wvis)); }, g.n_cand,
                 g.n_take, g.cand_lo, hist[wave], out + g.init_hi);
}

// The same for rows of at most 64 R candidates, their keys in registers (reg_topk_emit: candidate
// 64 i + lane is key i of the lane).
//
// What bounds it: for many rows VALU issue (about 1000 instructions per row of 2048, half the time) and the
// row's one load latency, for few rows latency alone; so a row holds no more slots than it has candidates
// and its loads are batched.  32 768 rows of 2045 block scores 120-125 us (pooling window scores into LDS
// and four radix passes there 730); window scores of 8000 rows of 30, 122, 247 and 1560 candidates 7.3,
// 12.3, 16.3 and 74 us (26, 34, 35 and 96 with at least 16 slots and all loads at once; 10.8, 18.6, 34 and
// 140 by radix passes), of 128 rows of 30 candidates 3.8 (9.4; 5.5).
template <int R, bool kPooled, bool kScores>
__global__ __launch_bounds__(256) void row_topk_kernel(SelectArgs a, int64_t n_rows) {
  __shared__ uint32_t list[4][64];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + wave;
  if (row >= n_rows) return;
  const int64_t p = a.q_pos0 + (int)(row % a.n_q);
  const RowGeom g = row_geom(p, a.n_init, a.n_local, a.k_total);
  int16_t* out = a.sel + row * a.k_total;
  emit_forced(out, g, a.k_total, lane);
  if (lane == 0) a.cnt[row] = (int16_t)(g.n_forced + g.n_take);
  out += g.init_hi;
  const int C = g.n_cand, n = g.n_take;
  if (n >= C) {
    for (int i = lane; i < C; i += kWave) out[i] = (int16_t)(g.cand_lo + i);
    return;
  }
  if (n <= 0) return;
  const float* sc = a.ws + row * a.ws_stride;
  // Slots past the row's candidates: key 0, below every score.  The loads are requested kBatch slots at a time
  // before the first is waited for, repeats of the last candidate past the end; the empty asm keeps the
  // compiler from moving each into a branch of its own.
  uint32_t key[R];
  if constexpr (kPooled) {
    constexpr int kBatch = R < 16 ? R : 16;
#pragma unroll
    for (int i0 = 0; i0 < R; i0 += kBatch) {
      float x[kBatch];
#pragma unroll
      for (int i = 0; i < kBatch; ++i) x[i] = sc[min(64 * (i0 + i) + lane, C - 1)];
#pragma unroll
      for (int i = 0; i < kBatch; ++i) {
        __asm__ __volatile__("" : "+v"(x[i]));
        key[i0 + i] = 64 * (i0 + i) + lane < C ? score_key(x[i]) : 0u;
      }
    }
  } else {  // block j's windows are 4 j - 1 .. 4 j + 3: five loads, repeats past the first and the last one
    constexpr int kBatch = R < 8 ? R : 8;
    constexpr WinGrid kGrid{32, 16};
    const int32_t wf = grid_win_lo(kGrid, g.cand_lo), wvis = grid_win_vis(kGrid, p);
#pragma unroll
    for (int i0 = 0; i0 < R; i0 += kBatch) {
      float x[kBatch][5];
#pragma unroll
      for (int i = 0; i < kBatch; ++i) {
        const int lo = 4 * (g.cand_lo + min(64 * (i0 + i) + lane, C - 1)) - 1;
#pragma unroll
        for (int u = 0; u < 5; ++u) x[i][u] = sc[max(min(lo + u, wvis), 0) - wf];
      }
#pragma unroll
      for (int i = 0; i < kBatch; ++i) {
#pragma unroll
        for (int u = 0; u < 5; ++u) __asm__ __volatile__("" : "+v"(x[i][u]));
        const float m = fmaxf(fmaxf(fmaxf(x[i][0], x[i][1]), fmaxf(x[i][2], x[i][3])), x[i][4]);
        key[i0 + i] = 64 * (i0 + i) + lane < C ? score_key(m) : 0u;
      }
    }
  }
  if constexpr (R == 1)
    lane_topk_emit(key[0], C, n, g.cand_lo, out);
  else
    reg_topk_emit<R, kScores>(key, C, n, g.cand_lo, out, list[wave]);
}

template <bool kPooled, bool kScores>
static hipError_t launch_topk(const SelectArgs& a, hipStream_t stream) {
  const int64_t rows = (int64_t)a.batch * a.n_kv_heads * a.n_q;
  const int C = row_geom(a.q_pos0 + a.n_q - 1, a.n_init, a.n_local, a.k_total).n_cand;  // the last row has the most
  const dim3 grid((unsigned)((rows + 3) / 4)), block(256);
  if constexpr (!kScores) {  // Forecast scores come here from 513 candidates on only
    if (C <= 512) {
      if (C <= 64)
        hipLaunchKernelGGL((row_topk_kernel<1, kPooled, false>), grid, block, 0, stream, a, rows);
      else if (C <= 128)
        hipLaunchKernelGGL((row_topk_kernel<2, kPooled, false>), grid, block, 0, stream, a, rows);
      else if (C <= 256)
        hipLaunchKernelGGL((row_topk_kernel<4, kPooled, false>), grid, block, 0, stream, a, rows);
      else
        hipLaunchKernelGGL((row_topk_kernel<8, kPooled, false>), grid, block, 0, stream, a, rows);
      return hipGetLastError();
    }
  }
  if (C <= 1024)
    hipLaunchKernelGGL((row_topk_kernel<16, kPooled, kScores>), grid, block, 0, stream, a, rows);
  else if (C <= 2048)
    hipLaunchKernelGGL((row_topk_kernel<32, kPooled, kScores>), grid, block, 0, stream, a, rows);
  else if (C <= kRowTopkMax)
    hipLaunchKernelGGL((row_topk_kernel<64, kPooled, kScores>), grid, block, 0, stream, a, rows);
  else
    hipLaunchKernelGGL(rowwise_topk_kernel<kPooled>, grid, block, 0, stream, a, rows);
  return hipGetLastError();
}

// Window scores in the workspace: on the one-key-per-block grid they are the blocks'.
template <bool kScores>
static hipError_t launch_window_topk(const SelectArgs& a, hipStream_t stream) {
  return grid_is_blocks(a.grid) ? launch_topk<true, kScores>(a, stream) : launch_topk<false, kScores>(a, stream);
}

// ---- fused decode path ---------------------------------------------------------------------

// One workgroup per decode row (batch, group): the Forecast GEMV over all scored windows into LDS,
// the max-pool of window scores to block scores (skipped for the one-key-per-block grid), then
// the block-wide top-k (value bins, the threshold bin ranked exactly) and an ordered emission.
// Scores never leave the CU.
template <bool kOnce>
__global__ __launch_bounds__(kDecThreads) void decode_select_kernel(SelectArgs a) {
  __shared__ float sc[kDecodeMaxCand];
  __shared__ __align__(16) uint32_t hist[kTopkLds];
  __shared__ int wave_cnt[kDecThreads / 64];
  __shared__ int pick[3];
  // workgroup x takes row x / n_groups of group x % n_groups, so that (with 8 | n_groups) the rows of a
  // group share an XCD's L2
  const int64_t n_groups = (int64_t)a.batch * a.n_kv_heads;
  const int64_t bm = blockIdx.x % n_groups, r = blockIdx.x / n_groups, row = bm * a.n_q + r;
  a.q_pos0 += r;
  a.kc += (bm - row) * a.nc_cap * kHeadDim;  // the row's keys, where decode_select_row looks for them
  decode_select_row<kOnce>(a, row, sc, hist, wave_cnt, pick, a.sel + row * a.k_total, a.cnt + row);
}

// Decode rows with their window scores already in the workspace (row stride ws_stride, window
// wf of the row at offset 0): one workgroup per row loads them into LDS, max-pools them to block
// scores and runs the block-wide top-k.  The second kernel of the split decode path.
__global__ __launch_bounds__(kDecThreads) void decode_topk_kernel(SelectArgs a) {
  __shared__ float sc[kDecodeMaxCand];
  __shared__ __align__(16) uint32_t hist[kTopkLds];
  __shared__ int wave_cnt[kDecThreads / 64];
  __shared__ int pick[3];
  const int64_t row = blockIdx.x;
  decode_topk_row(a, row, sc, hist, wave_cnt, pick, a.sel + row * a.k_total, a.cnt + row);
}

// Which kernels serve a select call.
enum SelectPath { kPathDecode, kPathDecodeSplit, kPathTile, kPathRowwise };

// Decode calls with fewer rows than CUs score each row with many workgroups (the row-wise score
// kernel, 256 windows each) and select with one workgroup per row; otherwise one fused workgroup
// per row.
constexpr int64_t kDecodeSplitRows = 256;
// Multi-row calls of few rows (verifying drafted tokens, the tail of a prompt) select like decode rows,
// one workgroup per row: at most two rounds (a CU holds one workgroup), of at most the windows that a full
// tile row has.  Measured, 16 to 256 rows, then 512 (us, this path against the tile kernels or, past 512
// candidates, the row-wise path): (64, 64) grid at 2K 5.7 and 8.6 against 10-11, 4K 7.1 and 10.2 against
// 10-13, 8K 6.9 and 12.4 against 11-17, 20K 7.3 and 13.3 against 12-23, 32K 7.7 and 14.2 against 20-22,
// 64K 12 and 22 against 20-36; (32, 16) grid at 2K 6.5 and 10.3 against 12-16, 4K 7.8 and 11.6 against
// 15-17, 8K 8.2 and 15.4 against 20-22, 20K 12 and 23 against 28-34, 32K 16 and 32 against 41-46.  1024
// rows at 20K 26 against 22-24 and 46 against 35-39.  At 4060 windows per row ((32, 16) grid at 64K) 27 and
// 52 for 256 and 512 rows against 23-39.
constexpr int64_t kFewRows = 512;
constexpr int64_t kFewRowsWindows = 4 * kSelTileMaxCand + 1;
// Multi-row calls on the row-wise path with at least this many rows score on MFMA.
constexpr int32_t kTileScoreMinRows = 16;

static SelectPath select_path(int64_t rows, int32_t n_q, int64_t q_pos0, int32_t n_init, int32_t n_local,
                              WinGrid grid) {
  const int64_t p = q_pos0 + n_q - 1;
  const RowGeom g = row_geom(p, n_init, n_local, 1 << 30);
  int32_t wf, wl;
  row_windows(g, grid, p, &wf, &wl);
  const int64_t nw = wl >= wf ? wl - wf + 1 : 0;
  // window scores and (for a windowed grid) block scores share the LDS score array
  const int64_t need = grid_is_blocks(grid) ? g.n_cand : nw + g.n_cand;
  if (n_q == 1) {
    if (need > kDecodeMaxCand) return kPathRowwise;
    return rows < kDecodeSplitRows && nw >= 1024 ? kPathDecodeSplit : kPathDecode;
  }
  if (rows <= kFewRows && nw <= kFewRowsWindows) return kPathDecode;  // at most 2561 floats
  // multi-row: the fused tile kernel serves up to kSelTileMaxCand candidates per row
  return g.n_cand <= kSelTileMaxCand ? kPathTile : kPathRowwise;
}

int select_decode_path(int64_t rows, int32_t n_q, int64_t q_pos0, int32_t n_init, int32_t n_local, WinGrid grid) {
  const SelectPath path = select_path(rows, n_q, q_pos0, n_init, n_local, grid);
  return path == kPathDecode ? 0 : path == kPathDecodeSplit ? 1 : -1;
}

hipError_t launch_decode_split_scores(const SelectArgs& a, hipStream_t stream) {
  const int64_t rows = (int64_t)a.batch * a.n_kv_heads;
  const RowGeom g = row_geom(a.q_pos0, a.n_init, a.n_local, a.k_total);
  int32_t wf, wl;
  row_windows(g, a.grid, a.q_pos0, &wf, &wl);
  if (g.n_cand <= 0 || wl < wf) return hipSuccess;
  const int n_chunks = (wl - wf + 1 + 255) / 256;
  return launch_rowwise_scores(a, rows, n_chunks, stream);
}

// The workspace that a call must bring depends on its rows' lengths alone: a call of few rows past the
// tile kernel's candidates needs the row-wise path's, though the decode kernel leaves it unused.
bool select_needs_scratch(int64_t rows, int32_t n_q, int64_t q_pos0, int32_t n_init, int32_t n_local, WinGrid grid) {
  if (n_q > 1) return row_geom(q_pos0 + n_q - 1, n_init, n_local, 1 << 30).n_cand > kSelTileMaxCand;
  const SelectPath path = select_path(rows, n_q, q_pos0, n_init, n_local, grid);
  return path == kPathRowwise || path == kPathDecodeSplit;
}

hipError_t launch_rowwise_topk(const SelectArgs& a, hipStream_t stream) { return launch_window_topk<false>(a, stream); }

hipError_t launch_select(const SelectArgs& a, hipStream_t stream) {
  const int64_t rows = (int64_t)a.batch * a.n_kv_heads * a.n_q;
  const SelectPath path = select_path(rows, a.n_q, a.q_pos0, a.n_init, a.n_local, a.grid);
  if (path == kPathDecode) {
    // several rows of a group share its keys through L2: 5 rows x 64 groups at 32K 31.6 us, with the
    // hint 36.1; 12 x 8 at 20K 12.1 against 12.5
    if (a.n_q == 1)
      hipLaunchKernelGGL(decode_select_kernel<true>, dim3((unsigned)rows), dim3(kDecThreads), 0, stream, a);
    else
      hipLaunchKernelGGL(decode_select_kernel<false>, dim3((unsigned)rows), dim3(kDecThreads), 0, stream, a);
    return hipGetLastError();
  }
  if (path == kPathTile) return launch_prefill_select(a, stream);
  const int64_t pl = a.q_pos0 + a.n_q - 1;
  const RowGeom gl = row_geom(pl, a.n_init, a.n_local, a.k_total);
  int32_t wf, wl;
  row_windows(gl, a.grid, pl, &wf, &wl);
  if (gl.n_cand > 0 && wl >= wf && a.n_q >= kTileScoreMinRows) {
    // many rows: 64-row units score on MFMA, each key fragment shared by the unit's rows
    hipError_t e = launch_block_scores(a, stream);
    return e != hipSuccess ? e : launch_topk<true, true>(a, stream);
  } else if (gl.n_cand > 0 && wl >= wf) {  // the last row scores the most windows
    const int n_chunks = (wl - wf + 1 + 255) / 256;
    hipError_t e = launch_rowwise_scores(a, rows, n_chunks, stream);
    if (e != hipSuccess) return e;
  }
  if (path != kPathDecodeSplit) return launch_window_topk<true>(a, stream);
  hipLaunchKernelGGL(decode_topk_kernel, dim3((unsigned)rows), dim3(kDecThreads), 0, stream, a);
  return hipGetLastError();
}

}  // namespace sparda
