// indexer_kl.hip -- the indexer-training loss of Sec. 4.2 (Eq. 6-7) and its gradient with respect
// to the Forecast rows, on synthetic tensors (the Forecast projection's own weight gradient is a
// plain GEMM of this gradient with the layer input, outside this file).
//
// Per query row at position p of group m (G query heads):
//   target     each head's softmax of sm_scale q_h . K~t_i over the fine (2, 1) windows complete at
//              p (window i = mean of keys i, i + 1), summed over the group; T_w = the largest such
//              sum over the fine windows lying inside position w of the prediction grid
//              ((32, 16): tokens [16 w, 16 w + 32)).
//   predicted  P = softmax over the positions complete at p of sm_scale F . K~p_w.
//   selected   S = the k_top largest T_w (ties: lower w) among positions inside candidate blocks.
//   loss       KL of the (k+1)-bucket partitions: t_c = T_c / sum T for c in S plus the rest bucket,
//              against P_c and R = sum of P outside S.
//   gradient   dL/dz_w = P_w - t_w in S, P_w (1 - t_rest / R) outside; dF = sm_scale sum_w dz_w K~p_w.
//
// Kernels:
//   pair_compress_kernel -- the (2, 1) windows of the raw keys into the workspace: float64 sum of
//                           the pair, one rounding to bf16 (as every compressed key).
//   head_stats_kernel, head_weights_kernel, or head_unit_kernel for few fine windows and units
//                           (head_tiles.hpp) -- for G in {1, 2, 4, 8, 16}: the target's shared weights
//                           for 64 / G rows at a time (64 (row, head) columns on 32x32x16 MFMA),
//                           max-pooled to segments of 16 fine windows in the workspace (2 floats per
//                           segment instead of one per fine window).
//   kl_predict_kernel    -- for the same G, beside the two launches: F . K~p of 64 rows at a time on
//                           MFMA into the workspace.
//   kl_row_kernel        -- one 512-thread workgroup per query row.  Target: the max-pool of those
//                           weights into the positions, or for other G 16-window x 16-head
//                           MFMA tiles (A = the windows, B = the group's query rows padded to 16
//                           columns), an online maximum and sum of 2^z per head, then a second
//                           pass that sums each window's normalised head weights across the
//                           columns and max-pools it into its positions in LDS (atomic max on the
//                           float bits: all values are >= 0).  Prediction: the logits of
//                           kl_predict_kernel (or a Forecast GEMV) and their softmax in LDS.  Selection: the block-wide
//                           top-k of select_block.hpp over the candidate positions.  Then
//                           the bucket sums, the loss and the gradient GEMV.
#include <math.h>

#include "device_util.hpp"
#include "launch.hpp"
#include "head_tiles.hpp"
#include "select_block.hpp"

namespace sparda {

// Limits (checked by the entry point): 16384 positions per row and k_top <= 4096, so that the row
// kernel's per-position LDS arrays (9 bytes per position plus 2 per top-k entry) fit one CU.

__global__ __launch_bounds__(256) void pair_compress_kernel(const uint16_t* __restrict__ k, uint16_t* __restrict__ kt,
                                                            int64_t t_cap, int64_t n_win, int64_t rows) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;  // (row, window, 16-byte chunk)
  const int64_t total = rows * n_win * 16;
  if (idx >= total) return;
  const int c = (int)(idx & 15);
  const int64_t rw = idx >> 4;
  const int64_t row = rw / n_win, i = rw - row * n_win;
  const uint16_t* src = k + (row * t_cap + i) * kHeadDim + 8 * c;
  const uint4 a = ld16(src), b = ld16(src + kHeadDim);
  const uint32_t aw[4] = {a.x, a.y, a.z, a.w}, bw[4] = {b.x, b.y, b.z, b.w};
  uint32_t o[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const double lo = ((double)bf16lo(aw[e]) + (double)bf16lo(bw[e])) * 0.5;  // exact, then one rounding
    const double hi = ((double)bf16hi(aw[e]) + (double)bf16hi(bw[e])) * 0.5;
    o[e] = (uint32_t)f64_to_bf16(lo) | ((uint32_t)f64_to_bf16(hi) << 16);
  }
  *reinterpret_cast<uint4*>(kt + (row * n_win + i) * kHeadDim + 8 * c) = make_uint4(o[0], o[1], o[2], o[3]);
}

struct KlArgs {
  const uint16_t* q;      // [B][Hq][n_q][D]
  const uint16_t* kt;     // [B][Hkv][nt][D] fine windows (workspace)
  const uint16_t* f;      // [B][Hkv][n_q][D]
  const uint16_t* kp;     // [B][Hkv][nc_cap][D] prediction windows
  float* loss;            // [B][Hkv][n_q]
  float* dF;              // [B][Hkv][n_q][D]
  float* sw;              // [B][Hkv][n_q][sw_stride] segment maxima of the shared target weights (workspace)
  const float* z;         // [B][Hkv][n_q][sw_stride] prediction logits (exp2 domain; workspace)
  int64_t sw_stride;
  int32_t lds_pos, lds_top;  // per-position LDS entries (>= 512, a multiple of 16) and top-k list entries
  int64_t nt, nc_cap, q_pos0;
  int32_t n_kv_heads, group_size, n_q, n_init, n_local, k_top;
  WinGrid grid;           // prediction grid
  float scale_log2;       // sm_scale * log2(e)
  float sm_scale;
};

__device__ __forceinline__ float block_sum_f(float x, float* red, int wave, int lane) {
  x = row16_sum(x);
  x += __shfl_xor(x, 16, kWave);
  x += __shfl_xor(x, 32, kWave);
  __syncthreads();
  if (lane == 0) red[wave] = x;
  __syncthreads();
  float s = 0.f;
#pragma unroll
  for (int w = 0; w < kDecThreads / 64; ++w) s += red[w];
  return s;
}

// Three sums over the workgroup in one round of barriers.  red: at least 3 * kDecThreads / 64 floats.
__device__ __forceinline__ void block_sum3_f(float (&x)[3], float* red, int wave, int lane) {
  constexpr int kWaves = kDecThreads / 64;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    x[i] = row16_sum(x[i]);
    x[i] += __shfl_xor(x[i], 16, kWave);
    x[i] += __shfl_xor(x[i], 32, kWave);
  }
  __syncthreads();
  if (lane == 0)
#pragma unroll
    for (int i = 0; i < 3; ++i) red[i * kWaves + wave] = x[i];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    x[i] = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) x[i] += red[i * kWaves + w];
  }
}

__device__ __forceinline__ float block_max_f(float x, float* red, int wave, int lane) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) x = fmaxf(x, __shfl_xor(x, d, kWave));
  __syncthreads();
  if (lane == 0) red[wave] = x;
  __syncthreads();
  float m = red[0];
#pragma unroll
  for (int w = 1; w < kDecThreads / 64; ++w) m = fmaxf(m, red[w]);
  return m;
}

// The prediction's logits (in the exp2 domain) of many rows on MFMA: a unit is 64 rows of one (batch,
// group) with their one Forecast head (head_tiles.hpp with G = 1), against the prediction positions.
__global__ __launch_bounds__(kHtThreads, 2) void kl_predict_kernel(HeadTileArgs a) {
  using namespace head_tiles;
  __shared__ __align__(16) char slots[2 * kHtSlot];
  const int lane = threadIdx.x & 63, n = lane & 31, h = lane >> 5;
  const Unit u = unit_of<1>(a);
  bf16x8 fa[2][8];
  load_rows<1>(a, u, fa);
  float* const out = a.out + ((int64_t)u.grp * a.n_q + u.r0) * a.out_stride;
  walk<1>(a, u, fa, slots, [&](int key0, f32x16 (&c)[2]) {
    int64_t stride = a.out_stride;
    __asm__ __volatile__("" : "+s"(stride));  // row addresses here: held across the loop they would spill
    if (key0 + n >= u.n_keys) return;
    float* d = out + (int64_t)h * stride + key0 + n;
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int row = 32 * mt + 2 * e;  // of lane half 0
        if (row + h < u.nr) d[row * stride] = c[mt][e] * a.scale_log2;
      }
  });
}

// kLogits: the row's logits are in a.z (kl_predict_kernel); otherwise it computes them itself.
// kPre: the segment maxima of the target's shared weights are in a.sw (head_tiles.hpp); the row
// max-pools them into its positions.  Otherwise the row computes them itself (16-window x 16-column MFMA tiles).
template <bool kPre, bool kLogits>
__global__ __launch_bounds__(kDecThreads) void kl_row_kernel(KlArgs a) {
  // Per-position arrays, sized by the host for the call's largest row (kl_lds_layout): the pooled
  // target (float bits for the atomic max), the predicted distribution, the top-k list and the
  // chosen flags.  A small footprint lets several rows share a CU.
  extern __shared__ __align__(16) float kl_lds[];
  float* Tp = kl_lds;
  float* Pp = kl_lds + a.lds_pos;
  int16_t* idx = reinterpret_cast<int16_t*>(Pp + a.lds_pos);
  uint8_t* chosen = reinterpret_cast<uint8_t*>(idx + a.lds_top);
  __shared__ __align__(16) uint32_t hist[kTopkLds];
  __shared__ int wave_cnt[kDecThreads / 64];
  __shared__ int pick[3];
  __shared__ float red[3 * (kDecThreads / 64)];
  __shared__ float red_m[kDecThreads / 64][16], red_s[kDecThreads / 64][16];
  const int64_t row = blockIdx.x;  // (b * Hkv + m) * n_q + r
  const int r = (int)(row % a.n_q);
  const int64_t bm = row / a.n_q;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = lane & 15, j = lane >> 4;
  const int G = a.group_size;
  const int64_t p = a.q_pos0 + r;
  const int N = grid_win_vis(a.grid, p) + 1;           // positions 0 .. N - 1 (host-checked)
  const int n_tw = (int)p;                              // fine windows 0 .. p - 1 are complete at p
  float zl = -INFINITY;  // the largest logit of the thread's positions

  // ---- target
  if (kPre) {
    // T_w = the largest shared weight among the fine windows inside position w: tokens [i, i + 2)
    // within [w s, w s + l), i.e. i in [w s, w s + l - 2]: l / 16 segments of 16 fine windows, the last
    // one without its last window; every position complete at p has them
    const float2* seg = reinterpret_cast<const float2*>(a.sw + row * a.sw_stride);
    const float* z = kLogits ? a.z + row * a.sw_stride : nullptr;  // the row's logits, from kl_predict_kernel
    const int gs = a.grid.s / 16, gl = a.grid.l / 16;
    for (int w = tid; w < N; w += kDecThreads) {
      float m = seg[w * gs + gl - 1].x;
      for (int i = 0; i < gl - 1; ++i) m = fmaxf(m, seg[w * gs + i].y);
      Tp[w] = m;
      if (kLogits) {
        const float zw = z[w];
        Pp[w] = zw;
        zl = fmaxf(zl, zw);
      }
      chosen[w] = 0;
    }
  } else {  // MFMA tiles of 16 fine windows x the group's heads
    for (int w = tid; w < N; w += kDecThreads) {
      Tp[w] = 0.f;
      chosen[w] = 0;
    }
    __syncthreads();
    bf16x8 qb[4];
    // columns past the group's heads read head 0 (a valid address) and are zeroed
    const uint16_t* qrow = a.q + ((bm * G + (n < G ? n : 0)) * a.n_q + r) * kHeadDim + 8 * j;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const uint4 v = ld16(qrow + 32 * ks);
      qb[ks] = as_bf16x8(n < G ? v : make_uint4(0u, 0u, 0u, 0u));
    }
    const uint16_t* kb = a.kt + bm * a.nt * kHeadDim + 8 * j;
    const int n_tiles = (n_tw + 15) >> 4;
    auto score = [&](int t, float (&z)[4]) {
      const int win = min(16 * t + n, n_tw - 1);
      uint4 w[4];
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) w[ks] = ld16(kb + (int64_t)win * kHeadDim + 32 * ks);
      f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) c = mfma16x16x32(as_bf16x8(w[ks]), qb[ks], c);
#pragma unroll
      for (int e = 0; e < 4; ++e) z[e] = 16 * t + 4 * j + e < n_tw ? c[e] * a.scale_log2 : -INFINITY;
    };
    float m_run = -INFINITY, s_run = 0.f;
    for (int t = wave; t < n_tiles; t += kDecThreads / 64) {
      float z[4];
      score(t, z);
      const float mn = fmaxf(m_run, fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3])));
      if (mn > -INFINITY) {
        s_run = s_run * exp2f(m_run - mn) + exp2f(z[0] - mn) + exp2f(z[1] - mn) + exp2f(z[2] - mn) + exp2f(z[3] - mn);
        m_run = mn;
      }
    }
    auto merge = [](float& m, float& s, float m2, float s2) {
      const float mn = fmaxf(m, m2);
      if (mn > -INFINITY) {
        s = s * exp2f(m - mn) + s2 * exp2f(m2 - mn);
        m = mn;
      }
    };
    merge(m_run, s_run, __shfl_xor(m_run, 16, kWave), __shfl_xor(s_run, 16, kWave));
    merge(m_run, s_run, __shfl_xor(m_run, 32, kWave), __shfl_xor(s_run, 32, kWave));
    if (lane < 16) {
      red_m[wave][n] = m_run;
      red_s[wave][n] = s_run;
    }
    __syncthreads();
    float M = red_m[0][n], S = red_s[0][n];
#pragma unroll
    for (int w = 1; w < kDecThreads / 64; ++w) merge(M, S, red_m[w][n], red_s[w][n]);
    const float inv = n < G ? 1.0f / S : 0.f;
    const int gl = a.grid.l, gs = a.grid.s;
    for (int t = wave; t < n_tiles; t += kDecThreads / 64) {
      float z[4];
      score(t, z);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float sh = row16_sum(n < G ? exp2f(z[e] - M) * inv : 0.f);
        const int i = 16 * t + 4 * j + e;
        if (n == e && i < n_tw) {
          // positions w with w s <= i and i + 2 <= w s + l
          const int w_hi = min(i / gs, N - 1);
          const int num = i + 2 - gl;
          const int w_lo = num <= 0 ? 0 : (num + gs - 1) / gs;
          for (int w = w_lo; w <= w_hi; ++w) atomicMax(reinterpret_cast<unsigned int*>(&Tp[w]), __float_as_uint(sh));
        }
      }
    }
  }
  __syncthreads();

  // ---- prediction: the logits, from kl_predict_kernel (above) or a Forecast GEMV over the positions (16
  // lanes per position), then their softmax.  A position's entries are read and written by its own
  // thread from here to the top-k, and between the top-k and the gradient.
  if (!kLogits) {
    const int c = lane & 15, rs = lane >> 4;
    float fv[8];
    {
      const uint4 w = ld16(a.f + (bm * a.n_q + r) * kHeadDim + 8 * c);
      fv[0] = bf16lo(w.x) * a.scale_log2; fv[1] = bf16hi(w.x) * a.scale_log2;
      fv[2] = bf16lo(w.y) * a.scale_log2; fv[3] = bf16hi(w.y) * a.scale_log2;
      fv[4] = bf16lo(w.z) * a.scale_log2; fv[5] = bf16hi(w.z) * a.scale_log2;
      fv[6] = bf16lo(w.w) * a.scale_log2; fv[7] = bf16hi(w.w) * a.scale_log2;
    }
    const uint16_t* kpb = a.kp + bm * a.nc_cap * kHeadDim + 8 * c;
    for (int base = wave * 4; base < N; base += (kDecThreads / 64) * 4) {
      const int w = base + rs;
      const uint4 k = ld16(kpb + (int64_t)min(w, N - 1) * kHeadDim);
      float d = fv[0] * bf16lo(k.x);
      d = fmaf(fv[1], bf16hi(k.x), d);
      d = fmaf(fv[2], bf16lo(k.y), d);
      d = fmaf(fv[3], bf16hi(k.y), d);
      d = fmaf(fv[4], bf16lo(k.z), d);
      d = fmaf(fv[5], bf16hi(k.z), d);
      d = fmaf(fv[6], bf16lo(k.w), d);
      d = fmaf(fv[7], bf16hi(k.w), d);
      d = row16_sum(d);
      if (c == 0 && w < N) Pp[w] = d;
    }
  }
  if (!kLogits) {
    __syncthreads();
    for (int w = tid; w < N; w += kDecThreads) zl = fmaxf(zl, Pp[w]);
  }
  const float zmax = block_max_f(zl, red, wave, lane);
  float el = 0.f;
  for (int w = tid; w < N; w += kDecThreads) {
    const float e = exp2f(Pp[w] - zmax);
    Pp[w] = e;
    el += e;
  }
  const float pinv = 1.0f / block_sum_f(el, red, wave, lane);

  // ---- the target's top-k among positions inside candidate blocks [n_init, blk(p) - n_local]
  const int blk = (int)(p / kBlock);
  const int tok_lo = a.n_init * kBlock, tok_hi = (blk - a.n_local + 1) * kBlock;
  const int c_lo = (tok_lo + a.grid.s - 1) / a.grid.s;
  const int c_hi = min(N - 1, tok_hi - a.grid.l >= 0 ? (tok_hi - a.grid.l) / a.grid.s : -1);
  const int C = c_hi >= c_lo ? c_hi - c_lo + 1 : 0;
  const int n_take = min(a.k_top, C);
  __syncthreads();
  if (n_take >= C) {
    for (int i = tid; i < C; i += kDecThreads) chosen[c_lo + i] = 1;
  } else if (n_take > 0) {
    block_topk_emit(Tp + c_lo, C, n_take, c_lo, idx, hist, wave_cnt, pick);
    __syncthreads();
    for (int i = tid; i < n_take; i += kDecThreads) chosen[idx[i]] = 1;
  }
  __syncthreads();

  // ---- buckets and loss
  float sums[3] = {0.f, 0.f, 0.f};  // the target, then target and prediction outside the chosen positions
  for (int w = tid; w < N; w += kDecThreads) {
    const float t = Tp[w], pw = Pp[w] * pinv;
    Pp[w] = pw;
    sums[0] += t;
    if (!chosen[w]) {
      sums[1] += t;
      sums[2] += pw;
    }
  }
  block_sum3_f(sums, red, wave, lane);
  const float Ttot = sums[0], R = sums[2];
  const float tinv = 1.0f / Ttot;
  const float t_rest = sums[1] / Ttot;
  const float rest_f = R > 0.f ? 1.0f - t_rest / R : 0.f;
  float kl = 0.f;
  for (int w = tid; w < N; w += kDecThreads) {
    const float pw = Pp[w];
    if (chosen[w]) {
      const float tc = Tp[w] * tinv;
      if (tc > 0.f) kl += tc * __logf(tc / pw);
      Pp[w] = pw - tc;
    } else {
      Pp[w] = pw * rest_f;
    }
  }
  kl = block_sum_f(kl, red, wave, lane);  // its barriers also make every position's weight visible
  if (tid == 0) a.loss[row] = kl + (t_rest > 0.f ? t_rest * __logf(t_rest / R) : 0.f);

  // ---- gradient: dF[d] = sm_scale sum_w g_w K~p_w[d].  The weights g replace P in LDS; lane l of
  // wavefront v takes dimensions 8 (l % 16) .. + 7 of positions 4 (v + 8 i) + l / 16, so a wavefront
  // load is 1 KiB of K~p and a position's weight one LDS read for 16 lanes (a 2-byte load, two LDS reads
  // and a flag per product before: 270 of the 785 us of the kernel at 2048 rows of 4094 positions).
  // What bounds the kernel is latency, four rows to a CU: eight loads are in flight per wavefront here,
  // and each pass over the positions above does all it can for its barrier (208 to 135 us; one load at a
  // time 208, four 138).
  {
    constexpr int kStep = (kDecThreads / 64) * 4, kBatch = 8;
    const int c = lane & 15, rs = lane >> 4;
    const uint16_t* kpb = a.kp + bm * a.nc_cap * kHeadDim + 8 * c;
    float acc[8] = {};
    for (int base = wave * 4; base < N; base += kBatch * kStep) {
      uint4 k[kBatch];
      float g[kBatch];
#pragma unroll
      for (int i = 0; i < kBatch; ++i) {
        const int w = base + i * kStep + rs, wc = min(w, N - 1);
        k[i] = ld16(kpb + (int64_t)wc * kHeadDim);
        g[i] = w < N ? Pp[wc] : 0.f;
      }
#pragma unroll
      for (int i = 0; i < kBatch; ++i) {
        acc[0] = fmaf(g[i], bf16lo(k[i].x), acc[0]);
        acc[1] = fmaf(g[i], bf16hi(k[i].x), acc[1]);
        acc[2] = fmaf(g[i], bf16lo(k[i].y), acc[2]);
        acc[3] = fmaf(g[i], bf16hi(k[i].y), acc[3]);
        acc[4] = fmaf(g[i], bf16lo(k[i].z), acc[4]);
        acc[5] = fmaf(g[i], bf16hi(k[i].z), acc[5]);
        acc[6] = fmaf(g[i], bf16lo(k[i].w), acc[6]);
        acc[7] = fmaf(g[i], bf16hi(k[i].w), acc[7]);
      }
    }
    // the wavefront's four position residues, then the wavefronts through LDS (the target scores are no
    // longer needed: at least 512 floats, so two rounds of four wavefronts)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      acc[i] += __shfl_xor(acc[i], 16, kWave);
      acc[i] += __shfl_xor(acc[i], 32, kWave);
    }
    float sum = 0.f;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      __syncthreads();
      if (wave / 4 == half && rs == 0)
#pragma unroll
        for (int i = 0; i < 8; ++i) Tp[(wave & 3) * kHeadDim + 8 * c + i] = acc[i];
      __syncthreads();
      if (tid < kHeadDim) sum += Tp[tid] + Tp[tid + 128] + Tp[tid + 256] + Tp[tid + 384];
    }
    if (tid < kHeadDim) a.dF[row * kHeadDim + tid] = a.sm_scale * sum;
  }
}

hipError_t launch_indexer_kl(const uint16_t* q, const uint16_t* k, const uint16_t* f, const uint16_t* kp,
                             uint16_t* kt_ws, float* sw_ws, float* loss, float* dF, int32_t batch, int32_t n_kv_heads,
                             int32_t group_size, int32_t n_q, int64_t q_pos0, int64_t t_cap, int64_t nc_cap,
                             int32_t n_init, int32_t n_local, int32_t k_top, WinGrid grid, float sm_scale,
                             hipStream_t stream) {
  const int64_t rows_g = (int64_t)batch * n_kv_heads;
  const int64_t nt = q_pos0 + n_q - 1;  // fine windows complete at the last row: 0 .. p - 1
  if (nt > 0) {
    const int64_t total = rows_g * nt * 16;
    hipLaunchKernelGGL(pair_compress_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream, k, kt_ws,
                       t_cap, nt, rows_g);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  KlArgs a;
  a.q = q;
  a.kt = kt_ws;
  a.f = f;
  a.kp = kp;
  a.loss = loss;
  a.dF = dF;
  a.nt = nt > 0 ? nt : 1;
  a.nc_cap = nc_cap;
  a.q_pos0 = q_pos0;
  a.n_kv_heads = n_kv_heads;
  a.group_size = group_size;
  a.n_q = n_q;
  a.n_init = n_init;
  a.n_local = n_local;
  a.k_top = k_top;
  a.grid = grid;
  a.sm_scale = sm_scale;
  a.scale_log2 = sm_scale * 1.4426950408889634f;
  a.sw = sw_ws;
  a.sw_stride = (a.nt + 3) & ~(int64_t)3;
  // the last row has the most positions; the gradient's reduction reuses 512 entries of Tp
  const int n_max = grid_win_vis(grid, q_pos0 + n_q - 1) + 1;
  a.lds_pos = n_max > 512 ? (n_max + 15) & ~15 : 512;
  a.lds_top = ((k_top < n_max ? k_top : n_max) + 8) & ~7;
  const size_t lds = (size_t)a.lds_pos * 2 * sizeof(float) + (size_t)a.lds_top * sizeof(int16_t) + (size_t)a.lds_pos;
  const int G = group_size;
  if (G == 1 || G == 2 || G == 4 || G == 8 || G == 16) {  // the target of 64 / G rows per MFMA unit
    HeadTileArgs t = {};
    t.q = q;
    t.keys = kt_ws;
    t.key_cap = a.nt;
    // the statistics of a row's heads stay in its gradient row (128 floats), which kl_row_kernel
    // overwrites at the end
    t.part = dF;
    t.part_stride = kHeadDim;
    t.out = sw_ws;
    t.out_stride = a.sw_stride;
    t.q_pos0 = q_pos0;
    t.n_groups = (int32_t)rows_g;
    t.n_q = n_q;
    t.grid = WinGrid{2, 1};
    t.scale_log2 = a.scale_log2;
    hipError_t e;
    if (head_units_fit(t, G, (int)nt)) {  // at most 63 positions, whose logits a row forms itself
      e = launch_head_units<head_tiles::kSegments>(t, G, (int)nt, stream);
      if (e != hipSuccess) return e;
      a.z = nullptr;
      hipLaunchKernelGGL((kl_row_kernel<true, false>), dim3((unsigned)(rows_g * n_q)), dim3(kDecThreads), lds, stream, a);
      return hipGetLastError();
    }
    plan_head_tiles(t, G, kHeadDim / (2 * G));
    e = launch_head_tiles<head_tiles::kSegments>(t, G, stream);
    if (e != hipSuccess) return e;
    // the logits of a row's positions after its segment maxima: of the fine windows' nt floats per row
    // the maxima take 2 per 16 and the logits 1 per 16 or 64
    a.z = sw_ws + 2 * ((a.nt + 15) / 16);
    HeadTileArgs z = {};
    z.q = f;
    z.keys = kp;
    z.key_cap = nc_cap;
    z.out = const_cast<float*>(a.z);
    z.out_stride = a.sw_stride;
    z.q_pos0 = q_pos0;
    z.n_groups = (int32_t)rows_g;
    z.n_q = n_q;
    z.grid = grid;
    z.scale_log2 = a.scale_log2;
    plan_head_tiles(z, 1, 64);
    hipLaunchKernelGGL(kl_predict_kernel, dim3((unsigned)((int64_t)z.n_groups * z.n_wg * z.n_chunks)), dim3(kHtThreads),
                       0, stream, z);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((kl_row_kernel<true, true>), dim3((unsigned)(rows_g * n_q)), dim3(kDecThreads), lds, stream, a);
  } else {
    hipLaunchKernelGGL((kl_row_kernel<false, false>), dim3((unsigned)(rows_g * n_q)), dim3(kDecThreads), lds, stream, a);
  }
  return hipGetLastError();
}

}  // namespace sparda
