// head_tiles.hpp -- per-head softmax weights over compressed keys, summed over a GQA group, for
// 64 (row, head) columns at a time on 32x32x16 MFMA.  Shared by the multi-head selector's
// multi-row path (Sec. 3, the InfLLM-V2 selector) and the indexer-training target (Sec. 4.2,
// Eq. 6), which apply the same per-head softmax and group sum to different keys.
//
// A unit is 64 / G rows of one (batch, group) with their G heads, owned by one wavefront: the A
// operand of two M-tiles of 32 (row, head) pairs; B = 32 keys.  Accumulator element e of lane
// (n, h) is pair (e, h) against key n, and the pairs are dealt so that a row's G heads are G
// consecutive elements of one lane: the sum over heads needs no exchange, and a row's weights of 32
// consecutive keys lie in 32 consecutive lanes, so they are stored (or max-pooled) along the keys.
// The dimension order of the contraction is free: lane half h of k-step 4 u + i holds dimensions
// 64 u + 32 h + 8 i .. + 7 of both operands.
//
// A workgroup's four wavefronts take up to four units (of the same group) over one chunk of keys,
// staged 128 at a time in two LDS slots straight from memory (one barrier per 128 keys), so that a key
// read from L2 serves up to 256 columns; with fewer units the wavefronts share a unit's keys.
// Chunks fill the chip when there are few units: two launches (few units of few keys take one, at the end
// of this file),
//  * head_stats_kernel: per column and chunk the maximum and sum of 2^z over the keys the column's
//    row sees (z = scale * log2 e * q . k), the first tile's maximum standing in for the running
//    maximum (a reference only has to keep the exponent range, not the precision), one (reference, sum)
//    per column into the caller's scratch;
//  * head_weights_kernel: merges a column's chunks, forms the products again and writes each row's
//    shared weights.
// What bounds it: VALU issue (about 5 slots per product for the exponential, its argument and the
// sum, against 0.25 MFMA instructions), then the second pass's stores.  Measured: the target of 256 rows
// of 8 groups, G = 4, against 65 535 fine windows 0.15 + 0.23 ms, 2.28 ms as one launch of 128
// workgroups whose lanes held keys along the accumulator (a shuffle per head and product, the exp2
// library call, 4-byte stores to 64 rows); the multi-head selector's 2048 rows against 4095 windows
// 96 + 117 us, 444 us.
#pragma once
#include "device_util.hpp"
#include "launch.hpp"

namespace sparda {

constexpr int kHtThreads = 256;
constexpr int kHtKeys = 128;                          // keys per LDS slot
constexpr int kHtSlot = kHtKeys * kHeadDim * 2;       // bytes

typedef float f32x16 __attribute__((ext_vector_type(16)));

struct HeadTileArgs {
  const uint16_t* q;      // bf16 [n_groups][G][n_q][128]
  const uint16_t* keys;   // bf16 [n_groups][key_cap][128]
  float* part;            // row r's statistics at part + r * part_stride: [chunk][sharing wavefront][head] (reference, sum)
  float* out;             // row r's weights at out + r * out_stride
  int64_t key_cap, part_stride, out_stride, q_pos0;
  int32_t n_groups, n_q;
  WinGrid grid;           // of the keys
  float scale_log2;
  int32_t unit_waves;     // units per workgroup: 1, 2 or 4 (the other wavefronts share their keys)
  int32_t n_wg;           // workgroups per (batch, group) and chunk
  int32_t n_chunks, chunk_keys;  // chunk_keys is a multiple of kHtKeys
  // the selector: rows take part only while they leave candidates out, and store the windows from the
  // first one that overlaps a candidate on (out[0] is that window)
  int32_t n_init, n_local, k_total;
};

namespace head_tiles {

enum Emit { kWindows, kSegments };  // what head_weights_kernel writes

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// Row (within the unit) and head of element e of lane half h in M-tile mt.
template <int G>
__device__ __forceinline__ int row_of(int mt, int e, int h) { return mt * (32 / G) + (e / G) * 2 + h; }
template <int G>
__device__ __forceinline__ int head_of(int e) { return e % G; }

// What every wavefront of a workgroup knows about its unit.
__device__ __forceinline__ int last_key(const HeadTileArgs& a, int row) {  // that row sees (-1: none)
  const int p = (int)a.q_pos0 + row + 1 - a.grid.l;
  return p >= 0 ? p >> __builtin_ctz(a.grid.s) : -1;  // the strides are powers of two
}

struct Unit {
  int grp, chunk, r0, nr;   // group, chunk, first row, rows
  int n_keys;               // keys the unit's last row sees
  int vis0;                 // last key the unit's first row sees
  int k_lo, k_hi;           // the workgroup's chunk, cut at the last key any of its units sees
  int share, n_share;       // this wavefront's part of the unit's 32-key tiles
  bool live;                // the unit exists
};

template <int G>
__device__ __forceinline__ Unit unit_of(const HeadTileArgs& a) {
  constexpr int U = 64 / G;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  Unit u;
  u.grp = blockIdx.x % a.n_groups;
  const int x = blockIdx.x / a.n_groups;
  u.chunk = x % a.n_chunks;
  const int wg = a.n_wg - 1 - x / a.n_chunks;  // latest rows (most keys) first
  const int n_units = (a.n_q + U - 1) / U;
  const int unit = wg * a.unit_waves + wave % a.unit_waves;
  u.n_share = 4 / a.unit_waves;
  u.share = wave / a.unit_waves;
  u.live = unit < n_units;
  u.r0 = min(unit, n_units - 1) * U;
  u.nr = min(U, a.n_q - u.r0);
  u.n_keys = last_key(a, u.r0 + u.nr - 1) + 1;
  u.vis0 = last_key(a, u.r0);
  const int last_row = min((wg * a.unit_waves + a.unit_waves) * U, a.n_q) - 1;
  u.k_lo = u.chunk * a.chunk_keys;
  u.k_hi = min(u.k_lo + a.chunk_keys, last_key(a, last_row) + 1);
  return u;
}

// The A operand: lane l supplies pair m = l % 32 (element e, half h of the accumulator layout).
template <int G>
__device__ __forceinline__ void load_rows(const HeadTileArgs& a, const Unit& u, bf16x8 (&fa)[2][8]) {
  const int lane = threadIdx.x & 63, m = lane & 31, half = lane >> 5;
  const int eh = (m >> 2) & 1, e = ((m >> 3) << 2) | (m & 3);
#pragma unroll
  for (int mt = 0; mt < 2; ++mt) {
    const int row = min(row_of<G>(mt, e, eh), u.nr - 1);
    const uint16_t* src = a.q + (((int64_t)u.grp * G + head_of<G>(e)) * a.n_q + u.r0 + row) * kHeadDim + 32 * half;
#pragma unroll
    for (int s = 0; s < 8; ++s) fa[mt][s] = as_bf16x8(ld16(src + 64 * (s >> 2) + 8 * (s & 3)));
  }
}

// Stages 128 keys from key k0 on (rows past the last key repeat it): wavefront w brings rows 32 w ..
// 32 w + 31, 4 rows per instruction.  Physical 16-byte piece x of row r holds logical piece
// x ^ (r % 16) ^ (r / 16 % 2): the B operand's reads (32 rows of one piece per lane half) then touch
// every bank once.
__device__ __forceinline__ void stage_keys(const uint16_t* keys, int k0, int n_keys, uint32_t slot) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int r4 = lane >> 4, piece = (lane & 15) ^ (lane >> 4);
  __asm__ __volatile__("" : "+v"(r4), "+v"(piece));  // the eight offsets here: held across the loop they would spill
#pragma unroll
  for (int i = 0; i < 8; ++i) {  // row 4 i + r4 of the wavefront's 32
    const int key = min(k0 + 32 * wave + 4 * i + r4, n_keys - 1);
    lds_load16(keys, (uint32_t)key * (kHeadDim * 2) + 16 * (piece ^ (4 * (i & 3)) ^ (i >> 2)), slot + (32 * wave + 4 * i) * 256);
  }
}

__device__ __forceinline__ void products(const bf16x8 (&fa)[2][8], const bf16x8 (&b)[8], f32x16 (&c)[2]) {
#pragma unroll
  for (int e = 0; e < 16; ++e) c[0][e] = c[1][e] = 0.f;
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    c[0] = mfma32(fa[0][s], b[s], c[0]);
    c[1] = mfma32(fa[1][s], b[s], c[1]);
  }
}

// The products of one 32-key tile (rows 32 t .. of a slot) with both M-tiles.
__device__ __forceinline__ void tile_products(const char* slot, int t, const bf16x8 (&fa)[2][8], f32x16 (&c)[2]) {
  const int lane = threadIdx.x & 63, n = lane & 31, h = lane >> 5;
  const char* row = slot + (32 * t + n) * 256;
  const int sw = (n & 15) ^ (n >> 4);
  bf16x8 b[8];
#pragma unroll
  for (int s = 0; s < 8; ++s)
    b[s] = as_bf16x8(*reinterpret_cast<const uint4*>(row + 16 * ((8 * (s >> 2) + 4 * h + (s & 3)) ^ sw)));
  products(fa, b, c);
}
// Products of keys that a row does not see become -inf (only the last tiles of a unit hold any).
template <int G>
__device__ __forceinline__ void mask_tile(const HeadTileArgs& a, const Unit& u, int key0, f32x16 (&c)[2]) {
  if (key0 + 31 <= u.vis0) return;
  const int key = key0 + (threadIdx.x & 31), h = (threadIdx.x >> 5) & 1;
  int r0 = u.r0;
  __asm__ __volatile__("" : "+s"(r0));  // every row's last key here: held across the loop they would spill
#pragma unroll
  for (int r = 0; r < 16 / G; ++r)
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
      const int row = min(row_of<G>(mt, r * G, h), u.nr - 1);
      const bool seen = key <= last_key(a, r0 + row);
#pragma unroll
      for (int i = 0; i < G; ++i) c[mt][r * G + i] = seen ? c[mt][r * G + i] : -INFINITY;
    }
}

// Walks the chunk: slots of 128 keys, one ahead, and the wavefront's tiles of each; f(key of lane n =
// 0, c) per tile, products of keys that a row does not see set to -inf.  Every wavefront of the workgroup calls it.
template <int G, class F>
__device__ __forceinline__ void walk(const HeadTileArgs& a, const Unit& u, const bf16x8 (&fa)[2][8], char* slots, F f) {
  const uint16_t* keys = a.keys + (int64_t)u.grp * a.key_cap * kHeadDim;
  const int n_stage = (u.k_hi - u.k_lo + kHtKeys - 1) / kHtKeys;
  const uint32_t slots_at = __builtin_amdgcn_readfirstlane(lds_address(slots));
  if (n_stage > 0) stage_keys(keys, u.k_lo, u.k_hi, slots_at);
  for (int st = 0; st < n_stage; ++st) {
    lds_loads_landed();  // this wavefront's part of the slot is here and its reads of the other returned
    __syncthreads();
    const char* now = slots + (st & 1) * kHtSlot;
    if (st + 1 < n_stage) stage_keys(keys, u.k_lo + (st + 1) * kHtKeys, u.k_hi, slots_at + ((st + 1) & 1) * kHtSlot);
    const int k0 = u.k_lo + st * kHtKeys;
    if (u.live) {
      for (int t = u.share; t < 4 && k0 + 32 * t < u.n_keys; t += u.n_share) {
        f32x16 c[2];
        tile_products(now, t, fa, c);
        const int key0 = k0 + 32 * t;
        mask_tile<G>(a, u, key0, c);
        f(key0, c);
      }
    }
  }
}

__device__ __forceinline__ float half_max(float x) {  // over the 32 lanes of a half
  x = fmaxf(x, dpp_f<0x128>(x));
  x = fmaxf(x, dpp_f<0x124>(x));
  x = fmaxf(x, dpp_f<0x122>(x));
  x = fmaxf(x, dpp_f<0x121>(x));
  return fmaxf(x, __shfl_xor(x, 16, kWave));
}
__device__ __forceinline__ float half_sum(float x) {
  x = row16_sum(x);
  return x + __shfl_xor(x, 16, kWave);
}

// True when the unit writes nothing: a selector unit whose rows all take every candidate.
__device__ __forceinline__ bool idle_unit(const HeadTileArgs& a, const Unit& u) {
  if (a.k_total <= 0) return false;
  const RowGeom g = row_geom(a.q_pos0 + u.r0 + u.nr - 1, a.n_init, a.n_local, a.k_total);
  return g.n_take >= g.n_cand;
}

}  // namespace head_tiles

template <int G>
__global__ __launch_bounds__(kHtThreads, 2) void head_stats_kernel(HeadTileArgs a) {
  using namespace head_tiles;
  __shared__ __align__(16) char slots[2 * kHtSlot];
  const int lane = threadIdx.x & 63, n = lane & 31, h = lane >> 5;
  Unit u = unit_of<G>(a);
  if (idle_unit(a, u)) u.live = false;
  bf16x8 fa[2][8];
  load_rows<G>(a, u, fa);
  float m[2][16], s[2][16];  // reference and sum of (row, head) pair (e, h) over this lane's keys
  {  // the reference: the maximum over the wavefront's first tile (uniform over the lanes of a half)
    const int key0 = u.k_lo + 32 * u.share;
    const uint16_t* src = a.keys + ((int64_t)u.grp * a.key_cap + max(min(key0 + n, u.n_keys - 1), 0)) * kHeadDim + 32 * h;
    bf16x8 b[8];
#pragma unroll
    for (int s8 = 0; s8 < 8; ++s8) b[s8] = as_bf16x8(ld16(src + 64 * (s8 >> 2) + 8 * (s8 & 3)));
    f32x16 c[2];
    products(fa, b, c);
    mask_tile<G>(a, u, key0, c);
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const float z = half_max(c[mt][e] * a.scale_log2);
        m[mt][e] = z > -INFINITY ? z : 0.f;
      }
  }
  // The sums against a fixed reference: exact up to the exponent range, so a chunk whose scores rise
  // more than 2^60 above it (no branch in the loop: checked at the end) is walked again for its true
  // maxima and once more for the sums.
  constexpr float kRange = 60.f;
  for (int again = 0;; ++again) {
    float top = -INFINITY;
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int e = 0; e < 16; ++e) s[mt][e] = 0.f;
    walk<G>(a, u, fa, slots, [&](int, f32x16 (&c)[2]) {
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const float z = fmaf(c[mt][e], a.scale_log2, -m[mt][e]);
          top = fmaxf(top, z);
          s[mt][e] += __builtin_amdgcn_exp2f(z);
        }
    });
    if (__syncthreads_or(top > kRange) == 0 || again) break;
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int e = 0; e < 16; ++e) s[mt][e] = -INFINITY;
    walk<G>(a, u, fa, slots, [&](int, f32x16 (&c)[2]) {
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int e = 0; e < 16; ++e) s[mt][e] = fmaxf(s[mt][e], c[mt][e] * a.scale_log2);
    });
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const float z = half_max(s[mt][e]);
        m[mt][e] = z > -INFINITY ? z : 0.f;
      }
    __syncthreads();  // the slots are free again
  }
  if (!u.live) return;
  // lane n < 16 of a half stores pair (e = n) of M-tile 0, lane n >= 16 pair (e = n - 16) of M-tile 1
  float mv = 0.f, sv = 0.f;
#pragma unroll
  for (int mt = 0; mt < 2; ++mt)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const float sum = half_sum(s[mt][e]);
      if (n == 16 * mt + e) {
        mv = m[mt][e];
        sv = sum;
      }
    }
  const int e = n & 15, row = row_of<G>(n >> 4, e, h);
  if (row < u.nr) {
    float* d = a.part + ((int64_t)u.grp * a.n_q + u.r0 + row) * a.part_stride +
               2 * ((u.chunk * u.n_share + u.share) * G + head_of<G>(e));
    d[0] = mv;
    d[1] = sv;
  }
}

// kSegments: per 16 keys the largest weight of the first 15 and of all 16, at out[2 segment] and + 1
// (16 + 15 consecutive keys are what a prediction position of the (32, 16) grid pools).
template <int G, int kEmit>
__global__ __launch_bounds__(kHtThreads, 2) void head_weights_kernel(HeadTileArgs a) {
  using namespace head_tiles;
  constexpr int R = 16 / G;  // rows per lane and M-tile
  __shared__ __align__(16) char slots[2 * kHtSlot];
  __shared__ float ref[4][64], inv_sum[4][64];
  const int lane = threadIdx.x & 63, n = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  Unit u = unit_of<G>(a);
  if (idle_unit(a, u)) u.live = false;
  // lane c merges column c (row c / G, head c % G) over the parts
  {
    const int row = min(lane / G, u.nr - 1), parts = a.n_chunks * u.n_share;
    const float* src = a.part + ((int64_t)u.grp * a.n_q + u.r0 + row) * a.part_stride + 2 * (lane % G);
    float M = 0.f, S = 0.f;
    for (int p = 0; u.live && p < parts; ++p) {
      const float m2 = src[2 * G * p], s2 = src[2 * G * p + 1];
      if (!(s2 > 0.f)) continue;
      const float mn = S > 0.f ? fmaxf(M, m2) : m2;
      S = S * __builtin_amdgcn_exp2f(M - mn) + s2 * __builtin_amdgcn_exp2f(m2 - mn);
      M = mn;
    }
    ref[wave][lane] = M;
    inv_sum[wave][lane] = S > 0.f ? 1.0f / S : 0.f;
  }
  bf16x8 fa[2][8];
  load_rows<G>(a, u, fa);
  wave_lds_sync();
  float m[2][16], inv[2][16];
#pragma unroll
  for (int mt = 0; mt < 2; ++mt)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int c = row_of<G>(mt, e, h) * G + head_of<G>(e);
      m[mt][e] = ref[wave][c];
      inv[mt][e] = inv_sum[wave][c];
    }
  int first_key = 0, last_key = 0x7fffffff;
  if (kEmit == kWindows) {  // the windows the last row selects from; an earlier row's extra ones are weight 0
    const int64_t p = a.q_pos0 + u.r0 + u.nr - 1;
    const RowGeom g = row_geom(p, a.n_init, a.n_local, a.k_total);
    row_windows(g, a.grid, p, &first_key, &last_key);
  }
  float* const out = a.out + ((int64_t)u.grp * a.n_q + u.r0) * a.out_stride;
  walk<G>(a, u, fa, slots, [&](int key0, f32x16 (&c)[2]) {
    const int key = key0 + n;
    int64_t stride = a.out_stride;
    __asm__ __volatile__("" : "+s"(stride));  // row addresses here: held across the loop they would spill
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int r = 0; r < R; ++r) {
        float w = 0.f;
#pragma unroll
        for (int i = 0; i < G; ++i) {
          const int e = r * G + i;
          w = fmaf(__builtin_amdgcn_exp2f(fmaf(c[mt][e], a.scale_log2, -m[mt][e])), inv[mt][e], w);
        }
        const int row = row_of<G>(mt, r * G, h);
        float* d = out + (mt * (32 / G) + 2 * r) * stride + (int64_t)h * stride;
        if (kEmit == kWindows) {
          if (row < u.nr && key >= first_key && key <= last_key) d[key - first_key] = w;
        } else {  // prefix maxima along the 16 lanes of a segment: lane 14 the first 15 keys, lane 15 all
          w = fmaxf(w, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(w), 0x111, 0xf, 0xf, true)));
          w = fmaxf(w, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(w), 0x112, 0xf, 0xf, true)));
          w = fmaxf(w, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(w), 0x114, 0xf, 0xf, true)));
          w = fmaxf(w, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(w), 0x118, 0xf, 0xf, true)));
          if (row < u.nr && (n & 15) >= 14) d[2 * (key >> 4) + (n & 15) - 14] = w;
        }
      }
  });
}

// Sizes the launch: as many chunks of keys as fill the chip with about four workgroups per CU, at most
// `max_parts` partials per column (what the caller's scratch holds).
inline void plan_head_tiles(HeadTileArgs& a, int G, int64_t max_parts) {
  const int U = 64 / G, n_units = (a.n_q + U - 1) / U;
  a.unit_waves = n_units >= 4 ? 4 : n_units >= 2 ? 2 : 1;
  while (a.unit_waves < 4 && 4 / a.unit_waves > max_parts) a.unit_waves *= 2;
  a.n_wg = (n_units + a.unit_waves - 1) / a.unit_waves;
  const int n_keys = grid_win_vis(a.grid, a.q_pos0 + a.n_q - 1) + 1;
  const int stages = n_keys > 0 ? (n_keys + kHtKeys - 1) / kHtKeys : 1;
  int64_t chunks = (1024 + (int64_t)a.n_groups * a.n_wg - 1) / ((int64_t)a.n_groups * a.n_wg);
  const int64_t fit = max_parts / (4 / a.unit_waves);
  if (chunks > fit) chunks = fit;
  if (chunks > (stages + 3) / 4) chunks = (stages + 3) / 4;  // at least 512 keys each
  if (chunks < 1) chunks = 1;
  const int per = (int)((stages + chunks - 1) / chunks);
  a.chunk_keys = per * kHtKeys;
  a.n_chunks = (stages + per - 1) / per;
}

template <int G, int kEmit>
hipError_t launch_head_tiles_g(const HeadTileArgs& a, hipStream_t stream) {
  const dim3 grid((unsigned)((int64_t)a.n_groups * a.n_wg * a.n_chunks)), block(kHtThreads);
  hipLaunchKernelGGL(head_stats_kernel<G>, grid, block, 0, stream, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((head_weights_kernel<G, kEmit>), grid, block, 0, stream, a);
  return hipGetLastError();
}

template <int kEmit>
hipError_t launch_head_tiles(const HeadTileArgs& a, int G, hipStream_t stream) {
  switch (G) {
    case 1: return launch_head_tiles_g<1, kEmit>(a, stream);
    case 2: return launch_head_tiles_g<2, kEmit>(a, stream);
    case 4: return launch_head_tiles_g<4, kEmit>(a, stream);
    case 8: return launch_head_tiles_g<8, kEmit>(a, stream);
    case 16: return launch_head_tiles_g<16, kEmit>(a, stream);
    default: return hipErrorInvalidValue;
  }
}

// ---- few keys: one launch ---------------------------------------------------------------------
//
// A workgroup takes one unit and forms its products once: up to kHuKeys keys, 32 per tile, dealt to eight
// wavefronts, which hold them (T tiles each) until the columns' maxima and sums have been exchanged
// through LDS.  The keys are the A operand and the columns the B operand, so that a lane's accumulators
// are keys of one column (element e of lane (n, h): key 8 (e / 4) + 4 h + e % 4 of the tile, column 32 nt +
// n) and the statistics need no exchange between lanes but the two halves; the sum over a row's heads is
// one DPP step per doubling.  Every unit that selects, and every training row, sees a key.
//
// What bounds it: latency (the rows, a wavefront's keys, two barriers, the stores), and from about one
// workgroup per CU on the reads of the keys, which no two units share.  The two launches above
// have both (and one launch whose four wavefronts formed every product twice was between them); us of
// this kernel, the two launches, that one launch: 16 rows of one group, 4 heads, 124 keys 10, 14, 12; 64
// rows of 2 groups against 249 keys 11.5, 24, 17 and against 499 15.4, 36, 26; 1000 rows of 8 groups,
// one head, 499 keys 21, 55, 35.  The target's segments take it too: the whole training call on 300 tokens,
// 100 rows of 2 groups, 4 heads 20.6, 43.3, 29.9.
constexpr int kHuThreads = 512;
constexpr int kHuWaves = kHuThreads / kWave;
constexpr int kHuTileKeys = 32;
constexpr int kHuMaxTiles = 4;  // per wavefront
constexpr int kHuKeys = kHuTileKeys * kHuWaves * kHuMaxTiles;

template <int G, int T, int kEmit>
__global__ __launch_bounds__(kHuThreads) void head_unit_kernel(HeadTileArgs a) {
  using namespace head_tiles;
  constexpr int U = 64 / G;
  __shared__ float red_m[kHuWaves][64], red_s[kHuWaves][64];
  const int lane = threadIdx.x & 63, n = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = blockIdx.x % a.n_groups;
  const int unit = (int)(gridDim.x / a.n_groups) - 1 - (int)(blockIdx.x / a.n_groups);  // latest rows first
  const int r0 = unit * U, nr = min(U, a.n_q - r0);
  int32_t lo = 0;  // kWindows: the first window that the rows select from
  if (kEmit == kWindows) {
    const int64_t p_last = a.q_pos0 + r0 + nr - 1;
    const RowGeom gl = row_geom(p_last, a.n_init, a.n_local, a.k_total);
    if (gl.n_take >= gl.n_cand) return;  // then every row of the unit takes all its candidates
    int32_t last;
    row_windows(gl, a.grid, p_last, &lo, &last);
  }
  const int n_keys = last_key(a, r0 + nr - 1) + 1, vis0 = last_key(a, r0);

  bf16x8 fb[2][8];
  int vis[2];  // last key that the column's row sees
#pragma unroll
  for (int nt = 0; nt < 2; ++nt) {
    const int c = 32 * nt + n, row = min(c / G, nr - 1);
    const uint16_t* src = a.q + (((int64_t)grp * G + c % G) * a.n_q + r0 + row) * kHeadDim + 32 * h;
#pragma unroll
    for (int s = 0; s < 8; ++s) fb[nt][s] = as_bf16x8(ld16(src + 64 * (s >> 2) + 8 * (s & 3)));
    vis[nt] = last_key(a, r0 + row);
  }
  const uint16_t* keys = a.keys + (int64_t)grp * a.key_cap * kHeadDim + 32 * h;
  f32x16 z[T][2];  // products, then 2^(scaled product - maximum)
  float m[2] = {-INFINITY, -INFINITY};
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int k0 = kHuTileKeys * (wave + kHuWaves * t);
#pragma unroll
    for (int e = 0; e < 16; ++e) z[t][0][e] = z[t][1][e] = 0.f;
    const uint16_t* src = keys + (int64_t)min(k0 + n, n_keys - 1) * kHeadDim;
    bf16x8 fa[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) fa[s] = as_bf16x8(ld16(src + 64 * (s >> 2) + 8 * (s & 3)));
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      z[t][0] = mfma32(fa[s], fb[0][s], z[t][0]);
      z[t][1] = mfma32(fa[s], fb[1][s], z[t][1]);
    }
    if (k0 + kHuTileKeys - 1 > vis0) {  // keys that some row does not see
#pragma unroll
      for (int nt = 0; nt < 2; ++nt)
#pragma unroll
        for (int e = 0; e < 16; ++e)
          if (k0 + 8 * (e >> 2) + 4 * h + (e & 3) > vis[nt]) z[t][nt][e] = -INFINITY;
    }
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
      for (int e = 0; e < 16; ++e) m[nt] = fmaxf(m[nt], z[t][nt][e]);
  }
#pragma unroll
  for (int nt = 0; nt < 2; ++nt) {
    m[nt] = fmaxf(m[nt], __shfl_xor(m[nt], 32, kWave));
    if (h == 0) red_m[wave][32 * nt + n] = m[nt];
  }
  __syncthreads();
  float s[2] = {0.f, 0.f};
#pragma unroll
  for (int nt = 0; nt < 2; ++nt) {
#pragma unroll
    for (int w = 0; w < kHuWaves; ++w) m[nt] = fmaxf(m[nt], red_m[w][32 * nt + n]);
    const float ref = m[nt] > -INFINITY ? m[nt] * a.scale_log2 : 0.f;  // a row without a key: weights 0
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        z[t][nt][e] = __builtin_amdgcn_exp2f(fmaf(z[t][nt][e], a.scale_log2, -ref));
        s[nt] += z[t][nt][e];
      }
    s[nt] += __shfl_xor(s[nt], 32, kWave);
    if (h == 0) red_s[wave][32 * nt + n] = s[nt];
  }
  __syncthreads();
#pragma unroll
  for (int nt = 0; nt < 2; ++nt) {
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < kHuWaves; ++w) sum += red_s[w][32 * nt + n];
    const float inv = sum > 0.f ? 1.0f / sum : 0.f;
    // each row's weights go to its first column's lane, which stores those that the row needs
    const int row = 32 / G * nt + n / G;
    int hi = -1;
    if (n % G == 0 && row < nr) {
      hi = n_keys - 1;
      if (kEmit == kWindows) {
        const int64_t p = a.q_pos0 + r0 + row;
        const RowGeom g = row_geom(p, a.n_init, a.n_local, a.k_total);
        int32_t first, wl;
        row_windows(g, a.grid, p, &first, &wl);
        hi = g.n_take < g.n_cand ? wl : -1;
      }
    }
    float* out = a.out + ((int64_t)grp * a.n_q + r0 + min(row, nr - 1)) * a.out_stride - lo;
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int k0 = kHuTileKeys * (wave + kHuWaves * t);
#pragma unroll
      for (int e0 = 0; e0 < 16; e0 += 8) {
        float w[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          w[i] = z[t][nt][e0 + i] * inv;
          if (G >= 2) w[i] += dpp_f<0xB1>(w[i]);    // lane ^ 1
          if (G >= 4) w[i] += dpp_f<0x4E>(w[i]);    // lane ^ 2
          if (G >= 8) w[i] += dpp_f<0x141>(w[i]);   // the other four of eight
          if (G >= 16) w[i] += dpp_f<0x140>(w[i]);  // the other eight of sixteen
        }
        if (kEmit == kWindows) {
#pragma unroll
          for (int q = 0; q < 8; q += 4) {
            const int key = k0 + 2 * (e0 + q) + 4 * h;
            if (key >= lo && key + 3 <= hi) {
              __builtin_memcpy(out + key, w + q, 4 * sizeof(float));  // one store, aligned to a float
            } else {
#pragma unroll
              for (int i = 0; i < 4; ++i)
                if (key + i >= lo && key + i <= hi) out[key + i] = w[q + i];
            }
          }
        } else {  // the segment's keys 0-3 and 8-11 lie in lane half 0, 4-7 and 12-15 in half 1
          float m15 = fmaxf(fmaxf(fmaxf(w[0], w[1]), fmaxf(w[2], w[3])), fmaxf(fmaxf(w[4], w[5]), w[6]));
          float m16 = fmaxf(m15, w[7]);
          if (h == 0) m15 = m16;
          m15 = fmaxf(m15, __shfl_xor(m15, 32, kWave));
          m16 = fmaxf(m16, __shfl_xor(m16, 32, kWave));
          const int key = k0 + 2 * e0;
          if (h == 0 && key <= hi) *reinterpret_cast<float2*>(out + 2 * (key >> 4)) = make_float2(m15, m16);
        }
      }
    }
  }
}

template <int G, int kEmit>
hipError_t launch_head_units_g(const HeadTileArgs& a, int n_keys, hipStream_t stream) {
  const dim3 grid((unsigned)((int64_t)a.n_groups * ((a.n_q + 64 / G - 1) / (64 / G)))), block(kHuThreads);
  constexpr int kRound = kHuTileKeys * kHuWaves;
  if (n_keys <= kRound)
    hipLaunchKernelGGL((head_unit_kernel<G, 1, kEmit>), grid, block, 0, stream, a);
  else if (n_keys <= 2 * kRound)
    hipLaunchKernelGGL((head_unit_kernel<G, 2, kEmit>), grid, block, 0, stream, a);
  else
    hipLaunchKernelGGL((head_unit_kernel<G, kHuMaxTiles, kEmit>), grid, block, 0, stream, a);
  return hipGetLastError();
}

// Where one launch of units is the faster: while the units that have to select fill the chip at most once
// (a wavefront's four tiles: one workgroup per CU) or twice (two tiles).  Measured, one launch against two
// (us), for 128, 504, 940 and 2000 such units: 499 keys 21 / 55, 33 / 43, -, 119 / 57; 124 to 249 keys
// 13 / 34, 21 / 28, 37 / 27, 54 / 38; 1017 keys 32 / 57, 51 / 45, -, 199 / 105.
inline bool head_units_fit(const HeadTileArgs& a, int G, int n_keys) {
  const int U = 64 / G;
  const int64_t first = (int64_t)a.k_total * kBlock - a.q_pos0;  // rows before it take every candidate
  const int64_t units = (a.n_q + U - 1) / U - (first > 0 ? first / U : 0);
  return n_keys <= kHuKeys && units * a.n_groups <= (n_keys <= kHuKeys / 2 ? 512 : 256);
}

template <int kEmit>
hipError_t launch_head_units(const HeadTileArgs& a, int G, int n_keys, hipStream_t stream) {
  switch (G) {
    case 1: return launch_head_units_g<1, kEmit>(a, n_keys, stream);
    case 2: return launch_head_units_g<2, kEmit>(a, n_keys, stream);
    case 4: return launch_head_units_g<4, kEmit>(a, n_keys, stream);
    case 8: return launch_head_units_g<8, kEmit>(a, n_keys, stream);
    default: return launch_head_units_g<16, kEmit>(a, n_keys, stream);
  }
}

}  // namespace sparda
