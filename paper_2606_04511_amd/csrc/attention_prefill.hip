// attention_prefill.hip -- block-sparse attention for many query rows of one chunk (chunked
// prefill): paper Sec. 4.1, Eq. 5, over the per-row attended sets of Eq. 1 (Alg. 1 selects per
// query token, so neighbouring rows attend different blocks).
//
// Work unit: a tile of 128/G consecutive query rows of one (batch, group), i.e. 128 query-head
// rows, on one 256-thread workgroup; two workgroups share a CU, so a block's barrier waits for 4
// wavefronts while the other workgroup's wavefronts keep the SIMDs busy.  Wavefront w owns
// query-head rows [32 w, 32 w + 32): two MFMA N-tiles of 16 query-heads (16/G rows each), whose
// online-softmax state and output accumulators stay in registers for the whole tile.
//   1. Each row's attended blocks become a bitmap in LDS (entries outside [0, blk(p)] are
//      dropped; a block listed twice sets one bit, so it is attended once).  Their union, in
//      ascending order, is the tile's block list.  The bitmaps and the list are dynamic LDS
//      sized by the call's last row.
//   2. The tile walks its block list.  Block j's 16 KiB of K and 16 KiB of V go from HBM straight into
//      one of two LDS slots (global_load_lds, once per tile), one block ahead of the math; one
//      barrier per block.  The rows' 16-byte pieces are XOR-swizzled so that every operand read is
//      conflict-free.  V stays as it lies in memory: P V reads it through the transposing LDS read.
//   3. A wavefront skips block j for an N-tile none of whose rows lists j.  Otherwise:
//        S^T = K Q^T on v_mfma_f32_16x16x32_bf16 (M = 16 tokens, N = 16 query-heads, K = 32
//        dims); query-heads whose row does not list j, and tokens after the row's position, are
//        masked; online softmax in the exp2 domain;
//        O^T += V^T P^T on the same MFMA (M = 16 head dims, N = 16 query-heads, K = 32 tokens); the
//        denominators sum P in float32, before it is rounded for the product.
//      P needs no data movement between the two products: k slot 4 x + i of lane group q is token
//      16 (2 s + x) + 4 q + i, the order in which an S^T accumulator lane holds its scores.
//
// What bounds it: issue.  Per visited N-tile a wavefront issues 32 MFMAs (512 cycles) and about 115
// VALU instructions, which overlap only in part (a probe: two VALU instructions hide under one
// 16-cycle MFMA, the third costs 8 cycles), and a block ends with its busiest wavefront (1.28 to
// 1.5 times the mean).  Reading every block from a 256 KiB footprint instead changes 4 %, so memory is
// not the limit.  A 32K prefill of 32 / 8 heads, k = 64, neighbouring rows sharing 0.8 of their
// Forecast variance: 3.87 ms, 529 TFLOP/s of attended pairs (5.91 ms with K and V staged through
// registers, V transposed on the way, and a branch around every product; 1.5 % less with the denominators
// summed by two MFMAs of the rounded P against ones, which holds fewer bits of them); the last 8192 rows
// of 32 / 2 heads, k = 96: 1.24 ms (1.97).  Tried and slower: eight wavefronts with a ring of four blocks
// and one barrier per block (4.70 ms); one wavefront bringing the blocks for 7, 11 or 15 others without
// barriers (4.0 ms; the ring is too short to even out the wavefronts; 1.12 ms at 16 heads per group);
// one N-tile per wavefront on 16 wavefronts (4.33 ms).
//
// Tiles with the most blocks run first; consecutive workgroups (spread over the XCDs by the
// dispatcher) take different groups, so each XCD's L2 serves one group's K and V.
#include <math.h>

#include "device_util.hpp"
#include "launch.hpp"

namespace sparda {

// The prefill attention's dynamic LDS (row bitmaps, union bitmap, union list).
extern __shared__ __align__(16) uint32_t pa_dyn[];

namespace {

constexpr int kPaWaves = 4;                // two workgroups share a CU
constexpr int kPaThreads = 64 * kPaWaves;
constexpr int kNt = 2;                     // N-tiles of 16 query-heads per wavefront
constexpr int kPaQh = 16 * kNt * kPaWaves; // query-head rows per tile
constexpr int kPaMaxBlocks = 4096;         // causal blocks a tile may span
constexpr int kPaSlot = 2 * kBlock * kHeadDim * 2;  // bytes of one slot: a block's K, then its V
constexpr int kPaStaticLds = 2 * kPaSlot + 16;      // the two slots, n_union
constexpr int kPaLdsMax = 160 * 1024;      // LDS of one CU
constexpr float kLog2eP = 1.4426950408889634f;

// Row bitmaps, union bitmap and union list live in dynamic LDS sized by the call (its last row's
// causal blocks): wc words per row bitmap.
__host__ __device__ inline int pa_dyn_lds_bytes(int rows, int nbt) {
  const int wc = (nbt + 31) >> 5;
  return ((4 * (rows * wc + wc) + 2 * nbt) + 15) & ~15;
}

template <int G>
__global__ __launch_bounds__(kPaThreads, 2) void prefill_attn_kernel(AttnArgs a, int n_tiles, int n_groups, int wc) {
  constexpr int TR = kPaQh / G;  // rows per tile
  constexpr int RN = 16 / G;     // rows per N-tile of 16 query-heads; two N-tiles per wavefront
  static_assert(16 % G == 0, "an N-tile holds whole rows");
  __shared__ __align__(16) uint16_t ring[2 * kPaSlot / 2];
  __shared__ int n_union;
  uint32_t* rbm = pa_dyn;                                   // [TR][wc] (a tile uses [TR][W])
  uint32_t* ubm = pa_dyn + TR * wc;                         // [wc]
  int16_t* ulist = reinterpret_cast<int16_t*>(ubm + wc);    // [wc * 32] >= nbt

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t bm = blockIdx.x % n_groups;
  const int tile = n_tiles - 1 - (int)(blockIdx.x / n_groups);
  const int r0 = tile * TR;
  const int nrows = min(TR, a.n_q - r0);
  const int64_t p0 = a.q_pos0 + r0;
  const int nbt = (int)((p0 + nrows - 1) / kBlock) + 1;  // causal blocks of the tile's last row
  const int W = (nbt + 31) >> 5;                         // bitmap words per row

  // ---- 1. per-row bitmaps and their union
  for (int i = tid; i < TR * W; i += kPaThreads) rbm[i] = 0u;  // rows past the chunk list nothing
  for (int i = tid; i < W; i += kPaThreads) ubm[i] = 0u;
  __syncthreads();
  {
    const int kt = a.k_total;
    for (int e = tid; e < nrows * kt; e += kPaThreads) {
      const int rl = e / kt, s = e - rl * kt;
      const int64_t row = bm * a.n_q + r0 + rl;
      const int n = min(max((int)a.cnt[row], 0), kt);
      if (s < n) {
        const int j = a.sel[row * kt + s];
        const int blk = (int)((p0 + rl) / kBlock);
        if (j >= 0 && j <= blk) {
          atomicOr(&rbm[rl * W + (j >> 5)], 1u << (j & 31));
          atomicOr(&ubm[j >> 5], 1u << (j & 31));
        }
      }
    }
  }
  __syncthreads();
  if (wave == 0) {
    int base = 0;
    for (int w0 = 0; w0 < W; w0 += 64) {
      const int w = w0 + lane;
      uint32_t bits = w < W ? ubm[w] : 0u;
      const int c = __popc(bits);
      const int incl = wave_incl_scan(c);
      int pos = base + incl - c;
      while (bits) {
        ulist[pos++] = (int16_t)(w * 32 + __builtin_ctz(bits));
        bits &= bits - 1u;
      }
      base += readlane_i(incl, 63);
    }
    if (lane == 0) n_union = base;
  }

  // ---- per-lane query-head columns: lane (c, q) is column c of both N-tiles, k-chunk q
  const int c = lane & 15, q = lane >> 4;
  const int rl = wave * kNt * RN + c / G;  // N-tile 0's row within the tile; N-tile 1's is RN rows on
  bf16x8 qf[kNt][4];
#pragma unroll
  for (int nt = 0; nt < kNt; ++nt) {
    const uint16_t* qrow = a.q + ((bm * G + c % G) * a.n_q + r0 + rl + nt * RN) * kHeadDim + 8 * q;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
      qf[nt][ks] = as_bf16x8(rl + nt * RN < nrows ? ld16(qrow + 32 * ks) : make_uint4(0u, 0u, 0u, 0u));
  }
  const int pr = (int)(p0 % kBlock) + rl;  // N-tile 0's column position, from the start of the tile's first block
  // z = zscale (q . k): a negative scale is folded into the query's sign bits (exact in bf16), so
  // that the block maximum of z is always zscale times the maximum of q . k.
  float zscale = a.sm_scale * kLog2eP;
  if (zscale < 0.f) {
    zscale = -zscale;
#pragma unroll
    for (int nt = 0; nt < kNt; ++nt)
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        uint4 w = __builtin_bit_cast(uint4, qf[nt][ks]);
        w.x ^= 0x80008000u;
        w.y ^= 0x80008000u;
        w.z ^= 0x80008000u;
        w.w ^= 0x80008000u;
        qf[nt][ks] = as_bf16x8(w);
      }
  }
  // a scale of zero (uniform weights): the smallest positive scale instead, so that masked scores
  // (-inf) keep weight 0
  if (zscale == 0.f) zscale = __FLT_MIN__;
  float m_run[kNt], l_run[kNt];
  f32x4 acc[kNt][8];
#pragma unroll
  for (int nt = 0; nt < kNt; ++nt) {
    m_run[nt] = -INFINITY;
    l_run[nt] = 0.f;
#pragma unroll
    for (int md = 0; md < 8; ++md) acc[nt][md] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // Online softmax with a lazily raised reference: P = 2^(z - m_run) keeps its relative precision in
  // bf16 and fp32 whatever m_run is, so m_run is set by a column's first block and moves only when a
  // block's maximum exceeds it by more than kHeadroom (log2 units), which ordinary logits rarely do
  // again.  The accumulators stay within 2^kHeadroom of their final size, so that values of V up to
  // 2^105 cannot overflow them (2^15 tokens attended); 64 instead of 8 measured the same.  The final normalisation by l,
  // accumulated against the same reference, makes the result exact.
  constexpr float kHeadroom = 8.f;
  const int blk0 = (int)(p0 / kBlock);  // blocks >= blk0 may hold tokens after some row's position
  // The chunk's last position.  Whatever the caches hold after it (NaN, say) must not meet the P = 0 of
  // those tokens in the matrix cores.
  const int chunk_last = (int)(a.q_pos0 + a.n_q - 1);

  // Operand addresses: K row 16 mt + c, piece (4 ks + q) ^ c; V rows 16 mt + 4 q + r (lane's r = c
  // / 4), dims 16 md + 4 (c % 4) .. + 3, piece (2 md + (c / 2) % 2) ^ 2 (row % 8).  Both swizzles
  // leave the address of ks or md one XOR away from that of 0; mt is an immediate offset.
  const int vt = 4 * q + (c >> 2);
  uint32_t ka0 = (uint32_t)(c * kHeadDim + 8 * (q ^ c)) * 2;
  uint32_t va0 = (uint32_t)(vt * kHeadDim + 8 * (((c >> 1) & 1) ^ (2 * (vt & 7))) + 4 * (c & 1)) * 2;

  // ---- staging: K and V rows go from HBM straight into LDS (16 bytes per lane, one 1 KiB
  // instruction per 4 token rows, no registers held); instruction u of wavefront w brings rows 16 u +
  // 4 w .. + 3 of both.  The LDS side of such a load is linear, so the bank swizzle is in which
  // 16-byte piece of its row a lane asks for: physical piece x of token t holds logical piece
  // x ^ (t % 16) of K, x ^ 2 (t % 8) of V.
  const int s_tok = 4 * wave + (lane >> 4);  // token mod 16
  const uint32_t k_off = (uint32_t)(s_tok * kHeadDim + 8 * ((lane & 15) ^ s_tok)) * 2;
  const uint32_t v_off = (uint32_t)(s_tok * kHeadDim + 8 * ((lane & 15) ^ (2 * (s_tok & 7)))) * 2;
  const char* kp = reinterpret_cast<const char*>(a.k + bm * a.t_cap * kHeadDim);
  const char* vp = reinterpret_cast<const char*>(a.v + bm * a.t_cap * kHeadDim);
  const uint32_t ring_at = __builtin_amdgcn_readfirstlane(lds_address(ring)) + wave * 1024;
  auto issue = [&](int j, int slot) {
    const int64_t off = (int64_t)j * (kBlock * kHeadDim * 2);
    const uint32_t d = ring_at + slot * kPaSlot;
#pragma unroll
    for (int u = 0; u < 4; ++u) lds_load16(kp + off + u * 4096, k_off, d + u * 4096);
    const int last_tok = chunk_last - j * kBlock;
    if (last_tok >= kBlock - 1) {
#pragma unroll
      for (int u = 0; u < 4; ++u) lds_load16(vp + off + u * 4096, v_off, d + kBlock * kHeadDim * 2 + u * 4096);
    } else {  // tokens past the chunk's end: its last token's V in their place
      int t = lane >> 4;
      __asm__ __volatile__("" : "+v"(t));  // the offsets here: held across the loop they would spill
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int back = max(16 * u + 4 * wave + t - last_tok, 0);
        lds_load16(vp + off, v_off + (uint32_t)((16 * u - back) * kHeadDim * 2), d + kBlock * kHeadDim * 2 + u * 4096);
      }
    }
  };

  __syncthreads();  // union list and bitmaps complete
  const int nu = n_union;

  // ---- the tile's blocks.  64 entries of the union list at a time: bit i of a row's mask says
  // whether the row lists entry base + i.  The loop over blocks updates the accumulators in one
  // place and the raise sits outside it: with both inside, the compiler moves all accumulators
  // between registers on every block.
  int it = 0, jv = 0;
  uint64_t any[kNt] = {}, mine[kNt] = {};
  auto scan = [&](int base) {
    const int n = min(64, nu - base);
    jv = ulist[base + min(lane, n - 1)];
#pragma unroll
    for (int nt = 0; nt < kNt; ++nt) any[nt] = 0ull;
#pragma unroll
    for (int r = 0; r < kNt * RN; ++r) {
      const uint64_t b = __ballot(lane < n && ((rbm[(wave * kNt * RN + r) * W + (jv >> 5)] >> (jv & 31)) & 1u));
      any[r / RN] |= b;
      if (c / G == r % RN) mine[r / RN] = b;
    }
  };
  if (nu > 0) {
    scan(0);
    issue(readlane_i(jv, 0), 0);
  }
  bool again = false;  // the block at `it` is resident already: taken up again after a raise
  for (;;) {
    bool raise = false;
    float bmax[kNt];
#pragma unroll
    for (int nt = 0; nt < kNt; ++nt) bmax[nt] = -INFINITY;
    for (; it < nu; ++it) {
      const int i = it & 63, j = readlane_i(jv, i);
      bool on[kNt], act[kNt];
#pragma unroll
      for (int nt = 0; nt < kNt; ++nt) {
        on[nt] = ((any[nt] >> i) & 1ull) != 0ull;
        act[nt] = ((mine[nt] >> i) & 1ull) != 0ull;
      }
      if (!again) {
        // this wavefront's rows of block it have landed and its reads of block it - 1 have returned;
        // then block it + 1 is requested into the other slot, which every wavefront has left
        lds_loads_landed();
        __builtin_amdgcn_s_barrier();
        __asm__ __volatile__("" ::: "memory");
        if (it + 1 < nu) {
          const int jn = i == 63 ? __builtin_amdgcn_readfirstlane((int)ulist[it + 1]) : readlane_i(jv, i + 1);
          issue(jn, (it + 1) & 1);
        }
      }
      again = false;
      if (!(on[0] || on[kNt - 1])) {
        if (i == 63 && it + 1 < nu) scan(it + 1);
        continue;
      }
      const char* kb = reinterpret_cast<const char*>(ring) + (it & 1) * kPaSlot;
      const char* vb = kb + kBlock * kHeadDim * 2;
      // the XORs are recomputed per block: held across the loop they would spill
      __asm__ __volatile__("" : "+v"(ka0), "+v"(va0));
      // S^T[token 16 mt + 4 q + i][column c]
      bf16x8 kf[4][4];
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
          kf[mt][ks] = as_bf16x8(*reinterpret_cast<const uint4*>(kb + 16 * mt * kHeadDim * 2 + (ka0 ^ (ks << 6))));
      f32x4 st[kNt][4];
      bool ask = false;
#pragma unroll
      for (int nt = 0; nt < kNt; ++nt) {
        if (!on[nt]) continue;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
          for (int mt = 0; mt < 4; ++mt)
            st[nt][mt] = mfma16x16x32(kf[mt][ks], qf[nt][ks], ks == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : st[nt][mt]);
        if (j >= blk0) {  // a diagonal block: no token after the row's position
          const int lim = min(pr + nt * RN - (j - blk0) * kBlock, kBlock - 1) - 4 * q;
#pragma unroll
          for (int mt = 0; mt < 4; ++mt)
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (16 * mt + i > lim) st[nt][mt][i] = -INFINITY;
        }
        float e = -INFINITY;
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
          e = fmaxf(e, fmaxf(fmaxf(st[nt][mt][0], st[nt][mt][1]), fmaxf(st[nt][mt][2], st[nt][mt][3])));
        bmax[nt] = act[nt] ? e * zscale : -INFINITY;
        ask |= bmax[nt] > m_run[nt] + kHeadroom;  // also on a column's first block
      }
      if (__ballot(ask) != 0ull) {
        raise = true;
        break;
      }
      __builtin_amdgcn_s_setprio(1);
      uint2 vf[4][4];
      auto read_v = [&](int h) {
#pragma unroll
        for (int md = 0; md < 4; ++md)
#pragma unroll
          for (int x = 0; x < 4; ++x) vf[md][x] = lds_read_tr16(vb + 16 * x * kHeadDim * 2 + (va0 ^ ((4 * h + md) << 5)));
      };
      read_v(0);
      bf16x8 pb[kNt][2];
#pragma unroll
      for (int nt = 0; nt < kNt; ++nt) {
        if (!on[nt]) continue;
        // z - m_run as one FMA; an inactive column gets -inf, hence P = 0
        const float off = act[nt] ? -m_run[nt] : -INFINITY;
        float pz[4][4];
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
          for (int i = 0; i < 4; ++i) pz[mt][i] = __builtin_amdgcn_exp2f(fmaf(st[nt][mt][i], zscale, off));
        float psum = 0.f;  // of the lane's tokens, before P is rounded
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
          for (int i = 0; i < 4; ++i) psum += pz[mt][i];
        l_run[nt] += psum;
        // B operand of k-step s2: slot 4 x + i holds token 16 (2 s2 + x) + 4 q + i
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
          uint4 w;
          w.x = pack_bf16(pz[2 * s2][0], pz[2 * s2][1]);
          w.y = pack_bf16(pz[2 * s2][2], pz[2 * s2][3]);
          w.z = pack_bf16(pz[2 * s2 + 1][0], pz[2 * s2 + 1][1]);
          w.w = pack_bf16(pz[2 * s2 + 1][2], pz[2 * s2 + 1][3]);
          pb[nt][s2] = as_bf16x8(w);
        }
      }
      __builtin_amdgcn_s_setprio(0);
      // O^T[dim 16 md + 4 q + i][column c] += V^T P^T
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (h == 1) read_v(1);
#pragma unroll
        for (int nt = 0; nt < kNt; ++nt) {
          if (!on[nt]) continue;
#pragma unroll
          for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
            for (int md = 0; md < 4; ++md)
              acc[nt][4 * h + md] = mfma16x16x32(as_bf16x8(make_uint4(vf[md][2 * s2].x, vf[md][2 * s2].y, vf[md][2 * s2 + 1].x, vf[md][2 * s2 + 1].y)),
                                                 pb[nt][s2], acc[nt][4 * h + md]);
        }
      }
      if (i == 63 && it + 1 < nu) scan(it + 1);
    }
    if (!raise) break;
    again = true;
#pragma unroll
    for (int nt = 0; nt < kNt; ++nt) {
      float m = bmax[nt];
      m = fmaxf(m, __shfl_xor(m, 16, 64));
      m = fmaxf(m, __shfl_xor(m, 32, 64));
      if (!(m > m_run[nt] + kHeadroom)) continue;
      const float alpha = __builtin_amdgcn_exp2f(m_run[nt] - m);
      m_run[nt] = m;
      l_run[nt] *= alpha;
#pragma unroll
      for (int md = 0; md < 8; ++md) acc[nt][md] *= alpha;
    }
  }

  // ---- normalise and store: lane (c, q) holds dims 16 md + 4 q + i of its column
#pragma unroll
  for (int nt = 0; nt < kNt; ++nt) {
    float l = l_run[nt];
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    if (rl + nt * RN >= nrows) continue;
    const float inv = l > 0.f ? 1.f / l : 0.f;
    uint16_t* orow = a.o + ((bm * G + c % G) * a.n_q + r0 + rl + nt * RN) * kHeadDim + 4 * q;
#pragma unroll
    for (int md = 0; md < 8; ++md) {
      const f32x4 v = acc[nt][md];
      uint2 w;
      w.x = (uint32_t)f32_to_bf16(v[0] * inv) | ((uint32_t)f32_to_bf16(v[1] * inv) << 16);
      w.y = (uint32_t)f32_to_bf16(v[2] * inv) | ((uint32_t)f32_to_bf16(v[3] * inv) << 16);
      *reinterpret_cast<uint2*>(orow + 16 * md) = w;
    }
  }
}

template <int G>
hipError_t launch_tiles(const AttnArgs& a, hipStream_t stream) {
  const int tr = kPaQh / G;
  const int n_tiles = (a.n_q + tr - 1) / tr;
  const int n_groups = a.batch * a.n_kv_heads;
  const int nbt = (int)((a.q_pos0 + a.n_q - 1) / kBlock) + 1;  // causal blocks of the call's last row
  hipLaunchKernelGGL(prefill_attn_kernel<G>, dim3((unsigned)((int64_t)n_groups * n_tiles)), dim3(kPaThreads),
                     pa_dyn_lds_bytes(tr, nbt), stream, a, n_tiles, n_groups, (nbt + 31) >> 5);
  return hipGetLastError();
}

}  // namespace

bool attn_uses_tiles(int32_t group_size, int32_t n_q, int64_t q_pos0) {
  if (n_q < 16 || group_size < 1 || group_size > 16 || 16 % group_size != 0) return false;
  const int64_t tr = kPaQh / group_size;
  // the call's last row decides the bitmap width; two workgroups share a CU while the dynamic
  // part stays within 16 KiB (contexts up to about 190K tokens at G = 4), one beyond
  const int64_t nbt = (q_pos0 + n_q - 1) / kBlock + 1;
  return nbt <= kPaMaxBlocks && kPaStaticLds + pa_dyn_lds_bytes((int)tr, (int)nbt) <= kPaLdsMax;
}

hipError_t launch_prefill_attn(const AttnArgs& a, hipStream_t stream) {
  switch (a.group_size) {
    case 1: return launch_tiles<1>(a, stream);
    case 2: return launch_tiles<2>(a, stream);
    case 4: return launch_tiles<4>(a, stream);
    case 8: return launch_tiles<8>(a, stream);
    case 16: return launch_tiles<16>(a, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace sparda
