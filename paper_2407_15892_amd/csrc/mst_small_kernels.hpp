// The GEMMs of the LM-head path (and the MLP's weight gradients) with the smaller block tiles of gemm_small.hpp, for
// problems whose 256 x 256 tiles would occupy a fraction of the chip: small hidden sizes or vocabularies, short
// mini-sequences.  What bounds the launches they replace is the time of a single tile -- the latency of its first loads,
// a few K steps, an epilogue of thousands of instructions per wave -- while most compute units have none.
// Measured per launch under a kernel trace, us, 256 x 256 tiles -> these: 512 rows, d = 256, V = 4096: forward 16.9 -> 8.0;
// 128 of the rows: dlogits 12.8 -> 5.3, dH with its reduce 18.4 -> 10.0, dW of 256 rows 10.3 (14.5 where it adds) -> 5.3.
// 300 rows, d = 512, V = 8000: forward 22.4 -> 12.1, dlogits 18.2 -> 11.4, dH 29.3 -> 15.0, dW 14.7 -> 10.7.  256 rows,
// d = 1024, V = 50257 (197 tiles of 256 in dlogits): 33.6 -> 47 in a loop of launches, so not there.
#pragma once
#include "mst_kernels.hpp"

#include <algorithm>
#include <cmath>

namespace mst {

// forward: 256 x 64 and 256 x 32 tiles, pipelined, one workgroup per compute unit (120 and 144 KB of LDS)
typedef CfgSmall<8, 2, 3, 3, true> TileFwd64;
typedef CfgSmall<8, 1, 4, 4, true> TileFwd32;
// 64 x 64: several workgroups on a compute unit, or pipelined for a lone one
typedef CfgSmall<2, 2, 3, 2, false> Tile64;
typedef CfgSmall<2, 2, 5, 5, true> Tile64Lone;

// Host: estimates in us of a launch with 256 x 256 tiles and with 64 x 64 ones (whichever pipeline `lone` says), fitted to
// the launches above and to 128 to 2000 rows, d = 256 to 4096, V = 4096 to 50257; they only have to rank the two.
inline double tiles_of(int64_t a, int64_t b, int64_t e) { return (double)((a + e - 1) / e) * (double)((b + e - 1) / e); }
inline double big_launch_us(double tiles, double ksteps) { return std::ceil(tiles / 256.0) * (1.25 * ksteps + 7.0); }
inline bool lone_small(double tiles) { return tiles <= 256.0; }
inline double small_launch_us(double tiles, double ksteps) {
  if (lone_small(tiles)) return 0.25 * ksteps + 3.5;
  const double y = tiles / 1024.0;                             // four workgroups on a compute unit
  return y > 1.0 ? y * (ksteps + 3.5) : (0.25 + 0.75 * y) * ksteps + 3.5;
}

// ---------------------------------------------------------------------------
// forward: 256 vocabulary entries x 32 TB rows per workgroup.  The vocabulary side stays 256 wide because the workspace
// holds one (max, sum-exp) pair per row and 256 entries; every pair is formed in the same order as by k_fwd_gemm_lse, so
// lse and loss keep their bits.
// ---------------------------------------------------------------------------
template <class C>
__global__ __launch_bounds__(C::kThreads, kSmallWavesPerSimd) void k_fwd_gemm_lse_small(
    const __bf16* __restrict__ Hc, const __bf16* __restrict__ W, const int* __restrict__ labels_c,
    int rows, int d, int V, int n_st, int n_vt, float2* __restrict__ part, size_t part_stride, float* __restrict__ tgt) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  static_assert(C::EA == kTile && C::TA == kTA16, "one pair per row and 256 vocabulary entries");
  int vt, st;
  if (!even_tile_of_block(blockIdx.x, n_vt, n_st, &vt, &st)) return;
  const int v0 = vt * kTile, s0 = st * C::EB;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wa = wave / C::WB, wb = wave % C::WB;

  f32x4 acc[C::TA][C::TB];
  zero_acc<C::TA, C::TB>(acc);
  {
    PanelKC16<C, C::EA, C::TA, true> pa;
    PanelKC16<C, C::EB, C::TB, false> pb;
    pa.init(W + (size_t)v0 * d, d, V - v0, d, wave, lane, wa);
    pb.init(Hc + (size_t)s0 * d, d, rows - s0, d, wave, lane, wb);
    gemm_mainloop_small<C>(acc, pa, pb, smem, 0, d);
  }
  lse_epilogue<C::TB>(acc, labels_c, rows, V, vt, s0, part, part_stride, tgt, wa, wb, lane, smem);
}

// ---------------------------------------------------------------------------
// backward 1: recomputed logits -> softmax - onehot, as k_bwd_gemm_dlogits (whole vocabulary)
// ---------------------------------------------------------------------------
template <class C>
__global__ __launch_bounds__(C::kThreads, kSmallWavesPerSimd) void k_bwd_gemm_dlogits_small(
    const __bf16* __restrict__ Hc, const __bf16* __restrict__ W, const int* __restrict__ labels_c,
    const float* __restrict__ lse_c, int rows, int d, int V, int ignore_index, int n_st, int n_vt,
    __bf16* __restrict__ G, int ldg) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  int vt, st;
  if (!even_tile_of_block(blockIdx.x, n_vt, n_st, &vt, &st)) return;
  const int v0 = vt * C::EA, s0 = st * C::EB;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wa = wave / C::WB, wb = wave % C::WB;

  f32x4 acc[C::TA][C::TB];
  zero_acc<C::TA, C::TB>(acc);
  {
    PanelKC16<C, C::EA, C::TA, true> pa;
    PanelKC16<C, C::EB, C::TB, false> pb;
    pa.init(W + (size_t)v0 * d, d, V - v0, d, wave, lane, wa);
    pb.init(Hc + (size_t)s0 * d, d, rows - s0, d, wave, lane, wb);
    gemm_mainloop_small<C>(acc, pa, pb, smem, 0, d);
  }

  // a lane holds, for each of its TB rows, the kPer consecutive entries from va on; the bf16 tile leaves through LDS (free
  // now; rows padded by 16 bytes) as whole rows
  constexpr int kPer = 4 * C::TA, kStageRow = C::EA * 2 + 16;
  const int va_tile = wa * (16 * C::TA) + kPer * (lane >> 4), va = v0 + va_tile;
  int y_u[C::TB];                       // all loads before the first is waited for
  float lse_u[C::TB];
#pragma unroll
  for (int u = 0; u < C::TB; ++u) {
    const int s_local = s0 + wb * (16 * C::TB) + 16 * u + (lane & 15), s_in = s_local < rows ? s_local : rows - 1;
    y_u[u] = labels_c[s_in];
    lse_u[u] = lse_c[s_in];
  }
#pragma unroll
  for (int u = 0; u < C::TB; ++u) {
    const int row = wb * (16 * C::TB) + 16 * u + (lane & 15);
    const int s_local = s0 + row;
    if (s_local >= rows) continue;
    const int y_abs = y_u[u];
    const bool valid = (y_abs != ignore_index) && ((unsigned)y_abs < (unsigned)V);
    const float lse_s = valid ? lse_u[u] : __builtin_inff();           // an ignored row: every p is exp2(-infinity)
    const int y_lane = valid ? y_abs - va : -1;
    char* srow = smem + row * kStageRow + va_tile * 2;
#pragma unroll
    for (int p = 0; p < C::TA / 2; ++p) {
      bf16x8 o;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float z = acc[2 * p + (e >> 2)][u][e & 3];
        float x = fast_exp2((z - lse_s) * kLog2e);
        if (va + 8 * p + e >= V) x = 0.f;
        if (8 * p + e == y_lane) x -= 1.0f;
        o[e] = (__bf16)x;
      }
      *reinterpret_cast<bf16x8*>(srow + 16 * p) = o;
    }
  }
  __syncthreads();
  constexpr int kLanesPerRow = C::EA / 8, kRowsPerPass = C::kThreads / kLanesPerRow;
  const int col = (threadIdx.x % kLanesPerRow) * 8;
  if (v0 + col < ldg) {
#pragma unroll
    for (int i = 0; i < C::EB / kRowsPerPass; ++i) {
      const int row = i * kRowsPerPass + threadIdx.x / kLanesPerRow;
      if (s0 + row < rows)
        *reinterpret_cast<bf16x8*>(G + (size_t)(s0 + row) * ldg + v0 + col) =
            *reinterpret_cast<const bf16x8*>(smem + row * kStageRow + col * 2);
    }
  }
}

// ---------------------------------------------------------------------------
// backward 2: dH_chunk = G W, one split of the contraction over V per group of tiles (as kDhSplit of dh_tile)
//   A side = hidden index j (W, K-strided, permuted: a lane holds 4 TA consecutive j), B side = chunk rows (G)
// ---------------------------------------------------------------------------
template <class C>
__device__ __forceinline__ void dh_tile_small(
    const __bf16* __restrict__ G, int ldg, const __bf16* __restrict__ W, int rows, int d, int V,
    int n_st, int n_jt, int n_split, int ksteps_per_split, const long long* __restrict__ n_valid, float grad_loss,
    float* __restrict__ partial /* [n_split][rows_stride][d] */, int rows_stride, __bf16* __restrict__ dHc, char* smem) {
  // splits are the slow coordinate: an XCD's workgroups share a range of W and of the columns of G
  int w, st;
  if (!even_tile_of_block(blockIdx.x, n_jt * n_split, n_st, &w, &st)) return;
  const int sp = w / n_jt, jt = w - sp * n_jt;
  const int j0 = jt * C::EA, s0 = st * C::EB;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wa = wave / C::WB, wb = wave % C::WB;
  const int k_begin = sp * ksteps_per_split * C::BK;
  int k_end = k_begin + ksteps_per_split * C::BK;
  if (k_end > V) k_end = V;

  f32x4 acc[C::TA][C::TB];
  zero_acc<C::TA, C::TB>(acc);
  {
    PanelKS16<C, C::EA, C::TA, true> pa;
    PanelKC16<C, C::EB, C::TB, false> pb;
    pa.init(W + j0, d, V, d - j0, wave, lane, wa);
    pb.init(G + (size_t)s0 * ldg, ldg, rows - s0, ldg, wave, lane, wb);
    gemm_mainloop_small<C>(acc, pa, pb, smem, k_begin, k_end);
  }
  const float gamma = n_split == 1 ? gamma_of(n_valid, grad_loss) : 1.f;
  const int jb = j0 + 16 * C::TA * wa + 4 * C::TA * (lane >> 4);
#pragma unroll
  for (int u = 0; u < C::TB; ++u) {
    const int s_local = s0 + wb * (16 * C::TB) + 16 * u + (lane & 15);
    if (s_local >= rows) continue;
#pragma unroll
    for (int p = 0; p < C::TA / 2; ++p) {                       // d % 8 == 0: a group of 8 is inside or outside
      if (jb + 8 * p >= d) continue;
      if (n_split == 1) {
        bf16x8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = (__bf16)(gamma * acc[2 * p + (e >> 2)][u][e & 3]);
        *reinterpret_cast<bf16x8*>(dHc + (size_t)s_local * d + jb + 8 * p) = o;
      } else {
        float* dst = partial + ((size_t)sp * rows_stride + s_local) * d + jb + 8 * p;
        *reinterpret_cast<f32x4*>(dst) = acc[2 * p][u];
        *reinterpret_cast<f32x4*>(dst + 4) = acc[2 * p + 1][u];
      }
    }
  }
}
template <class C>
__global__ __launch_bounds__(C::kThreads, kSmallWavesPerSimd) void k_bwd_gemm_dh_small(
    const __bf16* __restrict__ G, int ldg, const __bf16* __restrict__ W, int rows, int d, int V,
    int n_st, int n_jt, int n_split, int ksteps_per_split, const long long* __restrict__ n_valid, float grad_loss,
    float* __restrict__ partial, int rows_stride, __bf16* __restrict__ dHc) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  dh_tile_small<C>(G, ldg, W, rows, d, V, n_st, n_jt, n_split, ksteps_per_split, n_valid, grad_loss, partial, rows_stride, dHc, smem);
}

// ---------------------------------------------------------------------------
// backward 3: dW (+)= G^T H, row-major throughout.
//   A side = hidden index j (H, K-strided, permuted: a lane holds 4 TA consecutive j, 16-byte loads and stores),
//   B side = vocabulary (G, K-strided)
// ---------------------------------------------------------------------------
template <class C>
__device__ __forceinline__ void dw_tile_small(const __bf16* __restrict__ G, int ldg, int g_cols, const __bf16* __restrict__ Hc,
                                              int ldh, int rows, int d, int V, int vt, int jt, bool accumulate, float scale,
                                              float* __restrict__ dW, int ldw, char* smem) {
  const int v0 = vt * C::EB, j0 = jt * C::EA;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wa = wave / C::WB, wb = wave % C::WB;

  f32x4 acc[C::TA][C::TB];
  zero_acc<C::TA, C::TB>(acc);
  const int jb = j0 + 16 * C::TA * wa + 4 * C::TA * (lane >> 4);
  auto at = [&](int u) { return v0 + wb * (16 * C::TB) + 16 * u + (lane & 15); };
  if (accumulate) {
#pragma unroll
    for (int u = 0; u < C::TB; ++u)
#pragma unroll
      for (int t = 0; t < C::TA; ++t)
        if (at(u) < V && jb + 4 * t < d) acc[t][u] = *reinterpret_cast<const f32x4*>(dW + (size_t)at(u) * ldw + jb + 4 * t);
    // arrived before the first operand loads are counted (the main loops wait by count)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
    for (int t = 0; t < C::TA; ++t)
#pragma unroll
      for (int u = 0; u < C::TB; ++u) asm volatile("" : "+v"(acc[t][u]));
  }
  {
    PanelKS16<C, C::EA, C::TA, true> pa;
    PanelKS16<C, C::EB, C::TB> pb;
    pa.init(Hc + j0, ldh, rows, d - j0, wave, lane, wa);
    pb.init(G + v0, ldg, rows, g_cols - v0, wave, lane, wb);
    gemm_mainloop_small<C>(acc, pa, pb, smem, 0, rows);
  }
#pragma unroll
  for (int u = 0; u < C::TB; ++u)
#pragma unroll
    for (int t = 0; t < C::TA; ++t)
      if (at(u) < V && jb + 4 * t < d) *reinterpret_cast<f32x4*>(dW + (size_t)at(u) * ldw + jb + 4 * t) = acc[t][u] * scale;
}

template <class C>
__global__ __launch_bounds__(C::kThreads, kSmallWavesPerSimd) void k_bwd_gemm_dw_small(
    const __bf16* __restrict__ G, int ldg, const __bf16* __restrict__ Hc, int rows, int d, int V,
    int n_vt, int n_jt, int accumulate, int last, const long long* __restrict__ n_valid, float grad_loss,
    float* __restrict__ dW) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  int vt, jt;
  if (!even_tile_of_block(blockIdx.x, n_vt, n_jt, &vt, &jt)) return;
  const float scale = last ? gamma_of(n_valid, grad_loss) : 1.0f;
  dw_tile_small<C>(G, ldg, ldg, Hc, d, rows, d, V, vt, jt, accumulate != 0, scale, dW, d, smem);
}

// ---------------------------------------------------------------------------
// backward 2 and 3 from one launch: neither needs the other.  In the smallest problems a launch takes 4 to 6 us whatever
// it does, and the pair order has seven of them per pair of chunks; these two kernels make two of them.
//
// A pair of chunks leaves no room for fp32 partials of dH, so the contraction over V is split between the four waves of
// a workgroup instead and added up in LDS.  A wave's loads are bound by their latency (72 KB in flight on a compute unit,
// 1.4 us), and 64-byte row pieces cost as much as 128-byte ones, so the tile is 64 hidden indices wide, or 32 where that
// makes enough more workgroups.  512 rows, d = 256, V = 4096, M = 4: backward 65 us (14 launches) -> 31 (4).
// ---------------------------------------------------------------------------
// dH = gamma G W.   A side = hidden index j (W, K-strided), B side = rows (G)
template <class C>
__device__ __forceinline__ void dh_tile_ksplit(const __bf16* __restrict__ G, int ldg, const __bf16* __restrict__ W, int rows, int d,
                                               int V, int st, int jt, const long long* __restrict__ n_valid, float grad_loss,
                                               __bf16* __restrict__ dHc, char* smem) {
  const int j0 = jt * C::EA, s0 = st * C::EB;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  f32x4 acc[C::TA][C::TB];
  zero_acc<C::TA, C::TB>(acc);
  {
    PanelKS16<C, C::EA, C::TA> pa;
    PanelKC16<C, C::EB, C::TB, false> pb;
    pa.init(W + j0, d, V, d - j0, 0, lane, 0);
    pb.init(G + (size_t)s0 * ldg, ldg, rows - s0, ldg, 0, lane, 0);
    gemm_mainloop_ksplit<C>(acc, pa, pb, smem, wave, V);
  }
  // every wave's sums side by side in LDS ([row][j], rows padded by 16 bytes), added in the order of the waves
  constexpr int kRow = C::EA + 4;
  float* const sums = reinterpret_cast<float*>(smem);
#pragma unroll
  for (int u = 0; u < C::TB; ++u)
#pragma unroll
    for (int t = 0; t < C::TA; ++t)
      *reinterpret_cast<f32x4*>(sums + (wave * C::EB + 16 * u + (lane & 15)) * kRow + 16 * t + 4 * (lane >> 4)) = acc[t][u];
  __syncthreads();
  const float gamma = gamma_of(n_valid, grad_loss);
  constexpr int kPer = 8, kLanesPerRow = C::EA / kPer;
  for (int i = threadIdx.x; i < C::EB * kLanesPerRow; i += C::kThreads) {
    const int row = i / kLanesPerRow, col = i % kLanesPerRow * kPer;
    if (s0 + row >= rows || j0 + col >= d) continue;                  // d % 8 == 0
    f32x4 v[2] = {};
#pragma unroll
    for (int w = 0; w < C::kSplit; ++w)
#pragma unroll
      for (int h = 0; h < 2; ++h) v[h] += *reinterpret_cast<const f32x4*>(sums + (w * C::EB + row) * kRow + col + 4 * h);
    bf16x8 o;
#pragma unroll
    for (int e = 0; e < kPer; ++e) o[e] = (__bf16)(gamma * v[e >> 2][e & 3]);
    *reinterpret_cast<bf16x8*>(dHc + (size_t)(s0 + row) * d + j0 + col) = o;
  }
}

typedef CfgKSplit<2, 1, 3> TileKSplit32x16;      // hidden indices x rows; with their stages they fit into Tile64's LDS, or nearly
typedef CfgKSplit<4, 1, 2> TileKSplit64x16;
typedef CfgKSplit<4, 2, 2> TileKSplit64x32;

// the first dh_grid workgroups (a multiple of the XCD count): dH, the longer ones
template <class CH, class CW>
__global__ __launch_bounds__(CW::kThreads, kSmallWavesPerSimd) void k_bwd_gemm_dh_dw_small(
    const __bf16* __restrict__ G, int ldg, const __bf16* __restrict__ W, const __bf16* __restrict__ Hc, int rows, int d, int V,
    int n_sh, int n_jh, int dh_grid, int n_vt, int n_jt, int accumulate, int last, const long long* __restrict__ n_valid,
    float grad_loss, __bf16* __restrict__ dHc, float* __restrict__ dW) {
  static_assert(CH::kThreads == CW::kThreads, "one launch");
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  if ((int)blockIdx.x < dh_grid) {
    int jt, st;
    if (!even_tile_of_block(blockIdx.x, n_jh, n_sh, &jt, &st)) return;
    dh_tile_ksplit<CH>(G, ldg, W, rows, d, V, st, jt, n_valid, grad_loss, dHc, smem);
    return;
  }
  int vt, jt;
  if (!even_tile_of_block((int)blockIdx.x - dh_grid, n_vt, n_jt, &vt, &jt)) return;
  const float scale = last ? gamma_of(n_valid, grad_loss) : 1.0f;
  dw_tile_small<CW>(G, ldg, ldg, Hc, d, rows, d, V, vt, jt, accumulate != 0, scale, dW, d, smem);
}

// The same for a call of one chunk, where the free dlogits slot holds fp32 partials of dH (for k_bwd_dh_reduce).
template <class C>
__global__ __launch_bounds__(C::kThreads, kSmallWavesPerSimd) void k_bwd_gemm_dh_split_dw_small(
    const __bf16* __restrict__ G, int ldg, const __bf16* __restrict__ W, const __bf16* __restrict__ Hc, int rows, int d, int V,
    int n_sh, int n_jh, int n_split, int ksteps_per_split, int dh_grid, int n_vt, const long long* __restrict__ n_valid,
    float grad_loss, float* __restrict__ partial, __bf16* __restrict__ dHc, float* __restrict__ dW) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  if ((int)blockIdx.x < dh_grid) {
    dh_tile_small<C>(G, ldg, W, rows, d, V, n_sh, n_jh, n_split, ksteps_per_split, n_valid, grad_loss, partial, rows, dHc, smem);
    return;
  }
  int vt, jt;
  if (!even_tile_of_block((int)blockIdx.x - dh_grid, n_vt, n_jh, &vt, &jt)) return;
  dw_tile_small<C>(G, ldg, ldg, Hc, d, rows, d, V, vt, jt, false, gamma_of(n_valid, grad_loss), dW, d, smem);
}

}  // namespace mst
