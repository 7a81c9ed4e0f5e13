// Device kernels of the mini-sequence MLP path (gfx950).
//
// Per mini-sequence (chunk) of C rows, or group of rows (see forward_group and
// BackwardGroups in mst_mlp_api.hip), following Algorithm 1 (forward) and
// Algorithm 3 (backward with recomputation) of the paper, for the block
// O = (silu(X Wg^T) * (X Wu^T)) Wd^T of Theorem 1 / Appendix C:
//
//   forward   k_mlp_gateup<false>  gate and up tiles of the same (token, i) range side by side in the MFMA
//                                  accumulators; A = silu(G) * U taken from them, bf16 to the workspace
//             k_mlp_gemm_nt        O_chunk = A Wd^T
//   backward  k_mlp_gemm_nn        dA = dO_chunk Wd
//             k_mlp_gateup<true>   gate and up tiles again; dG = dA U silu'(G), dU = dA silu(G), A
//             k_mlp_gemm_nn        dX_chunk = dG Wg + dU Wu   (two contractions into one accumulator)
//             k_mlp_dw3            dWg += dG^T X, dWu += dU^T X, dWd += dO^T A   (the LM-head's dW tile body)
//             k_mlp_dx_dw3         the last two from one launch
//
// These use the 256 x 256 block tile main loop of gemm_tile.hpp; their namesakes ending in _small do the same with the
// smaller tiles of gemm_small.hpp.  Workgroups are mapped to tiles XCD by XCD.
#pragma once
#include "mst_small_kernels.hpp"

#include <type_traits>

namespace mst {

// Workgroup -> tile mapping of the 256 x 256 kernels: cut into 8 x 4 (slow x fast) super-tiles, XCD x owning
// super-tiles x, x + 8, ... (row-major order of super-tiles), so that the 32 workgroups resident on an XCD read 12
// distinct operand panels; or the even map of gemm_small.hpp, where whole super-tiles would give some XCDs a round of
// workgroups more than others, or where there is not even one full round.  Gate/up on 36 x 6 tiles (10
// super-tiles on 8 XCDs): 38 us instead of 64; down on 16 x 4 tiles (2 super-tiles, so 2 XCDs): 95 instead of 124.
// On 112 x 16 tiles (7 full rounds either way) the super-tiles are 0.8 % faster.
// A template argument of the kernels, so that the long launches carry one map only.
constexpr int kSuperSlow = 8, kSuperFast = 4;
inline int super_tiles(int n_slow, int n_fast) {
  return ((n_slow + kSuperSlow - 1) / kSuperSlow) * ((n_fast + kSuperFast - 1) / kSuperFast);
}
inline bool use_super_tiles(int n_slow, int n_fast) {
  constexpr int kPerRound = kSuperSlow * kSuperFast;                       // workgroups resident on an XCD
  const int per_xcd = (n_slow * n_fast + kNumXcd - 1) / kNumXcd;
  return per_xcd >= kPerRound && (super_tiles(n_slow, n_fast) + kNumXcd - 1) / kNumXcd == (per_xcd + kPerRound - 1) / kPerRound;
}
inline int mlp_grid(int n_slow, int n_fast) {
  if (!use_super_tiles(n_slow, n_fast)) return even_grid(n_slow, n_fast);
  return kNumXcd * ((super_tiles(n_slow, n_fast) + kNumXcd - 1) / kNumXcd) * kSuperSlow * kSuperFast;
}
__host__ __device__ inline bool super_tile_of_block(unsigned block, int n_slow, int n_fast, int* slow, int* fast) {
  const int ss = (n_slow + kSuperSlow - 1) / kSuperSlow, sf = (n_fast + kSuperFast - 1) / kSuperFast;
  const int x = block % kNumXcd, q = block / kNumXcd;
  const int super = x + kNumXcd * (q / (kSuperSlow * kSuperFast));
  const int inner = q % (kSuperSlow * kSuperFast);
  if (super >= ss * sf) return false;
  *slow = (super / sf) * kSuperSlow + inner / kSuperFast;
  *fast = (super % sf) * kSuperFast + inner % kSuperFast;
  return *slow < n_slow && *fast < n_fast;
}
template <bool kSuper>
__device__ __forceinline__ bool mlp_tile(int n_slow, int n_fast, int* slow, int* fast) {
  if (!kSuper) return even_tile_of_block(blockIdx.x, n_slow, n_fast, slow, fast);
  return super_tile_of_block(blockIdx.x, n_slow, n_fast, slow, fast);
}

__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
// logistic function; exp2 overflows to +inf for very negative g, whose reciprocal is 0
__device__ __forceinline__ float sigmoid_f(float g) { return fast_rcp(1.0f + fast_exp2(-g * kLog2e)); }

// ---------------------------------------------------------------------------
// gate / up projections of a chunk with the SwiGLU epilogue.
//   A side = intermediate index i, 128 per workgroup: the 256-row A panel holds, for each of the two
//   wave rows, 64 gate rows (MFMA tiles 0..3) and the 64 up rows of the same i (tiles 4..7), so gate and
//   up values of one (token, i) sit in the same lane and register of accumulators t and t + 4.
//   B side = chunk rows (tokens).  A lane owns 4 tokens and 16 consecutive i for each: 32-byte stores.
//   kBackward: dAG holds dA on entry and receives dG (same element, same lane); dU and A are written.
//   T: the 256 x 256 tile, or half of it on the A side (64 indices).
// ---------------------------------------------------------------------------
constexpr int kGateUpI = 128;   // intermediate indices per workgroup of large tiles
template <class T, bool kBackward, bool kSuper>
__global__ __launch_bounds__(kThreads) void k_mlp_gateup(
    const __bf16* __restrict__ Xc, const __bf16* __restrict__ Wg, const __bf16* __restrict__ Wu,
    int rows, int d, int I /* indices of this launch */, int ldi, int n_st, int n_it,
    __bf16* __restrict__ A, __bf16* __restrict__ dAG, __bf16* __restrict__ dU) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  constexpr int H = T::TA / 2, N = 4 * H;                       // gate tiles of a wave; consecutive indices of a lane
  int it, st;
  if (!mlp_tile<kSuper>(n_it, n_st, &it, &st)) return;
  const int i0 = it * (T::EA / 2), s0 = st * T::EB;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wa = wave >> 2, wb = wave & 3;

  f32x4 acc[T::TA][T::TB];
  zero_acc<T::TA, T::TB>(acc);
  PanelKC16<T, T::EA, T::TA, true> pa;
  PanelKC16<T, T::EB, T::TB, false> pb;
  {
    // A panel, per wave row of 16 TA LDS rows: MFMA tiles 0..H-1 are gate rows, tiles H..2H-1 the up rows of the same 16 H
    // intermediate indices; LDS row 16 t + 4 g + r holds index N g + 4 (t % H) + r, so that a lane's gate value
    // acc[t][u][r] and up value acc[t + H][u][r] belong to the same index and its N indices are consecutive.
    // As a loader, a wave fills an eighth of the LDS rows: they belong to one half (gate or up) of one wave row.
    const int half = wave * (T::EA / 8) / (16 * H);
    const int ib = i0 + 16 * H * (half >> 1);                   // first index of the loader's wave row
    const __bf16* src = ((half & 1) ? Wu : Wg) + (size_t)ib * d;
    int valid = I - ib;
    if (valid > 16 * H) valid = 16 * H;
    pa.init_map(src, d, valid, d, wave, lane, wa,
                [](int lrow) { return N * ((lrow >> 2) & 3) + 4 * ((lrow >> 4) % H) + (lrow & 3); }, false);
  }
  pb.init(Xc + (size_t)s0 * d, d, rows - s0, d, wave, lane, wb);
  gemm_mainloop_pp<T>(acc, pa, pb, smem, 0, d, wa);

  const int ib = i0 + 16 * H * wa + N * (lane >> 4);           // this lane's N consecutive intermediate indices
  constexpr int kPer = 8;                                      // of a load or store; I % 8 == 0: inside or outside
  auto row_of = [&](int u) { return s0 + wb * (16 * T::TB) + 16 * u + (lane & 15); };
  bf16x8 da[T::TB][N / kPer];
  if (kBackward) {                                             // all of them before the first store, which they could alias
#pragma unroll
    for (int u = 0; u < T::TB; ++u)
#pragma unroll
      for (int h = 0; h < N / kPer; ++h)
        if (row_of(u) < rows && ib + kPer * h < I)
          da[u][h] = *reinterpret_cast<const bf16x8*>(dAG + (size_t)row_of(u) * ldi + ib + kPer * h);
  }
#pragma unroll
  for (int u = 0; u < T::TB; ++u) {
    const int s_local = row_of(u);
    if (s_local >= rows || ib >= I) continue;
    const size_t off = (size_t)s_local * ldi + ib;
    bf16x8 a_o[N / kPer], g_o[N / kPer], u_o[N / kPer];
#pragma unroll
    for (int e = 0; e < N; ++e) {                              // index ib + e: tile e / 4, register e % 4
      const float g = acc[e >> 2][u][e & 3], up = acc[H + (e >> 2)][u][e & 3];
      const float sg = sigmoid_f(g);
      const float act = g * sg;                                // silu(g)
      a_o[e / kPer][e % kPer] = (__bf16)(act * up);
      if (kBackward) {
        const float dav = (float)da[u][e / kPer][e % kPer];
        g_o[e / kPer][e % kPer] = (__bf16)(dav * up * (sg * (1.0f + g * (1.0f - sg))));   // dA * U * silu'(G)
        u_o[e / kPer][e % kPer] = (__bf16)(dav * act);                                    // dA * silu(G)
      }
    }
#pragma unroll
    for (int h = 0; h < N / kPer; ++h)
      if (ib + kPer * h < I) {
        *reinterpret_cast<bf16x8*>(A + off + kPer * h) = a_o[h];
        if (kBackward) {
          *reinterpret_cast<bf16x8*>(dAG + off + kPer * h) = g_o[h];
          *reinterpret_cast<bf16x8*>(dU + off + kPer * h) = u_o[h];
        }
      }
  }
}

// ---------------------------------------------------------------------------
// out[s][n] = sum_k P[s][k] Q[n][k]      (both operands K-contiguous; used for O_chunk = A Wd^T)
//   A side = n (rows of Q, permuted so a lane holds 32 consecutive n), B side = s (rows of P)
// ---------------------------------------------------------------------------
template <class T, bool kSuper>
__global__ __launch_bounds__(kThreads) void k_mlp_gemm_nt(
    const __bf16* __restrict__ P, int ldp, const __bf16* __restrict__ Q, int ldq, int rows, int N, int K,
    int n_st, int n_nt, __bf16* __restrict__ out, int ldo) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  int nt, st;
  if (!mlp_tile<kSuper>(n_nt, n_st, &nt, &st)) return;
  const int n0 = nt * T::EA, s0 = st * T::EB;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wa = wave >> 2, wb = wave & 3;

  f32x4 acc[T::TA][T::TB];
  zero_acc<T::TA, T::TB>(acc);
  PanelKC16<T, T::EA, T::TA, true> pa;
  PanelKC16<T, T::EB, T::TB, false> pb;
  pa.init(Q + (size_t)n0 * ldq, ldq, N - n0, K, wave, lane, wa);
  pb.init(P + (size_t)s0 * ldp, ldp, rows - s0, K, wave, lane, wb);
  gemm_mainloop_pp<T>(acc, pa, pb, smem, 0, K, wa);
  store_rows_bf16<T>(acc, out, ldo, rows, N, s0, n0, wa, wb, wave, lane, smem);
}

template <class T, bool kSuper>
__global__ __launch_bounds__(kThreads) void k_mlp_gemm_nn(
    const __bf16* __restrict__ P1, const __bf16* __restrict__ Q1,
    const __bf16* __restrict__ P2, const __bf16* __restrict__ Q2,
    int ldp, int ldq, int rows, int N, int K, int n_st, int n_nt, __bf16* __restrict__ out, int ldo) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  int nt, st;
  if (!mlp_tile<kSuper>(n_nt, n_st, &nt, &st)) return;
  nn_tile<T>(P1, Q1, P2, Q2, ldp, ldq, rows, N, K, nt, st, out, ldo, smem);
}

// ---------------------------------------------------------------------------
// The same three GEMMs with the smaller tiles of gemm_small.hpp, for chunks whose 256 x 256 tiles would leave most of
// the chip idle (the rule and the measurements are at choose_tile in mst_mlp_api.hip); every output has the same bits.
// A side = i or n (32 TA of them per workgroup; gate/up: 16 TA indices, gate and up rows interleaved per wave as above),
// B side = 32 TB tokens.  The permuted A rows give a lane 4 TA consecutive n (2 TA consecutive i), which
// leave the accumulators as 16-byte (8-byte) stores straight to memory: the four lane quarters complete a 128-byte line.
// ---------------------------------------------------------------------------
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;

// kDa: dA is computed here too, not read: dA = dO Wd over the same indices and tokens (Wd K-strided), rounded to bf16 as in
// memory.  One launch less, for launches that are one short tile deep (see fuse_da in mst_mlp_api.hip).
struct DaProblem { const __bf16 *dO, *Wd; };      // [rows][d] of the chunk, [d][ldi]
template <class C, bool kBackward, bool kDa = false>
__global__ __launch_bounds__(C::kThreads, kSmallWavesPerSimd) void k_mlp_gateup_small(
    const __bf16* __restrict__ Xc, const __bf16* __restrict__ Wg, const __bf16* __restrict__ Wu,
    int rows, int d, int I /* indices of this launch */, int ldi, int n_st, int n_it,
    __bf16* __restrict__ A, __bf16* __restrict__ dAG, __bf16* __restrict__ dU, DaProblem da_in) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  constexpr int H = C::TA / 2;                                  // gate tiles of a wave; as many up tiles follow
  int it, st;
  if (!even_tile_of_block(blockIdx.x, n_it, n_st, &it, &st)) return;
  const int i0 = it * (C::EA / 2), s0 = st * C::EB;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wa = wave / C::WB, wb = wave % C::WB;

  constexpr int N = 4 * H;                                      // consecutive indices of a lane
  typedef __attribute__((ext_vector_type(N))) __bf16 vec;
  vec da_own[C::TB];
  if constexpr (kDa) {
    static_assert(H == 1 && C::NSA == C::NSB, "the indices of a lane are those of an unpermuted 16-row tile");
    typedef CfgSmall<H, C::TB, C::NSA, C::NSB, true, C::BK> CD;
    static_assert(CD::kLds <= C::kLds, "the same launch");
    f32x4 acc[CD::TA][CD::TB];
    zero_acc<CD::TA, CD::TB>(acc);
    PanelKS16<CD, CD::EA, CD::TA> pa;
    PanelKC16<CD, CD::EB, CD::TB, false> pb;
    pa.init(da_in.Wd + i0, ldi, d, I - i0, wave, lane, wa);
    pb.init(da_in.dO + (size_t)s0 * d, d, rows - s0, d, wave, lane, wb);
    gemm_mainloop_small<CD>(acc, pa, pb, smem, 0, d);
#pragma unroll
    for (int u = 0; u < C::TB; ++u)
#pragma unroll
      for (int e = 0; e < N; ++e) da_own[u][e] = (__bf16)acc[0][u][e];
  }

  f32x4 acc[C::TA][C::TB];
  zero_acc<C::TA, C::TB>(acc);
  {
    PanelKC16<C, C::EA, C::TA, true> pa;
    PanelKC16<C, C::EB, C::TB, false> pb;
    // a loader wave's LDS rows belong to one half (gate or up) of one wave row
    constexpr int kLoaderRows = C::EA / C::kWaves;
    const int half = wave * kLoaderRows / (16 * H);
    const int ib = i0 + 16 * H * (half >> 1);
    const __bf16* src = ((half & 1) ? Wu : Wg) + (size_t)ib * d;
    const int valid = I - ib < 16 * H ? I - ib : 16 * H;
    pa.init_map(src, d, valid, d, wave, lane, wa,
                [](int lrow) { return 4 * H * ((lrow >> 2) & 3) + 4 * ((lrow >> 4) % H) + (lrow & 3); }, false);
    pb.init(Xc + (size_t)s0 * d, d, rows - s0, d, wave, lane, wb);
    gemm_mainloop_small<C>(acc, pa, pb, smem, 0, d);
  }
  const int ib = i0 + 16 * H * wa + N * (lane >> 4);
  auto row_of = [&](int u) { return s0 + wb * (16 * C::TB) + 16 * u + (lane & 15); };
  vec da[C::TB];
  if (kBackward && !kDa) {                                      // all of them before the first store, which they could alias
#pragma unroll
    for (int u = 0; u < C::TB; ++u)
      if (row_of(u) < rows && ib < I) da[u] = *reinterpret_cast<const vec*>(dAG + (size_t)row_of(u) * ldi + ib);
  }
#pragma unroll
  for (int u = 0; u < C::TB; ++u) {
    const int s_local = row_of(u);
    if (s_local >= rows || ib >= I) continue;                   // I % 8 == 0 and N divides 8
    const size_t off = (size_t)s_local * ldi + ib;
    vec a_o, g_o, u_o;
#pragma unroll
    for (int e = 0; e < N; ++e) {
      const float g = acc[e >> 2][u][e & 3], up = acc[H + (e >> 2)][u][e & 3];
      const float sg = sigmoid_f(g);
      const float act = g * sg;
      a_o[e] = (__bf16)(act * up);
      if (kBackward) {
        const float dav = (float)(kDa ? da_own : da)[u][e];
        g_o[e] = (__bf16)(dav * up * (sg * (1.0f + g * (1.0f - sg))));
        u_o[e] = (__bf16)(dav * act);
      }
    }
    *reinterpret_cast<vec*>(A + off) = a_o;
    if (kBackward) {
      *reinterpret_cast<vec*>(dAG + off) = g_o;
      *reinterpret_cast<vec*>(dU + off) = u_o;
    }
  }
}

// a lane's 4 TA consecutive n (A side, permuted) of UB token rows, as bf16
template <class C>
__device__ __forceinline__ void store_small_bf16(const f32x4 (&acc)[C::TA][C::TB], __bf16* __restrict__ out, int ldo,
                                                 int rows, int N, int s0, int n0, int wa, int wb, int lane) {
  constexpr int kPer = C::TA == 1 ? 4 : 8;                        // N % 8 == 0: a store is inside or outside
  typedef __attribute__((ext_vector_type(kPer))) __bf16 vec;
  const int nb = n0 + 16 * C::TA * wa + 4 * C::TA * (lane >> 4);
#pragma unroll
  for (int u = 0; u < C::TB; ++u) {
    const int s_local = s0 + wb * (16 * C::TB) + 16 * u + (lane & 15);
    if (s_local >= rows) continue;
#pragma unroll
    for (int p = 0; p < 4 * C::TA / kPer; ++p) {
      vec o;
#pragma unroll
      for (int e = 0; e < kPer; ++e) o[e] = (__bf16)acc[(kPer * p + e) >> 2][u][e & 3];
      if (nb + kPer * p < N) *reinterpret_cast<vec*>(out + (size_t)s_local * ldo + nb + kPer * p) = o;
    }
  }
}

// out[s][n] = sum_k P[s][k] Q[n][k].   kLines: rows are not whole cache lines (PanelKC16Lines).
template <class C, bool kLines>
__global__ __launch_bounds__(C::kThreads, kSmallWavesPerSimd) void k_mlp_gemm_nt_small(
    const __bf16* __restrict__ P, int ldp, const __bf16* __restrict__ Q, int ldq, int rows, int N, int K,
    int n_st, int n_nt, __bf16* __restrict__ out, int ldo) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  int nt, st;
  if (!even_tile_of_block(blockIdx.x, n_nt, n_st, &nt, &st)) return;
  const int n0 = nt * C::EA, s0 = st * C::EB;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wa = wave / C::WB, wb = wave % C::WB;

  f32x4 acc[C::TA][C::TB];
  zero_acc<C::TA, C::TB>(acc);
  {
    std::conditional_t<kLines, PanelKC16Lines<C, C::EA, C::TA, true>, PanelKC16<C, C::EA, C::TA, true>> pa;
    std::conditional_t<kLines, PanelKC16Lines<C, C::EB, C::TB, false>, PanelKC16<C, C::EB, C::TB, false>> pb;
    pa.init(Q + (size_t)n0 * ldq, ldq, N - n0, K, wave, lane, wa);
    pb.init(P + (size_t)s0 * ldp, ldp, rows - s0, K, wave, lane, wb);
    gemm_mainloop_small<C>(acc, pa, pb, smem, 0, K);
  }
  store_small_bf16<C>(acc, out, ldo, rows, N, s0, n0, wa, wb, lane);
}

// out[s][n] = sum_k P1[s][k] Q1[k][n] (+ sum_k P2[s][k] Q2[k][n]).   kLines: rows of P are not whole cache lines.
template <class C, bool kLines = false>
__device__ __forceinline__ void nn_tile_small(
    const __bf16* __restrict__ P1, const __bf16* __restrict__ Q1,
    const __bf16* __restrict__ P2, const __bf16* __restrict__ Q2,
    int ldp, int ldq, int rows, int N, int K, int block, int n_st, int n_nt, __bf16* __restrict__ out, int ldo, char* smem) {
  int nt, st;
  if (!even_tile_of_block(block, n_nt, n_st, &nt, &st)) return;
  const int n0 = nt * C::EA, s0 = st * C::EB;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wa = wave / C::WB, wb = wave % C::WB;

  f32x4 acc[C::TA][C::TB];
  zero_acc<C::TA, C::TB>(acc);
  const int terms = P2 != nullptr ? 2 : 1;
  for (int term = 0; term < terms; ++term) {
    PanelKS16<C, C::EA, C::TA, (C::TA > 1)> pa;                   // one 16-row tile: the permutation is the identity
    std::conditional_t<kLines, PanelKC16Lines<C, C::EB, C::TB, false>, PanelKC16<C, C::EB, C::TB, false>> pb;
    pa.init((term ? Q2 : Q1) + n0, ldq, K, N - n0, wave, lane, wa);
    pb.init((term ? P2 : P1) + (size_t)s0 * ldp, ldp, rows - s0, K, wave, lane, wb);
    gemm_mainloop_small<C>(acc, pa, pb, smem, 0, K);
  }
  store_small_bf16<C>(acc, out, ldo, rows, N, s0, n0, wa, wb, lane);
}
template <class C, bool kLines>
__global__ __launch_bounds__(C::kThreads, kSmallWavesPerSimd) void k_mlp_gemm_nn_small(
    const __bf16* __restrict__ P1, const __bf16* __restrict__ Q1,
    const __bf16* __restrict__ P2, const __bf16* __restrict__ Q2,
    int ldp, int ldq, int rows, int N, int K, int n_st, int n_nt, __bf16* __restrict__ out, int ldo) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  nn_tile_small<C, kLines>(P1, Q1, P2, Q2, ldp, ldq, rows, N, K, blockIdx.x, n_st, n_nt, out, ldo, smem);
}

// ---------------------------------------------------------------------------
// the three weight gradients of a chunk from one launch: dWg (+)= dG^T X, dWu (+)= dU^T X, dWd (+)= dO^T A.
//   Each is a tile space of its own (the LM-head's dW tile body); the workgroup index selects the problem.
//   One launch instead of three leaves one partly filled last round of workgroups instead of three
//   (3 x 896 tiles = 10.5 rounds of 256 instead of 3 x 4 at the Llama3-8B shape).
// ---------------------------------------------------------------------------
struct DwProblem {
  const __bf16* G; int ldg;      // [rows][ldg], V columns used
  const __bf16* H; int ldh;      // [rows][ldh], d columns used
  int d, V, n_vt, n_jt, grid;    // grid: workgroups of this problem
  float* dW;                     // [V][d]
};
struct DwProblems { DwProblem p[3]; };
// kStoreOnly: the first group of rows only stores; later ones add to the stored sums; `more`: another one follows
template <bool kStoreOnly, bool kEven>
__device__ __forceinline__ void dw3_tile(int b, const DwProblems& ps, int rows, int more, char* smem) {
  int which = 0;
  if (b >= ps.p[0].grid) { b -= ps.p[0].grid; which = 1; if (b >= ps.p[1].grid) { b -= ps.p[1].grid; which = 2; } }
  const DwProblem& q = ps.p[which];
  int vt, jt;
  // 8 x 4 rectangles walked group by group of 4 fast tiles (measured 0.7 % faster here than the LM-head's 4 x 8 bands)
  if (!launch_tile<8, 4, 4>(kEven, b, q.n_vt, q.n_jt, &vt, &jt)) return;
  dw_tile(q.G, q.ldg, q.ldg, q.H, q.ldh, rows, q.d, q.V, vt, jt, kStoreOnly ? 0 : 1, more, 1.0f, q.dW, q.d, smem);
}
template <bool kStoreOnly, bool kEven>
__global__ __launch_bounds__(kThreads) void k_mlp_dw3(DwProblems ps, int rows, int more) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  dw3_tile<kStoreOnly, kEven>(blockIdx.x, ps, rows, more, smem);
}

// dX = dG Wg + dU Wu and the weight gradients of a chunk from one launch: neither needs the other.  On its own dX is a
// single, partly filled round of long tiles (its contraction is 2 I), or of smaller, slower ones that fill the chip; here
// its large tiles occupy some compute units while the others work through the short tiles of the weight gradients, whose
// stores then also overlap with MFMAs.  First dx.grid workgroups: dX, the longer ones, dealt out evenly over the XCDs.
// T: 256 x 256, or half of that on the A side (hidden index) where whole tiles would be the end of the launch.
// Both launches -> one, us: 1024 rows, d = 4096, I = 14336: 638 -> 570 (half tiles); 2048 rows of it 1050 -> 940 (whole);
// 1668 rows, d = 1544, I = 5384: 206 -> 170 (half).
// With whole tiles the launch has 36 bytes of scratch per lane, for eight registers that nn_tile spills across its first
// term's main loop, once per tile (as in k_mlp_gemm_nn); the weight-gradient tiles spill nothing.
struct DxProblem {
  const __bf16 *dG, *Wg, *dU, *Wu;   // [rows][I], [I][d]
  int d, I, n_st, n_jt, grid;        // grid: workgroups of this problem, a multiple of the XCD count
  __bf16* dX;                        // [rows][d]
};
template <bool kStoreOnly, bool kEven, class T>
__global__ __launch_bounds__(kThreads) void k_mlp_dx_dw3(DxProblem x, DwProblems ps, int rows, int more) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  if ((int)blockIdx.x < x.grid) {
    int jt, st;
    if (!even_tile_of_block(blockIdx.x, x.n_jt, x.n_st, &jt, &st)) return;
    nn_tile<T>(x.dG, x.Wg, x.dU, x.Wu, x.I, x.d, rows, x.d, x.I, jt, st, x.dX, x.d, smem);
    return;
  }
  dw3_tile<kStoreOnly, kEven>((int)blockIdx.x - x.grid, ps, rows, more, smem);
}

// the same with 64 x 64 tiles, for problems too small to occupy the chip with large ones (mst_small_kernels.hpp)
template <class C>
__device__ __forceinline__ void dw3_tile_small(int b, const DwProblems& ps, int rows, int accumulate, char* smem) {
  int which = 0;
  if (b >= ps.p[0].grid) { b -= ps.p[0].grid; which = 1; if (b >= ps.p[1].grid) { b -= ps.p[1].grid; which = 2; } }
  const DwProblem& q = ps.p[which];
  int vt, jt;
  if (!even_tile_of_block(b, q.n_vt, q.n_jt, &vt, &jt)) return;
  dw_tile_small<C>(q.G, q.ldg, q.ldg, q.H, q.ldh, rows, q.d, q.V, vt, jt, accumulate != 0, 1.0f, q.dW, q.d, smem);
}
template <class C>
__global__ __launch_bounds__(C::kThreads, kSmallWavesPerSimd) void k_mlp_dw3_small(DwProblems ps, int rows, int accumulate) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  dw3_tile_small<C>(blockIdx.x, ps, rows, accumulate, smem);
}
// and with dX beside them (CX: its tile).  dX has the workgroups from dx_from on; the others, before and behind, are those
// of the weight gradients (dx_from is 0 or all of theirs).
template <class CX, class CW, bool kLines>
__global__ __launch_bounds__(CW::kThreads, kSmallWavesPerSimd) void k_mlp_dx_dw3_small(DxProblem x, DwProblems ps, int rows, int accumulate,
                                                                                      int dx_from) {
  static_assert(CX::kThreads == CW::kThreads, "one launch");
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int b = (int)blockIdx.x - dx_from;
  if (b >= 0 && b < x.grid) {
    nn_tile_small<CX, kLines>(x.dG, x.Wg, x.dU, x.Wu, x.I, x.d, rows, x.d, x.I, b, x.n_st, x.n_jt, x.dX, x.d, smem);
    return;
  }
  dw3_tile_small<CW>(b < 0 ? (int)blockIdx.x : b - x.grid, ps, rows, accumulate, smem);
}

}  // namespace mst
