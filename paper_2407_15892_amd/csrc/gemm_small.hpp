// Smaller block tiles for launches that would leave most compute units without a 256 x 256 tile.
//
// A workgroup owns a (32 TA) x (16 TB WB) output tile.  Panels, fragments and MFMA order are those of gemm_tile16.hpp
// and every output is summed over K in the same order as in the 256 x 256 kernels, so results do not depend on the
// tile a launch was given, bit for bit (a split of K between groups of waves would be up to a quarter faster with 128
// to 256 tiles, but its sums would depend on the rows of a chunk, that is on M).
//
// What bounds it: a 128 x 128 tile moves twice the bytes per flop of a 256 x 256 one from L2 into LDS (64 flop per byte,
// about what one compute unit's load path and matrix cores balance at), a 64 x 64 tile four times; these tiles pay
// where the large ones leave compute units idle or spend their time on first loads and epilogues.
#pragma once
#include "gemm_tile.hpp"
#include "gemm_tile16.hpp"

namespace mst {

// wave grid 2 x WB, wave tile (16 TA) x (16 TB), NSA and NSB LDS stages of the two panels
template <int TA_, int TB_, int WB_, int NSA_, int NSB_>
struct CfgSmall {
  static constexpr int WA = 2, WB = WB_, TA = TA_, TB = TB_, BK = 64;
  static constexpr int NSA = NSA_, NSB = NSB_;
  static_assert(NSB >= 2 && (NSA == NSB || NSA == NSB + 1), "the wait in the main loop counts on this");
  static constexpr int kWaves = WA * WB, kThreads = 64 * kWaves;
  static constexpr int EA = 16 * TA * WA, EB = 16 * TB * WB;
  static constexpr int kPanelA = EA * BK * 2, kPanelB = EB * BK * 2;
  static constexpr int kLds = NSA * kPanelA + NSB * kPanelB;
  static constexpr int kKK = BK / 32;
  static constexpr bool kPingPong = kWaves == 8;         // two waves per SIMD, half a step apart (see gemm_mainloop_pp)
  static_assert(kLds <= 163840, "all of a compute unit's LDS at most");
  typedef f32x4 Acc;
  __device__ __forceinline__ static Acc mma(bf16x8 a, bf16x8 b, Acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
};

// One K step: a memory phase (loads of the later stages between the fragment reads of this one), then the MFMAs.  With
// four waves a barrier per step keeps them together and a second workgroup on the compute unit fills the gaps; with
// eight the two halves alternate, one barrier per phase.
template <class C, class PA, class PB>
__device__ __forceinline__ void gemm_mainloop_small(f32x4 (&acc)[C::TA][C::TB], const PA& pa, const PB& pb, char* smem,
                                                    int k_begin, int k_end, int group) {
  // In step kt a wave issues its B loads for step kt + NSB - 1, then its A loads for step kt + NSA - 1; the wait that
  // opens the next step leaves everything in flight that was issued after that step's own panels.
  constexpr int kAhead = (C::NSB - 2) * (PA::SPW + PB::SPW) + (C::NSA > C::NSB ? PA::SPW : 0);
  const uint32_t ldsA = lds_addr_of(smem), ldsB = ldsA + C::NSA * C::kPanelA;
  const char* smemB = smem + C::NSA * C::kPanelA;
  const int nk = (k_end - k_begin + C::BK - 1) / C::BK;
#pragma unroll
  for (int j = 0; j < C::NSA - 1; ++j) {
    const int jb = j - (C::NSA - C::NSB);
    if (jb >= 0) pb.issue(ldsB + jb * C::kPanelB, k_begin + jb * C::BK);
    pa.issue(ldsA + j * C::kPanelA, k_begin + j * C::BK);
  }
  wait_vmcnt<kAhead>();
  __builtin_amdgcn_s_barrier();
  if (C::kPingPong && group == 1) __builtin_amdgcn_s_barrier();
  int ca = 0, cb = 0;
  int ka = k_begin + (C::NSA - 1) * C::BK, kb = k_begin + (C::NSB - 1) * C::BK;
  for (int kt = 0; kt < nk; ++kt) {
    // ---- memory phase
    int na = ca + C::NSA - 1; if (na >= C::NSA) na -= C::NSA;
    int nb = cb + C::NSB - 1; if (nb >= C::NSB) nb -= C::NSB;
    const char* a_panel = smem + ca * C::kPanelA;
    const char* b_panel = smemB + cb * C::kPanelB;
    bf16x8 a[C::kKK][C::TA], b[C::kKK][C::TB];
    constexpr int kLoads = PB::SPW + PA::SPW, kFrags = C::kKK * (C::TA + C::TB);
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      if (j < PB::SPW) pb.issue_one(j, ldsB + nb * C::kPanelB, kb);
      else pa.issue_one(j - PB::SPW, ldsA + na * C::kPanelA, ka);
#pragma unroll
      for (int f = j * kFrags / kLoads; f < (j + 1) * kFrags / kLoads; ++f) {
        const int kk = f / (C::TA + C::TB), r = f % (C::TA + C::TB);
        if (r < C::TA) a[kk][r] = pa.frag(a_panel, r, kk);
        else b[kk][r - C::TA] = pb.frag(b_panel, r - C::TA, kk);
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (C::kPingPong && group == 1) wait_vmcnt<kAhead>();   // the other half reads the next stages behind the next barrier
    __builtin_amdgcn_sched_barrier(0);
    if (C::kPingPong) {
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
    }
    // ---- compute phase
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int kk = 0; kk < C::kKK; ++kk)
#pragma unroll
      for (int t = 0; t < C::TA; ++t)
#pragma unroll
        for (int uu = 0; uu < C::TB; ++uu) {
          const int u = (t & 1) ? C::TB - 1 - uu : uu;
          acc[t][u] = C::mma(a[kk][t], b[kk][u], acc[t][u]);
        }
    __builtin_amdgcn_s_setprio(0);
    if (!C::kPingPong || group == 0) wait_vmcnt<kAhead>();
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    ca = ca + 1 == C::NSA ? 0 : ca + 1;
    cb = cb + 1 == C::NSB ? 0 : cb + 1;
    ka += C::BK;
    kb += C::BK;
  }
  if (C::kPingPong && group == 0) __builtin_amdgcn_s_barrier();
  wait_vmcnt<0>();
  __syncthreads();
}

// Workgroup -> tile map: every XCD gets an equal, contiguous share of the tiles, ordered in bands of eight fast tiles, so
// that the 32 workgroups resident on an XCD form a 4 x 8 rectangle (or, with fewer fast tiles, a taller one).
__host__ __device__ inline bool even_tile_of_block(int block, int n_slow, int n_fast, int* slow, int* fast) {
  constexpr int kBand = 8;
  const int total = n_slow * n_fast, per_xcd = (total + 7) / 8;
  const int w = (block % 8) * per_xcd + block / 8;
  if (block / 8 >= per_xcd || w >= total) return false;
  const int band = w / (n_slow * kBand), f0 = band * kBand;
  const int fs = n_fast - f0 < kBand ? n_fast - f0 : kBand;
  const int r = w - n_slow * f0;
  *slow = r / fs;
  *fast = f0 + r - *slow * fs;
  return true;
}
inline int even_grid(int n_slow, int n_fast) { return 8 * ((n_slow * n_fast + 7) / 8); }

}  // namespace mst
