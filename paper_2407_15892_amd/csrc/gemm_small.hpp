// Smaller block tiles for launches that would leave most compute units without a 256 x 256 tile.
//
// A workgroup of four waves (2 x 2) owns a (32 TA) x (32 TB) output tile.  Panels, fragments and MFMA order are those of
// gemm_tile16.hpp and every output is summed over K in the same order as in the 256 x 256 kernels, so results do not
// depend on the tile a launch was given, bit for bit (a split of K between groups of waves would be up to a quarter
// faster with 128 to 256 tiles, but its sums would depend on the rows of a chunk, that is on M).  The one exception is
// the LM-head's dH, whose contraction is split between launches' workgroups in any case: the number of splits is chosen
// with the tile, and with it the order of the fp32 sums.
//
// What bounds it: waiting that nobody fills.  A lone workgroup has one wave per SIMD; in lone 128 x 128 tiles (1024 tokens,
// d = 4096, I = 14336: down, 137 us) it spends 31 % of its time at waits and barriers and 29 % on its turn to issue, and the
// matrix cores are busy 40 % of the clocks.  LDS is not the limit (active a fifth of the clocks, no bank conflicts), nor is
// L2 by itself (13.7 TB/s, 81 % of the requests hit), but a 128 x 128 tile moves twice the bytes per flop out of it that a
// 256 x 256 one does, and a 64 x 64 tile twice as much again.
// These tiles pay where the large ones leave compute units idle or spend their time on first loads and epilogues.
#pragma once
#include "gemm_tile.hpp"
#include "gemm_tile16.hpp"

namespace mst {

// Second launch bound of every kernel with these tiles (256 threads): at two waves per SIMD a wave has at most 256 registers,
// and the compiler then keeps accumulators in ordinary ones.  In accumulation registers they were moved about within the main
// loop: gate/up with 128 x 128 tiles had 64 moves and dependent pairs of MFMAs in a K step of 32 (234 instructions -> 132).
// Forward of 130 tokens, d = 3072, I = 8192: 62 us -> 58; of 353, d = 2096, I = 5768: 77 -> 73; of 1000, d = 3072: 149 -> 145;
// step of 512, d = 256, I = 896, M = 2: 41.8 -> 41.2; LM-head forward of 64 rows, d = 4096, V = 128256: 211 -> 206.  The pipelined
// ones use 90 to 256; only the 256 x 64 forward tile spills, two registers across its loop.
constexpr int kSmallWavesPerSimd = 2;

// wave tile (16 TA) x (16 TB), NSA and NSB LDS stages of the two panels; kPipelined: see the two main loops
template <int TA_, int TB_, int NSA_, int NSB_, bool kPipelined_, int BK_ = 64>
struct CfgSmall {
  static constexpr int WA = 2, WB = 2, TA = TA_, TB = TB_, BK = BK_;
  static constexpr int NSA = NSA_, NSB = NSB_;
  static constexpr bool kPipelined = kPipelined_;
  static constexpr int kWaves = WA * WB, kThreads = 64 * kWaves;
  static constexpr int EA = 16 * TA * WA, EB = 16 * TB * WB;
  static constexpr int kPanelA = EA * BK * 2, kPanelB = EB * BK * 2;
  static constexpr int kLds = NSA * kPanelA + NSB * kPanelB;
  static constexpr int kKK = BK / 32;
  static_assert(kLds <= 163840, "all of a compute unit's LDS at most");
  typedef f32x4 Acc;
  __device__ __forceinline__ static Acc mma(bf16x8 a, bf16x8 b, Acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
};

// For compute units that hold two or more workgroups.  A K step is a memory phase (loads of the later stages between the
// fragment reads of this one), then the MFMAs, with one barrier; another workgroup fills the gaps.  In step kt a wave
// issues its B loads for step kt + 1, then its A loads for step kt + 2, which stay in flight over the next wait.
template <class C, class PA, class PB>
__device__ __forceinline__ void gemm_mainloop_shared(f32x4 (&acc)[C::TA][C::TB], const PA& pa, const PB& pb, char* smem,
                                                     int k_begin, int k_end) {
  static_assert(C::NSA == 3 && C::NSB == 2, "three A stages, two B stages");
  constexpr int kAhead = PA::SPW;
  const uint32_t ldsA = lds_addr_of(smem), ldsB = ldsA + C::NSA * C::kPanelA;
  const char* smemB = smem + C::NSA * C::kPanelA;
  const int nk = (k_end - k_begin + C::BK - 1) / C::BK;
  pa.issue(ldsA, k_begin);
  pb.issue(ldsB, k_begin);
  pa.issue(ldsA + C::kPanelA, k_begin + C::BK);
  wait_vmcnt<kAhead>();
  __builtin_amdgcn_s_barrier();
  int ca = 0, cb = 0;
  int kb = k_begin + C::BK, ka = kb + C::BK;
  for (int kt = 0; kt < nk; ++kt) {
    int na = ca + C::NSA - 1; if (na >= C::NSA) na -= C::NSA;
    const int nb = cb ^ 1;
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
    __builtin_amdgcn_sched_barrier(0);
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
    wait_vmcnt<kAhead>();
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    ca = ca + 1 == C::NSA ? 0 : ca + 1;
    cb ^= 1;
    kb += C::BK;
    ka += C::BK;
  }
  wait_vmcnt<0>();
  __syncthreads();
}

// For a workgroup that has its compute unit to itself: one wave per SIMD, so nothing else issues MFMAs while it reads.
// Each step therefore reads the fragments of the next one into a second set of registers between its own MFMAs (a
// quarter wave of slack per load: 4 MFMAs after every load and its share of the reads).
//
// Stages, of NS per panel: step kt reads stage kt + 1, loads stage kt + NS - 1 into the place of stage kt - 1 (whose
// fragments every wave has in registers, as its MFMAs of step kt - 1 needed them before the barrier), and stages
// kt + 2 .. kt + NS - 2 are in flight at its wait.  Panels whose fragments come from two stages (PanelKC16Lines) have one
// stage less in flight.  64 x 64 tiles, NS = 5, 512 tokens, d = 2048, I = 5632: dX 41 us
// against 57 with the loop above, down 22 against 27; 128 x 128, NS = 4, 1668 tokens, d = 1544, I = 5384: dX 91
// against 120, down 52 against 58.
template <class C, class PA, class PB>
__device__ __forceinline__ void gemm_mainloop_pipelined(f32x4 (&acc)[C::TA][C::TB], const PA& pa, const PB& pb, char* smem,
                                                        int k_begin, int k_end) {
  constexpr int NS = C::NSA, kBehind = PA::kLines || PB::kLines ? 1 : 0;       // stages that a step reads behind its own
  static_assert(C::NSA == C::NSB && C::NSA >= 3 + 2 * kBehind, "as many stages of both panels");
  constexpr int kLoads = PB::SPW + PA::SPW, kFrags = C::kKK * (C::TA + C::TB), kMma = C::kKK * C::TA * C::TB;
  const uint32_t ldsA = lds_addr_of(smem), ldsB = ldsA + NS * C::kPanelA;
  const char* smemB = smem + NS * C::kPanelA;
  const int nk = (k_end - k_begin + C::BK - 1) / C::BK;
#pragma unroll
  for (int j = 0; j < NS - 1; ++j) {
    pb.issue(ldsB + j * C::kPanelB, k_begin + j * C::BK);
    pa.issue(ldsA + j * C::kPanelA, k_begin + j * C::BK);
  }
  wait_vmcnt<(NS - 2 - kBehind) * kLoads>();
  __builtin_amdgcn_s_barrier();
  typedef bf16x8 FragsA[C::kKK][C::TA];
  typedef bf16x8 FragsB[C::kKK][C::TB];
  FragsA a0, a1;
  FragsB b0, b1;
#pragma unroll
  for (int kk = 0; kk < C::kKK; ++kk) {
#pragma unroll
    for (int t = 0; t < C::TA; ++t) a0[kk][t] = pa.frag(smem, smem + C::kPanelA, t, kk);
#pragma unroll
    for (int u = 0; u < C::TB; ++u) b0[kk][u] = pb.frag(smemB, smemB + C::kPanelB, u, kk);
  }
  int rd = 1, ld = NS - 1, kl = k_begin + (NS - 1) * C::BK;      // stage to read, stage to load, its k
  auto step = [&](FragsA& a, FragsB& b, FragsA& an, FragsB& bn) {
    wait_vmcnt<(NS - 3 - kBehind) * kLoads>();
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    const int next = rd + 1 == NS ? 0 : rd + 1;
    const char *a_panel = smem + rd * C::kPanelA, *a_next = smem + next * C::kPanelA;
    const char *b_panel = smemB + rd * C::kPanelB, *b_next = smemB + next * C::kPanelB;
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      if (j < PB::SPW) pb.issue_one(j, ldsB + ld * C::kPanelB, kl);
      else pa.issue_one(j - PB::SPW, ldsA + ld * C::kPanelA, kl);
#pragma unroll
      for (int f = j * kFrags / kLoads; f < (j + 1) * kFrags / kLoads; ++f) {
        const int kk = f / (C::TA + C::TB), r = f % (C::TA + C::TB);
        if (r < C::TA) an[kk][r] = pa.frag(a_panel, a_next, r, kk);
        else bn[kk][r - C::TA] = pb.frag(b_panel, b_next, r - C::TA, kk);
      }
#pragma unroll
      for (int m = j * kMma / kLoads; m < (j + 1) * kMma / kLoads; ++m) {
        const int kk = m / (C::TA * C::TB), t = m / C::TB % C::TA, uu = m % C::TB;
        const int u = (t & 1) ? C::TB - 1 - uu : uu;
        acc[t][u] = C::mma(a[kk][t], b[kk][u], acc[t][u]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    rd = next;
    ld = ld + 1 == NS ? 0 : ld + 1;
    kl += C::BK;
  };
  int kt = 0;
  for (; kt + 2 <= nk; kt += 2) {
    step(a0, b0, a1, b1);
    step(a1, b1, a0, b0);
  }
  if (kt < nk) step(a0, b0, a1, b1);
  wait_vmcnt<0>();
  __syncthreads();
}

template <class C, class PA, class PB>
__device__ __forceinline__ void gemm_mainloop_small(f32x4 (&acc)[C::TA][C::TB], const PA& pa, const PB& pb, char* smem,
                                                    int k_begin, int k_end) {
  if constexpr (C::kPipelined) gemm_mainloop_pipelined<C>(acc, pa, pb, smem, k_begin, k_end);
  else gemm_mainloop_shared<C>(acc, pa, pb, smem, k_begin, k_end);
}

// One wave's share of a contraction, for tiles whose K is split between the four waves of a workgroup: wave w takes the
// K steps (of 32) w, w + 4, w + 8, ...  Every wave has LDS stages of its own and waits for nobody.
//
// In step s the fragments of step s are in registers; the stage they came from is loaded anew with step s + NS, those of
// step s + 1 are read between the MFMAs, and the steps s + 2 .. s + NS are in flight.
template <int TA_, int TB_, int NS_>
struct CfgKSplit {
  static constexpr int TA = TA_, TB = TB_, BK = 32, NS = NS_;
  static constexpr int kWaves = 1, kSplit = 4, kThreads = 64 * kSplit;      // kWaves: of a panel's loaders
  static constexpr int EA = 16 * TA, EB = 16 * TB;
  static constexpr int kPanelA = EA * BK * 2, kPanelB = EB * BK * 2;
  static constexpr int kLds = kSplit * NS * (kPanelA + kPanelB);
  static constexpr int kKK = 1;
  typedef f32x4 Acc;
};
template <class C, class PA, class PB>
__device__ __forceinline__ void gemm_mainloop_ksplit(f32x4 (&acc)[C::TA][C::TB], const PA& pa, const PB& pb, char* smem,
                                                     int wave, int k) {
  constexpr int NS = C::NS, kLoads = PA::SPW + PB::SPW, kStride = C::kSplit * C::BK;
  const int n_step = (k + kStride - 1) / kStride;
  char* const mine = smem + wave * NS * (C::kPanelA + C::kPanelB);
  const uint32_t lds = lds_addr_of(mine);
  auto issue = [&](int slot, int s) {
    const uint32_t at = lds + slot * (C::kPanelA + C::kPanelB);
    const int k0 = s * kStride + wave * C::BK;
    pb.issue(at + C::kPanelA, k0);
    pa.issue(at, k0);
  };
  bf16x8 a0[C::TA], b0[C::TB], a1[C::TA], b1[C::TB];
  auto read = [&](int slot, bf16x8 (&a)[C::TA], bf16x8 (&b)[C::TB]) {
    const char* at = mine + slot * (C::kPanelA + C::kPanelB);
#pragma unroll
    for (int u = 0; u < C::TB; ++u) b[u] = pb.frag(at + C::kPanelA, u, 0);
#pragma unroll
    for (int t = 0; t < C::TA; ++t) a[t] = pa.frag(at, t, 0);
  };
#pragma unroll
  for (int j = 0; j < NS; ++j) issue(j, j);
  wait_vmcnt<(NS - 1) * kLoads>();
  read(0, a0, b0);
  int slot = 0;
  auto step = [&](int s, bf16x8 (&a)[C::TA], bf16x8 (&b)[C::TB], bf16x8 (&an)[C::TA], bf16x8 (&bn)[C::TB]) {
    const int next = slot + 1 == NS ? 0 : slot + 1;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");          // this step's fragments are out of their stage
    issue(slot, s + NS);
    wait_vmcnt<(NS - 1) * kLoads>();
    read(next, an, bn);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < C::TA; ++t)
#pragma unroll
      for (int uu = 0; uu < C::TB; ++uu) {
        const int u = (t & 1) ? C::TB - 1 - uu : uu;
        acc[t][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[t], b[u], acc[t][u], 0, 0, 0);
      }
    __builtin_amdgcn_sched_barrier(0);
    slot = next;
  };
  int s = 0;
  for (; s + 2 <= n_step; s += 2) {
    step(s, a0, b0, a1, b1);
    step(s + 1, a1, b1, a0, b0);
  }
  if (s < n_step) step(s, a0, b0, a1, b1);
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
__host__ __device__ inline int even_grid(int n_slow, int n_fast) { return 8 * ((n_slow * n_fast + 7) / 8); }

}  // namespace mst
