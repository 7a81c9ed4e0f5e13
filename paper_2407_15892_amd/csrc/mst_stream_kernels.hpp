// Backward of the LM-head for small hidden sizes: dlogits never leave the compute unit.
//
// The two gradient products are formed by workgroups that own part of the output and stream the other operand past it:
//
//   dW   owners: vocabulary entries;  stream: the rows of H           dW[v] = gamma sum_s G[s][v] H[s]
//   dH   owners: rows;                stream: the vocabulary (of W)   dH[s] = gamma sum_v G[s][v] W[v]
//
// A wave holds its owners' operand rows in registers.  Per step of 32 stream rows it multiplies them with the stream (the
// logits), turns those into G = softmax - onehot in place, rounded to bf16 as in memory, and multiplies G with the same
// stream rows again, now along the other index.  Both products read one LDS copy of the stream rows: the logits by rows
// (ds_read_b128), the gradient transposed (ds_read_b64_tr_b16).  The accumulators of the first product are the operand of
// the second as they are: lane quarter g holds G of its owner (lane % 16) for the stream rows 4 g .. 4 g + 3 and 16 + 4 g ..
// 16 + 4 g + 3, and the transposed reads fetch the stream rows in that order.
//
// Every logit is formed once more than with dlogits in memory (8 S d V flop instead of 6).  In return there is one launch (and
// dH's reduce) instead of two or three per pair of mini-sequences or block, whose size the workspace limits, and a logit's K
// loop of four to eight steps of 64 has no epilogue through memory: with d = 256 a 256 x 256 tile of dlogits takes 5 us of
// main loop and 7 at its ends.  Backward calls, us, before -> this: 512 rows, d = 256, V = 4096, M = 4: 31.0 -> 16.2; 1706,
// 256, 38336, 6: 283 -> 139; 4096, 384, 32000, 16: 826 -> 439; 5470, 512, 15850, 21: 899 -> 630; 8192, 256, 65536, 64: 2375 -> 895
// (1230 TFLOP/s).
//
// What bounds it: with two workgroups on a compute unit the 64 MFMAs of a wave and step (1024 clocks), the exponentials (450
// to 600 clocks, overlapped with the other wave's MFMAs) and the LDS reads (each fragment feeds OT MFMAs).  Of the clocks of the
// last of these calls the matrix cores are busy 54 %, LDS 42 % (a third of that bank conflicts), of the third call 40 and 62 %; waves
// wait to issue for 40 % of their time and at waits and barriers for 24 %.  In the first one, whose launch takes 15 us (and dH's
// sum 4), the ends of the workgroups are all (8 and 12 %).  Fragments are read a few MFMAs ahead by hand: left to the compiler
// every read was waited for at once (1706 rows: 211 us).  d > 512 would need more accumulators than two waves per SIMD have;
// there dlogits in memory are the better way.
#pragma once
#include "mst_small_kernels.hpp"

namespace mst {

// DK: hidden sizes up to this; OT: 16-owner tiles of a wave; NWS: the rings that share out the stream's steps, 4 / NWS waves
// and their owners each; NST: stages of 32 stream rows in a ring.
template <int DK_, int OT_, int NWS_, int NST_>
struct CfgStream {
  static constexpr int DK = DK_, OT = OT_, NWS = NWS_, NST = NST_;
  static constexpr int kWaves = 4, kThreads = 64 * kWaves, NWO = kWaves / NWS;
  static constexpr int kOwners = 16 * OT * NWO, kStep = 32;
  static constexpr int RB = DK * 2;                              // bytes of a stream row in LDS
  static constexpr int kPanel = kStep * RB, kStage = kPanel + 512;   // rows, then their log-sum-exps and labels (256 bytes each)
  static constexpr int kRing = NST * kStage;
  static constexpr int kSumRow = DK + 4;
  static constexpr int kSums = NWS > 1 ? NWS * kOwners * kSumRow * 4 : 0;
  static constexpr int kLds = NWS * kRing > kSums ? NWS * kRing : kSums;
  static constexpr int NK = DK / 32, NT = DK / 16;               // K steps of the logits, column tiles of the gradient
  static constexpr int kIssue = kPanel / 1024 / NWO;             // panel loads of a wave and stage
  static_assert(DK % 128 == 0 && NST >= 2 && kLds <= 163840 && kIssue * NWO * 1024 == kPanel, "whole loads; fits");
};

__device__ __forceinline__ void dma4(__amdgpu_buffer_rsrc_t rsrc, uint32_t voffset, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dword %1, %2, 0 offen lds"
               :: "s"(lds_addr), "v"(voffset), "s"(rsrc) : "memory");
}

// A ring's stream rows: loads of a stage, fragments for both products.
template <class C>
struct StreamPanel {
  __amdgpu_buffer_rsrc_t rsrc;
  uint32_t voff[C::kIssue];
  uint32_t ok_mask, ld_bytes, slot0;
  uint32_t rd, rt;

  // XOR swizzle of the 16-byte chunk index by the row, for both kinds of reads: sixteen lanes read sixteen rows at one
  // chunk (all sixteen values differ), and 32 lanes read eight rows at a pair of chunks (the upper three bits differ).  A third
  // of the clocks that LDS works are conflicts all the same.
  __device__ __forceinline__ static uint32_t swz(uint32_t row) { return ((row & 7) << 1) | ((row >> 3) & 1); }

  __device__ __forceinline__ void init(const void* base, int d, int rows, int wave_of_ring, int lane) {
    ld_bytes = (uint32_t)d * 2;
    rsrc = make_rsrc_uniform(base, (uint32_t)rows * ld_bytes);
    slot0 = wave_of_ring * C::kIssue;
    ok_mask = 0;
#pragma unroll
    for (int i = 0; i < C::kIssue; ++i) {
      const uint32_t at = (slot0 + i) * 1024 + lane * 16, row = at / C::RB, chunk = (at % C::RB / 16) ^ swz(row);
      voff[i] = row * ld_bytes + chunk * 16;
      ok_mask |= ((int)chunk * 8 < d ? 1u : 0u) << i;
    }
    const uint32_t g = lane >> 4, i16 = lane & 15, q = i16 & 3;
    rd = i16 * C::RB + ((g ^ swz(i16)) * 16);
    const uint32_t krow = 4 * g + (i16 >> 2);
    rt = krow * C::RB + (((q >> 1) ^ swz(krow)) * 16) + (q & 1) * 8;
  }
  __device__ __forceinline__ void issue(uint32_t stage_lds, uint32_t row0) const {
#pragma unroll
    for (int i = 0; i < C::kIssue; ++i)
      dma16(rsrc, ((ok_mask >> i) & 1u) ? voff[i] + row0 * ld_bytes : kOutOfRange, stage_lds + (slot0 + i) * 1024);
  }
  // Chunk indices are XORed into the lane's offset: stages and rows are multiples of the 256 bytes that the swizzle permutes.
  typedef __attribute__((address_space(3))) const char* lds_ptr;
  // rows 16 t + lane % 16, k = 32 kk + 8 (lane / 16) .. + 7
  __device__ __forceinline__ bf16x8 by_row(uint32_t stage_lds, int t, int kk) const {
    typedef __attribute__((address_space(3))) const bf16x8* vec_ptr;
    return *(vec_ptr)((lds_ptr)(uintptr_t)((stage_lds + rd) ^ (64u * (kk & 3))) + (kk >> 2) * 256 + t * (16 * C::RB));
  }
  // column 16 n + lane % 16 of rows 4 g .. + 3 and 16 + 4 g .. + 3
  __device__ __forceinline__ bf16x8 transposed(uint32_t stage_lds, int n) const {
    typedef __attribute__((address_space(3))) i16x4* vec_ptr;
    const lds_ptr at = (lds_ptr)(uintptr_t)((stage_lds + rt) ^ (32u * (n & 7))) + (n >> 3) * 256;
    i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((vec_ptr)(at));
    i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((vec_ptr)(at + 16 * C::RB));
    i16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
  }
};

typedef __attribute__((ext_vector_type(4))) int i32x4;

struct StreamProblem {
  const __bf16 *H, *W;             // [S][d], [V][d]
  const int* labels;
  const float* lse;
  int S, d, V, ignore_index;
  const long long* n_valid;
  float grad_loss;
};

// One workgroup's owners from `o0` on, over the stream rows [begin, end).  kDw: which of the two products (see above).
// store(owner, column, sums of four columns)
template <class C, bool kDw, class Store>
__device__ __forceinline__ void stream_tile(const StreamProblem& p, int o0, int begin, int end, char* smem, Store store) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ring = wave / C::NWO, wo = wave % C::NWO;
  const int g = lane >> 4, c = lane & 15;
  const int n_own = kDw ? p.V : p.S;
  const int own0 = o0 + wo * (16 * C::OT);
  char* const mine = smem + ring * C::kRing;
  const uint32_t lds = lds_addr_of(mine);

  StreamPanel<C> stream;
  const int length = end > begin ? end - begin : 0;
  stream.init((kDw ? p.H : p.W) + (size_t)begin * p.d, p.d, length, wo, lane);
  const uint32_t rows_bytes = (uint32_t)length * 4u;
  const __amdgpu_buffer_rsrc_t lse_rsrc = make_rsrc_uniform(p.lse + begin, rows_bytes), label_rsrc = make_rsrc_uniform(p.labels + begin, rows_bytes);
  constexpr int kLoads = C::kIssue + (kDw ? 2 : 0);
  auto issue = [&](int slot, int step) {
    const uint32_t row0 = (uint32_t)(step * C::NWS + ring) * C::kStep, at = lds + slot * C::kStage;
    stream.issue(at, row0);
    if (kDw) {                     // of 64 rows, of which 32 are this step's; every wave of a ring writes the same
      dma4(lse_rsrc, (row0 + lane) * 4u, at + C::kPanel);
      dma4(label_rsrc, (row0 + lane) * 4u, at + C::kPanel + 256);
    }
  };
  const int n_step = (length + C::kStep * C::NWS - 1) / (C::kStep * C::NWS);
#pragma unroll
  for (int j = 0; j < C::NST - 1; ++j) issue(j, j);

  // the owners' rows: B operand of the logits (lane: owner c of a tile, eight k's of quarter g)
  bf16x8 own[C::OT][C::NK];
  {
    const __bf16* const src = (kDw ? p.W : p.H) + (size_t)own0 * p.d;
    const int left = n_own - own0;
    const __amdgpu_buffer_rsrc_t rsrc = make_rsrc_uniform(src, (uint32_t)(left < 0 ? 0 : left < 16 * C::OT ? left : 16 * C::OT) * (uint32_t)p.d * 2u);
#pragma unroll
    for (int o = 0; o < C::OT; ++o)
#pragma unroll
      for (int kk = 0; kk < C::NK; ++kk) {
        const int k = 32 * kk + 8 * g;
        own[o][kk] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(
            rsrc, k < p.d ? ((uint32_t)(16 * o + c) * (uint32_t)p.d + (uint32_t)k) * 2u : kOutOfRange, 0, 0));
      }
  }
  float own_lse[C::OT];            // dH: of the owner rows
  int own_label[C::OT];
  if (!kDw) {
#pragma unroll
    for (int o = 0; o < C::OT; ++o) {
      const int s = own0 + 16 * o + c, s_in = s < p.S ? s : p.S - 1;
      const int y = p.labels[s_in];
      const bool valid = y != p.ignore_index && (unsigned)y < (unsigned)p.V;
      own_lse[o] = valid ? p.lse[s_in] : __builtin_inff();       // an ignored row: every p is exp2(-infinity)
      own_label[o] = valid ? y : -1;
    }
  }
  // everything above has arrived, so that the waits below count this loop's loads only
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
  for (int o = 0; o < C::OT; ++o)
#pragma unroll
    for (int kk = 0; kk < C::NK; ++kk) asm volatile("" : "+v"(own[o][kk]));

  constexpr int kAhead1 = 2, kAhead2 = C::OT * C::DK > 384 ? 3 : 6;    // fragments read ahead of their MFMAs
  f32x4 acc[C::OT][C::NT];         // columns 16 n + 4 g + r of owner c
  zero_acc<C::OT, C::NT>(acc);
  int slot = 0;
  for (int step = 0; step < n_step; ++step) {
    const int behind = slot == 0 ? C::NST - 1 : slot - 1;          // the stage of the step before, to be loaded anew
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if constexpr (C::NWO > 1) {
      wait_vmcnt<(C::NST - 2) * kLoads>();
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      issue(behind, step + C::NST - 1);
    } else {
      issue(behind, step + C::NST - 1);
      wait_vmcnt<(C::NST - 1) * kLoads>();
    }
    __builtin_amdgcn_sched_barrier(0);
    const char* const stage = mine + slot * C::kStage;

    const uint32_t stage_lds = lds + slot * C::kStage;

    f32x4 z[2][C::OT];             // logits: stream rows 16 t + 4 g + r, owner c
    zero_acc<2, C::OT>(z);
    {
      bf16x8 a[kAhead1 + 1][2];
#pragma unroll
      for (int kk = 0; kk < kAhead1; ++kk)
#pragma unroll
        for (int t = 0; t < 2; ++t) a[kk][t] = stream.by_row(stage_lds, t, kk);
#pragma unroll
      for (int kk = 0; kk < C::NK; ++kk) {
        if (kk + kAhead1 < C::NK)
#pragma unroll
          for (int t = 0; t < 2; ++t) a[(kk + kAhead1) % (kAhead1 + 1)][t] = stream.by_row(stage_lds, t, kk + kAhead1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int o = 0; o < C::OT; ++o)
            z[t][o] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[kk % (kAhead1 + 1)][t], own[o][kk], z[t][o], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    bf16x8 b[kAhead2 + 1];         // the first fragments of the second product, on their way while G is formed
#pragma unroll
    for (int n = 0; n < kAhead2; ++n) b[n] = stream.transposed(stage_lds, n);
    __builtin_amdgcn_sched_barrier(0);

    __builtin_amdgcn_s_setprio(1);
    const int row0 = begin + (step * C::NWS + ring) * C::kStep;   // of the stream
    f32x4 lse_t[2];
    if (kDw) {
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        lse_t[t] = *reinterpret_cast<const f32x4*>(stage + C::kPanel + 64 * t + 16 * g);
        const i32x4 y = *reinterpret_cast<const i32x4*>(stage + C::kPanel + 256 + 64 * t + 16 * g);
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (y[r] == p.ignore_index || (unsigned)y[r] >= (unsigned)p.V) lse_t[t][r] = __builtin_inff();
      }
    }
    // does any of these logits belong to a label?  For most steps none does.
    bool label_here;
    if (kDw) {
      const int y = *reinterpret_cast<const int*>(stage + C::kPanel + 256 + 4 * (lane & 31));
      label_here = __ballot((unsigned)(y - own0) < (unsigned)(16 * C::OT)) != 0;
    } else {
      bool any = false;
#pragma unroll
      for (int o = 0; o < C::OT; ++o) any |= (unsigned)(own_label[o] - row0) < (unsigned)C::kStep;
      label_here = __ballot(any) != 0;
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int o = 0; o < C::OT; ++o)
#pragma unroll
        for (int r = 0; r < 4; ++r) z[t][o][r] = fast_exp2((z[t][o][r] - (kDw ? lse_t[t][r] : own_lse[o])) * kLog2e);
    if (label_here) {
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        i32x4 y;                   // dW: of stream rows; those past the end read as 0, and their rows of H as zeros
        if (kDw) y = *reinterpret_cast<const i32x4*>(stage + C::kPanel + 256 + 64 * t + 16 * g);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int at = kDw ? (y[r] == p.ignore_index ? -1 : y[r] - own0) : row0 + 16 * t + 4 * g + r;
#pragma unroll
          for (int o = 0; o < C::OT; ++o)
            z[t][o][r] -= at == (kDw ? 16 * o + c : own_label[o]) ? 1.0f : 0.0f;
        }
      }
    }
    if (!kDw && row0 + C::kStep > end) {       // entries past the end: their W rows are read as zeros, and p must be finite
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (row0 + 16 * t + 4 * g + r >= end) {
#pragma unroll
            for (int o = 0; o < C::OT; ++o) z[t][o][r] = 0.f;
          }
    }
    bf16x8 gfrag[C::OT];
#pragma unroll
    for (int o = 0; o < C::OT; ++o)
#pragma unroll
      for (int e = 0; e < 8; ++e) gfrag[o][e] = (__bf16)z[e >> 2][o][e & 3];
    __builtin_amdgcn_s_setprio(0);
#pragma unroll
    for (int n = 0; n < C::NT; ++n) {
      if (n + kAhead2 < C::NT) b[(n + kAhead2) % (kAhead2 + 1)] = stream.transposed(stage_lds, n + kAhead2);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int o = 0; o < C::OT; ++o)
        acc[o][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[n % (kAhead2 + 1)], gfrag[o], acc[o][n], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    slot = slot + 1 == C::NST ? 0 : slot + 1;
  }
  wait_vmcnt<0>();
  if constexpr (C::NWS == 1) {
#pragma unroll
    for (int o = 0; o < C::OT; ++o)
#pragma unroll
      for (int n = 0; n < C::NT; ++n) store(own0 + 16 * o + c, 16 * n + 4 * g, acc[o][n]);
  } else {
    // the rings' sums side by side in LDS, added in the order of the rings
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __syncthreads();
    float* const sums = reinterpret_cast<float*>(smem);
#pragma unroll
    for (int o = 0; o < C::OT; ++o)
#pragma unroll
      for (int n = 0; n < C::NT; ++n)
        *reinterpret_cast<f32x4*>(sums + (ring * C::kOwners + wo * (16 * C::OT) + 16 * o + c) * C::kSumRow + 16 * n + 4 * g) = acc[o][n];
    __syncthreads();
    for (int i = threadIdx.x; i < C::kOwners * (C::DK / 4); i += C::kThreads) {
      const int o = i / (C::DK / 4), col = i % (C::DK / 4) * 4;
      f32x4 v = *reinterpret_cast<const f32x4*>(sums + o * C::kSumRow + col);
#pragma unroll
      for (int w = 1; w < C::NWS; ++w) v += *reinterpret_cast<const f32x4*>(sums + (w * C::kOwners + o) * C::kSumRow + col);
      store(o0 + o, col, v);
    }
  }
}

// dH has the dh_grid workgroups from dh_from on (0, or all of dW's: the longer ones come first): n_split shares of the
// vocabulary (of `per_split` entries, a multiple of 32) side by side, fp32 partials for k_bwd_dh_reduce, or bf16 if there is
// one.  The others: dW.  CH, CW: their configurations.
template <class CH, class CW>
__global__ __launch_bounds__(CH::kThreads, CH::kLds > 81920 || CW::kLds > 81920 ? 1 : 2) void k_bwd_stream(
    StreamProblem p, int dh_from, int dh_grid, int n_split, int per_split, float* __restrict__ partial, __bf16* __restrict__ dH,
    float* __restrict__ dW) {
  static_assert(CH::kThreads == CW::kThreads, "one launch");
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int b = (int)blockIdx.x - dh_from;
  if (b >= 0 && b < dh_grid) {
    int sp, rt;                    // an XCD's workgroups share their parts of W
    if (!even_tile_of_block(b, n_split, (p.S + CH::kOwners - 1) / CH::kOwners, &sp, &rt)) return;
    const int begin = sp * per_split, end = begin + per_split < p.V ? begin + per_split : p.V;
    const float gamma = n_split == 1 ? gamma_of(p.n_valid, p.grad_loss) : 1.f;
    stream_tile<CH, false>(p, rt * CH::kOwners, begin, end, smem, [&](int s, int col, f32x4 v) {
      if (s >= p.S || col >= p.d) return;
      if (n_split > 1) {
        *reinterpret_cast<f32x4*>(partial + ((size_t)sp * p.S + s) * p.d + col) = v;
        return;
      }
      typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
      bf16x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = (__bf16)(gamma * v[e]);
      *reinterpret_cast<bf16x4*>(dH + (size_t)s * p.d + col) = o;
    });
    return;
  }
  int vt, one;
  if (!even_tile_of_block(b < 0 ? (int)blockIdx.x : b - dh_grid, (p.V + CW::kOwners - 1) / CW::kOwners, 1, &vt, &one)) return;
  const float gamma = gamma_of(p.n_valid, p.grad_loss);
  stream_tile<CW, true>(p, vt * CW::kOwners, 0, p.S, smem, [&](int v, int col, f32x4 x) {
    if (v < p.V && col < p.d) *reinterpret_cast<f32x4*>(dW + (size_t)v * p.d + col) = x * gamma;
  });
}

}  // namespace mst
