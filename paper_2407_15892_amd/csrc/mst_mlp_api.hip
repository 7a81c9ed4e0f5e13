// Host side of the mini-sequence MLP library: argument validation, the chunk
// schedule over the M mini-sequences (Algorithm 1 lines 1-5 and Algorithm 3
// lines 1-7 of the paper: partition, loop, concatenate / accumulate), workspace
// carving, launches, and the optional per-kernel event timing.
#include "../../include/mst_mlp.h"
#include "host_util.hpp"
#include "launch_model.hpp"
#include "mst_mlp_kernels.hpp"

#include <cmath>
#include <mutex>
#include <type_traits>

namespace {

using namespace mst;
using mst_host::misaligned;

struct Plan {
  int64_t S, d, I;
  int M;
  int C;            // rows per chunk = ceil(S / M)
  size_t slot;      // bytes of one chunk-sized bf16 [C, I] buffer
};

mst_status make_plan(int64_t S, int64_t d, int64_t I, int32_t M, Plan* p) {
  if (S <= 0 || d <= 0 || I <= 0) return MST_ERR_BAD_SHAPE;
  if (d % 8 != 0 || I % 8 != 0) return MST_ERR_BAD_SHAPE;
  if (M < 1 || (int64_t)M > S) return MST_ERR_BAD_M;
  if (I * d >= (int64_t(1) << 31) || d >= (int64_t(1) << 22) || I >= (int64_t(1) << 22)) return MST_ERR_BAD_SHAPE;
  const int64_t C = (S + M - 1) / M;
  if (C * I >= (int64_t(1) << 30) || C * d >= (int64_t(1) << 30)) return MST_ERR_BAD_SHAPE;
  p->S = S; p->d = d; p->I = I; p->M = M;
  p->C = (int)C;
  p->slot = mst_host::align_up((size_t)C * I * 2, 256);
  return MST_OK;
}

mst_host::Profiler g_prof;
struct Scope : mst_host::Scope {
  Scope(hipStream_t s, int k) : mst_host::Scope(g_prof, s, k) {}
};

// The smaller tiles of gemm_small.hpp: 128 x 128 and 64 x 64 with several workgroups on a compute unit (80 and 40 KB of
// LDS: two and four), and both software-pipelined for launches that have a compute unit for every workgroup.
typedef CfgSmall<4, 4, 3, 2, false> Tile128;
typedef CfgSmall<4, 4, 4, 4, true> Tile128Lone;      // Tile64, Tile64Lone: mst_small_kernels.hpp
typedef CfgSmall<2, 2, 5, 5, true, 128> Tile64Long;  // K steps of 128: half as many barriers in a long contraction
typedef CfgSmall<1, 1, 5, 5, true, 128> Tile32;      // 32 x 32, for products of a few 64 x 64 tiles

template <class C, class Set>
void set_small_attributes(Set set) {
  set((const void*)k_mlp_gateup_small<C, false>);
  set((const void*)k_mlp_gateup_small<C, true>);
  set((const void*)k_mlp_gemm_nt_small<C, false>);
  set((const void*)k_mlp_gemm_nn_small<C, false>);
}

template <class T, class Set>
void set_dx_dw3_attributes(Set set) {
  set((const void*)k_mlp_dx_dw3<false, false, T>);
  set((const void*)k_mlp_dx_dw3<true, false, T>);
  set((const void*)k_mlp_dx_dw3<false, true, T>);
  set((const void*)k_mlp_dx_dw3<true, true, T>);
}

mst_host::PerDeviceOnce g_attr_once;
bool set_kernel_attributes() {   // on the current device
  bool ok = true;
  auto set = [&ok](const void* f) {
    if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes) != hipSuccess) ok = false;
  };
  set((const void*)k_mlp_gateup<Tile16, false, false>);
  set((const void*)k_mlp_gateup<Tile16, false, true>);
  set((const void*)k_mlp_gateup<Tile16, true, false>);
  set((const void*)k_mlp_gateup<Tile16, true, true>);
  set((const void*)k_mlp_gateup<Tile16Half, false, false>);
  set((const void*)k_mlp_gateup<Tile16Half, true, false>);
  set((const void*)k_mlp_gemm_nt<Tile16, false>);
  set((const void*)k_mlp_gemm_nt<Tile16, true>);
  set((const void*)k_mlp_gemm_nt<Tile16Half, false>);
  set_small_attributes<Tile128>(set);
  set_small_attributes<Tile128Lone>(set);
  set_small_attributes<Tile64>(set);
  set_small_attributes<Tile64Lone>(set);
  set_small_attributes<Tile64Long>(set);
  set((const void*)k_mlp_gemm_nt_small<Tile32, false>);
  set((const void*)k_mlp_gemm_nt_small<Tile64Lone, true>);
  set((const void*)k_mlp_gemm_nn_small<Tile32, false>);
  set((const void*)k_mlp_gemm_nn_small<Tile64Lone, true>);
  set((const void*)k_mlp_gateup_small<Tile64Lone, true, true>);
  set((const void*)k_mlp_dx_dw3_small<Tile64Lone, Tile64Lone, false>);
  set((const void*)k_mlp_dx_dw3_small<Tile64Lone, Tile64Lone, true>);
  set((const void*)k_mlp_dx_dw3_small<Tile32, Tile64Lone, false>);
  set((const void*)k_mlp_gemm_nn<Tile16, false>);
  set((const void*)k_mlp_gemm_nn<Tile16, true>);
  set((const void*)k_mlp_dw3_small<Tile64>);
  set((const void*)k_mlp_dw3_small<Tile64Lone>);
  set((const void*)k_mlp_dw3<false, false>);
  set((const void*)k_mlp_dw3<true, false>);
  set((const void*)k_mlp_dw3<false, true>);
  set((const void*)k_mlp_dw3<true, true>);
  set_dx_dw3_attributes<Tile16>(set);
  set_dx_dw3_attributes<Tile16Half>(set);
  set_dx_dw3_attributes<Tile16Quarter>(set);
  return ok;
}

mst_status check_launch() { return hipGetLastError() == hipSuccess ? MST_OK : MST_ERR_LAUNCH; }

mst_status prepare_device() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return MST_ERR_NO_DEVICE;
  if (!g_attr_once.run(dev, set_kernel_attributes)) {
    (void)hipGetLastError();
    return MST_ERR_LAUNCH;
  }
  return MST_OK;
}

bool overlap(const void* a, size_t na, const void* b, size_t nb) {
  const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
  return x < y + nb && y < x + na;
}

// The forward's next launch pair: `rows` rows from the first of the `left` on, and where their A goes.  Rows are independent
// (O has the same bits for every grouping), so a pair of launches takes as many rows as there is memory for their A: in the
// workspace, where a caller hands in more than the forward needs (a training step's one workspace has the backward's three
// chunks), or in the rows of O behind the group, which nobody has written yet, where that makes fewer groups.  One chunk of a
// small block is far from a round of tiles, and a launch takes 4 us whatever it does.  Chunk by chunk -> this: step of 512
// rows, d = 256, I = 896, M = 2: 41.4 us -> 33.9; of 5003, d = 1544, I = 5384, M = 3: 1214 -> 1135; forward alone of 31999,
// d = 416, I = 1160, M = 77: 819 -> 286.  Of 120 calls with two or more chunks, d = 256 to 3840: 0.35 to 1.0, the steps 0.89
// in the mean, the forwards alone 0.83.
struct ForwardGroup { int64_t rows; bool in_output; };
ForwardGroup forward_group(const Plan& p, int64_t left, size_t workspace_bytes, bool output_is_free) {
  const int64_t most = std::min(((int64_t(1) << 30) - 1) / p.I, ((int64_t(1) << 30) - 1) / p.d);   // 32-bit offsets
  const int64_t room = std::min((int64_t)(workspace_bytes / (2 * (size_t)p.I)), most);             // >= C
  if (left <= room) return {left, false};
  auto groups = [room](int64_t rows) { return (rows + room - 1) / room; };
  const int64_t behind = output_is_free ? std::min(left * p.d / (p.I + p.d), most) : 0;            // behind * I <= (left - behind) * d
  if (1 + groups(left - behind) < groups(left)) return {behind, true};
  return {(left + groups(left) - 1) / groups(left), false};                                        // what is left in equal groups
}

// The backward's groups of rows, likewise: of dG, dU and A of a group, up to three are kept in the rows of dX behind it, and
// the workspace then holds those of one and a half times or three times the rows of a chunk.  The groups are the order in which
// the weight gradients are summed, so they depend on the shape alone: of a larger workspace only what the call needs is used.
// The largest group is kept as small as the number of groups allows; without fewer groups than chunks they are the chunks.  Backward, us, chunk
// by chunk -> this: 22592 rows, d = 616, I = 1560, M = 37: 1436 -> 1044; 32128, 640, 2264, 50: 2381 -> 1678; 20288, 1760, 5776, 12:
// 3750 -> 3496.  Groups as large as fit, where that makes no fewer of them: 8128, 1376, 3760, 4: 788 -> 820.
struct BackwardGroups {
  const Plan& p;
  int64_t room[4];                // rows whose dG, dU and A fit with k of them in dX: of the workspace (a chunk with none)
  int64_t cap;                    // most rows of a group
  bool in_dx;
  BackwardGroups(const Plan& plan, bool dx_is_free) : p(plan), in_dx(false) {
    const int64_t most = std::min(((int64_t(1) << 30) - 1) / p.I, ((int64_t(1) << 30) - 1) / p.d);        // 32-bit offsets
    room[0] = cap = p.C;
    for (int k = 1; k < 3; ++k) room[k] = std::min((int64_t)(slot(k) / (2 * (size_t)p.I)), most);
    room[3] = most;
    const int64_t n = (p.S + p.C - 1) / p.C;
    if (n < 4 || !dx_is_free) return;
    in_dx = true;
    cap = most;
    const int64_t fewest = count();
    if (fewest >= n) {
      in_dx = false;
      cap = p.C;
      return;
    }
    int64_t low = (p.S + fewest - 1) / fewest - 1, high = 0;
    for (int k = 0; k <= 3; ++k) high = std::max(high, fits(p.S, k));      // the largest group there can be
    while (high - low > 32) {     // the smallest cap with which there are no more of them
      cap = (low + high) / 2;
      (count() > fewest ? low : high) = cap;
    }
    cap = high;
  }
  size_t slot(int k) const { return 3 * p.slot / (size_t)(3 - k) / 256 * 256; }   // a buffer's share of the workspace
  int64_t fits(int64_t left, int k) const { return k ? std::min(room[k], left * p.d / (k * p.I + p.d)) : room[0]; }   // k rows I <= (left - rows) d
  int64_t next(int64_t left, int* k) const {            // rows of the next group; how many of its buffers are in dX
    const int64_t most = std::min(left, cap);
    *k = 0;
    for (int j = 1; j <= 3 && in_dx && fits(left, *k) < most; ++j)
      if (fits(left, j) > fits(left, *k)) *k = j;
    return std::min(most, fits(left, *k));
  }
  int64_t count() const {
    int64_t n = 0;
    int k;
    for (int64_t left = p.S; left > 0; ++n) left -= next(left, &k);
    return n;
  }
};

// Which block tile a GEMM of n_a x n_b outputs (A side: weights, B side: tokens) and `ksteps` K steps of 64 runs with.
// The figures are microseconds fitted to launches of the three kinds (gate/up, down, dA/dX) at 64 to 3000 tokens,
// d = 256 to 4096, I = 896 to 14336; they only have to rank the tiles, and every tile gives the same bits:
//   256 x 256      1.25 per K step (1.4 with K-strided weights) + 7 (first loads, epilogue), in whole rounds of kNumCu
//   128 x 128      1.0 per K step + 4 for two workgroups on a compute unit; further rounds overlap.  3000 tokens,
//                  d = 768, I = 2304: dA 17 us (432 tiles) against 26 (108 of 256)
//   128 x 128 lone 0.55 per K step + 3.2, up to kNumCu tiles.  1024 tokens, d = 4096, I = 14336: down 140 us (256 tiles)
//                  against 308 (64 tiles of 256), dX 266 against 607
//   128 x 256      0.68 per K step + 5, one round: between the 128 x 128 tiles that need two on a compute unit and the large
//                  ones that leave half of them idle.  Gate/up of 200 tokens, d = 4096, I = 14336: 65 us (448 tiles of
//                  128 x 128) -> 60 (224), down of 1300 tokens of it 182 -> 137; with two rounds slower than large tiles,
//                  with K-strided weights as fast as 128 x 128.  Behind full rounds of large tiles: forward of 1024 tokens,
//                  I = 11008: 265 us -> 253
//                  The estimates favour 128 x 128 too much: up to 1.12 of theirs (gate/up; down 1.02) 128 x 256 is taken.  24 and
//                  9 shapes between 1 and that: forward calls 0.84 to 1.02, 0.93 in the mean (231 tokens, d = 3304, I = 8400:
//                  96 us -> 81) and 0.86 to 1.02, 0.93; beyond it 0.96 to 1.10 (gate/up, 1.0 in the mean), 0.86 to 1.07 (down)
//   64 x 64        0.45 (few workgroups on a compute unit) to 0.85 (four) per K step + 2.5.  1536 tokens, d = 1536,
//                  I = 4608: down 38 us (576 tiles) against 79 (36 of 256).  Too low behind large tiles: gate/up of 1668
//                  tokens below is taken at 16.6, a trace has 20.9 (182 lone 128 x 128 tiles would be 17.0 by their line)
//   64 x 64 lone   0.24 per K step + 2.5.  256 tokens, d = 256, I = 896: down 5.5 against 18; 200 tokens, d = 4096,
//                  I = 14336: down 63 against 250 (16 tiles of 256), dX 129 against 523
//   64 x 64 long   the same with K steps of 128, 0.22 per 64 + 3.5, for one workgroup per compute unit: the down of 200
//                  tokens 53, of 512 tokens (d = 2048, I = 5632) 21.6 against 22.5; slower at fewer than 64 K steps
//   32 x 32        0.11 per 64 (0.17 with K-strided weights) + 3 where there are few 64 x 64 tiles (more than 128, or 64
//                  K-strided, move too much through L2 for this): half of the LDS traffic and a quarter of the MFMAs per K
//                  step, on four times the compute units.  Forward of 64 tokens, d = 2048, I = 6000: 33 us -> 22, of 500, d = 640, I = 1800:
//                  18.9 -> 15; backward of 178 tokens, d = 520, I = 1456: 35 -> 30.  Not for gate/up (pairs of row tiles),
//                  and not for three rows of them (65 to 96 tokens) that are more than a round and more than 60000 K steps
//                  in all: 39 forward calls there, d = 3200 to 4096, took 0.96 to 1.10 of their time with 64 x 64 tiles, 1.06
//                  in the mean; 52 below that line 0.83 to 1.06, 0.98; 97 to 128 tokens 0.88 to 1.07, 0.97
// Where the large tiles end in a partly filled round, whole columns of them may make up the full rounds and a second
// launch the rest with smaller tiles: gate/up of 1668 tokens, d = 1544, I = 5384 (301 large tiles) as 252 large and 675 of
// 64 x 64: step of 5003 tokens 1.31 -> 1.23 ms; dA of 4096 tokens, I = 14336 (896 tiles) as 768 large and 512 of
// 128 x 128: 376 us against 412.  With all compute units busy a K step takes 1.36, with the K-strided weights of dA and
// dX 1.4 also where some are idle; not split, by this, are the 1376 tiles of gate/up at I = 11008 (2 % slower split).
enum TileKind { kBig, k128, k128Lone, k64, k64Lone, k64Long, k32, kHalf };   // MST_MLP_TILE_* of the header, in this order
struct TileChoice {
  TileKind kind;      // of the whole, or of what follows the first `head` columns
  int64_t head;       // A-side extent, a multiple of 256, that large tiles cover in a launch of its own (0: none)
  double us;          // of the tile that the ranking is about: of 128 x 128 where 128 x 256 is taken in its place
};
enum Weights { kGateUp, kContiguous, kStrided };                 // gate/up, down, dA and dX
double half_us(double k) { return 0.68 * k + 5.0; }                // a round of 128 x 256 tiles
TileChoice choose_whole(int64_t n_a, int64_t n_b, int64_t ksteps, Weights w) {
  const bool strided = w == kStrided;
  const double k = (double)ksteps;
  TileChoice best = {kBig, 0, std::ceil(tiles_of(n_a, n_b, 256) / kNumCu) * ((strided ? 1.4 : 1.25) * k + 7.0)};
  auto consider = [&](TileKind kind, double t) {
    if (t < best.us) best = {kind, 0, t};
  };
  const double x = tiles_of(n_a, n_b, 128) / (2.0 * kNumCu), y = tiles_of(n_a, n_b, 64) / (4.0 * kNumCu);
  if (x <= 0.5) consider(k128Lone, 0.55 * k + 3.2);
  else consider(k128, (x >= 1.5 ? x : x > 1.0 ? 1.5 : 0.3 + 0.7 * x) * (k + 4.0));
  consider(k64, (y > 1.0 ? 0.85 * y : y > 0.25 ? 0.3 + 0.4 * y : 0.45) * k + 2.5);
  if (y <= 0.25 && ksteps >= 64) consider(k64Long, 0.22 * k + 3.5);
  if (!strided && std::ceil((double)n_a / 128.0) * std::ceil((double)n_b / 256.0) <= kNumCu) {
    const double t = half_us(k);
    if (best.kind == k128 && t <= (w == kGateUp ? 1.12 : 1.02) * best.us) best.kind = kHalf;
    consider(kHalf, t);
  }
  const double n32 = tiles_of(n_a, n_b, 32);
  const bool thin = n_b > 64 && n_b <= 96 && n32 > kNumCu && n32 * k >= 60000.0;
  if (w != kGateUp && !thin && tiles_of(n_a, n_b, 64) <= (strided ? 64.0 : 128.0)) consider(k32, (strided ? 0.17 : 0.11) * k + 3.0);
  if (y <= 0.5) consider(k64Lone, 0.24 * (y > 0.25 ? 4.0 * y : 1.0) * k + 2.5);
  return best;
}
TileChoice choose_tile(int64_t n_a, int64_t n_b, int64_t ksteps, Weights w) {
  const TileChoice whole = choose_whole(n_a, n_b, ksteps, w);
  const int64_t t_a = (n_a + kTile - 1) / kTile, t_b = (n_b + kTile - 1) / kTile;
  const int64_t full = t_a * t_b / kNumCu * kNumCu, cols = full / t_b;       // full rounds; columns of tiles in them
  if (cols == 0 || cols == t_a) return whole;
  const TileChoice rest = choose_whole(n_a - cols * kTile, n_b, ksteps, w);
  const double t = (double)(full / kNumCu) * ((w == kStrided ? 1.4 : 1.36) * (double)ksteps + 7.0) + rest.us + 2.0;
  const double below = rest.kind == kHalf && rest.us >= half_us((double)ksteps) ? 0.97 : 1.0;   // at 0.98 to 1 they took 0.99 to 1.04
  return rest.kind != kBig && t < below * whole.us ? TileChoice{rest.kind, cols * kTile, t} : whole;
}

// the choices of the four products of a chunk of `rows` rows
int64_t ksteps_of(int64_t k) { return (k + kBK - 1) / kBK; }
TileChoice gateup_tile(int64_t rows, int64_t d, int64_t I) { return choose_tile(2 * I, rows, ksteps_of(d), kGateUp); }
// Lone 64 x 64 tiles load rows that are not whole cache lines line by line (PanelKC16Lines), the other tiles fetch their lines
// twice.  Down of 800 rows, d = 2048: 45 us at I = 7168, at 7176 66 -> 45; 507 rows, d = 2688, I = 7120: 64 -> 45.  With that they
// are faster than 128 x 128 tiles in a long contraction that has a few more of those than compute units.  Forwards timed with
// both: 80 of up to 1144 tiles of 64 x 64 took 0.77 to 1.02 of their time, 0.90 in the mean (1421 rows, d = 2752, I = 6952: 220 us
// -> 176), 26 of 1887 to 2040 1.04 to 1.24 (2400, 3216, 9248: 396 -> 450), and there is nothing between: up to five rounds.  Where
// rows begin on a line or half way into one (K % 64 == 32) half as much is to gain: 8 of up to four rounds 0.88 to 0.99, 11 of more
// 0.99 to 1.07, 1.03 in the mean.
// With K steps of 128, which straddle half as many lines, the panels gained
// nothing (64 x 64: 62 us either way) or lost (32 x 32: 10.1 us -> 13.1, one stage less ahead), in larger tiles there is no
// stage of LDS left for them.  Forward of 38 shapes, d = 320 to 3072: 0.77 to 0.95 with more tiles than compute units; with
// fewer, where a stage less ahead costs as much as the lines, 0.96 to 1.06, so not there.
// The same for the rows of dG, dU and dO in dX's and dA's lone 64 x 64 tiles: 33 backward calls with dX beside small tiles of the
// weight gradients 0.94 to 1.06 of their time, 0.97 in the mean; 793 rows, d = 1336, I = 3368, dX alone: 151 us -> 142.
bool whole_lines(int64_t K) { return K % 64 == 0; }
bool by_lines(int64_t tiles, int64_t K, const void* p, const void* q) {
  return tiles > kNumCu && (!whole_lines(K) || misaligned(p, 128) || misaligned(q, 128));
}
TileChoice nt_tile(int64_t rows, int64_t N, int64_t K) {
  TileChoice c = choose_tile(N, rows, ksteps_of(K), kContiguous);
  if (c.kind == k128 && c.head == 0 && !whole_lines(K) && ksteps_of(K) >= 60 &&
      tiles_of(N, rows, 64) <= (K % 64 == 32 ? 4.0 : 5.0) * kNumCu)
    c.kind = k64Lone;
  return c;
}
TileChoice nn_tile(int64_t rows, int64_t N, int64_t K, int terms) { return choose_tile(N, rows, terms * ksteps_of(K), kStrided); }

// The weight gradients have one tile kind for all groups of rows: what the large tiles keep between them is not row-major.
struct DwChoice { bool small, lone, even; };
DwChoice dw_choice(int64_t C, int64_t d, int64_t I) {
  const double tiles64 = 3.0 * tiles_of(I, d, 64), ksteps = (double)ksteps_of(C);
  const int n_it = (int)((I + kTile - 1) / kTile), n_dt = (int)((d + kTile - 1) / kTile);
  auto share = [&](bool even) { return 2 * xcd_share(n_it, n_dt, even) + xcd_share(n_dt, n_it, even); };
  DwChoice c;
  c.small = small_launch_us(tiles64, ksteps) < big_launch_us(3.0 * tiles_of(I, d, 256), ksteps);
  c.lone = lone_small(tiles64);
  c.even = c.small || uneven_over_xcds(n_it) || uneven_over_xcds(n_dt) || saves_a_round(share(false), share(true));
  return c;
}

TileKind dw_tile(const DwChoice& c) { return c.small ? (c.lone ? k64Lone : k64) : kBig; }

// dA computed by gate/up's backward launch: where both are one short tile deep, a launch less is worth more than the
// second contraction in it.  Up to 16 K steps: backward of 256 tokens, d = 256, I = 896: 22.4 -> 19.6 us; of 256, d = 1024,
// I = 2816: 46.7 -> 45.2; from 24 on nothing (100 tokens, d = 1536) to 3 % slower (64, d = 4096).
bool fuse_da(int64_t rows, int64_t d, int64_t I) {
  const TileChoice c = gateup_tile(rows, d, I);
  return c.kind == k64Lone && c.head == 0 && ksteps_of(d) <= 16;
}

// Whether dX shares the launch of the chunk's weight gradients, and with which tile (MST_MLP_DX_* of the header).
//
// Small tiles: both in one launch of lone 64 x 64 tiles, dX in 32 x 32 ones where few (72 in a shared launch; 78 take as
// long either way).  Over 47 shapes of 64 to 8000 rows, d = 152 to 768, the backward call took 0.67 to 1.00 of its time with
// two launches (256 rows, d = 256, I = 896: 22.4 -> 16.2 us; 300, d = 656, I = 2000: 46 -> 37).
//
// Large tiles: a K step of a half tile takes 0.8 us, 0.9 with all compute units busy; K-strided weights as at choose_whole.
// Over twenty shapes of 200 to 4096 rows, d = 1024 to 4096, one and two chunks, both ways timed: the backward call took
// 0.87 to 1.01 of its time with two launches, 0.96 in the mean, and nowhere was the other tile more than 1.5 % faster.
// kShared: a shared launch must be this much cheaper (what is left alone, 4096 rows, d = 4096: both take the same).
// A later chunk keeps two launches where one row of large tiles holds it and its 64 x 64 tiles of dX fit a round: the weight
// gradients are bound by the sums that they read and write again, dX's K steps take 1.0 to 1.25 us beside them and not 0.8,
// and they are the end of the launch.  212 steps of 2 to 5 chunks of up to 256 rows, d = 1800 to 4096, took 0.98 to 1.20 of
// their time with two launches, 1.03 in the mean (4 x 244 rows, d = 4096, I = 14336: 2.49 ms, 2.65 with one); 67 with d
// above 4096 0.93 to 1.13, 0.99.
// 128 x 128 tiles of dX (Tile16Quarter): a K step takes 0.58 beside the weight gradients, so its contraction over 2 I, which no
// other workgroup can help with, ends sooner than in a half tile, for 1.4 times its compute unit time.  Backward of 3 chunks of
// 888 rows, d = 1776, I = 6936: 869 us -> 708; of 707 rows, d = 1504, I = 5208: 182 -> 142.  70 backward calls of 1 to 3 chunks
// of 100 to 7000 rows, d = 792 to 4016, each timed with every kind: 0.953 of their time without this one in the mean, 0.77 to
// 1.02, and 0.6 % behind the fastest kind.  kQuarter: its estimate is a tenth too high.  Those had I = 2.5 to 4 d; not taken
// below 2 d, where the contraction is no longer than the weight gradients' tiles.  kQuarterBusy: of 1100 rows on that is so only
// where the launch waits for the chain, not where it has nearly as much work as all compute units can do in that time: of 180
// calls of 1 to 7 chunks 18 keep their other tile for this, which took 0.94 to 1.09 of their time with quarter tiles, 1.02 in the
// mean (16999 rows, d = 1336, I = 4848, M = 7: 2072 us, 2252 with them); the others took 0.92 in the mean.  kQuarterLater: nor
// for later chunks that wait for the chain and whose dX would have a launch of its own: 14 that this turns back took 0.96 to 1.06
// of their time with quarter tiles, 1.02 in the mean (1390, 1976, 7736, 5: 1016 us, 1073), 50 others 0.71 to 1.03, 0.91.  200 more
// calls that take quarter tiles by all this: 0.91 in the mean, eleven of them 1.02 to 1.08.
constexpr double kShared = 0.98, kQuarter = 0.9, kQuarterBusy = 0.96, kQuarterLater = 0.97;
enum DxKind { kDxOwn, kDxWhole, kDxHalf, kDx64, kDx32, kDxQuarter };
DxKind choose_dx(int64_t rows, int64_t d, int64_t I, bool accumulate, const DwChoice& dw) {
  if (dw.small) {
    const TileChoice own = nn_tile(rows, d, I, 2);
    if (own.kind < k64 || own.head) return kDxOwn;
    return tiles_of(d, rows, 64) <= 72.0 ? kDx32 : kDx64;
  }
  if (accumulate && rows <= kTile && tiles_of(d, kTile, 64) <= kNumCu) return kDxOwn;
  auto tiles = [&](int64_t a, int64_t b, int64_t e, int64_t f = kTile) { return (a + e - 1) / e * ((b + f - 1) / f); };
  const int64_t n_dw = 2 * tiles(I, d, kTile) + tiles(d, I, kTile);
  const TileCost c = dw_cost(rows, accumulate);
  const double bytes = (accumulate ? 24.0 : 12.0) * (double)(I * d), ksteps = 2.0 * (double)ksteps_of(I);
  const double own = kShared * (nn_tile(rows, d, I, 2).us + 2.0 + launch_us(n_dw, c, bytes));
  const double whole = launch_us(tiles(d, rows, kTile), TileCost{ksteps, 7.0, 1.4, 1.5}, n_dw, c, bytes);
  const double half = launch_us(tiles(d, rows, Tile16Half::EA), TileCost{ksteps, 7.0, 0.8, 0.9}, n_dw, c, bytes);
  const int64_t n_q = tiles(d, rows, Tile16Quarter::EA, Tile16Quarter::EB);
  const TileCost c_q = {ksteps, 7.0, 0.58, 0.65};
  double quarter = launch_us(n_q, c_q, n_dw, c, bytes);
  const bool busy = quarter <= 1.2 * ((double)n_q * c_q.busy() + (double)n_dw * c.busy()) / kNumCu;
  quarter *= busy && rows >= 1100 ? kQuarterBusy : !busy && accumulate && own < std::min(whole, half) ? kQuarterLater : kQuarter;
  const double best = std::min(whole, I >= 2 * d ? std::min(half, quarter) : half);
  if (best > own) return kDxOwn;
  return best == whole ? kDxWhole : best == half ? kDxHalf : kDxQuarter;
}
int dx_tile(DxKind dx) { return dx == kDxQuarter ? kDxHalf : dx; }       // MST_MLP_DX_* of the header
int dx_tile_rows(DxKind dx) {
  switch (dx) {
    case kDxWhole: case kDxHalf: return kTile;
    case kDxQuarter: return Tile16Quarter::EB;
    case kDx64: return Tile64Lone::EB;
    case kDx32: return Tile32::EB;
    default: return 0;
  }
}
template <class T>
void launch_dx_dw3(hipStream_t st, DxProblem x, const DwProblems& ps, int rows, bool even, bool accumulate, int more) {
  x.n_jt = (x.d + T::EA - 1) / T::EA;
  x.n_st = (rows + T::EB - 1) / T::EB;
  x.grid = even_grid(x.n_jt, x.n_st);
  const auto kernel = even ? (accumulate ? k_mlp_dx_dw3<false, true, T> : k_mlp_dx_dw3<true, true, T>)
                           : (accumulate ? k_mlp_dx_dw3<false, false, T> : k_mlp_dx_dw3<true, false, T>);
  hipLaunchKernelGGL(kernel, dim3(x.grid + ps.p[0].grid + ps.p[1].grid + ps.p[2].grid), dim3(kThreads), kLdsBytes, st,
                     x, ps, rows, more);
}

template <class CX>
void launch_dx_dw3_small(hipStream_t st, DxProblem x, const DwProblems& ps, int rows, int accumulate) {
  typedef Tile64Lone CW;
  x.n_jt = (x.d + CX::EA - 1) / CX::EA;
  x.n_st = (rows + CX::EB - 1) / CX::EB;
  x.grid = even_grid(x.n_jt, x.n_st);
  const int dw_grid = ps.p[0].grid + ps.p[1].grid + ps.p[2].grid;
  // The longer tiles first, where not all workgroups are resident at once (two per compute unit): behind dX the weight
  // gradients' are dealt out as slots come free, two to one unit while others idle.  dX first, 57 steps with more than 512
  // tiles of dX and 129 to 256 of the weight gradients took 1.06 of their time with two launches in the mean, up to 1.21 (9764
  // rows, d = 256, I = 816: 114 us -> 137); with the longer first 38 with more than 512 of dX took 0.89 to 0.99, 0.93.
  const bool dw_first = 2 * ksteps_of(x.I) < ksteps_of(rows) && x.grid + dw_grid > 2 * kNumCu;
  constexpr bool kCan = std::is_same_v<CX, Tile64Lone>;
  const bool lines = kCan && by_lines(x.grid + dw_grid, x.I, x.dG, x.dU);
  hipLaunchKernelGGL((lines ? k_mlp_dx_dw3_small<CX, CW, kCan> : k_mlp_dx_dw3_small<CX, CW, false>), dim3(x.grid + dw_grid), dim3(CW::kThreads),
                     CX::kLds > CW::kLds ? CX::kLds : CW::kLds, st, x, ps, rows, accumulate, dw_first ? dw_grid : 0);
}

// A = silu(X Wg^T) * (X Wu^T) of a chunk, or its backward (dA given)
template <class C, bool kBackward, bool kDa = false>
void launch_gateup_small(hipStream_t st, const __bf16* X, const __bf16* Wg, const __bf16* Wu, int rows, int d, int n_i, int ldi,
                         __bf16* A, __bf16* dAG, __bf16* dU, DaProblem da = DaProblem{}) {
  const int n_it = (n_i + C::EA / 2 - 1) / (C::EA / 2), n_st = (rows + C::EB - 1) / C::EB;
  hipLaunchKernelGGL((k_mlp_gateup_small<C, kBackward, kDa>), dim3(even_grid(n_it, n_st)), dim3(C::kThreads), C::kLds, st,
                     X, Wg, Wu, rows, d, n_i, ldi, n_st, n_it, A, dAG, dU, da);
}
template <bool kBackward>
void launch_gateup(hipStream_t st, const __bf16* X, const __bf16* Wg, const __bf16* Wu, int rows, int d, int I,
                   __bf16* A, __bf16* dAG, __bf16* dU) {
  const TileChoice c = gateup_tile(rows, d, I);
  const int i0 = (int)(c.head / 2), n_i = I - i0;               // the second launch's indices
  auto large = [&](auto tile, auto super, int i_first, int n) {
    typedef decltype(tile) T;
    const int n_it = (n + T::EA / 2 - 1) / (T::EA / 2), n_st = (rows + T::EB - 1) / T::EB;
    const size_t w = (size_t)i_first * d;
    hipLaunchKernelGGL((k_mlp_gateup<T, kBackward, decltype(super)::value>), dim3(decltype(super)::value ? mlp_grid(n_it, n_st) : even_grid(n_it, n_st)),
                       dim3(kThreads), kLdsBytes, st, X, Wg + w, Wu + w, rows, d, n, I, n_st, n_it,
                       A + i_first, kBackward ? dAG + i_first : nullptr, kBackward ? dU + i_first : nullptr);
  };
  if (c.kind == kBig || i0) {
    const int n = i0 ? i0 : I;
    if (use_super_tiles((n + kGateUpI - 1) / kGateUpI, (rows + kTile - 1) / kTile)) large(Tile16{}, std::true_type{}, 0, n);
    else large(Tile16{}, std::false_type{}, 0, n);
  }
  if (c.kind == kHalf) return large(Tile16Half{}, std::false_type{}, i0, n_i);
  Wg += (size_t)i0 * d;
  Wu += (size_t)i0 * d;
  A += i0;
  if (kBackward) { dAG += i0; dU += i0; }
  switch (c.kind) {
    case k128: return launch_gateup_small<Tile128, kBackward>(st, X, Wg, Wu, rows, d, n_i, I, A, dAG, dU);
    case k128Lone: return launch_gateup_small<Tile128Lone, kBackward>(st, X, Wg, Wu, rows, d, n_i, I, A, dAG, dU);
    case k64: return launch_gateup_small<Tile64, kBackward>(st, X, Wg, Wu, rows, d, n_i, I, A, dAG, dU);
    case k64Lone: return launch_gateup_small<Tile64Lone, kBackward>(st, X, Wg, Wu, rows, d, n_i, I, A, dAG, dU);
    case k64Long: return launch_gateup_small<Tile64Long, kBackward>(st, X, Wg, Wu, rows, d, n_i, I, A, dAG, dU);
    default: return;
  }
}

// out[rows][N] = P Q^T, P [rows][K], Q [N][K]
template <class C>
void launch_nt_small(hipStream_t st, const __bf16* P, const __bf16* Q, int rows, int N, int K, __bf16* out, int ldo) {
  const int n_nt = (N + C::EA - 1) / C::EA, n_st = (rows + C::EB - 1) / C::EB;
  constexpr bool kCan = std::is_same_v<C, Tile64Lone>;
  const bool lines = kCan && by_lines(n_nt * n_st, K, P, Q);
  hipLaunchKernelGGL((lines ? k_mlp_gemm_nt_small<C, kCan> : k_mlp_gemm_nt_small<C, false>), dim3(even_grid(n_nt, n_st)), dim3(C::kThreads),
                     C::kLds, st, P, K, Q, K, rows, N, K, n_st, n_nt, out, ldo);
}
void launch_nt(hipStream_t st, const __bf16* P, const __bf16* Q, int rows, int N, int K, __bf16* out) {
  const TileChoice c = nt_tile(rows, N, K);
  const int n0 = (int)c.head;
  if (c.kind == kBig || n0) {
    const int n_nt = ((n0 ? n0 : N) + kTile - 1) / kTile, n_st = (rows + kTile - 1) / kTile;
    hipLaunchKernelGGL((use_super_tiles(n_nt, n_st) ? k_mlp_gemm_nt<Tile16, true> : k_mlp_gemm_nt<Tile16, false>), dim3(mlp_grid(n_nt, n_st)), dim3(kThreads), kLdsBytes, st,
                       P, K, Q, K, rows, N, K, n_st, n_nt, out, N);
  }
  Q += (size_t)n0 * K;
  out += n0;
  switch (c.kind) {
    case kHalf: {
      const int n_nt = (N - n0 + Tile16Half::EA - 1) / Tile16Half::EA, n_st = (rows + Tile16Half::EB - 1) / Tile16Half::EB;
      hipLaunchKernelGGL((k_mlp_gemm_nt<Tile16Half, false>), dim3(even_grid(n_nt, n_st)), dim3(kThreads), kLdsBytes, st,
                         P, K, Q, K, rows, N - n0, K, n_st, n_nt, out, N);
      return;
    }
    case k128: return launch_nt_small<Tile128>(st, P, Q, rows, N - n0, K, out, N);
    case k128Lone: return launch_nt_small<Tile128Lone>(st, P, Q, rows, N - n0, K, out, N);
    case k64: return launch_nt_small<Tile64>(st, P, Q, rows, N - n0, K, out, N);
    case k64Lone: return launch_nt_small<Tile64Lone>(st, P, Q, rows, N - n0, K, out, N);
    case k64Long: return launch_nt_small<Tile64Long>(st, P, Q, rows, N - n0, K, out, N);
    case k32: return launch_nt_small<Tile32>(st, P, Q, rows, N - n0, K, out, N);
    default: return;
  }
}

// out[rows][N] = P1 Q1 (+ P2 Q2), P: [rows][K], Q: [K][N]
template <class C>
void launch_nn_small(hipStream_t st, const __bf16* P1, const __bf16* Q1, const __bf16* P2, const __bf16* Q2,
                     int rows, int N, int K, int ldq, __bf16* out) {
  const int n_nt = (N + C::EA - 1) / C::EA, n_st = (rows + C::EB - 1) / C::EB;
  constexpr bool kCan = std::is_same_v<C, Tile64Lone>;
  const bool lines = kCan && by_lines(n_nt * n_st, K, P1, P2 ? P2 : P1);
  hipLaunchKernelGGL((lines ? k_mlp_gemm_nn_small<C, kCan> : k_mlp_gemm_nn_small<C, false>), dim3(even_grid(n_nt, n_st)), dim3(C::kThreads),
                     C::kLds, st, P1, Q1, P2, Q2, K, ldq, rows, N, K, n_st, n_nt, out, ldq);
}
void launch_nn(hipStream_t st, const __bf16* P1, const __bf16* Q1, const __bf16* P2, const __bf16* Q2,
               int rows, int N, int K, __bf16* out) {
  const TileChoice c = nn_tile(rows, N, K, P2 ? 2 : 1);
  const int n0 = (int)c.head;
  if (c.kind == kBig || n0) {
    const int n = n0 ? n0 : N, n_nt = (n + kTile - 1) / kTile, n_st = (rows + kTile - 1) / kTile;
    hipLaunchKernelGGL((use_super_tiles(n_nt, n_st) ? k_mlp_gemm_nn<Tile16, true> : k_mlp_gemm_nn<Tile16, false>), dim3(mlp_grid(n_nt, n_st)), dim3(kThreads), kLdsBytes, st,
                       P1, Q1, P2, Q2, K, N, rows, n, K, n_st, n_nt, out, N);
  }
  Q1 += n0;
  if (Q2) Q2 += n0;
  out += n0;
  switch (c.kind) {
    case k128: return launch_nn_small<Tile128>(st, P1, Q1, P2, Q2, rows, N - n0, K, N, out);
    case k128Lone: return launch_nn_small<Tile128Lone>(st, P1, Q1, P2, Q2, rows, N - n0, K, N, out);
    case k64: return launch_nn_small<Tile64>(st, P1, Q1, P2, Q2, rows, N - n0, K, N, out);
    case k64Lone: return launch_nn_small<Tile64Lone>(st, P1, Q1, P2, Q2, rows, N - n0, K, N, out);
    case k64Long: return launch_nn_small<Tile64Long>(st, P1, Q1, P2, Q2, rows, N - n0, K, N, out);
    case k32: return launch_nn_small<Tile32>(st, P1, Q1, P2, Q2, rows, N - n0, K, N, out);
    default: return;
  }
}

// tile: 256 or 64; even: dealt out evenly over the XCDs (always so with the small ones)
DwProblem dw_problem(const __bf16* G, int ldg, const __bf16* H, int ldh, int d, int V, float* dW, int tile, bool even) {
  DwProblem q;
  q.G = G; q.ldg = ldg; q.H = H; q.ldh = ldh; q.d = d; q.V = V;
  q.n_vt = (V + tile - 1) / tile;
  q.n_jt = (d + tile - 1) / tile;
  q.grid = launch_grid(even, q.n_vt, q.n_jt);
  q.dW = dW;
  return q;
}

}  // namespace

extern "C" {

const char* mst_mlp_version(void) { return "mst-mlp 0.1 (gfx950)"; }

int32_t mst_mlp_suggest_m(int64_t S, int64_t d, int64_t I) {
  if (S <= 0 || d <= 0 || I <= 0) return 0;
  int64_t m = (2 * S + d) / (2 * d);             // S / d to the nearest integer: chunk size C = d
  if (m < 1) m = 1;
  if (m > S) m = S;
  if (m > 0x7fffffff) m = 0x7fffffff;
  return (int32_t)m;
}

mst_status mst_mlp_workspace_bytes(int64_t S, int64_t d, int64_t I, int32_t M, size_t* fwd_bytes, size_t* bwd_bytes) {
  Plan p;
  mst_status s = make_plan(S, d, I, M, &p);
  if (s != MST_OK) return s;
  if (fwd_bytes) *fwd_bytes = p.slot;
  if (bwd_bytes) *bwd_bytes = 3 * p.slot;
  return MST_OK;
}

mst_status mst_mlp_fwd(const void* X, const void* Wg, const void* Wu, const void* Wd,
                       int64_t S, int64_t d, int64_t I, int32_t M,
                       void* workspace, size_t workspace_bytes, void* O, void* stream) {
  Plan p;
  mst_status s = make_plan(S, d, I, M, &p);
  if (s != MST_OK) return s;
  if (!X || !Wg || !Wu || !Wd || !O) return MST_ERR_NULL_POINTER;
  if (!workspace || workspace_bytes < p.slot) return MST_ERR_WORKSPACE;
  if (misaligned(X, 16) || misaligned(Wg, 16) || misaligned(Wu, 16) || misaligned(Wd, 16) || misaligned(O, 16) ||
      misaligned(workspace, 256))
    return MST_ERR_ALIGNMENT;
  if ((s = prepare_device()) != MST_OK) return s;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const __bf16* Xb = static_cast<const __bf16*>(X);
  const __bf16* Wgb = static_cast<const __bf16*>(Wg);
  const __bf16* Wub = static_cast<const __bf16*>(Wu);
  const __bf16* Wdb = static_cast<const __bf16*>(Wd);
  __bf16* Ob = static_cast<__bf16*>(O);
  const size_t x_bytes = (size_t)S * d * 2, w_bytes = (size_t)I * d * 2;
  const bool output_is_free = !overlap(O, x_bytes, X, x_bytes) && !overlap(O, x_bytes, Wg, w_bytes) &&
                              !overlap(O, x_bytes, Wu, w_bytes) && !overlap(O, x_bytes, Wd, w_bytes);
  // Algorithm 1: loop over groups of rows (whole or parts of mini-sequences); each lands in its row range of O (the concatenation
  // of line 5)
  for (int64_t r0 = 0; r0 < p.S;) {
    const ForwardGroup g = forward_group(p, p.S - r0, workspace_bytes, output_is_free);
    const int rows = (int)g.rows;
    __bf16* const A = g.in_output ? Ob + p.S * p.d - g.rows * p.I : static_cast<__bf16*>(workspace);
    {
      Scope sc(st, MST_MLP_K_GATEUP);
      launch_gateup<false>(st, Xb + r0 * p.d, Wgb, Wub, rows, (int)p.d, (int)p.I, A, nullptr, nullptr);
    }
    {
      Scope sc(st, MST_MLP_K_DOWN);
      launch_nt(st, A, Wdb, rows, (int)p.d, (int)p.I, Ob + r0 * p.d);
    }
    r0 += g.rows;
  }
  return check_launch();
}

mst_status mst_mlp_bwd(const void* X, const void* Wg, const void* Wu, const void* Wd, const void* dO,
                       int64_t S, int64_t d, int64_t I, int32_t M,
                       void* workspace, size_t workspace_bytes,
                       void* dX, float* dWg, float* dWu, float* dWd, void* stream) {
  Plan p;
  mst_status s = make_plan(S, d, I, M, &p);
  if (s != MST_OK) return s;
  if (!X || !Wg || !Wu || !Wd || !dO || !dX || !dWg || !dWu || !dWd) return MST_ERR_NULL_POINTER;
  if (!workspace || workspace_bytes < 3 * p.slot) return MST_ERR_WORKSPACE;
  if (misaligned(X, 16) || misaligned(Wg, 16) || misaligned(Wu, 16) || misaligned(Wd, 16) || misaligned(dO, 16) ||
      misaligned(dX, 16) || misaligned(dWg, 16) || misaligned(dWu, 16) || misaligned(dWd, 16) || misaligned(workspace, 256))
    return MST_ERR_ALIGNMENT;
  if ((s = prepare_device()) != MST_OK) return s;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const __bf16* Xb = static_cast<const __bf16*>(X);
  const __bf16* Wgb = static_cast<const __bf16*>(Wg);
  const __bf16* Wub = static_cast<const __bf16*>(Wu);
  const __bf16* Wdb = static_cast<const __bf16*>(Wd);
  const __bf16* dOb = static_cast<const __bf16*>(dO);
  __bf16* dXb = static_cast<__bf16*>(dX);
  char* ws = static_cast<char*>(workspace);
  const int dI = (int)p.I, dd = (int)p.d;
  const size_t x_bytes = (size_t)S * d * 2, w_bytes = (size_t)I * d * 2;
  const bool dx_is_free = !overlap(dX, x_bytes, X, x_bytes) && !overlap(dX, x_bytes, dO, x_bytes) && !overlap(dX, x_bytes, Wg, w_bytes) &&
                          !overlap(dX, x_bytes, Wu, w_bytes) && !overlap(dX, x_bytes, Wd, w_bytes);
  const BackwardGroups groups(p, dx_is_free);
  const DwChoice dw = dw_choice(std::min(groups.cap, p.S), p.d, p.I);

  // Algorithm 3: loop over groups of rows, likewise; their dX lands in its row range, the weight gradients accumulate
  for (int64_t r0 = 0; r0 < p.S;) {
    int in_dx = 0;
    const int rows = (int)groups.next(p.S - r0, &in_dx);
    __bf16* buf[3];                                             // dA, then dG in place; dU; A
    for (int k = 0; k < 3; ++k)
      buf[k] = k < in_dx ? dXb + p.S * p.d - (k + 1) * (int64_t)rows * p.I
                         : reinterpret_cast<__bf16*>(ws + (k - in_dx) * groups.slot(in_dx));
    __bf16 *const bufG = buf[0], *const bufU = buf[1], *const bufA = buf[2];
    const bool more = r0 + rows < p.S;
    const __bf16* Xc = Xb + r0 * p.d;
    const __bf16* dOc = dOb + r0 * p.d;
    const int acc = r0 > 0 ? 1 : 0;
    const bool da_in_gateup = fuse_da(rows, p.d, p.I);
    if (!da_in_gateup) {
      Scope sc(st, MST_MLP_K_DA);
      launch_nn(st, dOc, Wdb, nullptr, nullptr, rows, dI, dd, bufG);
    }
    {
      Scope sc(st, MST_MLP_K_GATEUP_BWD);
      if (da_in_gateup)
        launch_gateup_small<Tile64Lone, true, true>(st, Xc, Wgb, Wub, rows, dd, dI, dI, bufA, bufG, bufU, DaProblem{dOc, Wdb});
      else
        launch_gateup<true>(st, Xc, Wgb, Wub, rows, dd, dI, bufA, bufG, bufU);
    }
    const DxKind dx = choose_dx(rows, p.d, p.I, acc != 0, dw);
    if (dx == kDxOwn) {
      Scope sc(st, MST_MLP_K_DX);
      launch_nn(st, bufG, Wgb, bufU, Wub, rows, dd, dI, dXb + r0 * p.d);
    }
    {
      Scope sc(st, MST_MLP_K_DW);
      const int tile = dw.small ? Tile64::EA : kTile;
      DwProblems ps;
      ps.p[0] = dw_problem(bufG, dI, Xc, dd, dd, dI, dWg, tile, dw.even);     // dWg [I][d] (+)= dG^T X
      ps.p[1] = dw_problem(bufU, dI, Xc, dd, dd, dI, dWu, tile, dw.even);     // dWu [I][d] (+)= dU^T X
      ps.p[2] = dw_problem(dOc, dd, bufA, dI, dI, dd, dWd, tile, dw.even);    // dWd [d][I] (+)= dO^T A
      const dim3 grid(ps.p[0].grid + ps.p[1].grid + ps.p[2].grid);
      DxProblem x = {};
      x.dG = bufG; x.Wg = Wgb; x.dU = bufU; x.Wu = Wub;
      x.d = dd; x.I = dI; x.dX = dXb + r0 * p.d;
      if (dx == kDx64 || dx == kDx32) {
        (dx == kDx32 ? launch_dx_dw3_small<Tile32> : launch_dx_dw3_small<Tile64Lone>)(st, x, ps, rows, acc);
      } else if (dx != kDxOwn) {
        (dx == kDxHalf ? launch_dx_dw3<Tile16Half> : dx == kDxQuarter ? launch_dx_dw3<Tile16Quarter> : launch_dx_dw3<Tile16>)(st, x, ps, rows, dw.even, acc != 0, more ? 1 : 0);
      } else if (dw.small) {
        if (dw.lone)
          hipLaunchKernelGGL(k_mlp_dw3_small<Tile64Lone>, grid, dim3(Tile64Lone::kThreads), Tile64Lone::kLds, st, ps, rows, acc);
        else
          hipLaunchKernelGGL(k_mlp_dw3_small<Tile64>, grid, dim3(Tile64::kThreads), Tile64::kLds, st, ps, rows, acc);
      } else {
        const auto kernel = dw.even ? (acc ? k_mlp_dw3<false, true> : k_mlp_dw3<true, true>)
                                 : (acc ? k_mlp_dw3<false, false> : k_mlp_dw3<true, false>);
        hipLaunchKernelGGL(kernel, grid, dim3(kThreads), kLdsBytes, st, ps, rows, more ? 1 : 0);
      }
    }
    r0 += rows;
  }
  return check_launch();
}

mst_status mst_mlp_tile_info(int64_t rows, int64_t d, int64_t I, int64_t* info) {
  Plan p;
  const mst_status s = make_plan(rows, d, I, 1, &p);
  if (s != MST_OK) return s;
  if (!info) return MST_ERR_NULL_POINTER;
  auto put = [&](int at, TileChoice c, int64_t n_a, int per_tile) {   // per_tile: indices of a column of large tiles
    const int64_t head = c.head / kTile * per_tile, n = head ? head : n_a;
    info[at] = c.kind;
    info[at + 1] = head;
    info[at + 2] = (c.kind == kBig || head) && use_super_tiles((int)((n + per_tile - 1) / per_tile), (int)((rows + kTile - 1) / kTile));
  };
  put(0, gateup_tile(rows, d, I), I, kGateUpI);
  put(3, nt_tile(rows, d, I), d, kTile);
  put(6, nn_tile(rows, I, d, 1), I, kTile);
  put(9, nn_tile(rows, d, I, 2), d, kTile);
  const DwChoice dw = dw_choice(rows, d, I);
  info[12] = dw_tile(dw);
  info[13] = dw.even;
  return MST_OK;
}

int32_t mst_mlp_dx_tile(int64_t rows, int64_t d, int64_t I, int32_t first) {
  Plan p;
  if (make_plan(rows, d, I, 1, &p) != MST_OK) return -1;
  return dx_tile(choose_dx(rows, d, I, !first, dw_choice(rows, d, I)));
}

int32_t mst_mlp_dx_tile_rows(int64_t rows, int64_t d, int64_t I, int32_t first) {
  Plan p;
  if (make_plan(rows, d, I, 1, &p) != MST_OK) return -1;
  return dx_tile_rows(choose_dx(rows, d, I, !first, dw_choice(rows, d, I)));
}

int64_t mst_mlp_fwd_groups(int64_t S, int64_t d, int64_t I, int32_t M, size_t workspace_bytes, int32_t output_overlaps,
                           int64_t room, int64_t* info) {
  Plan p;
  if (make_plan(S, d, I, M, &p) != MST_OK || workspace_bytes < p.slot || room < 0 || (room && !info)) return -1;
  int64_t n = 0;
  for (int64_t left = S; left > 0; ++n) {
    const ForwardGroup g = forward_group(p, left, workspace_bytes, !output_overlaps);
    left -= g.rows;
    if (n >= room) continue;
    info[2 * n] = g.rows;
    info[2 * n + 1] = g.in_output;
  }
  return n;
}

int64_t mst_mlp_bwd_groups(int64_t S, int64_t d, int64_t I, int32_t M, int32_t dx_overlaps, int64_t room, int64_t* info) {
  Plan p;
  if (make_plan(S, d, I, M, &p) != MST_OK || room < 0 || (room && !info)) return -1;
  const BackwardGroups groups(p, !dx_overlaps);
  const DwChoice dw = dw_choice(std::min(groups.cap, S), d, I);
  int64_t n = 0;
  for (int64_t left = S; left > 0; ++n) {
    int in_dx = 0;
    const int64_t rows = groups.next(left, &in_dx);
    const DxKind dx = choose_dx(rows, d, I, left < S, dw);
    left -= rows;
    if (n >= room) continue;
    const int64_t values[6] = {rows, in_dx, dx_tile(dx), dx_tile_rows(dx), fuse_da(rows, d, I), dw_tile(dw)};
    std::copy(values, values + 6, info + 6 * n);
  }
  return n;
}

int32_t mst_mlp_line_panels(int64_t rows, int64_t d, int64_t I) {
  Plan p;
  if (make_plan(rows, d, I, 1, &p) != MST_OK) return -1;
  auto lone = [&](TileChoice c, int64_t N, int64_t K) { return c.kind == k64Lone && by_lines((int64_t)tiles_of(N - c.head, rows, 64), K, nullptr, nullptr); };
  const DwChoice dw = dw_choice(rows, d, I);
  const DxKind dx = choose_dx(rows, d, I, false, dw);
  const int n_d = (int)((d + 63) / 64), n_i = (int)((I + 63) / 64), n_s = (int)((rows + 63) / 64);
  const int64_t shared = even_grid(n_d, n_s) + 2 * even_grid(n_i, n_d) + even_grid(n_d, n_i);
  return (lone(nt_tile(rows, d, I), d, I) ? MST_MLP_LINES_DOWN : 0) |
         (!fuse_da(rows, d, I) && lone(nn_tile(rows, I, d, 1), I, d) ? MST_MLP_LINES_DA : 0) |
         ((dx == kDxOwn ? lone(nn_tile(rows, d, I, 2), d, I) : dx == kDx64 && by_lines(shared, I, nullptr, nullptr)) ? MST_MLP_LINES_DX : 0);
}

int32_t mst_mlp_da_in_gateup(int64_t rows, int64_t d, int64_t I) {
  Plan p;
  if (make_plan(rows, d, I, 1, &p) != MST_OK) return -1;
  return fuse_da(rows, d, I) ? 1 : 0;
}

int32_t mst_mlp_tile_grid(int32_t n_slow, int32_t n_fast) {
  if (n_slow < 1 || n_fast < 1 || (int64_t)n_slow * n_fast > (1 << 28)) return -1;
  return mlp_grid(n_slow, n_fast);
}

int32_t mst_mlp_tile_of_workgroup(int32_t n_slow, int32_t n_fast, int32_t workgroup, int32_t* slow, int32_t* fast) {
  const int32_t grid = mst_mlp_tile_grid(n_slow, n_fast);
  if (grid < 0 || workgroup < 0 || workgroup >= grid || !slow || !fast) return -1;
  int s = 0, f = 0;
  const bool ok = use_super_tiles(n_slow, n_fast) ? super_tile_of_block(workgroup, n_slow, n_fast, &s, &f)
                                                  : even_tile_of_block(workgroup, n_slow, n_fast, &s, &f);
  *slow = s;
  *fast = f;
  return ok ? 1 : 0;
}

mst_status mst_mlp_profile_enable(int every) {
  g_prof.enable(every);
  return MST_OK;
}

mst_status mst_mlp_profile_collect(double* ms_per_kind, int64_t* launches_per_kind, int64_t* issued_per_kind) {
  return g_prof.collect(MST_MLP_PROFILE_KINDS, ms_per_kind, launches_per_kind, issued_per_kind) ? MST_OK : MST_ERR_LAUNCH;
}

const char* mst_mlp_profile_kind_name(int kind) {
  static const char* names[MST_MLP_PROFILE_KINDS] = {"gateup", "down", "da", "gateup_bwd", "dx", "dw"};
  return (kind >= 0 && kind < MST_MLP_PROFILE_KINDS) ? names[kind] : "?";
}

}  // extern "C"
