// Host side of the mini-sequence LM-head + cross-entropy library: argument
// validation, the chunk schedule over the M mini-sequences (Algorithm 2 lines
// 1-3 and Algorithm 4 lines 1-4 of the paper: partition, then loop; for the
// backward also the choice between that loop and blocks of rows x vocabulary
// windows of the same size), workspace carving, launches, and the optional
// per-kernel event timing.
#include "../../include/mst_lmhead.h"
#include "host_util.hpp"
#include "launch_model.hpp"
#include "mst_small_kernels.hpp"
#include "mst_stream_kernels.hpp"

#include <algorithm>
#include <atomic>
#include <mutex>

namespace {

using namespace mst;

constexpr int kMaxDhSplit = 64;
constexpr int kMaxWindows = 64;      // most vocabulary windows the block schedule considers
constexpr int kMaxBlockSplit = 8;    // most splits of a window's dH contraction

// Override of the backward order, per calling thread: a caller that forces an order cannot change the
// summation order of a call another thread is making at the same time.
thread_local int t_bwd_schedule = MST_BWD_SCHEDULE_AUTO;

using mst_host::align_up;
using mst_host::misaligned;

struct Plan {
  int64_t S, d, V;
  int M;
  int C;            // rows per chunk = ceil(S / M)
  int n_chunks;     // non-empty chunks = ceil(S / C)
  int64_t fwd_group_rows;   // rows whose log-sum-exp partials are merged by one launch: a whole number of chunks
  int ldg;          // leading dimension of the dlogits workspace (V rounded up to 8)
  int n_vt;         // vocabulary tiles
  int n_jt;         // hidden tiles
  int n_st;         // row tiles of a full chunk
  int dh_split;     // splits of the dH contraction over V
  int dh_ksteps;    // K steps (of kBK) per split
  // pair order: 64 x 64 tiles instead of 256 x 256 ones, per launch kind (mst_small_kernels.hpp)
  bool small_dlogits, small_dh, small_dw;
  int small_dh_split, small_dh_ksteps;
  int joint;        // pair order: dH and dW from one launch, dlogits of a pair from another (MST_PAIR_* of the header)
  double joint_us;
  // forward workspace (byte offsets)
  size_t f_nll, f_tgt, f_part, f_total;
  // backward workspace: two dlogits slots of one chunk each (bf16), contiguous
  size_t b_slot;      // bytes of one slot = C * ldg * 2
  size_t b_total;     // 2 * b_slot: what the call needs when lse and n_valid are supplied
  size_t b_ctl;       // offset of the control block used when n_valid is not supplied (aligned, after the slots)
  size_t b_lse;       // offset of the lse scratch used when lse is not supplied
  size_t b_fwd;       // offset of the forward region used when lse is not supplied
  size_t b_total_max; // bytes needed when neither lse nor n_valid is supplied
  // Block schedule of the backward pass (used when blk_use): the same b_total bytes hold dlogits of blk_rows rows
  // by blk_win_tiles * kTile vocabulary entries (bf16, leading dimension blk_ldg) and, behind it, fp32 dH sums of
  // blk_rows x d.  blk_n_rb row blocks x blk_n_win vocabulary windows cover S x V.
  bool blk_use;
  bool blk_fused;     // dH and dW of a block from one launch
  int blk_rows, blk_n_rb, blk_win_tiles, blk_n_win, blk_ldg;
  int blk_split;      // splits of a window's dH contraction, each with running sums of its own
  size_t blk_acc;     // byte offset of the dH sums
  double est_pairs_us, est_blocks_us;   // the cost model's figures (for the record; see choose_schedule)
  // Neither order: dlogits formed where they are used (MST_STREAMED_* of the header, 0: not so)
  int streamed;
  int stream_split, stream_per_split;   // shares of dH's contraction, vocabulary entries of each
};

// ------------------------------------------------------------------ backward schedule
// Both schedules recompute each logit once and keep at most b_total bytes of dlogits alive; they differ in
// which block of the S x V dlogits matrix is alive at a time and therefore in how often the fp32 gradients
// are read back and rewritten:
//   pairs   (Algorithm 4 as printed, two mini-sequences per dW pass): blocks of 2C rows x all of V.
//           dW is read and rewritten once per pair after the first; dH is final after each chunk.
//   blocks  R rows x one window of the vocabulary, R as large as the same bytes allow (dlogits of the block
//           plus fp32 dH sums of its rows).  dW of a window accumulates over the row blocks (none to add when
//           R covers S), dH of a row block accumulates over the windows (S*d*4 bytes, far smaller than dW when
//           V >> d).
// The estimate counts rounds of kNumCu workgroups per launch at a nominal time per K step, plus the fp32
// gradient traffic at a nominal bandwidth; it only has to rank the candidates.  The automatic choice looks at more
// block shapes afterwards (choose_split_blocks).
constexpr double kUsPerKStep = 1.5;      // one 256 x 256 x 64 block-tile step with one workgroup per CU
constexpr double kRmwBytesPerUs = 4.0e6; // fp32 read-modify-write streams next to a running GEMM
double rounds_us(int64_t tiles, int64_t k) {
  return (double)((tiles + kNumCu - 1) / kNumCu) * (double)((k + kBK - 1) / kBK) * kUsPerKStep;
}

// Block shapes with splits of dH's contraction, or with a single window.  With few row tiles (1024 rows x 4096: 64 tiles
// of dH) the unsplit dH tiles of a block are too few and too long to share a launch with its dW tiles, so the printed
// order with its read-modify-write of dW per pair used to be taken: S = 1024, d = 4096, V = 128256, M = 4: step 4.6 ms,
// with two splits and four windows 3.4 ms.
//
// The model is that of launch_model.hpp, with a tile's ends, in microseconds: dlogits 6; dH sums 8, and 8 more where they
// are read; dW as there.
TileCost dlogits_cost(int64_t d) { return tile_cost(d, 6.0); }
TileCost dh_cost(int64_t k, bool add) { return tile_cost(k, add ? 16.0 : 8.0); }

double pairs_us(const Plan* p) {
  const int64_t S = p->S, d = p->d, V = p->V, C = p->C;
  const double w_all = 2.0 * (double)V * (double)d;                        // bytes of W
  const int split = p->small_dh ? p->small_dh_split : p->dh_split;
  auto chunk = [&](int64_t rows) {
    const int64_t n_st = (rows + kTile - 1) / kTile;
    const double g = 2.0 * (double)rows * (double)V, part = 4.0 * (double)split * (double)(rows * d);
    double t = p->small_dlogits ? small_launch_us(tiles_of(rows, V, 64), (double)((d + kBK - 1) / kBK))
                                : launch_us(n_st * p->n_vt, dlogits_cost(d), w_all + g);
    t += p->small_dh ? small_launch_us(tiles_of(rows, d, 64) * split, (double)p->small_dh_ksteps)
                     : launch_us(n_st * p->n_jt * split, dh_cost((int64_t)p->dh_ksteps * kBK, false), w_all + g + part);
    return split > 1 ? t + 4.0 + part / kHbmBytesPerUs : t;
  };
  auto dw = [&](int64_t rows, bool add) {
    return p->small_dw ? small_launch_us(tiles_of(V, d, 64), (double)((rows + kBK - 1) / kBK))
                       : launch_us((int64_t)p->n_vt * p->n_jt, dw_cost(rows, add), (add ? 4.0 : 2.0) * w_all);
  };
  const int64_t last = S - (int64_t)(p->n_chunks - 1) * C;                 // rows of the last chunk
  const int n_pairs = (p->n_chunks + 1) / 2;
  const int64_t last_pair = p->n_chunks % 2 ? last : C + last;
  double t = (double)(p->n_chunks - 1) * chunk(C) + chunk(last);
  t += n_pairs > 1 ? dw(2 * C, false) + (double)(n_pairs - 2) * dw(2 * C, true) + dw(last_pair, true) : dw(last_pair, false);
  return t;
}

// Joint launches of the pair order, for problems whose launches all take 64 x 64 tiles.  Microseconds, fitted to launches of
// 64 to 2400 rows, d = 256 to 2112, V = 2012 to 23326: dlogits of the pair as one launch; dH + dW the longer of one dH
// workgroup by itself (5, and a time per 128 vocabulary entries by its tile) and the dH loads (16 TB/s; 64-byte pieces cost
// half as much again) on top of the time of dW.  A call of one chunk can keep the split partials of dH instead: its separate
// launches less 2, unless few tiles of dW have a contraction over so many rows that their pipelined form, which they have in a
// launch of their own, is worth more (0.45 against 0.25 per K step).  500 calls of one chunk, both ways: 133 in separate
// launches by this rule took 0.98 to 1.77 of their time in one, 1.26 in the mean (27903 rows, d = 16, V = 55: 102 us, 180
// in one), the others 0.89 to 1.11, 0.98.
// kJoint: of 104 shapes timed in every form none takes longer than with separate launches (0.82 of that in the mean), and
// the form taken is 0.5 % behind the fastest one in the mean, 8 % at most.
constexpr double kJoint = 0.95;
struct JointTile { int j, rows, piece; double step; };
constexpr JointTile kJointTiles[] = {{TileKSplit32x16::EA, TileKSplit32x16::EB, 48, 0.22},
                                     {TileKSplit64x16::EA, TileKSplit64x16::EB, 64, 0.27},
                                     {TileKSplit64x32::EA, TileKSplit64x32::EB, 64, 0.40}};
double ksplit_us(const Plan* p, const JointTile& t, int64_t rows) {
  const int64_t n = (rows + t.rows - 1) / t.rows * ((p->d + t.j - 1) / t.j);
  const double loads = (double)n * (t.piece + t.rows) * 2.0 * (double)p->V / 16.0e6;
  const double dw = small_launch_us(std::max(257.0, tiles_of(p->V, p->d, 64)), (double)((rows + kBK - 1) / kBK));
  return 1.0 + small_launch_us(tiles_of(rows, p->V, 64), (double)((p->d + kBK - 1) / kBK)) +
         std::max(5.0 + t.step * (double)((p->V + 127) / 128), loads + dw);
}
void choose_joint(Plan* p) {
  p->joint = 0;
  if (!p->small_dlogits || !p->small_dh || !p->small_dw) return;
  p->joint_us = pairs_us(p);
  if (p->n_chunks == 1) {
    const double kw = (double)((p->S + kBK - 1) / kBK), kh = (double)p->small_dh_ksteps;
    const double apart = 2.0 + small_launch_us(tiles_of(p->S, p->d, 64) * p->small_dh_split, kh) +
                         small_launch_us(tiles_of(p->V, p->d, 64), kw);
    if (0.45 * std::max(kw, kh) + 3.5 <= apart) {
      p->joint = MST_PAIR_SPLIT;
      p->joint_us -= 2.0;
    }
  }
  double best = kJoint * p->joint_us;
  for (int k = 0; k < 3; ++k) {
    double t = 0.0;
    for (int64_t r0 = 0; r0 < p->S; r0 += 2 * (int64_t)p->C)
      t += ksplit_us(p, kJointTiles[k], std::min(2 * (int64_t)p->C, p->S - r0));
    if (t >= best) continue;
    p->joint = MST_PAIR_KSPLIT_32X16 + k;
    p->joint_us = best = t;
  }
}

double blocks_us(const Plan* p, int64_t R, int n_rb, int win_tiles, int n_win, int split) {
  const int64_t S = p->S, d = p->d, V = p->V, win = (int64_t)win_tiles * kTile;
  auto block = [&](int64_t rows, int64_t cols, bool dw_add, bool dh_add) {
    const int64_t n_st = (rows + kTile - 1) / kTile, tiles_w = (cols + kTile - 1) / kTile;
    const double w_bytes = 2.0 * (double)(cols * d), g_bytes = 2.0 * (double)(rows * cols);
    const double sum_bytes = n_win > 1 || split > 1 ? 4.0 * (double)split * (double)(n_st * p->n_jt) * (kTile * kTile) : 0.0;
    return launch_us(n_st * tiles_w, dlogits_cost(d), w_bytes + g_bytes) +
           launch_us(n_st * p->n_jt * split, dh_cost((cols + split - 1) / split, dh_add), tiles_w * p->n_jt, dw_cost(rows, dw_add),
                     w_bytes + g_bytes + (dw_add ? 4.0 : 2.0) * w_bytes + (dh_add ? 2.0 : 1.0) * sum_bytes);
  };
  auto row_block = [&](int64_t rows, bool dw_add) {           // its first, middle and last window, its reduce
    const int64_t last = V - (int64_t)(n_win - 1) * win;
    double t = block(rows, n_win > 1 ? win : last, dw_add, false);
    if (n_win > 2) t += (double)(n_win - 2) * block(rows, win, dw_add, true);
    if (n_win > 1) t += block(rows, last, dw_add, true);
    if (split > 1) t += 4.0 + 4.0 * (double)split * (double)(rows * d) / kHbmBytesPerUs;
    return t;
  };
  double t = row_block(n_rb > 1 ? R : S, false);
  if (n_rb > 2) t += (double)(n_rb - 2) * row_block(R, true);
  if (n_rb > 1) t += row_block(S - (int64_t)(n_rb - 1) * R, true);
  return t;
}

// Looks for a block shape with one window, or with dH's contraction split, that beats `p`'s choice so far by more than
// the model is good for, and for a block shape chosen so far that the pair order beats.  Not where two rounds of dH tiles
// fill the chip as it is: the shapes of the long configurations are the ones measured.  1 to 12 us of host time for steps
// of 80 us to 6 ms: more windows than eight past the first count that leaves one row block only make the windows smaller.
//
// The choice so far does not know the 64 x 64 tiles of the pair order, so it has to be able to go back: 712 rows,
// d = 1920, V = 6637, M = 2: backward 289 us in blocks, 119 in pairs.  kPairsBelow: of 68 shapes timed in both orders,
// pairs below 0.8 of the blocks' estimate took 0.31 to 0.91 of the time (35 shapes); from 0.8 to 1 it was 0.88 to 1.11
// (33), either way round.
constexpr double kPairsBelow = 0.8;
void choose_split_blocks(Plan* p) {
  const int64_t S = p->S, d = p->d;
  if (p->blk_use && (int64_t)(p->blk_rows / kTile) * p->n_jt >= 2 * kNumCu) return;
  const double pairs = p->joint ? p->joint_us : pairs_us(p);
  const double so_far = p->blk_use ? blocks_us(p, p->blk_rows, p->blk_n_rb, p->blk_win_tiles, p->blk_n_win, 1) : pairs;
  double best = 0.95 * std::min(so_far, pairs);
  double cheapest = p->blk_use ? so_far : 0.0;                             // of all block shapes (0: none fits)
  bool found = false;
  for (int split = 1; split <= kMaxBlockSplit; split *= 2) {
    int one_row_block_from = 0;
    for (int n_win = 1; n_win <= kMaxWindows && n_win <= p->n_vt; ++n_win) {
      if (one_row_block_from && n_win > one_row_block_from + 8) break;
      const int win_tiles = (p->n_vt + n_win - 1) / n_win;
      if (split > win_tiles) break;
      if ((p->n_vt + win_tiles - 1) / win_tiles != n_win) continue;        // same partition as a smaller count
      const int64_t ldg_w = (int64_t)win_tiles * kTile;
      const int64_t per_row = ldg_w * 2 + (n_win > 1 || split > 1 ? (int64_t)split * p->n_jt * kTile * 4 : 0);
      if (p->b_total < 256 + (size_t)per_row * kTile) continue;
      int64_t R = (int64_t)((p->b_total - 256) / (size_t)per_row) / kTile * kTile;
      const int64_t S_up = (S + kTile - 1) / kTile * kTile;
      if (R > S_up) R = S_up;
      const int n_rb = (int)((S + R - 1) / R);
      if (n_rb == 1 && !one_row_block_from) one_row_block_from = n_win;
      R = ((S + n_rb - 1) / n_rb + kTile - 1) / kTile * kTile;
      if (R * ldg_w >= (int64_t(1) << 30) || R * d >= (int64_t(1) << 30)) continue;   // 32-bit offsets inside a block
      const double t = blocks_us(p, R, n_rb, win_tiles, n_win, split);
      if (cheapest == 0.0 || t < cheapest) cheapest = t;
      if (t < best) {
        best = t;
        found = true;
        p->blk_use = true;
        p->blk_fused = true;
        p->blk_rows = (int)R; p->blk_n_rb = n_rb; p->blk_win_tiles = win_tiles; p->blk_n_win = n_win;
        p->blk_ldg = (int)ldg_w;
        p->blk_split = split;
        p->blk_acc = align_up((size_t)R * ldg_w * 2, 256);
      }
    }
  }
  if (!found && p->blk_use && pairs < kPairsBelow * so_far) p->blk_use = false;
  p->est_pairs_us = pairs;
  p->est_blocks_us = found ? best : p->blk_use ? so_far : cheapest;
}

// The pair order with one launch for the pair's dlogits and one for its dH and dW, dH in 128 x 128 tiles over the whole
// vocabulary (k_bwd_gemm_dh128_dw): two launches instead of seven, for pairs that are less than a few rounds of tiles, as long
// as a dH tile's chain of V / 64 K steps is not much longer than dW's work.  Backward, us: 3094 rows, d = 2696, V = 12307, M = 6:
// 1374 -> 762; 1232, 2096, 14469, 4: 590 -> 351; 2980, 824, 7045, 4: 298 -> 184; but, where it is not taken, 1700, 1472, 9339, 6:
// 288 -> 300.
// Microseconds: a K step of a dH tile 0.55, 0.65 with all compute units busy, 8 for its ends; dlogits and dW as above.  Of 70
// shapes of 219 to 19863 rows, d = 408 to 3112, V = 4117 to 69139, timed both ways, this estimate takes it for 12, at 0.56 to
// 0.90 of their time, and the choice is 0.4 % behind the faster way in the mean; 30 others that it takes 0.54 to 1.00, 0.79.
// kDh128Blocks: blocks are a little faster than
// estimated; four shapes of 0.7 to 0.95 of their estimate took 0.94 to 1.06 of their time.
constexpr double kDh128Pairs = 0.95, kDh128Blocks = 0.7;
bool small_pair_dlogits(const Plan& p, int64_t rows) {
  const double k = (double)((p.d + kBK - 1) / kBK);
  return small_launch_us(tiles_of(rows, p.V, 64), k) < big_launch_us(tiles_of(rows, p.V, kTile), k);
}
double dh128_us(const Plan* p, int64_t rows, bool add) {
  const double w_all = 2.0 * (double)p->V * (double)p->d, g = 2.0 * (double)rows * (double)p->V;
  const double dlogits = small_pair_dlogits(*p, rows) ? small_launch_us(tiles_of(rows, p->V, 64), (double)((p->d + kBK - 1) / kBK))
                                                      : launch_us((rows + kTile - 1) / kTile * p->n_vt, dlogits_cost(p->d), w_all + g);
  return dlogits + launch_us((int64_t)tiles_of(rows, p->d, Tile16Quarter::EA),
                             TileCost{(double)((p->V + kBK - 1) / kBK), 8.0, 0.55, 0.65},
                             (int64_t)p->n_vt * p->n_jt, dw_cost(rows, add), w_all + g + (add ? 4.0 : 2.0) * w_all);
}
void choose_dh128(Plan* p) {
  if (p->small_dlogits && p->small_dh && p->small_dw) return;                        // has joint launches of its own
  if (2 * (int64_t)p->C * p->ldg >= (int64_t(1) << 30)) return;                      // 32-bit offsets inside a pair
  if (p->blk_use && (int64_t)(p->blk_rows / kTile) * p->n_jt >= 2 * kNumCu) return;
  double t = 0.0;
  for (int64_t r0 = 0; r0 < p->S; r0 += 2 * (int64_t)p->C) t += dh128_us(p, std::min(2 * (int64_t)p->C, p->S - r0), r0 > 0);
  if (t >= (p->blk_use ? kDh128Blocks * p->est_blocks_us : kDh128Pairs * pairs_us(p))) return;
  p->joint = MST_PAIR_DH128;
  p->blk_use = false;
  p->est_pairs_us = t;
}

int64_t dh_split_room(const Plan* p) { return ((int64_t)p->C * p->ldg * 2) / ((int64_t)p->C * p->d * 4); }

// Splits of the pair order's dH: among the counts that fit (at most `most`, at most one per K step, partials must fit into
// the dlogits slot that is free at that moment: dh_split_room) the one with the fullest rounds
// of workgroups, with a small penalty per split for the fp32 partials it adds.
int best_dh_split(const Plan* p, int ksteps, int most) {
  const int out_tiles = p->n_st * p->n_jt;
  const int64_t room = dh_split_room(p);
  int split = 1;
  double best = -1.0;
  for (int s = 1; s <= most && s <= ksteps && (s == 1 || s <= room); ++s) {
    const int wgs = out_tiles * s;
    const int rounds = (wgs + kNumCu - 1) / kNumCu;
    const double score = (double)wgs / ((double)rounds * kNumCu) - 0.002 * s;
    if (score > best) { best = score; split = s; }
  }
  const int per = (ksteps + split - 1) / split;
  return (ksteps + per - 1) / per;
}

// ---- backward without dlogits in memory (mst_stream_kernels.hpp), for 128 < d <= 512 and the automatic order only
typedef CfgStream<256, 2, 1, 4> Stream256;          // 128 owners, two workgroups on a compute unit
typedef CfgStream<256, 1, 1, 4> Stream256Narrow;    // 64 owners
typedef CfgStream<256, 1, 4, 2> Stream256SplitH;    // 16 and 32 owners, whose waves share out the stream: for few owners
typedef CfgStream<256, 2, 4, 2> Stream256SplitW;
typedef CfgStream<384, 1, 1, 3> Stream384;          // 64 owners
typedef CfgStream<384, 1, 2, 2> Stream384Split;     // 32 owners
typedef CfgStream<512, 1, 1, 2> Stream512;
typedef CfgStream<512, 1, 2, 2> Stream512Split;

typedef void (*StreamLaunch)(hipStream_t, const StreamProblem&, int split, int per_split, float*, __bf16*, float*);
template <class CH, class CW>
void launch_streamed(hipStream_t st, const StreamProblem& q, int split, int per_split, float* partial, __bf16* dH, float* dW) {
  const int dh_grid = even_grid(split, (q.S + CH::kOwners - 1) / CH::kOwners), dw_grid = even_grid((q.V + CW::kOwners - 1) / CW::kOwners, 1);
  const bool dw_first = q.S > per_split;               // steps of a workgroup
  hipLaunchKernelGGL((k_bwd_stream<CH, CW>), dim3(dh_grid + dw_grid), dim3(CH::kThreads), CH::kLds > CW::kLds ? CH::kLds : CW::kLds, st,
                     q, dw_first ? dw_grid : 0, dh_grid, split, per_split, partial, dH, dW);
}
// Microseconds: a step of a workgroup by itself, a step's share of a compute unit with all of them busy, the ends of a
// workgroup (in steps), the launch.  Fitted to 260 shapes of 64 to 32768 rows, d = 136 to 512, V = 1000 to 128000, every
// form with 1 to 64 splits (within 4 to 8 % rms; the form and split taken are 2.5 % behind the fastest in the mean).  The chain is
// that of the XCD that has most workgroups: 154 of dW and 100 of dH are 254 in all, but 20 + 13 on one XCD, a second round (308
// rows, d = 256, V = 4928: 23.1 us in five splits, 16.1 in four; 120 shapes whose form or split this changes: 0.90 in the mean, 0.69
// to 1.21).  A step of dW takes up to 1.7 times that where its 16 OT entries are likely to be labels; operands, dW and partials at
// 2.5 TB/s.
struct StreamForm { int dk, owners_h, owners_w, ot_w, rings, per_cu; double step, busy, ends, fixed; StreamLaunch launch; };
template <class CH, class CW>
constexpr StreamForm stream_form(double step, double busy, double ends, double fixed) {
  static_assert(CH::NWS == CW::NWS && CH::DK == CW::DK, "one launch");
  return {CH::DK, CH::kOwners, CW::kOwners, CW::OT, CH::NWS, CH::kLds > 81920 ? 1 : 2, step, busy, ends, fixed, launch_streamed<CH, CW>};
}
constexpr StreamForm kStreamForms[] = {                // MST_STREAMED_*, from 1 on, in this order
    stream_form<Stream256, Stream256>(0.89, 0.80, 0.0, 8.5),
    stream_form<Stream256Narrow, Stream256Narrow>(0.63, 0.52, 0.0, 6.0),
    stream_form<Stream256SplitH, Stream256SplitW>(0.62, 0.66, 7.1, 1.1),
    stream_form<Stream384, Stream384>(0.84, 0.77, 0.0, 5.9),
    stream_form<Stream384Split, Stream384Split>(1.00, 0.90, 4.0, 2.8),
    stream_form<Stream512, Stream512>(1.09, 1.00, 2.0, 3.2),
    stream_form<Stream512Split, Stream512Split>(1.32, 1.20, 3.1, 2.8)};
double stream_us(const Plan* p, const StreamForm& f, int split, int per_split) {
  auto up = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
  const int64_t n_h = up(p->S, f.owners_h) * split, n_w = up(p->V, f.owners_w);
  const double by_label = 1.0 + 0.7 * std::min(1.0, 512.0 * f.ot_w / (double)p->V);
  const double t_h = (double)up(per_split, 32 * f.rings) + f.ends, t_w = ((double)up(p->S, 32 * f.rings) + f.ends) * by_label;
  const double partials = split > 1 ? 4.0 * (double)split * (double)(p->S * p->d) : 0.0;
  const int64_t units = (int64_t)kXcdCu * f.per_cu, x_h = up(n_h, kNumXcd), x_w = up(n_w, kNumXcd);   // of the XCD that has most
  const double chain = f.step * (t_w > t_h ? span_us(x_w, t_w, x_h, t_h, units) : span_us(x_h, t_h, x_w, t_w, units));
  const double busy = f.busy * ((double)n_h * t_h + (double)n_w * t_w) / kNumCu, bytes = (8.0 * (double)(p->V * p->d) + partials) / 2.5e6;
  const double t = f.fixed + std::cbrt(chain * chain * chain + busy * busy * busy + bytes * bytes * bytes);     // the longest, smoothed
  return split > 1 ? t + 3.5 + partials / kHbmBytesPerUs : t;
}
// Taken where it is estimated this much below the order that would run.  The estimates of blocks are 8 % too high in the mean;
// those of joint launches 3 us a pair where pairs are short, their last launch being less than a round of short tiles; and of
// one chunk with split partials beside dW the sum over many splits of few rows costs more than estimated.  750 shapes that this
// takes, of 32 to 32768 rows, V = 300 to 128256, took 0.67 of that order's time in the mean, ten of them 1.04 to 1.11; without the
// 3 us and the limit of splits 35 of 300 calls of up to 3000 rows took 1.02 to 1.28 (99 rows, d = 192, V = 5908, M = 1: 15.5 us, 19.3
// streamed).  Blocks from 0.78 to 0.82 of theirs: 60 shapes 0.74 to 1.07.
constexpr double kStreamedPairs = 0.9, kStreamedJoint = 0.9, kStreamedBlocks = 0.82, kShortPair = 20.5, kShortPairLess = 3.0;
constexpr int kStreamedSplits = 10;
void choose_streamed(Plan* p) {
  const int64_t S = p->S, d = p->d, V = p->V;
  if (d <= 128 || d > 512 || S * d >= (int64_t(1) << 30) || V * d >= (int64_t(1) << 30)) return;   // 32-bit byte offsets of whole operands
  int64_t room = (int64_t)(p->b_total / ((size_t)(S * d) * 4));
  double best = kStreamedPairs * p->est_pairs_us;
  if (p->blk_use) {
    best = kStreamedBlocks * p->est_blocks_us;
  } else if (p->joint == MST_PAIR_SPLIT) {
    best = kStreamedJoint * p->est_pairs_us;
    room = std::min(room, (int64_t)kStreamedSplits);
  } else if (p->joint && p->joint != MST_PAIR_DH128) {
    const double pairs = (double)((p->n_chunks + 1) / 2);
    best = kStreamedJoint * (p->est_pairs_us - (p->est_pairs_us < kShortPair * pairs ? kShortPairLess * pairs : 0.0));
  }
  for (int k = 0; k < (int)(sizeof(kStreamForms) / sizeof(kStreamForms[0])); ++k) {
    const StreamForm& f = kStreamForms[k];
    if (f.dk < d || f.dk - d >= (f.dk == 256 ? 256 : 128)) continue;
    for (const int n : {1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 20, 24, 32, 48, 64}) {
      if (n > 1 && n > room) break;
      const int per_split = (int)(((V + n - 1) / n + 31) / 32 * 32), split = (int)((V + per_split - 1) / per_split);   // all begin inside V
      if (split != n) continue;
      const double t = stream_us(p, f, split, per_split);
      if (t >= best) continue;
      best = t;
      p->streamed = k + 1;
      p->stream_split = split;
      p->stream_per_split = per_split;
    }
  }
}

void choose_schedule(Plan* p, int forced) {
  choose_joint(p);
  const int64_t S = p->S, d = p->d, V = p->V, C = p->C;
  const int n_vt = p->n_vt, n_jt = p->n_jt;
  // pairs (the estimate is calibrated for at most 16 splits of dH)
  const int ksteps = (int)((V + kBK - 1) / kBK), split = best_dh_split(p, ksteps, 16);
  double pairs = 0.0;
  for (int ia = 0; ia < p->n_chunks; ia += 2) {
    int64_t rows_pair = 0;
    for (int i = ia; i < ia + 2 && i < p->n_chunks; ++i) {
      const int64_t rows = (S - (int64_t)i * C) < C ? (S - (int64_t)i * C) : C;
      const int64_t n_st = (rows + kTile - 1) / kTile;
      rows_pair += rows;
      pairs += rounds_us(n_st * n_vt, d);                                                  // dlogits
      pairs += rounds_us(n_st * n_jt * split, (int64_t)((ksteps + split - 1) / split) * kBK);   // dH
      if (split > 1) pairs += 2.0 * (double)(split * rows * d * 4) / kRmwBytesPerUs;
    }
    pairs += rounds_us((int64_t)n_vt * n_jt, rows_pair);                                   // dW
    pairs += (double)((ia > 0 ? 8 : 4) * V * d) / kRmwBytesPerUs;
  }
  p->est_pairs_us = pairs;
  // blocks: for every window count, the largest row block that fits, then rows balanced over the blocks
  p->blk_use = false;
  p->blk_fused = false;
  p->est_blocks_us = 0.0;
  double best = 0.0;
  for (int n_win = 2; n_win <= kMaxWindows && n_win <= n_vt; ++n_win) {
    const int win_tiles = (n_vt + n_win - 1) / n_win;
    const int n_win_eff = (n_vt + win_tiles - 1) / win_tiles;
    if (n_win_eff != n_win) continue;                       // same partition as a smaller count
#ifdef MST_FORCE_WINDOWS                                    // measurement builds: rank by measurement, not by the model
    if (n_win != MST_FORCE_WINDOWS) continue;
#endif
    const int64_t ldg_w = (int64_t)win_tiles * kTile;
    const int64_t per_row = ldg_w * 2 + (int64_t)n_jt * kTile * 4;   // dlogits + fp32 dH sums (whole column tiles)
    if (p->b_total < 256 + (size_t)per_row * kTile) continue;
    int64_t R = (int64_t)((p->b_total - 256) / (size_t)per_row) / kTile * kTile;
    const int64_t S_up = (S + kTile - 1) / kTile * kTile;
    if (R > S_up) R = S_up;
    const int n_rb = (int)((S + R - 1) / R);
    R = ((S + n_rb - 1) / n_rb + kTile - 1) / kTile * kTile;
    if (R * ldg_w >= (int64_t(1) << 30) || R * d >= (int64_t(1) << 30)) continue;   // 32-bit offsets inside a block
    double t = 0.0;
    for (int rb = 0; rb < n_rb; ++rb) {
      const int64_t rows = (S - rb * R) < R ? (S - rb * R) : R;
      const int64_t n_st = (rows + kTile - 1) / kTile;
      for (int w = 0; w < n_win; ++w) {
        const int64_t tiles_w = (w + 1) * win_tiles <= n_vt ? win_tiles : n_vt - w * win_tiles;
        const int64_t cols = tiles_w * kTile < V - (int64_t)w * ldg_w ? tiles_w * kTile : V - (int64_t)w * ldg_w;
        t += rounds_us(n_st * tiles_w, d);                                                 // dlogits
        t += (double)((w > 0 ? 4 : 0) + (w + 1 < n_win ? 4 : 2)) * (double)(rows * d) / kRmwBytesPerUs;
        t += (double)((rb > 0 ? 8 : 4) * cols * d) / kRmwBytesPerUs;
        t += rounds_us(n_st * n_jt, cols) + rounds_us(tiles_w * n_jt, rows);               // dH, dW
      }
    }
    // One launch for the dH and the dW tiles of a block (BLOCKS_FUSED): a partly filled last round of dH workgroups is
    // topped up with dW tiles, and one launch boundary per block goes away.  Measured: -0.25 to -0.4 % of the step where
    // both tile counts fill whole rounds anyway (512 and 1008 tiles), -1.5 to -2 % where they do not (896 dH tiles = 3.5
    // rounds; 496).  The automatic choice always takes it; the block shapes are ranked as separate launches.
    const bool fuse = forced == MST_BWD_SCHEDULE_BLOCKS_FUSED || forced == MST_BWD_SCHEDULE_AUTO;
    const double t_pick = t;
    if (!p->blk_use || t_pick < best) {
      best = t_pick;
      p->blk_use = true;
      p->blk_fused = fuse;
      p->blk_rows = (int)R; p->blk_n_rb = n_rb; p->blk_win_tiles = win_tiles; p->blk_n_win = n_win;
      p->blk_ldg = (int)ldg_w;
      p->blk_split = 1;
      p->blk_acc = align_up((size_t)R * ldg_w * 2, 256);
    }
  }
  p->est_blocks_us = best;
  if (forced == MST_BWD_SCHEDULE_PAIRS) {
    p->blk_use = false;
    choose_dh128(p);
  }
  else if (forced == MST_BWD_SCHEDULE_AUTO) {
    if (!(best < pairs)) p->blk_use = false;
    choose_split_blocks(p);
    choose_dh128(p);
    choose_streamed(p);
  }
  // MST_BWD_SCHEDULE_BLOCKS and _BLOCKS_FUSED keep the best block shape whenever one fits
}

// `forced`: one of the MST_BWD_SCHEDULE_* values; only the backward's block shape depends on it.
// `fwd_cap`: if non-zero, the forward's groups of mini-sequences are shortened until the forward workspace fits
// into that many bytes (one mini-sequence per group at least; the caller checks f_total against the cap).
// `schedule`: whether the backward's order and block shape are needed.
mst_status make_plan(int64_t S, int64_t d, int64_t V, int32_t M, Plan* p, int forced = MST_BWD_SCHEDULE_AUTO,
                     size_t fwd_cap = 0, bool schedule = true) {
  if (S <= 0 || d <= 0 || V <= 0) return MST_ERR_BAD_SHAPE;
  if (d % 8 != 0) return MST_ERR_BAD_SHAPE;
  if (M < 1 || (int64_t)M > S) return MST_ERR_BAD_M;
  if (V * d >= (int64_t(1) << 31) || d >= (int64_t(1) << 22)) return MST_ERR_BAD_SHAPE;
  const int64_t C = (S + M - 1) / M;
  const int64_t ldg = (V + 7) / 8 * 8;
  if (C * ldg >= (int64_t(1) << 30) || C * d >= (int64_t(1) << 30)) return MST_ERR_BAD_SHAPE;
  p->S = S; p->d = d; p->V = V; p->M = M;
  p->C = (int)C;
  p->n_chunks = (int)((S + C - 1) / C);
  p->ldg = (int)ldg;
  p->n_vt = (int)((V + kTile - 1) / kTile);
  p->n_jt = (int)((d + kTile - 1) / kTile);
  p->n_st = (int)((C + kTile - 1) / kTile);
  // dH: few output tiles, long contraction -> split V so that the workgroups fill whole rounds of kNumCu (one workgroup
  // is resident per CU)
  const int out_tiles = p->n_st * p->n_jt;
  const int ksteps = (int)((V + kBK - 1) / kBK);
  const int64_t room = dh_split_room(p);
  const int split = best_dh_split(p, ksteps, kMaxDhSplit);
  p->dh_ksteps = (ksteps + split - 1) / split;
  p->dh_split = (ksteps + p->dh_ksteps - 1) / p->dh_ksteps;

  // Small problems: 64 x 64 tiles where they are estimated faster.  For dH that is ranked with its split count: splits
  // cost a reduce launch (4 us and the partials).
  {
    const double kd = (double)((d + kBK - 1) / kBK);
    p->small_dlogits = small_launch_us(tiles_of(C, V, 64), kd) < big_launch_us(tiles_of(C, V, 256), kd);
    const int64_t pair = p->n_chunks > 1 ? 2 * C : C;
    const double kw = (double)((pair + kBK - 1) / kBK);
    p->small_dw = small_launch_us(tiles_of(V, d, 64), kw) < big_launch_us(tiles_of(V, d, 256), kw);
    auto reduce_us = [&](int s) { return s > 1 ? 4.0 + (double)s * (double)(C * d) * 8.0 / 4.6e6 : 0.0; };
    double t_best = big_launch_us((double)out_tiles * p->dh_split, (double)p->dh_ksteps) + reduce_us(p->dh_split);
    p->small_dh = false;
    p->small_dh_split = p->small_dh_ksteps = 0;
    for (int s = 1; s <= 16 && s <= ksteps && (s == 1 || s <= room); s *= 2) {
      const int per = (ksteps + s - 1) / s;
      const double t = small_launch_us(tiles_of(C, d, 64) * s, (double)per) + reduce_us(s);
      if (t < t_best) {
        t_best = t;
        p->small_dh = true;
        p->small_dh_ksteps = per;
        p->small_dh_split = (ksteps + per - 1) / per;
      }
    }
  }

  // Forward: one GEMM launch per mini-sequence; the (max, sum) pairs per row and vocabulary tile of a group of
  // consecutive mini-sequences are merged by one launch.  A group is as many chunks as fit, with their pairs,
  // into half of one fp32 logits chunk (all of them at the paper-shaped configurations).
  {
    const int64_t per_chunk = ((int64_t)p->n_vt * 8 + 4) * C;
    int64_t g = (C * ldg * 2) / per_chunk;
    if (fwd_cap) {
      const int64_t fixed = (int64_t)sizeof(Control) + (S * 4 + 255) / 256 * 256 + 512;   // control, nll, padding
      const int64_t by_cap = ((int64_t)fwd_cap - fixed) / per_chunk;
      if (g > by_cap) g = by_cap;
    }
    if (g < 1) g = 1;
    if (g > p->n_chunks) g = p->n_chunks;
    p->fwd_group_rows = g * C;
  }
  size_t off = sizeof(Control);
  p->f_nll = off;  off = align_up(off + (size_t)S * 4, 256);
  p->f_tgt = off;  off = align_up(off + (size_t)p->fwd_group_rows * 4, 256);
  p->f_part = off; off = align_up(off + (size_t)p->n_vt * p->fwd_group_rows * 8, 256);
  p->f_total = off;

  p->b_slot = (size_t)C * ldg * 2;
  p->b_total = 2 * p->b_slot;
  p->b_ctl = align_up(p->b_total, 256);
  p->b_lse = p->b_ctl + sizeof(Control);
  p->b_fwd = p->b_lse + align_up((size_t)S * 4, 256);
  p->b_total_max = p->b_fwd + p->f_total;
  p->streamed = 0;
  if (schedule) choose_schedule(p, forced);
  return MST_OK;
}

// ------------------------------------------------------------------ profiling
mst_host::Profiler g_prof;
struct Scope : mst_host::Scope {
  Scope(hipStream_t s, int k) : mst_host::Scope(g_prof, s, k) {}
};

mst_host::PerDeviceOnce g_attr_once, g_shape_once;
// The tile maps and the schedule's cost model are written for the whole chip: kNumCu compute units in kNumXcd
// XCDs.  A partitioned device (fewer compute units behind one HIP device) would be mis-tiled, so it is refused.
bool device_is_whole_chip(int dev) {
  int cus = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return false;
  return cus == kNumCu;
}
bool set_kernel_attributes() {   // on the current device
  bool ok = true;
  auto set = [&ok](const void* f) {
    if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes) != hipSuccess) ok = false;
  };
  set((const void*)k_fwd_gemm_lse<false>);
  set((const void*)k_fwd_gemm_lse<true>);
  set((const void*)k_fwd_gemm_lse_small<TileFwd64>);
  set((const void*)k_fwd_gemm_lse_small<TileFwd32>);
  set((const void*)k_fwd_gemm_lse_rows128);
  set((const void*)k_bwd_gemm_dlogits_small<Tile64>);
  set((const void*)k_bwd_gemm_dlogits_small<Tile64Lone>);
  set((const void*)k_bwd_gemm_dh_small<Tile64>);
  set((const void*)k_bwd_gemm_dh_small<Tile64Lone>);
  set((const void*)k_bwd_gemm_dw_small<Tile64>);
  set((const void*)k_bwd_gemm_dw_small<Tile64Lone>);
  set((const void*)k_bwd_gemm_dh_dw_small<TileKSplit32x16, Tile64>);
  set((const void*)k_bwd_gemm_dh_dw_small<TileKSplit64x16, Tile64>);
  set((const void*)k_bwd_gemm_dh_dw_small<TileKSplit64x32, Tile64>);
  set((const void*)k_bwd_gemm_dh_split_dw_small<Tile64>);
  set((const void*)k_bwd_stream<Stream256, Stream256>);
  set((const void*)k_bwd_stream<Stream256Narrow, Stream256Narrow>);
  set((const void*)k_bwd_stream<Stream256SplitH, Stream256SplitW>);
  set((const void*)k_bwd_stream<Stream384, Stream384>);
  set((const void*)k_bwd_stream<Stream384Split, Stream384Split>);
  set((const void*)k_bwd_stream<Stream512, Stream512>);
  set((const void*)k_bwd_stream<Stream512Split, Stream512Split>);
  set((const void*)k_bwd_gemm_dlogits<false>);
  set((const void*)k_bwd_gemm_dlogits<true>);
  set((const void*)k_bwd_gemm_dh<false>);
  set((const void*)k_bwd_gemm_dh<true>);
  set((const void*)k_bwd_gemm_dw<false, false>);
  set((const void*)k_bwd_gemm_dw<true, false>);
  set((const void*)k_bwd_gemm_dw<false, true>);
  set((const void*)k_bwd_gemm_dw<true, true>);
  set((const void*)k_bwd_gemm_dh_dw<false, false>);
  set((const void*)k_bwd_gemm_dh_dw<true, false>);
  set((const void*)k_bwd_gemm_dh_dw<false, true>);
  set((const void*)k_bwd_gemm_dh_dw<true, true>);
  set((const void*)k_bwd_gemm_dh128_dw<false, false>);
  set((const void*)k_bwd_gemm_dh128_dw<true, false>);
  set((const void*)k_bwd_gemm_dh128_dw<false, true>);
  set((const void*)k_bwd_gemm_dh128_dw<true, true>);
  return ok;
}

auto dlogits_kernel(bool even) { return even ? k_bwd_gemm_dlogits<true> : k_bwd_gemm_dlogits<false>; }
auto dw_kernel(bool store_only, bool even) {
  return even ? (store_only ? k_bwd_gemm_dw<true, true> : k_bwd_gemm_dw<false, true>)
              : (store_only ? k_bwd_gemm_dw<true, false> : k_bwd_gemm_dw<false, false>);
}

mst_status check_launch() { return hipGetLastError() == hipSuccess ? MST_OK : MST_ERR_LAUNCH; }

mst_status prepare_device() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return MST_ERR_NO_DEVICE;
  if (!g_shape_once.run(dev, [dev] { return device_is_whole_chip(dev); })) {
    (void)hipGetLastError();
    return MST_ERR_NO_DEVICE;
  }
  if (!g_attr_once.run(dev, set_kernel_attributes)) {
    (void)hipGetLastError();
    return MST_ERR_LAUNCH;
  }
  return MST_OK;
}

// Rows of the forward's tiles (256 vocabulary entries wide; the same bits): the fewest of 32, 64 and 128 with which every
// workgroup has a compute unit to itself, else 256.  The groups after the first are not larger.  256 -> 128 rows: 200 rows,
// d = 4096, V = 32000: 83 us -> 64; 1000 rows, d = 512, V = 8000: 23 -> 19.  64 -> 32: 250 rows, d = 1024, V = 4000: 17.4 -> 13.3.
int forward_tile_rows(const Plan& p) {
  const int64_t rows = p.S < p.fwd_group_rows ? p.S : p.fwd_group_rows;
  for (const int e : {32, 64, 128})
    if ((rows + e - 1) / e * p.n_vt <= kNumCu) return e;
  return kTile;
}
// The forward's large launch is persistent (TileFeed) where it takes long: balancing the XCDs is worth 2 % of it, the queues'
// launch, the first fetch and the synchronisation per tile cost 10 to 20 us.  Rounds of tiles times K steps, persistent or not:
// 1984 (4096 rows, d = 4096, V = 128256) 2860 us against 2878, 647: 1096 against 1117, 592: the same, 499: 773 against 755,
// 128 (200 rows, d = 4096, V = 128256): 252 against 234.
constexpr int64_t kPersistentSteps = 600;
int64_t forward_group_rows(const Plan& p, int64_t g0) { return std::min(p.S - g0, p.fwd_group_rows); }
int forward_row_tiles(const Plan& p, int64_t g0, int tile_rows) {
  return (int)((forward_group_rows(p, g0) + tile_rows - 1) / tile_rows);
}
bool persistent_forward(const Plan& p) {                           // decided by the first group
  const int64_t grid = xcd_grid_2d(p.n_vt, forward_row_tiles(p, 0, kTile));
  return forward_tile_rows(p) == kTile && (grid + kNumCu - 1) / kNumCu * ((p.d + kBK - 1) / kBK) >= kPersistentSteps;
}

// One workgroup finishes the forward call: a row per thread, its pairs in registers.  At 8192 pairs (512 rows, V = 4096) the
// call takes 12.5 us instead of 15.0, at 9600 15.2 instead of 17.1, at 32000 1 us more.
bool finalize_in_one(const Plan& p) {
  return p.S <= 1024 && p.S <= p.fwd_group_rows && p.n_vt <= kFinOneTiles && p.S * p.n_vt <= 12288;
}

// forward pass over all chunks: writes lse (if non-null) and nll (if non-null)
// `ctl`: its queues serve persistent forward launches (nullptr: one workgroup per tile)
mst_status run_forward_chunks(const Plan& p, const __bf16* H, const __bf16* W, const int32_t* labels,
                              int ignore_index, char* ws, float* lse, float* nll, hipStream_t st, Control* ctl = nullptr, bool finalize = true) {
  float* tgt = reinterpret_cast<float*>(ws + p.f_tgt);
  float2* part = reinterpret_cast<float2*>(ws + p.f_part);
  const size_t stride = (size_t)p.fwd_group_rows;
  const int tile_rows = forward_tile_rows(p);
  int* queue = ctl && persistent_forward(p) ? ctl->queue : nullptr;
  int queue_base = 0;
  if (queue) {
    Scope sc(st, MST_K_LABEL_SCAN);
    hipLaunchKernelGGL(k_clear_queues, dim3(1), dim3(64), 0, st, ctl);
  }
  for (int64_t g0 = 0; g0 < p.S; g0 += p.fwd_group_rows) {
    const int64_t g_rows = forward_group_rows(p, g0);
    // One launch for the group's mini-sequences.  Rows are independent and no logits are stored, so the row tiles
    // of the launch need not respect the boundaries between the mini-sequences of the group: a mini-sequence
    // shorter than a 256-row tile costs no idle tile rows, and every row's result is bit-identical for every M.
    const int n_st = forward_row_tiles(p, g0, tile_rows);
    if (tile_rows == kTile) {
      Scope sc(st, MST_K_FWD_GEMM_LSE);
      const bool even = !queue && forward_even_map(p.n_vt, n_st);
      const int tiles = launch_grid(even, p.n_vt, n_st);
      const int grid = queue && tiles > kNumCu ? kNumCu : tiles;
      hipLaunchKernelGGL(even ? k_fwd_gemm_lse<true> : k_fwd_gemm_lse<false>, dim3(grid), dim3(kThreads), kLdsBytes, st,
                         H + g0 * p.d, W, labels + g0, (int)g_rows, (int)p.d, (int)p.V, n_st, p.n_vt,
                         part, stride, tgt, queue, queue_base);
      queue_base += tiles / kNumXcd + grid;
    } else {
      Scope sc(st, MST_K_FWD_GEMM_LSE);
      const auto kernel = tile_rows == 128 ? k_fwd_gemm_lse_rows128
                        : tile_rows == 64 ? k_fwd_gemm_lse_small<TileFwd64> : k_fwd_gemm_lse_small<TileFwd32>;
      const int threads = tile_rows == 128 ? kThreads : TileFwd64::kThreads;
      const int lds = tile_rows == 128 ? Tile16Rows128::kLds : tile_rows == 64 ? TileFwd64::kLds : TileFwd32::kLds;
      hipLaunchKernelGGL(kernel, dim3(even_grid(p.n_vt, n_st)), dim3(threads), lds, st,
                         H + g0 * p.d, W, labels + g0, (int)g_rows, (int)p.d, (int)p.V, n_st, p.n_vt, part, stride, tgt);
    }
    if (finalize) {
      Scope sc(st, MST_K_LSE_FINALIZE);
      hipLaunchKernelGGL(k_lse_finalize, dim3((unsigned)((g_rows + kFinRows - 1) / kFinRows)), dim3(kFinRows * kFinGroups), 0, st,
                         part, stride, p.n_vt, tgt, labels + g0, (int)g_rows, (int)p.V, ignore_index,
                         lse ? lse + g0 : nullptr, nll ? nll + g0 : nullptr);
    }
  }
  return check_launch();
}

// dH and dW of the rows whose dlogits are at G, one launch of small tiles
template <class CH>
void launch_ksplit(hipStream_t st, const Plan& p, const __bf16* G, const __bf16* W, const __bf16* H, int rows, int accumulate,
                   int last, const long long* n_valid, float grad_loss, __bf16* dH, float* dW) {
  const int n_sh = (rows + CH::EB - 1) / CH::EB, n_jh = (int)((p.d + CH::EA - 1) / CH::EA), dh_grid = even_grid(n_jh, n_sh);
  const int n_vh = (int)((p.V + Tile64::EB - 1) / Tile64::EB), n_jw = (int)((p.d + Tile64::EA - 1) / Tile64::EA);
  hipLaunchKernelGGL((k_bwd_gemm_dh_dw_small<CH, Tile64>), dim3(dh_grid + even_grid(n_vh, n_jw)), dim3(Tile64::kThreads),
                     CH::kLds > Tile64::kLds ? CH::kLds : Tile64::kLds, st, G, p.ldg, W, H, rows, (int)p.d, (int)p.V,
                     n_sh, n_jh, dh_grid, n_vh, n_jw, accumulate, last, n_valid, grad_loss, dH, dW);
}

mst_status check_forward_alignment(const void* H, const void* W, const int32_t* labels, const float* loss,
                                   const float* lse, const int64_t* n_valid) {
  if (misaligned(H, 16) || misaligned(W, 16) || misaligned(lse, 4) || misaligned(labels, 4) || misaligned(loss, 4) ||
      misaligned(n_valid, 8))
    return MST_ERR_ALIGNMENT;
  return MST_OK;
}

// everything the forward call enqueues, on workspace `ws` of p.f_total bytes
mst_status enqueue_forward(const Plan& p, const void* H, const void* W, const int32_t* labels, int32_t ignore_index,
                           char* ws, float* loss, float* lse, int64_t* n_valid, void* stream) {
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  float* nll = reinterpret_cast<float*>(ws + p.f_nll);
  const bool one = finalize_in_one(p);
  const mst_status s = run_forward_chunks(p, static_cast<const __bf16*>(H), static_cast<const __bf16*>(W), labels, ignore_index,
                                          ws, lse, nll, st, reinterpret_cast<Control*>(ws), !one);
  if (s != MST_OK) return s;
  Scope sc(st, MST_K_LOSS_REDUCE);
  if (one) {
    hipLaunchKernelGGL(k_finalize_loss, dim3(1), dim3(1024), 0, st, reinterpret_cast<const float2*>(ws + p.f_part),
                       (size_t)p.fwd_group_rows, p.n_vt, reinterpret_cast<const float*>(ws + p.f_tgt), labels, (int)p.S, (int)p.V,
                       ignore_index, lse, loss, reinterpret_cast<long long*>(n_valid));
  } else {
    hipLaunchKernelGGL(k_loss_reduce, dim3(1), dim3(1024), 0, st, nll, labels, (long long)p.S, (int)p.V, ignore_index, loss,
                       reinterpret_cast<long long*>(n_valid));
  }
  return check_launch();
}

// Scratch of the entry point that allocates nothing: one array per GPU, part of the code object, alive until
// the process ends.  Its name is only a host-side handle; the device address is asked for once per device
// (with that device current) and kept, and only that address is ever handed to a kernel.
__device__ __align__(256) static unsigned char scratch[MST_STATIC_SCRATCH_BYTES];
std::mutex g_scratch_mu;
char* g_scratch_ptr[mst_host::PerDeviceOnce::kMaxDevices] = {};
char* static_scratch_of_current_device() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= mst_host::PerDeviceOnce::kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
      (void)hipGetLastError();
      return nullptr;
    }
    g_scratch_ptr[dev] = static_cast<char*>(ptr);
  }
  return g_scratch_ptr[dev];
}

}  // namespace

extern "C" {

const char* mst_strerror(mst_status s) {
  switch (s) {
    case MST_OK: return "ok";
    case MST_ERR_NULL_POINTER: return "a required pointer is NULL";
    case MST_ERR_BAD_SHAPE: return "bad shape: S, d, V must be positive, d % 8 == 0, d < 2^22, V*d < 2^31, ceil(S/M)*V < 2^30";
    case MST_ERR_BAD_M: return "M must satisfy 1 <= M <= S";
    case MST_ERR_WORKSPACE: return "workspace is NULL or too small (see mst_workspace_bytes)";
    case MST_ERR_ALIGNMENT: return "pointer alignment: H, W, dH, dW 16 bytes; workspace 256 bytes; n_valid 8 bytes; labels, lse, loss 4 bytes";
    case MST_ERR_LAUNCH: return "the HIP runtime refused a kernel launch or attribute";
    case MST_ERR_NO_DEVICE: return "no current HIP device, or it is not a whole 256-CU gfx950 chip";
    default: return "unknown status";
  }
}

const char* mst_version(void) { return "mst-lmhead 0.1 (gfx950)"; }

int32_t mst_suggest_m(int64_t S, int64_t d, int64_t V) {
  if (S <= 0 || d <= 0 || V <= 0) return 0;
  int64_t m = (2 * V + d) / (2 * d);             // V / d to the nearest integer
  const int64_t by_rows = S / kTile;             // most chunks that still have one full block tile of rows
  if (m > by_rows) m = by_rows;
  if (m < 1) m = 1;
  if (m > 0x7fffffff) m = 0x7fffffff;
  return (int32_t)m;
}

mst_status mst_mfma_probe(int32_t blocks, int32_t iters, float scale, float* sink, void* stream) {
  if (blocks < 1 || blocks > (1 << 20) || iters < 1 || iters > (1 << 20)) return MST_ERR_BAD_SHAPE;
  if (!sink) return MST_ERR_NULL_POINTER;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return MST_ERR_NO_DEVICE;
  hipLaunchKernelGGL(k_mfma_probe, dim3(blocks), dim3(kThreads), 0, reinterpret_cast<hipStream_t>(stream),
                     sink, iters, scale);
  return check_launch();
}

mst_status mst_shift_labels(const int32_t* labels_in, int64_t B, int64_t L, int32_t ignore_index,
                            int32_t* labels_out, void* stream) {
  if (B <= 0 || L <= 0 || B >= (int64_t(1) << 40) / L) return MST_ERR_BAD_SHAPE;
  if (!labels_in || !labels_out) return MST_ERR_NULL_POINTER;
  if (misaligned(labels_in, 4) || misaligned(labels_out, 4)) return MST_ERR_ALIGNMENT;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return MST_ERR_NO_DEVICE;
  const long long n = (long long)(B * L);
  hipLaunchKernelGGL(k_shift_labels, dim3((unsigned)((n + 255) / 256)), dim3(256), 0,
                     reinterpret_cast<hipStream_t>(stream), labels_in, n, (long long)L, ignore_index, labels_out);
  return check_launch();
}

mst_status mst_workspace_bytes(int64_t S, int64_t d, int64_t V, int32_t M, size_t* fwd_bytes, size_t* bwd_bytes) {
  Plan p;
  mst_status s = make_plan(S, d, V, M, &p, MST_BWD_SCHEDULE_AUTO, 0, false);
  if (s != MST_OK) return s;
  if (fwd_bytes) *fwd_bytes = p.f_total;
  if (bwd_bytes) *bwd_bytes = p.b_total;
  return MST_OK;
}

mst_status mst_lmhead_ce_fwd(const void* H, const void* W, const int32_t* labels, int64_t S, int64_t d, int64_t V,
                             int32_t ignore_index, int32_t M, void* workspace, size_t workspace_bytes,
                             float* loss, float* lse, int64_t* n_valid, void* stream) {
  Plan p;
  mst_status s = make_plan(S, d, V, M, &p, MST_BWD_SCHEDULE_AUTO, 0, false);
  if (s != MST_OK) return s;
  if (!H || !W || !labels || !loss) return MST_ERR_NULL_POINTER;
  if (!workspace || workspace_bytes < p.f_total) return MST_ERR_WORKSPACE;
  if (misaligned(workspace, 256)) return MST_ERR_ALIGNMENT;
  if ((s = check_forward_alignment(H, W, labels, loss, lse, n_valid)) != MST_OK) return s;
  if ((s = prepare_device()) != MST_OK) return s;
  return enqueue_forward(p, H, W, labels, ignore_index, static_cast<char*>(workspace), loss, lse, n_valid, stream);
}

mst_status mst_lmhead_ce_fwd_static(const void* H, const void* W, const int32_t* labels, int64_t S, int64_t d, int64_t V,
                                    int32_t ignore_index, int32_t M, float* loss, float* lse, int64_t* n_valid,
                                    void* stream) {
  Plan p;
  mst_status s = make_plan(S, d, V, M, &p, MST_BWD_SCHEDULE_AUTO, (size_t)MST_STATIC_SCRATCH_BYTES, false);
  if (s != MST_OK) return s;
  if (!H || !W || !labels || !loss) return MST_ERR_NULL_POINTER;
  if (p.f_total > (size_t)MST_STATIC_SCRATCH_BYTES) return MST_ERR_WORKSPACE;   // one mini-sequence alone is too large
  if ((s = check_forward_alignment(H, W, labels, loss, lse, n_valid)) != MST_OK) return s;
  if ((s = prepare_device()) != MST_OK) return s;
  char* ws = static_scratch_of_current_device();
  if (!ws) return MST_ERR_LAUNCH;
  return enqueue_forward(p, H, W, labels, ignore_index, ws, loss, lse, n_valid, stream);
}

mst_status mst_lmhead_ce_bwd(const void* H, const void* W, const int32_t* labels, int64_t S, int64_t d, int64_t V,
                             int32_t ignore_index, int32_t M, float grad_loss, const float* lse,
                             const int64_t* n_valid, void* workspace, size_t workspace_bytes,
                             void* dH, float* dW, void* stream) {
  Plan p;
  mst_status s = make_plan(S, d, V, M, &p, t_bwd_schedule);
  if (s != MST_OK) return s;
  if (!H || !W || !labels || !dH || !dW) return MST_ERR_NULL_POINTER;
  const size_t need = !lse ? p.b_total_max : (!n_valid ? p.b_lse : p.b_total);
  if (!workspace || workspace_bytes < need) return MST_ERR_WORKSPACE;
  if (misaligned(H, 16) || misaligned(W, 16) || misaligned(dH, 16) || misaligned(workspace, 256) ||
      misaligned(lse, 4) || misaligned(dW, 16) || misaligned(labels, 4) || misaligned(n_valid, 8))
    return MST_ERR_ALIGNMENT;
  if ((s = prepare_device()) != MST_OK) return s;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
  const __bf16* Hb = static_cast<const __bf16*>(H);
  const __bf16* Wb = static_cast<const __bf16*>(W);
  const long long* nv = reinterpret_cast<const long long*>(n_valid);
  if (!nv) {
    Control* ctl = reinterpret_cast<Control*>(ws + p.b_ctl);
    Scope sc(st, MST_K_LABEL_SCAN);
    hipLaunchKernelGGL(k_label_scan, dim3(1), dim3(1024), 0, st, labels, (long long)S, (int)V, ignore_index, ctl);
    nv = &ctl->n_valid_checked;   // -1 if a label is outside [0, V): dH and dW then come out NaN
  }
  if (!lse) {
    // no saved log-sum-exp: run the forward's pass first, in the tail of the workspace
    float* lse_tmp = reinterpret_cast<float*>(ws + p.b_lse);
    s = run_forward_chunks(p, Hb, Wb, labels, ignore_index, ws + p.b_fwd, lse_tmp, nullptr, st);
    if (s != MST_OK) return s;
    lse = lse_tmp;
  }
  __bf16* slot[2] = {reinterpret_cast<__bf16*>(ws), reinterpret_cast<__bf16*>(ws + p.b_slot)};
  __bf16* dHb = static_cast<__bf16*>(dH);
  if (p.streamed) {
    float* const partial = reinterpret_cast<float*>(ws);
    {
      Scope sc(st, MST_K_BWD_GEMM_DLOGITS);
      const StreamProblem q = {Hb, Wb, labels, lse, (int)S, (int)d, (int)V, ignore_index, nv, grad_loss};
      kStreamForms[p.streamed - 1].launch(st, q, p.stream_split, p.stream_per_split, partial, dHb, dW);
    }
    if (p.stream_split > 1) {
      Scope sc(st, MST_K_BWD_DH_REDUCE);
      const size_t n = (size_t)S * d;
      hipLaunchKernelGGL(k_bwd_dh_reduce, dim3((unsigned)((n / 8 + 255) / 256)), dim3(256), 0, st, partial, p.stream_split, n, n, nv,
                         grad_loss, dHb);
    }
    return check_launch();
  }

  auto rows_of = [&](int i) { const int64_t r0 = (int64_t)i * p.C; return (int)((p.S - r0) < p.C ? (p.S - r0) : p.C); };
  auto dlogits = [&](int i, int rows, __bf16* G) {        // of `rows` rows from chunk i on
    const int64_t r0 = (int64_t)i * p.C;
    const int n_st = (rows + kTile - 1) / kTile;
    Scope sc(st, MST_K_BWD_GEMM_DLOGITS);
    if (p.joint == MST_PAIR_DH128 ? small_pair_dlogits(p, rows) : p.small_dlogits) {
      const int n_vh = (int)((p.V + Tile64::EA - 1) / Tile64::EA), n_sh = (rows + Tile64::EB - 1) / Tile64::EB;
      const bool lone = lone_small((double)n_vh * n_sh);
      hipLaunchKernelGGL(lone ? k_bwd_gemm_dlogits_small<Tile64Lone> : k_bwd_gemm_dlogits_small<Tile64>,
                         dim3(even_grid(n_vh, n_sh)), dim3(Tile64::kThreads), lone ? Tile64Lone::kLds : Tile64::kLds, st,
                         Hb + r0 * p.d, Wb, labels + r0, lse + r0, rows, (int)p.d, (int)p.V, ignore_index, n_sh, n_vh, G, p.ldg);
      return;
    }
    const bool even = use_even_map(p.n_vt, n_st);
    hipLaunchKernelGGL(dlogits_kernel(even), dim3(launch_grid(even, p.n_vt, n_st)), dim3(kThreads), kLdsBytes, st,
                       Hb + r0 * p.d, Wb, labels + r0, lse + r0, rows, (int)p.d, (int)p.V, 0, (int)p.V, ignore_index,
                       n_st, p.n_vt, G, p.ldg);
  };
  auto dh_reduce = [&](int i, int rows, const void* partial, int split) {
    Scope sc(st, MST_K_BWD_DH_REDUCE);
    const size_t n = (size_t)rows * p.d;
    hipLaunchKernelGGL(k_bwd_dh_reduce, dim3((unsigned)((n / 8 + 255) / 256)), dim3(256), 0, st,
                       static_cast<const float*>(partial), split, (size_t)p.C * p.d, n, nv, grad_loss, dHb + (int64_t)i * p.C * p.d);
  };
  auto grad_h = [&](int i, const __bf16* G, void* partial_space) {
    const int64_t r0 = (int64_t)i * p.C;
    const int rows = rows_of(i), n_st = (rows + kTile - 1) / kTile;
    float* partial = static_cast<float*>(partial_space);
    const int split = p.small_dh ? p.small_dh_split : p.dh_split;
    {
      Scope sc(st, MST_K_BWD_GEMM_DH);
      if (p.small_dh) {
        const int n_jh = (int)((p.d + Tile64::EA - 1) / Tile64::EA), n_sh = (rows + Tile64::EB - 1) / Tile64::EB;
        const bool lone = lone_small((double)n_jh * n_sh * split);
        hipLaunchKernelGGL(lone ? k_bwd_gemm_dh_small<Tile64Lone> : k_bwd_gemm_dh_small<Tile64>,
                           dim3(even_grid(n_jh * split, n_sh)), dim3(Tile64::kThreads), lone ? Tile64Lone::kLds : Tile64::kLds, st,
                           G, p.ldg, Wb, rows, (int)p.d, (int)p.V, n_sh, n_jh, split, p.small_dh_ksteps, nv, grad_loss,
                           partial, p.C, dHb + r0 * p.d);
      } else {
        hipLaunchKernelGGL(k_bwd_gemm_dh<false>, dim3(xcd_grid(n_st * p.n_jt * p.dh_split)), dim3(kThreads), kLdsBytes, st,
                           G, p.ldg, Wb, rows, (int)p.d, (int)p.V, n_st, p.n_jt, p.dh_split, p.dh_ksteps, kDhSplit,
                           nv, grad_loss, partial, p.C, dHb + r0 * p.d);
      }
    }
    if (split > 1) dh_reduce(i, rows, partial, split);
  };
  auto grad_w = [&](int i_first, int i_last, int rows) {
    const int64_t r0 = (int64_t)i_first * p.C;
    Scope sc(st, MST_K_BWD_GEMM_DW);
    if (p.small_dw) {
      const int n_vh = (int)((p.V + Tile64::EB - 1) / Tile64::EB), n_jh = (int)((p.d + Tile64::EA - 1) / Tile64::EA);
      const bool lone = lone_small((double)n_vh * n_jh);
      hipLaunchKernelGGL(lone ? k_bwd_gemm_dw_small<Tile64Lone> : k_bwd_gemm_dw_small<Tile64>,
                         dim3(even_grid(n_vh, n_jh)), dim3(Tile64::kThreads), lone ? Tile64Lone::kLds : Tile64::kLds, st,
                         slot[0], p.ldg, Hb + r0 * p.d, rows, (int)p.d, (int)p.V, n_vh, n_jh, i_first > 0 ? 1 : 0,
                         i_last == p.n_chunks - 1 ? 1 : 0, nv, grad_loss, dW);
      return;
    }
    const bool even = use_even_map(p.n_vt, p.n_jt);
    hipLaunchKernelGGL(dw_kernel(i_first == 0, even), dim3(launch_grid(even, p.n_vt, p.n_jt)),
                       dim3(kThreads), kLdsBytes, st,
                       slot[0], p.ldg, Hb + r0 * p.d, rows, (int)p.d, (int)p.V, p.n_vt, p.n_jt,
                       i_last == p.n_chunks - 1 ? 1 : 0, nv, grad_loss, dW);
  };

  if (p.blk_use) {
    // Block schedule: for each block of rows, walk the vocabulary windows.  Per (row block, window):
    //   dlogits of the block -> workspace | dH sums of the row block (+)= G W_window | dW_window (+)= G^T H_block
    // dH of a row block is final after its last window, dW of a window after the last row block; both
    // accumulate in a fixed order.
    __bf16* G = reinterpret_cast<__bf16*>(ws);
    float* dh_sums = reinterpret_cast<float*>(ws + p.blk_acc);
    auto launch_dh_reduce_tiles = [&](int n_st, int rows, int64_t r0) {
      Scope sc(st, MST_K_BWD_DH_REDUCE);
      const int waves = n_st * p.n_jt * kTA16 * Tile16::kWaves;       // a multiple of the 4 of a workgroup
      hipLaunchKernelGGL(k_bwd_dh_reduce_tiles, dim3(waves / 4), dim3(256), 0, st, dh_sums, p.blk_split, n_st, p.n_jt, rows,
                         (int)p.d, nv, grad_loss, dHb + r0 * p.d);
    };
    for (int rb = 0; rb < p.blk_n_rb; ++rb) {
      const int64_t r0 = (int64_t)rb * p.blk_rows;
      const int rows = (int)((p.S - r0) < p.blk_rows ? (p.S - r0) : p.blk_rows);
      const int n_st = (rows + kTile - 1) / kTile;
      for (int w = 0; w < p.blk_n_win; ++w) {
        const int t0 = w * p.blk_win_tiles;
        const int tiles_w = t0 + p.blk_win_tiles <= p.n_vt ? p.blk_win_tiles : p.n_vt - t0;
        const int64_t v_base = (int64_t)t0 * kTile;
        const int Vw = (int)((p.V - v_base) < (int64_t)tiles_w * kTile ? (p.V - v_base) : (int64_t)tiles_w * kTile);
        {
          Scope sc(st, MST_K_BWD_GEMM_DLOGITS);
          const bool even = use_even_map(tiles_w, n_st);
          hipLaunchKernelGGL(dlogits_kernel(even), dim3(launch_grid(even, tiles_w, n_st)), dim3(kThreads), kLdsBytes, st,
                             Hb + r0 * p.d, Wb + v_base * p.d, labels + r0, lse + r0, rows, (int)p.d, Vw, (int)v_base,
                             (int)p.V, ignore_index, n_st, tiles_w, G, p.blk_ldg);
        }
        const bool last_win = w == p.blk_n_win - 1;
        const int mode = p.blk_split > 1 ? (w == 0 ? kDhFirst : kDhAdd)
                                         : (w == 0 ? (last_win ? kDhOnly : kDhFirst) : (last_win ? kDhLast : kDhAdd));
        const int dw_last = rb == p.blk_n_rb - 1 ? 1 : 0;
        if (p.blk_fused) {
          Scope sc(st, MST_K_BWD_GEMM_DH_DW);
          auto dh_share = [&](bool even) {
            return even ? xcd_share(p.blk_split * p.n_jt, n_st, true) : p.blk_split * xcd_share(n_st, p.n_jt, false);
          };
          auto share = [&](bool even) { return dh_share(even) + xcd_share(tiles_w, p.n_jt, even); };
          const bool both = saves_a_round(share(false), share(true));
          const bool dh_even = both || uneven_over_xcds(n_st) || saves_a_round(dh_share(false), dh_share(true));
          const bool dw_even = both || use_even_map(tiles_w, p.n_jt);
          const bool general = p.blk_split > 1 || dh_even || dw_even;
          const int dh_grid = dh_grid_2d(dh_even, p.blk_split, n_st, p.n_jt);
          hipLaunchKernelGGL(general ? (rb > 0 ? k_bwd_gemm_dh_dw<false, true> : k_bwd_gemm_dh_dw<true, true>)
                                     : (rb > 0 ? k_bwd_gemm_dh_dw<false, false> : k_bwd_gemm_dh_dw<true, false>),
                             dim3(dh_grid + launch_grid(dw_even, tiles_w, p.n_jt)), dim3(kThreads), kLdsBytes, st,
                             G, p.blk_ldg, Wb + v_base * p.d, Hb + r0 * p.d, rows, (int)p.d, Vw, n_st, tiles_w, p.n_jt,
                             dh_grid, mode, dw_last, nv, grad_loss, dh_sums, p.blk_rows, dHb + r0 * p.d,
                             dW + v_base * p.d, p.blk_split, dh_even ? 1 : 0, dw_even ? 1 : 0);
          if (last_win && p.blk_split > 1) launch_dh_reduce_tiles(n_st, rows, r0);
        } else {
          {
            Scope sc(st, MST_K_BWD_GEMM_DH);
            const bool even = use_even_map(n_st, p.n_jt);
            hipLaunchKernelGGL(even ? k_bwd_gemm_dh<true> : k_bwd_gemm_dh<false>, dim3(dh_grid_2d(even, 1, n_st, p.n_jt)), dim3(kThreads), kLdsBytes, st,
                               G, p.blk_ldg, Wb + v_base * p.d, rows, (int)p.d, Vw, n_st, p.n_jt, 1, (Vw + kBK - 1) / kBK, mode,
                               nv, grad_loss, dh_sums, p.blk_rows, dHb + r0 * p.d);
          }
          {
            Scope sc(st, MST_K_BWD_GEMM_DW);
            const bool even = use_even_map(tiles_w, p.n_jt);
            hipLaunchKernelGGL(dw_kernel(rb == 0, even), dim3(launch_grid(even, tiles_w, p.n_jt)),
                               dim3(kThreads), kLdsBytes, st,
                               G, p.blk_ldg, Hb + r0 * p.d, rows, (int)p.d, Vw, tiles_w, p.n_jt,
                               dw_last, nv, grad_loss, dW + v_base * p.d);
          }
        }
      }
    }
    return check_launch();
  }

  // Algorithm 4's loop over mini-sequences, two at a time: the chunk pair (A, B) shares one dW pass.
  //   dlogits(A) -> slot 0 | dH(A), partials in slot 1 | dlogits(B) -> slot 1 | dW += [G_A; G_B]^T [H_A; H_B]
  //   | dH(B), partials in slot 0
  if (p.joint == MST_PAIR_SPLIT) {
    const int rows = (int)p.S, split = p.small_dh_split;
    const int n_vh = (int)((p.V + Tile64::EB - 1) / Tile64::EB), n_jh = (int)((p.d + Tile64::EA - 1) / Tile64::EA);
    const int n_sh = (rows + Tile64::EB - 1) / Tile64::EB, dh_grid = even_grid(n_jh * split, n_sh);
    dlogits(0, rows, slot[0]);
    {
      Scope sc(st, MST_K_BWD_GEMM_DH_DW);
      hipLaunchKernelGGL(k_bwd_gemm_dh_split_dw_small<Tile64>, dim3(dh_grid + even_grid(n_vh, n_jh)), dim3(Tile64::kThreads),
                         Tile64::kLds, st, slot[0], p.ldg, Wb, Hb, rows, (int)p.d, (int)p.V, n_sh, n_jh, split, p.small_dh_ksteps,
                         dh_grid, n_vh, nv, grad_loss, reinterpret_cast<float*>(slot[1]), dHb, dW);
    }
    if (split > 1) dh_reduce(0, rows, slot[1], split);
    return check_launch();
  }
  if (p.joint == MST_PAIR_DH128) {
    const bool even = use_even_map(p.n_vt, p.n_jt);
    for (int ia = 0; ia < p.n_chunks; ia += 2) {          // the two slots are contiguous: the pair's dlogits are one matrix
      const int64_t r0 = (int64_t)ia * p.C;
      const int rows = (int)std::min(2 * (int64_t)p.C, p.S - r0);
      const int n_sq = (rows + Tile16Quarter::EB - 1) / Tile16Quarter::EB, n_jq = (int)((p.d + Tile16Quarter::EA - 1) / Tile16Quarter::EA);
      dlogits(ia, rows, slot[0]);
      Scope sc(st, MST_K_BWD_GEMM_DH_DW);
      const auto kernel = even ? (ia > 0 ? k_bwd_gemm_dh128_dw<false, true> : k_bwd_gemm_dh128_dw<true, true>)
                               : (ia > 0 ? k_bwd_gemm_dh128_dw<false, false> : k_bwd_gemm_dh128_dw<true, false>);
      const int dh_grid = even_grid(n_jq, n_sq);
      hipLaunchKernelGGL(kernel, dim3(dh_grid + launch_grid(even, p.n_vt, p.n_jt)), dim3(kThreads), kLdsBytes, st, slot[0], p.ldg, Wb,
                         Hb + r0 * p.d, rows, (int)p.d, (int)p.V, n_sq, n_jq, dh_grid, p.n_vt, p.n_jt, ia + 2 >= p.n_chunks ? 1 : 0,
                         nv, grad_loss, dHb + r0 * p.d, dW);
    }
    return check_launch();
  }
  if (p.joint) {
    // the two slots are contiguous: the pair's dlogits are one matrix
    for (int ia = 0; ia < p.n_chunks; ia += 2) {
      const int64_t r0 = (int64_t)ia * p.C;
      const int rows = (int)std::min(2 * (int64_t)p.C, p.S - r0);
      dlogits(ia, rows, slot[0]);
      Scope sc(st, MST_K_BWD_GEMM_DH_DW);
      const auto launch = p.joint == MST_PAIR_KSPLIT_32X16 ? launch_ksplit<TileKSplit32x16>
                        : p.joint == MST_PAIR_KSPLIT_64X16 ? launch_ksplit<TileKSplit64x16> : launch_ksplit<TileKSplit64x32>;
      launch(st, p, slot[0], Wb, Hb + r0 * p.d, rows, ia > 0 ? 1 : 0, ia + 2 >= p.n_chunks ? 1 : 0, nv, grad_loss, dHb + r0 * p.d, dW);
    }
    return check_launch();
  }
  for (int ia = 0; ia < p.n_chunks; ia += 2) {
    const int ib = ia + 1;
    dlogits(ia, rows_of(ia), slot[0]);
    grad_h(ia, slot[0], slot[1]);
    if (ib < p.n_chunks) {
      dlogits(ib, rows_of(ib), slot[1]);
      grad_w(ia, ib, p.C + rows_of(ib));
      grad_h(ib, slot[1], slot[0]);
    } else {
      grad_w(ia, ia, rows_of(ia));
    }
  }
  return check_launch();
}

mst_status mst_set_bwd_schedule(int32_t schedule) {
  if (schedule < MST_BWD_SCHEDULE_AUTO || schedule > MST_BWD_SCHEDULE_BLOCKS_FUSED) return MST_ERR_BAD_SHAPE;
  t_bwd_schedule = schedule;
  return MST_OK;
}

mst_status mst_bwd_schedule_info(int64_t S, int64_t d, int64_t V, int32_t M, int64_t* info) {
  return mst_bwd_schedule_info_for(S, d, V, M, t_bwd_schedule, info);
}

mst_status mst_bwd_schedule_info_for(int64_t S, int64_t d, int64_t V, int32_t M, int32_t schedule, int64_t* info) {
  if (!info) return MST_ERR_NULL_POINTER;
  if (schedule < MST_BWD_SCHEDULE_AUTO || schedule > MST_BWD_SCHEDULE_BLOCKS_FUSED) return MST_ERR_BAD_SHAPE;
  Plan p;
  const mst_status s = make_plan(S, d, V, M, &p, schedule);
  if (s != MST_OK) return s;
  info[0] = p.blk_use ? (p.blk_fused ? MST_BWD_SCHEDULE_BLOCKS_FUSED : MST_BWD_SCHEDULE_BLOCKS) : MST_BWD_SCHEDULE_PAIRS;
  info[1] = p.blk_use ? p.blk_rows : 2 * (int64_t)p.C;
  info[2] = p.blk_use ? p.blk_n_rb : (p.n_chunks + 1) / 2;
  info[3] = p.blk_use ? (int64_t)p.blk_win_tiles * kTile : p.V;
  info[4] = p.blk_use ? p.blk_n_win : 1;
  info[5] = p.blk_use ? p.blk_split : p.joint == MST_PAIR_DH128 ? 1 : p.joint && p.joint != MST_PAIR_SPLIT ? TileKSplit64x16::kSplit : p.small_dh ? p.small_dh_split : p.dh_split;
  info[6] = (int64_t)p.est_pairs_us;
  info[7] = (int64_t)p.est_blocks_us;
  return MST_OK;
}

int32_t mst_tile_of_workgroup(int32_t n_slow, int32_t n_fast, int32_t order, int32_t workgroup, int32_t* slow,
                              int32_t* fast) {
  if (n_slow < 1 || n_fast < 1 || workgroup < 0 || !slow || !fast || order < 0 || order > 1) return -1;
  if (workgroup >= xcd_grid_2d(n_slow, n_fast)) return -1;
  int s = 0, f = 0;
  const bool ok = order == 0
      ? xcd_tile_of_block<kXcdRectSlow, kXcdRectFast, kXcdSuper>(workgroup, n_slow, n_fast, &s, &f)
      : xcd_tile_of_block<kXcdRectSlow, kXcdRectFast, kXcdRectFast>(workgroup, n_slow, n_fast, &s, &f);
  *slow = s;
  *fast = f;
  return ok ? 1 : 0;
}

int32_t mst_tile_grid(int32_t n_slow, int32_t n_fast) {
  if (n_slow < 1 || n_fast < 1 || (int64_t)xcd_grid_2d(n_slow, 1) * n_fast > 0x7fffffff) return -1;
  return xcd_grid_2d(n_slow, n_fast);
}

int32_t mst_dh_tile_grid(int32_t even, int32_t n_split, int32_t n_row_tiles, int32_t n_col_tiles) {
  if (n_split < 1 || n_row_tiles < 1 || n_col_tiles < 1) return -1;
  if ((int64_t)n_split * n_col_tiles * (kNumXcd * (((int64_t)n_row_tiles + kNumXcd - 1) / kNumXcd)) > 0x7ffffff0) return -1;
  return dh_grid_2d(even != 0, n_split, n_row_tiles, n_col_tiles);
}

int32_t mst_dh_tile_of_workgroup(int32_t even, int32_t n_split, int32_t n_row_tiles, int32_t n_col_tiles, int32_t workgroup,
                                 int32_t* split, int32_t* row_tile, int32_t* col_tile) {
  const int32_t grid = mst_dh_tile_grid(even, n_split, n_row_tiles, n_col_tiles);
  if (grid < 0 || workgroup < 0 || workgroup >= grid || !split || !row_tile || !col_tile) return -1;
  int sp = 0, st = 0, jt = 0;
  const bool ok = dh_tile_of_block(even != 0, workgroup, n_split, n_row_tiles, n_col_tiles, &sp, &st, &jt);
  *split = sp;
  *row_tile = st;
  *col_tile = jt;
  return ok ? 1 : 0;
}

int32_t mst_forward_tile_rows(int64_t S, int64_t d, int64_t V, int32_t M) {
  Plan p;
  if (make_plan(S, d, V, M, &p, MST_BWD_SCHEDULE_AUTO, 0, false) != MST_OK) return -1;
  return forward_tile_rows(p);
}

int32_t mst_forward_launch(int64_t S, int64_t d, int64_t V, int32_t M) {
  Plan p;
  if (make_plan(S, d, V, M, &p, MST_BWD_SCHEDULE_AUTO, 0, false) != MST_OK) return -1;
  if (persistent_forward(p)) return MST_FORWARD_QUEUES;
  const bool even = forward_tile_rows(p) < kTile || forward_even_map(p.n_vt, forward_row_tiles(p, 0, kTile));
  return even ? MST_FORWARD_EVEN : MST_FORWARD_RECTANGLES;
}

int32_t mst_pair_launches(int64_t S, int64_t d, int64_t V, int32_t M) {
  Plan p;
  if (make_plan(S, d, V, M, &p, MST_BWD_SCHEDULE_PAIRS) != MST_OK) return -1;
  return p.joint;
}

int32_t mst_bwd_streamed(int64_t S, int64_t d, int64_t V, int32_t M, int32_t* splits) {
  Plan p;
  if (make_plan(S, d, V, M, &p) != MST_OK) return -1;
  if (splits) *splits = p.streamed ? p.stream_split : 0;
  return p.streamed;
}

mst_status mst_tile_info(int64_t S, int64_t d, int64_t V, int32_t M, int64_t* info) {
  if (!info) return MST_ERR_NULL_POINTER;
  Plan p;
  const mst_status s = make_plan(S, d, V, M, &p, MST_BWD_SCHEDULE_AUTO, 0, false);
  if (s != MST_OK) return s;
  info[0] = forward_tile_rows(p);
  info[1] = p.small_dlogits ? Tile64::EA : kTile;
  info[2] = p.small_dh ? Tile64::EA : kTile;
  info[3] = p.small_dw ? Tile64::EA : kTile;
  return MST_OK;
}

mst_status mst_profile_enable(int every) {
  g_prof.enable(every);
  return MST_OK;
}

mst_status mst_profile_collect(double* ms_per_kind, int64_t* launches_per_kind, int64_t* issued_per_kind) {
  return g_prof.collect(MST_PROFILE_KINDS, ms_per_kind, launches_per_kind, issued_per_kind) ? MST_OK : MST_ERR_LAUNCH;
}

const char* mst_profile_kind_name(int kind) {
  static const char* names[MST_PROFILE_KINDS] = {
      "label_scan", "fwd_gemm_lse", "lse_finalize", "loss_reduce",
      "bwd_gemm_dlogits", "bwd_gemm_dh", "bwd_dh_reduce", "bwd_gemm_dw", "bwd_gemm_dh_dw"};
  return (kind >= 0 && kind < MST_PROFILE_KINDS) ? names[kind] : "?";
}

}  // extern "C"
