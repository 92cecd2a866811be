// Tile shape and k-split choice of every matrix product of a surrogate, and the
// split-K workspace that follows from it.  Free of HIP, so that the workspace
// bound can be checked on the CPU over whole ranges of rows.
#pragma once

#include <algorithm>
#include <cstdint>
#include <vector>

#include "intmath.h"

namespace ot {

constexpr int kMaxSmallK = 16;   // layer 1 with in <= 16 uses the small-K kernels

// Tile shapes (4 wavefronts each): 128 x 128, 64 x 128, 64 x 64 on fp32 MFMAs;
// 128 x 128, 64 x 128, 64 x 64, 32 x 256 and 64 x 256 on three bf16 terms
// (gemm_f32x3.h).
enum Cfg : int { kC128x128 = 0, kC64x128 = 1, kC64x64 = 2, kX128 = 3, kX64 = 4, kX32W = 5, kX64W = 6, kX64x128 = 7 };

inline int64_t tiles_of(int cfg, int64_t M, int64_t N) {
  switch (cfg) {
    case kC128x128: return ceil_div(M, 128) * ceil_div(N, 128);
    case kC64x128: return ceil_div(M, 64) * ceil_div(N, 128);
    case kX128: return ceil_div(M, 128) * ceil_div(N, 128);
    case kX64x128: return ceil_div(M, 64) * ceil_div(N, 128);
    case kX32W: return ceil_div(M, 32) * ceil_div(N, 256);
    case kX64W: return ceil_div(M, 64) * ceil_div(N, 256);
    default: return ceil_div(M, 64) * ceil_div(N, 64);
  }
}

struct Plan {
  int cfg = kC64x64;
  int64_t splits = 1;     // k ranges actually launched
  int64_t asked = 1;      // before the ranges were rounded to k tiles (>= splits)
  int64_t k_chunk = 0;
  int64_t blocks = 0;
};

// The plan on three bf16 terms, or false where the fp32 MFMA kernel is as good:
// below 4e8 flops launch and fill time dominate (49 x 15766 x 242: forward 18
// against 20 us, gradients even or slower), a weight gradient over fewer than 128 rows is bound by its
// Adam epilogue (1000000 x 256 over 10 rows: 1146 us on fp32 MFMAs, 1168 here),
// and fewer than 192 blocks leave CUs idle.  Forward products are never split
// here (their partials would need scratch that surrogate_predict_noalloc's
// callers did not have to fit); 64 x 128 tiles when they give two blocks per CU
// (1024 x 10000 x 256 with the MSE epilogue: 55 us, 67 on 64 x 64 tiles), else 64 x
// 64 (331 x 6561 x 437, the same: 34 us, 35 on 64 x 128).  Backward products are split until about 512 blocks
// (two 128 x 128 blocks share a CU; more would queue behind them: 10000 x 256
// over 1024 rows in 3 splits 39 us, in 4 47 us).
// any_size: without the rule on flops (for bounds over a range of sizes).
inline bool make_plan_x3(int64_t M, int64_t N, int64_t K, bool backward, Plan* p, bool any_size = false) {
  constexpr int64_t kCUs = 256;
  if (!any_size && 2.0 * M * N * K < 4e8) return false;
  const int wide = M <= 32 ? kX32W : kX64W;
  if (!backward) {
    if (M <= 64 && tiles_of(wide, M, N) >= kCUs) p->cfg = wide;
    else p->cfg = tiles_of(kX64x128, M, N) >= 2 * kCUs ? kX64x128 : kX64;
    if (tiles_of(p->cfg, M, N) < kCUs - 64) return false;
    p->splits = 1;
  } else {
    p->cfg = (M <= 64 && N > 128) ? wide : (M <= 64 || N <= 64) ? kX64 : kX128;
    const int64_t t = tiles_of(p->cfg, M, N);
    p->splits = std::max<int64_t>(1, std::min<int64_t>(2 * kCUs / t, K / 128));
    if (t * p->splits < kCUs - 64 || K < 128) return false;
  }
  p->asked = p->splits;
  p->k_chunk = round_up(ceil_div(K, p->splits), 16);
  p->splits = std::max<int64_t>(1, ceil_div(K, p->k_chunk));
  p->blocks = tiles_of(p->cfg, M, N) * p->splits;
  return true;
}

// Tile and k-split choice on fp32 MFMAs (measured on MI355X at the surrogate's shapes).
// Whole tiles per CU matter more than tile size: a launch whose block count
// leaves some CUs a block more than others loses that fraction, so the plan
// aims for about 4 blocks per CU (960+) with 64 x 128 tiles, splits long k
// ranges (>= 4096) over 128 x 128 tiles, splits medium ones over 64 x 64
// tiles (>= 256 deep per split), and splits short problems down to 32-deep
// ranges until every CU has a block.  The MSE epilogue needs whole sums and
// is never split.
inline Plan make_plan_f32(int64_t M, int64_t N, int64_t K, bool allow_split) {
  constexpr int64_t kCUs = 256;
  Plan p;
  if (tiles_of(kC64x128, M, N) >= 960 || !allow_split) {
    p.cfg = kC64x128;
    if (tiles_of(kC64x128, M, N) < kCUs) p.cfg = kC64x64;
    if (!allow_split && tiles_of(kC64x64, M, N) < kCUs) p.cfg = kC64x64;
  } else if (K >= 4096) {
    p.cfg = kC128x128;
    const int64_t t = tiles_of(kC128x128, M, N);
    while (t * p.splits < 2 * kCUs - 32 && K / (2 * p.splits) >= 256) p.splits *= 2;
  } else {
    p.cfg = kC64x64;
    const int64_t t = tiles_of(kC64x64, M, N);
    while (t * p.splits < 960 && K / (2 * p.splits) >= 256) p.splits *= 2;
    if (t * p.splits < kCUs)
      while (t * p.splits < kCUs && K / (2 * p.splits) >= 32) p.splits *= 2;
  }
  p.asked = p.splits;
  p.k_chunk = round_up(ceil_div(K, p.splits), 16);
  p.splits = std::max<int64_t>(1, ceil_div(K, p.k_chunk));
  p.blocks = tiles_of(p.cfg, M, N) * p.splits;
  return p;
}

// The plan of an fp32 product.
inline Plan make_plan(int64_t M, int64_t N, int64_t K, bool allow_split, bool backward = false) {
  Plan p;
  return make_plan_x3(M, N, K, backward, &p) ? p : make_plan_f32(M, N, K, allow_split);
}

// bf16 tiles: for large products the pipelined 256 x 128 kernel (k tile 32,
// direct-to-LDS loads, two blocks per CU), its 128 x 256 shape for up to 128
// rows, or the ping-pong 256 x 256 kernel (eight wavefronts, one block per CU);
// 128 x 128 (4 x 4 fragments per wave) and 64 x 64 (2 x 2) with a k tile of 32
// otherwise.
enum CfgB : int { kB128 = 0, kB64 = 1, kBPipe = 2, kBPipeW = 3, kBPipeH = 4 };
constexpr int kBK = 32;
constexpr int kPipeBK = 32;

inline int64_t tiles_b(int cfg, int64_t M, int64_t N) {
  if (cfg == kBPipe) return ceil_div(M, 256) * ceil_div(N, 128);
  if (cfg == kBPipeW) return ceil_div(M, 256) * ceil_div(N, 256);
  if (cfg == kBPipeH) return ceil_div(M, 128) * ceil_div(N, 256);
  return cfg == kB128 ? ceil_div(M, 128) * ceil_div(N, 128) : ceil_div(M, 64) * ceil_div(N, 64);
}

// Rows of a tile.
inline int64_t tile_rows_b(int cfg) {
  return (cfg == kBPipe || cfg == kBPipeW) ? 256 : (cfg == kB128 || cfg == kBPipeH) ? 128 : 64;
}

enum class Prod : int { Forward, InputGrad, WeightGrad };

// Wide forward products (about a tile per CU or more) are not split.  Up to 64
// rows they stream the weights through 64 x 64 tiles (predictions of 1000000 x 1024:
// 367 us at 1 row, 571 on 128 x 128; 537 and 618 at 64 rows, where 128 x 256 tiles
// would take 494), up to 128 through the pipelined kernel's 128 x 256 (100 rows: 508
// us, 655 on 128 x 128, 718 on 64 x 64), above through the ping-pong kernel's 256 x 256 (200
// rows, 1000000 x 2048: 1246 against 2115 us on 128 x 128, 1417 on 128 x 256);
// rows past the operand are read from its last one.
// Input gradients: over long k ranges the ping-pong kernel in splits until about two
// blocks per CU, keeping at least 32 k tiles per split (200 x 1024, k 200000: 110
// against 369 us on 128 x 128); else 256 x 128 tiles of the pipelined kernel with at
// least 10 k tiles per split (512 x 512, k 19616: 23 against 38 us; from k of 4096 on,
// which hidden layers rarely reach: below it ranges of 32 k tiles as before, since each
// other order of a hidden gradient's sums moves a few values to the next bf16 value, which
// the layers before it pass on, 1.9e-4 of the outputs of a 2048-2048-2048 net after one
// step); 128 x 256 tiles up to 128 rows (64 x 1024, k 300000: 125 against 178 us; 100
// x 512, k 200000: 45 against 66).
// Others with the 32-deep k tile kernels when k is a multiple of 32 and the tiles
// give about one block per CU or more (forward products keep 32 k tiles per
// split, so that their partials stay as small as they were), else 128 x 128 tiles
// when they give about two blocks per CU; long k ranges are split over 128 x 128
// tiles, shorter ones over 64 x 64.
// pipe_ok: the 32-deep k tile kernels may be used (they have no row-sum output).
inline Plan make_plan_b(int64_t M, int64_t N, int64_t K, bool allow_split, Prod prod, bool pipe_ok = true) {
  constexpr int64_t kCUs = 256;
  Plan p;
  auto plan = [&](int cfg, int64_t sp) {
    p.cfg = cfg;
    p.asked = sp;
    p.k_chunk = round_up(ceil_div(K, sp), kPipeBK);
    p.splits = std::max<int64_t>(1, ceil_div(K, p.k_chunk));
    p.blocks = tiles_b(cfg, M, N) * p.splits;
    return p;
  };
  const bool deep = pipe_ok && K % kPipeBK == 0;
  if (prod == Prod::Forward) {
    if (M <= 64 && tiles_b(kB64, M, N) >= kCUs - 16) return plan(kB64, 1);
    if (deep && N >= 256 && M > 64 && M <= 128 && tiles_b(kBPipeH, M, N) >= kCUs - 16) return plan(kBPipeH, 1);
    if (deep && N >= 256 && M > 128 && tiles_b(kBPipeW, M, N) >= kCUs - 16) return plan(kBPipeW, 1);
  }
  if (deep && allow_split && M >= (prod == Prod::InputGrad ? 129 : 256) && N >= 256) {
    const int64_t t = tiles_b(kBPipeW, M, N);
    int64_t sp = 1;
    while (t * sp < 2 * kCUs - 32 && K / (2 * sp) >= 32 * kPipeBK) sp *= 2;
    if (sp > 1 && t * sp >= kCUs - 16) return plan(kBPipeW, sp);
  }
  if (deep && allow_split && prod == Prod::InputGrad && M <= 128 && N >= 128) {
    const int64_t t = tiles_b(kBPipeH, M, N);
    int64_t sp = 1;
    while (t * sp < (M <= 32 ? 2 * kCUs - 32 : kCUs - 16) && K / (2 * sp) >= 10 * kPipeBK) sp *= 2;
    if (t * sp >= kCUs - 16) return plan(kBPipeH, sp);
  }
  if (deep && M >= (prod == Prod::InputGrad ? 129 : 256) && N >= 128) {
    const int64_t t = tiles_b(kBPipe, M, N);
    int64_t sp = 1;
    if (allow_split)
      while (t * sp < 4 * kCUs - 64 && K / (2 * sp) >= (prod == Prod::InputGrad && K >= 4096 ? 10 : 32) * kPipeBK)
        sp *= 2;
    if (t * sp >= kCUs - 16) return plan(kBPipe, sp);
  }
  const int64_t t128 = tiles_b(kB128, M, N);
  if (t128 >= 2 * kCUs - 32) {
    p.cfg = kB128;
  } else if (!allow_split) {
    p.cfg = t128 >= kCUs - 16 ? kB128 : kB64;
  } else {
    p.cfg = K >= 4096 ? kB128 : kB64;
    const int64_t t = tiles_b(p.cfg, M, N);
    while (t * p.splits < 2 * kCUs - 32 && K / (2 * p.splits) >= 256) p.splits *= 2;
    if (t * p.splits < kCUs)
      while (t * p.splits < kCUs && K / (2 * p.splits) >= 64) p.splits *= 2;
  }
  p.asked = p.splits;
  p.k_chunk = round_up(ceil_div(K, p.splits), kBK);
  p.splits = std::max<int64_t>(1, ceil_div(K, p.k_chunk));
  p.blocks = tiles_b(p.cfg, M, N) * p.splits;
  return p;
}

// What decides which products a net runs and how they are planned.
struct NetShape {
  std::vector<int64_t> widths;   // of the input and the layers 1..L
  bool bf16 = false;
  bool small_hidden = false;     // hidden layers of an fp32 net in the narrow-layer kernels
  bool fuse_out = false;         // output-layer Adam in its weight gradient

  int L() const { return (int)widths.size() - 1; }
  // Whether layer l's (1..L) forward, weight gradient, input gradient are matrix
  // products (the others run in the small-K and narrow-layer kernels).
  bool forward_product(int l) const {
    return l == L() || !(bf16 ? l == 1 : small_hidden || (l == 1 && widths[0] <= kMaxSmallK));
  }
  bool wgrad_product(int l) const {
    return !(small_hidden && l < L()) && !(l == 1 && widths[0] <= kMaxSmallK);
  }
  bool igrad_product(int l) const { return l >= 2 && !(small_hidden && l < L()); }
  // k range of layer l's input gradient (a bf16 dY is padded to whole k tiles)
  int64_t igrad_k(int l) const { return bf16 && l == L() ? round_up(widths[l], kPipeBK) : widths[l]; }
};

// Rows of one prediction pass when train steps take up to `rows` rows.  At least
// kPassRows, so that a prediction of more rows than the batch reads the output
// weights once (40 rows after batches of 10, 1000000 x 256 fp32: 340 us instead of 4
// x 250), as far as the hidden activations fit kPassBytes (a hidden layer of a
// million units has 4 MB a row; nets of up to 65,536 hidden units keep all 256).
constexpr int64_t kPassRows = 256;
constexpr int64_t kPassBytes = 64 << 20;
inline int64_t pass_rows(const NetShape& net, int64_t rows) {
  int64_t row_bytes = 1;
  for (int l = 1; l < net.L(); ++l) row_bytes += round_up(net.widths[l], 8) * (net.bf16 ? 2 : 4);
  return std::max(rows, std::min(kPassRows, kPassBytes / row_bytes));
}

// Floats of split-K partial products and of partial row sums.
struct SplitNeed {
  int64_t partials = 0, rowsums = 0;
  void add(int64_t splits, int64_t M, int64_t N, bool rowsum) {
    if (splits <= 1) return;
    partials = std::max(partials, splits * M * round_up(N, 4));
    if (rowsum) rowsums = std::max(rowsums, splits * M);
  }
};

// Every product that may be split in a prediction pass over m rows (train
// false) or in a train step on m rows besides.  fn(M, N, K, prod, pipe_ok, rowsum).
template <class F>
inline void for_split_products(const NetShape& net, int64_t m, bool train, F fn) {
  const int L = net.L();
  for (int l = 1; l <= L; ++l) {
    const int64_t in = net.widths[l - 1], out = net.widths[l];
    if (net.forward_product(l)) fn(m, out, in, Prod::Forward, true, false);
    if (!train) continue;
    if (net.igrad_product(l)) fn(m, in, net.igrad_k(l), Prod::InputGrad, true, false);
    if (net.wgrad_product(l) && !(net.bf16 && net.fuse_out && l == L)) {
      const bool rowsum = !net.bf16 || l < L;
      fn(out, in, m, Prod::WeightGrad, !rowsum, rowsum);
    }
  }
}

// The split-K workspace of any train step on up to `rows` rows and any prediction
// pass of up to `act_rows` (>= rows) rows.
//
// It is fixed when the surrogate's workspaces are made and never grows: a captured
// step or prediction holds its address, and a call under capture cannot allocate.
// Plans change with the number of rows at multiples of 32 or one above one (and, in
// fp32, with the flops, so both fp32 plans count); in between, the ranges asked for
// grow with it, except that a bf16 weight gradient has plans of its own over whole k
// tiles of 32 rows.  So the largest row counts of each group of 32 with and without
// its last one bound the group.
inline SplitNeed split_need(const NetShape& net, int64_t rows, int64_t act_rows) {
  SplitNeed need;
  auto at = [&](int64_t m) {
    for_split_products(net, m, m <= rows, [&](int64_t M, int64_t N, int64_t K, Prod prod, bool pipe_ok, bool rowsum) {
      if (net.bf16) {
        need.add(make_plan_b(M, N, K, true, prod, pipe_ok).asked, M, N, rowsum);
        return;
      }
      Plan p;
      if (make_plan_x3(M, N, K, prod != Prod::Forward, &p, true)) need.add(p.asked, M, N, rowsum);
      need.add(make_plan_f32(M, N, K, true).asked, M, N, rowsum);
    });
  };
  for (int64_t m = 32; m < act_rows + 32; m += 32) {
    if (std::min(m, act_rows) > 1) at(std::min(m, act_rows) - 1);
    at(std::min(m, act_rows));
  }
  if (rows > 1) at(rows - 1);
  at(rows);
  return need;
}

}  // namespace ot
