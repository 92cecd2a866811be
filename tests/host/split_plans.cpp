// The split-K workspace bound (plan.h) against every plan it has to cover: for
// each net, all row counts of train steps and prediction passes.  Prints one
// line a net: the bound, the largest need and what asked for it.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>

#include "plan.h"

using namespace ot;

static SplitNeed need_of(const NetShape& net, int64_t m, bool train) {
  SplitNeed n;
  for_split_products(net, m, train, [&](int64_t M, int64_t N, int64_t K, Prod prod, bool pipe_ok, bool rowsum) {
    const Plan p = net.bf16 ? make_plan_b(M, N, K, true, prod, pipe_ok) : make_plan(M, N, K, true, prod != Prod::Forward);
    if (p.splits > p.asked || p.splits * p.k_chunk < K || (p.splits - 1) * p.k_chunk >= K) {
      std::printf("bad plan of %lld x %lld x %lld\n", (long long)M, (long long)N, (long long)K);
      std::exit(1);
    }
    // the launches have three-term tiles for these only: forward ones are never split
    const bool forward = prod == Prod::Forward;
    if (!net.bf16 && ((forward && (p.cfg == kX128 || (p.cfg > kC64x64 && p.splits > 1))) ||
                      (!forward && p.cfg == kX64x128))) {
      std::printf("tiles %d of %lld x %lld x %lld\n", p.cfg, (long long)M, (long long)N, (long long)K);
      std::exit(1);
    }
    n.add(p.splits, M, N, rowsum);
  });
  return n;
}

static void check(const NetShape& net, int64_t rows, int64_t act_rows) {
#ifdef TRAIN_ONLY     // the workspace of the train steps alone, as if predictions never split
  const SplitNeed bound = need_of(net, rows, true);
#else
  const SplitNeed bound = split_need(net, rows, act_rows);
#endif
  SplitNeed most;
  for (int64_t m = 1; m <= std::max(rows, act_rows); ++m) {
    const SplitNeed n = need_of(net, m, m <= rows);
    if (n.partials > bound.partials || n.rowsums > bound.rowsums) {
      std::printf("%lld rows (batch %lld) of", (long long)m, (long long)rows);
      for (int64_t w : net.widths) std::printf(" %lld", (long long)w);
      std::printf(" ask for %lld + %lld, above %lld + %lld\n", (long long)n.partials, (long long)n.rowsums,
                  (long long)bound.partials, (long long)bound.rowsums);
      std::exit(1);
    }
    most.partials = std::max(most.partials, n.partials);
    most.rowsums = std::max(most.rowsums, n.rowsums);
  }
  std::printf("%s", net.bf16 ? "bf16" : "fp32");
  for (int64_t w : net.widths) std::printf(" %lld", (long long)w);
  std::printf(" batch %lld: %lld + %lld for %lld + %lld\n", (long long)rows, (long long)bound.partials,
              (long long)bound.rowsums, (long long)most.partials, (long long)most.rowsums);
  // the bound is above what some call asks for by no more than one product's 512 blocks of 128 x 128
  if (bound.partials > most.partials + 512 * 128 * 128 || bound.rowsums > most.rowsums + 512 * 128) std::exit(2);
}

static NetShape net(std::vector<int64_t> w, bool bf16, bool fuse = true) {
  const bool small = !bf16 && w.size() == 4 && w[0] <= 16 && w[1] <= 256 && w[2] <= 256;
  return {std::move(w), bf16, small, fuse};
}

int main() {
  // prediction passes: 256 rows or the batch, fewer where wide hidden layers take over 64 MB
  const int64_t act = pass_rows(net({6, 64, 64, 256}, false), 32);
  if (act != 256 || pass_rows(net({6, 2048, 2048, 2048, 1000000}, true), 1024) != 1024 ||
      pass_rows(net({6, 32768, 32760, 8}, false), 1) != 256 || pass_rows(net({6, 1000000, 1}, false), 1) != 16 ||
      pass_rows(net({6, 1000000, 1}, true), 3) != 33 || pass_rows(net({6, 1 << 26, 1}, false), 1) != 1) {
    std::printf("pass rows\n");
    return 1;
  }
  check(net({6, 64, 64, 256}, false), 32, act);
  check(net({6, 256, 256, 10000}, false), 1024, 1024);
  check(net({6, 300, 437, 6561}, false), 331, 331);
  check(net({6, 256, 256, 1000000}, false), 10, act);
  check(net({24, 9001}, false), 1000, 1000);
  check(net({6, 512, 512, 19600}, true), 512, 512);
  check(net({6, 1024, 1024, 1000000}, true), 512, 512);
  check(net({6, 2048, 2048, 2048, 1000000}, true), 1024, 1024);
  check(net({6, 1024, 1024, 1000000}, true, false), 1, act);
  check(net({6, 500, 4096, 4100, 300}, true, false), 4200, 4200);
  check(net({6, 500, 4096, 4100, 300}, false), 4200, 4200);
  std::mt19937_64 rng(7);
  auto pick = [&](double lo, double hi) {
    return (int64_t)(lo * std::exp(std::uniform_real_distribution<double>(0, std::log(hi / lo))(rng)));
  };
  for (int i = 0; i < 400; ++i) {
    const bool bf16 = rng() % 2;
    std::vector<int64_t> w{bf16 || rng() % 4 ? 6 : pick(1, 300)};
    for (int l = 1 + (int)(rng() % 3); l > 0; --l) w.push_back(rng() % 3 ? pick(4, 5000) : 32 * pick(1, 128));
    w.push_back(rng() % 3 ? pick(1, 2000000) : 32 * pick(1, 40000));
    const int64_t rows = pick(1, 3000);
    const NetShape shape = net(w, bf16, rng() % 2);
    check(shape, rows, pass_rows(shape, rows));
  }
  std::printf("ok\n");
}
