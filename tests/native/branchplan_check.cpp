// Cuts of the wide branches' scratch over random plans and scratch sizes: a
// range and one tile always fit, ranges cover the atoms, and scratch for
// everything gives one range.
#include <cmath>
#include <cstdio>
#include <random>

#include "branchplan.h"

int main() {
  std::mt19937_64 g(7);
  auto log_uniform = [&](double lo, double hi) {
    return lo * std::exp(std::uniform_real_distribution<double>(0, std::log(hi / lo))(g));
  };
  long long many = 0;
  for (int t = 0; t < 200000; ++t) {
    BranchPlan p;
    p.y_row = (size_t)log_uniform(128, 8192) & ~(size_t)63;
    p.dyh_row = t % 3 ? 0 : (size_t)log_uniform(64, 524288) & ~(size_t)63;
    p.tile = (size_t)log_uniform(4096, 8e6);
    p.TM = t % 2 ? 32 : 128;
    const int N = (int)log_uniform(1, 2e6);
    const int heads = t % 3 ? 1 : 16;
    p.tiles = (long long)N * heads / p.TM + heads;
    const size_t least = branch_scratch_min(p, N), full = branch_scratch_full(p, N);
    if (full < least) return std::printf("full < least\n"), 1;
    const size_t sizes[] = {least, least + (size_t)log_uniform(1, 1e9), full, full + full / 4};
    for (size_t s : sizes) {
      const int n = branch_range(p, N, s);
      if (n < 1 || n > N) return std::printf("range %d of %d\n", n, N), 1;
      if (branch_range_bytes(p, n) + p.tile > s)
        return std::printf("N %d n %d: %zu + %zu > %zu\n", N, n, branch_range_bytes(p, n), p.tile, s), 1;
      const int k = (N + n - 1) / n;
      if (k > 1) ++many;
      if (k > 1 && n < p.TM / 2) return std::printf("ranges of %d\n", n), 1;
    }
    const size_t rows = branch_range_bytes(p, N), all = (size_t)p.tiles * p.tile;
    if (rows <= BRANCH_SCRATCH_TARGET && all <= BRANCH_SCRATCH_TARGET && branch_range(p, N, full) != N)
      return std::printf("all of %d fits, range %d\n", N, branch_range(p, N, full)), 1;
  }
  std::printf("ok, %lld cuts in several ranges\n", many);
  return many > 1000 ? 0 : 1;
}
