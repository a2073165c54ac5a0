// Sizes of the dedispersed tiles (frbx_plan.h): every launch stays within the
// int arithmetic of the kernels, also at the largest counts that are admitted.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>

#include "../paper_1801_02391_amd/csrc/frbx_plan.h"

static long n_checks = 0;
#define CHECK(x)                                                        \
  do {                                                                  \
    ++n_checks;                                                         \
    if (!(x)) {                                                         \
      std::printf("line %d: %s\n", __LINE__, #x);                       \
      std::exit(1);                                                     \
    }                                                                   \
  } while (0)

int main() {
  using namespace frbx;
  // what a launch of n tasks computes in int: work-groups of up to eight,
  // the last task of the last work-group, one more sweep of 1024 of them
  CHECK((kLaunchMost + 7) / 8 * 8 + 8 * 1024 + 7 < (int64_t(1) << 31));
  std::mt19937_64 rng(1);
  auto logint = [&](int64_t lo, int64_t hi) {
    std::uniform_real_distribution<double> u(std::log(double(lo)), std::log(double(hi) + 1));
    return std::min<int64_t>(hi, std::max<int64_t>(lo, int64_t(std::exp(u(rng)))));
  };
  for (int k = 0; k < 200000; ++k) {
    const int D = int(logint(1, 65536)), B = int(logint(1, 1000));
    const int64_t S = logint(1, int64_t(1) << 30), R = logint(1, 64);
    const size_t per = size_t(logint(64, int64_t(1) << 34)), most = size_t(logint(1, int64_t(1) << 38));
    const int dt = tile_trials(most, per, D, S * R);
    CHECK(dt >= 1 && dt <= D && (dt == 1 || (size_t(dt) * per <= most && int64_t(dt) * S * R <= kLaunchMost)));
    const int all = whole_baselines(dt, per, D, B, S * R, most);
    CHECK(all == dt || (dt == D && all % D == 0 && all / D <= B));
    CHECK(all == dt || (size_t(all) * per <= most && int64_t(all) * S * R <= kLaunchMost));
  }
  // at the limit itself and one task beyond it
  CHECK(tile_trials(size_t(1) << 40, 64, 2, kLaunchMost / 2) == 2);
  CHECK(tile_trials(size_t(1) << 40, 64, 2, kLaunchMost / 2 + 1) == 1);
  CHECK(whole_baselines(1, 64, 1, 2, kLaunchMost / 2, size_t(1) << 40) == 2);
  CHECK(whole_baselines(1, 64, 1, 2, kLaunchMost / 2 + 1, size_t(1) << 40) == 1);
  CHECK(tile_trials(1 << 20, 0, 5, 0) == 1 && whole_baselines(5, 0, 5, 3, 0, 1 << 20) == 5);
  std::printf("ok %ld\n", n_checks);
  return 0;
}
