// Host check of the time-split rules (splits.h): prints, for each shape given
// as "N F units slots fused solve_us_per_sample T" on stdin, the splits and
// the bytes of their partial images.  With an argument: how often SplitMemo
// works out the rule in 1000 calls that go through that many run lengths (and,
// in turn, both forms of the run).
#include <cstdio>
#include <cstdlib>

#include "splits.h"

int main(int argc, char** argv) {
  if (argc > 1) {
    const int lengths = std::atoi(argv[1]);
    epic::SplitMemo memo;
    for (int k = 0; k < 1000; ++k) {
      const epic::SplitShape d{64, 128, 256, 128, 8, k % lengths % 2 == 1, 40.0};
      const int T = 1000 + 700 * (k % lengths);
      if (memo.get(d, T) != epic::splits_by_steps(d, T)) return 1;
    }
    std::printf("%u\n", memo.worked_out());
    return 0;
  }
  epic::SplitShape d{};
  int fused;
  double per_sample, T;
  long long units, slots;
  d.n_cu = 256;
  while (std::scanf("%d %d %lld %lld %d %lf %lf", &d.N, &d.F, &units, &slots, &fused, &per_sample, &T) == 7) {
    d.units = units;
    d.slots = slots;
    d.fused = fused != 0;
    d.solve_us = fused ? per_sample * T : 0.0;
    const long long s = epic::splits_by_steps(d, int64_t(T));
    std::printf("%lld %lld\n", s, s * d.F * d.N * d.N * 4);
  }
  return 0;
}
