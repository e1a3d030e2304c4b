// Host check of the time-split rules (splits.h): prints, for each shape given
// as "N F units slots fused solve_us_per_sample T" on stdin, the splits and
// the bytes of their partial images.
#include <cstdio>

#include "splits.h"

int main() {
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
