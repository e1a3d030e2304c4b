// How many workgroups share a channel's samples ("time splits"): host rules,
// no device code.  Each split writes a partial image of its own, so the count
// also sets the scratch a run needs.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <limits>

namespace epic {

struct SplitShape {
  int N, F, n_cu;
  int64_t units;      // workgroups of one split: channels x class groups
  int64_t slots;      // frames a workgroup images at once, each into accumulators of its own
  bool fused;         // imaging items of the fused run, else a launch of its own
  double solve_us;    // fused: one channel's solve

  bool operator==(const SplitShape& o) const {
    return N == o.N && F == o.F && n_cu == o.n_cu && units == o.units && slots == o.slots && fused == o.fused &&
           solve_us == o.solve_us;
  }
};

// Time splits per channel for a target of `wg` workgroups, keeping >= 8 frames
// per slot; at 64 x 64 (the two-waves-per-SIMD engines: eight waves) >= 16
// frames per wave, which repays a workgroup's set-up and reduction (the
// 1000-sample differentiable workload: 31 splits 1.20 ms, 8 splits 1.08 ms),
// rounded up to whole rounds of workgroups over the CUs (one imaging
// workgroup per CU).
inline int64_t splits_for_target(const SplitShape& d, int64_t T, int64_t wg) {
  const int N = d.N;
  const int64_t units = d.units;
  int64_t s = (wg + units - 1) / units;
  const int64_t per_split = N == 64 ? 8 * 16 : N >= 128 ? 8 : 8 * 4 * (64 / N);
  s = std::min<int64_t>(s, std::max<int64_t>(1, T / per_split));
  if (units * s > d.n_cu) {
    const int64_t rounds = (units * s + d.n_cu - 1) / d.n_cu;
    s = std::min<int64_t>((rounds * d.n_cu + units - 1) / units, std::max<int64_t>(1, T));
  }
  return std::max<int64_t>(1, s);
}

// The most splits splits_by_steps gives, whatever the run's length: 12 rounds of
// the CUs (3072 workgroups on 256, those of the largest fused shapes), so that the
// partial images stay under 50 MB at 64 x 64, 0.2 GB at 128 x 128 and 0.4 GB at
// 256 x 256 (beyond 3072 workgroups, one image per channel).
inline int64_t most_splits(const SplitShape& d) {
  return std::max<int64_t>(1, (12 * int64_t(d.n_cu) + d.units - 1) / d.units);
}

// The fewest splits that keep the rounding of the image sums where the rule by
// workgroups has it (2048 of them, two rounds of the CUs for the paired 64 x 64
// engine, half as many splits again in the fused run).  T frames in n FP32
// accumulators per pixel, added in FP64, are off by sqrt(T / 3) / n of one
// rounding; that rule's accumulators (four waves' up to 32 x 32, eight in the
// fused run) were also added in FP32 within a workgroup, sqrt(slots / 3) of one
// averaged over the splits.  A quarter of a rounding's variance is allowed in any
// case, since the transforms and FP32 gains weigh some six.
//   Error against exact sums, 64 channels of 250 samples, by splits: 128 x 128, 512
// antennas, 1: 1.8e-7, 2: 1.2e-7, 6: 8.5e-8, 12: 8.1e-8, 32: 7.8e-8; 256 x 256, 2048
// antennas, 2: 1.8e-7, 6: 1.2e-7, 16: 1.03e-7, 64: 9.3e-8.
inline int64_t splits_for_rounding(const SplitShape& d, int64_t T) {
  int64_t s = splits_for_target(d, T, d.N == 64 && d.slots == 8 && !d.fused ? 2 * int64_t(d.n_cu) : 2048);
  if (d.fused) s = (3 * s + 1) / 2;
  const double slots = d.N <= 32 ? (d.fused ? 8.0 : 4.0) * (64 / d.N) : double(d.slots), n = slots * double(s);
  const double var = std::max(0.25, double(T) / 3.0 / (n * n) + (slots > 1 ? slots / 3.0 / double(s) : 0.0));
  return int64_t(std::ceil(std::sqrt(double(T) / 3.0 / var) / double(d.slots) - 1e-6));
}

// Time splits per channel from what a workgroup does: steps of `slots` frames,
// and a set-up and reduction worth one step more in a launch of its own, three
// (1.5 up to 32 x 32) as an item of the fused run.
//   A launch of its own takes its rounds of workgroups over the CUs times
//   (steps + 1): 32 x 32, 48 channels x 700: 5 splits 53 us, 4 62, 8 63, 11
//   (the rule by workgroups) 68; 64 x 64, 64 channels x 1000: 4 splits 221 us, 7
//   253.  256 x 256, 2048 antennas, 64 channels x 250, with its solve, would take
//   2.05 ms at 2 splits, 2.19 at the 16 that the rounding asks for.
//   The fused run's workgroups pull items one after another, those that solve
//   from `late` steps on (their channel's solve): LWA shape 22 splits 4.66 ms,
//   24 4.72, 16 4.77; 32 x 32, 75 channels x 1501: 16 splits 264 us, 23
//   370.
inline int splits_by_steps(const SplitShape& d, int64_t T) {
  const bool fused = d.fused;
  const int N = d.N;
  const int64_t units = d.units, slots = d.slots, steps = (T + slots - 1) / slots, most = std::min(steps, most_splits(d));
  const double setup = !fused ? 1.0 : N <= 32 ? 1.5 : 3.0;
  // the solve of a channel in steps
  const double step_us = N <= 32 ? 5.0 : N == 64 ? 6.8 : slots == 2 ? 9.0 : 14.0;
  const double late = d.solve_us / step_us;
  const int64_t solvers = std::min<int64_t>(d.F, d.n_cu - 1);
  // at most 256 frames in one FP32 accumulator, since rounding grows with them (HERA
  // shape, 1000: 4.8e-7, 250: 1.4e-7), as far as the bound on the partial images allows
  const int64_t least = std::min(std::max((steps + 255) / 256, splits_for_rounding(d, T)), most);
  int64_t best = least;
  double cost = std::numeric_limits<double>::max();
  auto consider = [&](int64_t s) {
    s = std::max(least, std::min(s, most));
    const double len = double(((T + s - 1) / s + slots - 1) / slots) + setup;
    const int64_t items = units * s;
    double c;
    if (!fused) {
      c = double((items + d.n_cu - 1) / d.n_cu) * len;
    } else {
      // the earliest end of an item by which all are done; the first items
      // wait for the solves to get through their samples
      const double first = late / double(s), end = double(items) * len;
      auto done = [&](double t) {
        return double(d.n_cu - solvers) * std::floor(std::max(0.0, t - first) / len) +
               double(solvers) * std::floor(std::max(0.0, t - late) / len);
      };
      const double t0 = (end + double(solvers) * std::min(late, end) + double(d.n_cu - solvers) * std::min(first, end)) / d.n_cu;
      c = std::numeric_limits<double>::max();
      for (int k = 0; k < 3; ++k) {
        const double e1 = first + len * (std::floor(std::max(0.0, t0 - first) / len) + k),
                     e2 = late + len * (std::floor(std::max(0.0, t0 - late) / len) + k);
        for (double e : {e1, e2})
          if (done(e + 1e-6 * len) >= double(items)) c = std::min(c, e);
      }
      if (c > 1e300) c = t0 + 2 * len;
      c = std::max(c, late + len);   // a channel's last item waits for its last interval
    }
    // the partial images' reduction: a launch whose threads read them one after
    // another, eight at a time, at 5 TB/s at best
    c += double(s) * (0.04 + double(d.F) * N * N * 4.0 / 5e6) / step_us;
    if (c < cost) {
      cost = c;
      best = s;
    }
  };
  for (int64_t k = 1; k <= 24; ++k) {
    consider(k);
    consider(k * d.n_cu / units);                 // k rounds of workgroups
    consider((T + k * slots - 1) / (k * slots));   // k steps each
  }
  return int(best);
}

// splits_by_steps of the shapes and run lengths seen last, so that a program with a
// few of them works it out once each (0.8 us of the host's time, 6 us for the
// fused run).
class SplitMemo {
 public:
  int get(const SplitShape& d, int64_t T) {
    for (const Entry& e : e_)
      if (e.T == T && e.d == d) return e.splits;
    Entry& e = e_[next_++ % kEntries];
    e = Entry{T, d, splits_by_steps(d, T)};
    return e.splits;
  }
  unsigned worked_out() const { return next_; }

 private:
  struct Entry {
    int64_t T = -1;
    SplitShape d{};
    int splits = 1;
  };
  static constexpr unsigned kEntries = 8;
  Entry e_[kEntries];
  unsigned next_ = 0;
};

}  // namespace epic
