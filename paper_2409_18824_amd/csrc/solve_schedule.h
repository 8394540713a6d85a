// The schedule of a plain FP64 solve: which passes its sweeps run in, which
// residuals they carry, and how many sweeps the host queues between two looks
// at the device's flag.  Host arithmetic only.
#pragma once

#include <algorithm>
#include <cmath>
#include <numeric>

namespace j3d {

// Chunk length (in sweeps) that keeps the device busy for about 2 ms.
inline long long chunk_sweeps(long long points, double bytes_per_point, long long multiple) {
  const double t = std::max(3e-6, bytes_per_point * (double)points / 5e12);
  long long n = (long long)std::ceil(2e-3 / t);
  n = std::max<long long>(n, 1);
  n = std::min<long long>(n, 1 << 16);
  n = ((n + multiple - 1) / multiple) * multiple;
  return n;
}

// Passes of `step` sweeps.  Three-sweep passes run straight through the
// sweeps: the residual of a check is fused into the pass that forms its
// iterate, at that stage of the pass, whose input stays in its array until the
// check's verdict is known (every later kernel skips its work once a check has
// converged), so the checked iterate can be formed again; with checks after
// every sweep they carry all three residuals.  (At the end of a range a
// shorter pass stops before a check it would hold past its input.)  With a
// step of one or two a check group of c sweeps opens with one pass of c mod
// step sweeps (none when step divides c), which carries the check's residual,
// and continues in passes of step sweeps.
struct SolveSchedule {
  long long c;     // sweeps from check to check
  long long step;  // sweeps per pass
  bool all3;       // three-sweep passes with the residuals of all three of their input iterates

  struct Pass {
    int len;    // sweeps
    int stage;  // the residual it carries is that of the iterate after this many of them; -1: none,
                // 3: those of its input and both intermediate iterates
  };

  // The pass that starts after sw sweeps of a range that ends at `to`.
  Pass next(long long sw, long long to) const {
    if (step != 3) {
      const long long p = sw % c, lead = c % step;
      const long long len = std::min(p == 0 && lead != 0 ? lead : step, c - p);
      return Pass{(int)std::min(len, to - sw), p == 0 ? 0 : -1};
    }
    if (all3) return to - sw >= 3 ? Pass{3, 3} : Pass{1, 0};
    int len = (int)std::min<long long>(3, to - sw), stage = -1;
    for (int o = 0; o < len; ++o) {
      if ((sw + o) % c != 0) continue;
      if (stage < 0)
        stage = o;
      else
        len = o;  // the next check opens the next pass
    }
    if (stage > 0 && len < 3) return Pass{stage, -1};
    return Pass{len, stage};
  }

  bool straight() const { return step == 3 && (c >= 3 || all3); }
  // The schedule repeats after `period` sweeps.
  long long period() const { return straight() ? std::lcm(c, 3LL) : c; }
  long long period_passes() const {
    return straight() ? period() / 3 : step == 3 ? 1 : (c % step != 0 ? 1 : 0) + c / step;
  }

  // Chunks of `sweeps` sweeps, made of units of `unit`.  A chunk begins at a
  // check and is the same passes wherever it begins.  Its units are whole
  // periods with an even number of passes, which leave the iterate in the
  // array it was in.  Where those overshoot the 2 ms more than twice (checks a
  // long way apart, at a distance that three does not divide), they are check
  // groups instead, and a chunk's last pass may be a shorter one, which is at
  // most one pass in a hundred.  A converged solve has up to two chunks of
  // empty launches left: 40^3 with check_every = 1000, converged at the first
  // check, 2.5 ms of them in chunks of 3000 sweeps, 0.95 ms in chunks of 1000.
  struct Chunks {
    long long unit, sweeps;
  };
  Chunks chunks(long long points) const {
    const long long per = period(), pp = period_passes();
    const double bytes = 24.0 * (double)pp / (double)per;
    const long long unit = pp % 2 == 0 ? per : 2 * per;
    const long long target = chunk_sweeps(points, bytes, 1);
    const Chunks whole{unit, chunk_sweeps(points, bytes, unit)}, groups{c, chunk_sweeps(points, bytes, c)};
    return straight() && whole.sweeps > 2 * target && groups.sweeps >= 300 ? groups : whole;
  }
};

}  // namespace j3d
