"""The host's schedule of a plain FP64 solve, compiled from its header alone."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2409_18824_amd", "csrc")

MAIN = r"""
#include <cstdio>
#include "solve_schedule.h"
using namespace j3d;
// lines of "c step all3 points": chunk unit, chunk length, its passes and the passes of 50 chunks' sweeps in one
// range, as len:stage lists
int main() {
  long long c, step, all3, points;
  while (std::scanf("%lld %lld %lld %lld", &c, &step, &all3, &points) == 4) {
    const SolveSchedule s{c, step, all3 != 0};
    const auto k = s.chunks(points);
    std::printf("%lld %lld", k.unit, k.sweeps);
    for (long long sw = 0; sw < k.sweeps;) {
      const auto p = s.next(sw, k.sweeps);
      std::printf(" %d:%d", p.len, p.stage);
      sw += p.len;
    }
    long long straight = 0;
    for (long long sw = 0; sw < 50 * k.sweeps; ++straight) sw += s.next(sw, 50 * k.sweeps).len;
    std::printf(" %lld\n", straight);
  }
}
"""


@pytest.fixture(scope="module")
def schedule(tmp_path_factory):
    d = tmp_path_factory.mktemp("schedule")
    src, exe = d / "main.cpp", d / "main"
    src.write_text(MAIN)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC, str(src), "-o", str(exe)])

    def ask(cases):
        text = "\n".join("%d %d %d %d" % q for q in cases) + "\n"
        out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
        got = []
        for line in out:
            w = line.split()
            passes = [tuple(int(v) for v in q.split(":")) for q in w[2:-1]]
            got.append((int(w[0]), int(w[1]), passes, int(w[-1])))
        return got
    return ask


CADENCES = [1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 20, 25, 49, 50, 51, 97, 99, 100, 200, 250, 251, 256, 333, 500, 667, 668, 998,
            999, 1000, 1001, 2000, 5000]
POINTS = [1, 40 ** 3, 100 ** 3, 181 * 143 * 160, 256 ** 3, 512 ** 3]


def cases():
    for points in POINTS:
        for c in CADENCES:
            yield c, min(c, 3), 0, points
            for step in (1, 2):
                yield c, step, 0, points
        yield 1, 3, 1, points


def test_passes_of_a_chunk_carry_every_check_once(schedule):
    qs = list(cases())
    for (c, step, all3, points), (unit, n, passes, _) in zip(qs, schedule(qs)):
        at, checks = 0, []
        for length, stage in passes:
            assert 1 <= length <= 3
            checks += [at, at + 1, at + 2] if stage == 3 else [at + stage] if stage >= 0 else []
            assert stage in (-1, 0) or length == 3  # later stages' residuals are a three-sweep pass's
            at += length
        assert at == n and n % c == 0, (c, step, points)
        assert checks == list(range(0, n, c)), (c, step, points)
        assert n % unit == 0
        if unit != c:
            assert len(passes) % 2 == 0


def test_chunks_stay_near_two_milliseconds(schedule):
    """A converged solve has up to two chunks of empty launches left.  2 ms are
    at most 667 sweeps: a chunk of a small grid is at most twice that or one
    check group (three and six of them before), and that of any grid at most
    300 sweeps and six groups of fewer than 300.  Shorter passes at the ends of
    chunks add at most 1 % to the passes."""
    qs = list(cases())
    for (c, step, all3, points), (unit, n, passes, straight) in zip(qs, schedule(qs)):
        if step != 3:
            continue
        assert n <= max(2 * 667, c) or (points > 100 ** 3 and c < 300 and n <= 300 + 6 * c), (c, points, n)
        assert 50 * len(passes) <= 1.01 * straight, (c, points, len(passes), straight)
