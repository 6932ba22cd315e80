"""The rule by which the timed kernel choice rules candidates out (csrc/choose.h), run on
made-up durations: without noise the fastest candidate always wins, whatever its place in
the list, the events' own cost and the cost of a kernel's first launch."""
import os
import shutil
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2201_12931_amd", "csrc")
MAIN = r"""
#include <cstdio>
#include "choose.h"
// input: trials, then per trial: n reps overhead, n times (duration, first-use cost)
int main() {
  int trials;
  if (scanf("%d", &trials) != 1) return 1;
  while (trials--) {
    int n, reps;
    double over;
    if (scanf("%d %d %lf", &n, &reps, &over) != 3) return 1;
    std::vector<double> T(n), first(n);
    for (int i = 0; i < n; ++i)
      if (scanf("%lf %lf", &T[i], &first[i]) != 2) return 1;
    int launches = 0;
    auto timed = [&](int i, int k, float* ms) {
      *ms = (float)(over + k * T[i] + first[i]);
      first[i] = 0.0;
      launches += k;
      return 0;
    };
    std::vector<float> ms;
    if (hexmg::time_candidates(n, reps, timed, &ms)) return 1;
    printf("%d %d\n", (int)(std::min_element(ms.begin(), ms.end()) - ms.begin()), launches);
  }
  return 0;
}
"""


def test_fastest_candidate_wins(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if not cxx:
        pytest.skip("no C++ compiler")
    (tmp_path / "main.cpp").write_text(MAIN)
    exe = str(tmp_path / "main")
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", CSRC, str(tmp_path / "main.cpp"), "-o", exe], check=True)
    rng = np.random.default_rng(3)
    # an 8 us launch after a 9 us one, between events that cost 10 us
    trials = [(12, 10.0, [9.0, 8.0], [40.0, 40.0])]
    for _ in range(400):
        n = int(rng.integers(2, 60))
        T = rng.uniform(3.0, 30.0, n) * (1.0 + 1e-3 * np.arange(n))
        trials.append((int(rng.choice([3, 12])), float(rng.uniform(0.0, 30.0)), list(T), list(rng.uniform(0.0, 60.0, n))))
    text = f"{len(trials)}\n"
    for reps, over, T, first in trials:
        text += f"{len(T)} {reps} {over}\n" + "\n".join(f"{t} {c}" for t, c in zip(T, first)) + "\n"
    r = subprocess.run([exe], input=text, capture_output=True, text=True, check=True)
    rows = [tuple(map(int, line.split())) for line in r.stdout.splitlines()]
    assert len(rows) == len(trials)
    for (reps, over, T, first), (best, launches) in zip(trials, rows):
        assert best == int(np.argmin(T)), (reps, over, T, first)
        assert launches <= len(T) * (1 + reps)
