// Timing of the candidate kernels of one level (host code without HIP, so that it can be
// run on made-up durations).
#pragma once

#include <algorithm>
#include <vector>

namespace hexmg {

// Times n candidates by `reps` launches each: ms[i] receives the duration of candidate i's
// launches, 1e30 where a shorter sample ruled it out.
// timed(i, k, &ms) launches candidate i k times back to back between two events and returns a
// status (0: go on).  Each candidate is launched once unjudged (its first use and cold caches),
// then reps / 3 times: a candidate that takes 1.25 times as long for these as the fastest
// has taken for as many is timed no further (such samples repeat within a few per cent), the
// others are launched the rest of the times.  Samples that are compared hold the same number
// of launches and of intervals, so the events' own cost, which can exceed a small launch,
// brings them nearer each other and never rules a faster candidate out (a single launch
// scaled by reps against the total of reps launches would).
template <typename Timed>
int time_candidates(int n, int reps, Timed&& timed, std::vector<float>* ms) {
  const int probe = std::max(1, reps / 3);
  float fastest = 1e30f;
  ms->assign(n, 1e30f);
  for (int i = 0; i < n; ++i) {
    float t = 0.f;
    if (int e = timed(i, 1, &t)) return e;
    if (int e = timed(i, probe, &t)) return e;
    if (t > 1.25f * fastest) continue;
    fastest = std::min(fastest, t);
    float rest = 0.f;
    if (reps > probe)
      if (int e = timed(i, reps - probe, &rest)) return e;
    (*ms)[i] = t + rest;
  }
  return 0;
}

}  // namespace hexmg
