// Host-side checks of the static schedules: whether a shape's class schedules and stage rows are
// valid, by running their rounds without costs.
#pragma once

#include <algorithm>
#include <vector>

#include "octo_device.hpp"

namespace octo {

// Steps of the ideal stage pipeline of MERGE (largest ideal start + 1) for S stages, or 0 if some
// link would need more than two slots: every value of micro-batch m must be consumed in an
// earlier step than the one that produces micro-batch m + 2 of its link (sr_entry). Longest-path
// times of the unit-cost pipeline, each stage running the interleaved order at v = 1.
inline int stage_steps(int S, int M, int split) {
  std::vector<int> st((size_t)2 * S * M, -1);  // start of F(s, m), then B(s, m)
  auto at = [&](int kind, int s, int m) -> int& { return st[((size_t)kind * S + s) * M + m]; };
  const int durB = split ? 1 : 2, n = (split ? 3 : 2) * M;
  std::vector<GenInter> g(S);
  std::vector<int> pos(S, 0), clock(S, 0);
  for (int s = 0; s < S; ++s) g[s].init(S, 1, M, s, split, split ? s : 0);
  int steps = 0;
  for (bool go = true; go;) {
    go = false;
    for (int s = 0; s < S; ++s)
      for (; pos[s] < n; ++pos[s], go = true) {
        const int kind = g[s].kind, m = g[s].m;
        int in = 0;  // the producer's end
        if (kind == KF && s > 0) {
          if (at(KF, s - 1, m) < 0) break;
          in = at(KF, s - 1, m) + 1;
        } else if (kind == KB && s < S - 1) {
          if (at(KB, s + 1, m) < 0) break;
          in = at(KB, s + 1, m) + durB;
        }
        const int t = std::max(clock[s], in);
        if (kind != KW) at(kind, s, m) = t;
        clock[s] = t + (kind == KB ? durB : 1);
        steps = std::max(steps, t + 1);
        g[s].advance(true);
      }
  }
  for (int s = 0; s < S; ++s)
    for (int m = 0; m + 2 < M; ++m) {
      if (s < S - 1 && at(KF, s + 1, m) >= at(KF, s, m + 2)) return 0;
      if (s > 0 && at(KB, s - 1, m) >= at(KB, s, m + 2)) return 0;
    }
  return steps;
}

// Whether k_static_build's schedule of the interleaved order (looped, P devices, v stages each) is
// valid: the same lockstep rounds, counting the values alive between their producer's and their
// reader's round.
inline bool inter_schedule_fits(int P, int M, int v, int split) {
  if (v >= 2 && M % P != 0) return true;  // no such record is valid
  const int S = P * v, n = (split ? 3 : 2) * v * M, neg = sc_neg(sc_slots(P, v));
  std::vector<char> done((size_t)2 * S * M, 0);
  std::vector<GenInter> g(P);
  std::vector<int> pos(P, 0);
  std::vector<size_t> now;
  for (int c = 0; c < P; ++c) g[c].init(P, v, M, c, split, split ? c : 0);
  int live = 0, left = P;
  for (int round = 0; left > 0; ++round) {
    if (round >= sc_round_cap(P, M, v)) return false;
    now.clear();
    for (int c = 0; c < P; ++c) {
      if (pos[c] == n) continue;
      const int kind = g[c].kind, m = g[c].m, s = c + g[c].k * P;
      const int ps = kind == KF ? s - 1 : kind == KB ? s + 1 : -1;
      const bool cross = ps >= 0 && ps < S;
      if (cross && !done[((size_t)kind * S + ps) * M + m]) continue;
      if (cross && P > 1) --live;  // read, and nobody else's
      if (kind != KW) now.push_back(((size_t)kind * S + s) * M + m);
      if (P > 1 && ((kind == KF && s < S - 1) || (kind == KB && s > 0))) ++live;
      if (++pos[c] == n) --left;
      g[c].advance(true);
    }
    if (live > neg) return false;
    for (size_t x : now) done[x] = 1;
  }
  return true;
}

}  // namespace octo
