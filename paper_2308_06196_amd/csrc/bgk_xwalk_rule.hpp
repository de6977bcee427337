// bgk_xwalk_rule.hpp -- which solvers run their stages by the x walk
// (bgk_xwalk.hpp), and the length of the runs. Host code without kernels.
#pragma once

#include <cstdlib>

#include <algorithm>

#include "bgk_device.hpp"

namespace bgk {

// (dimension, order, precision) that walk
#define BGK_XWALK_CASES \
  BGK_CASE(2, 3, 1) BGK_CASE(2, 3, 2) BGK_CASE(3, 1, 0) BGK_CASE(3, 1, 1) BGK_CASE(3, 1, 2) \
  BGK_CASE(3, 2, 2)

inline int xwalk_key(const DevGeom& g, int precision) {
  return g.dim * 100 + (g.n1 - 1) * 10 + precision;
}

// Share of the waves whose velocities all move with their chunk's walk.
inline double carried_share(const DevGeom& g) {
  int waves = 0, carried = 0;
  auto positive = [&](int j) {
    int b[3];
    slot_nodes(g, j, b);
    return (g.vlo[0] + b[0] * g.du[0]) * g.scale[0] > 0.0;
  };
  for (int j0 = 0; j0 < g.nv; j0 += 64, ++waves) {
    const bool up = positive(j0 / kBlock * kBlock);
    bool all = true;
    for (int j = j0; all && j < j0 + 64 && j < g.nv; ++j) all = positive(j) == up;
    carried += all;
  }
  return (double)carried / waves;
}

// Runs of about 8 elements on quadrilaterals (FP32, 32^2 box, us per launch,
// runs of 4, 8, 16, 32: 551, 541, 549, 556), 16 on hexahedra (p = 1 Taylor-Green
// box, FP64, 8 and 16: 738, 726), and not so long that fewer than about 4096
// work-groups are left (16 x 5 x 5 elements on 24^3 velocities, p = 1, FP64, 0
// (per element), 4, 8, 16: 314, 253, 258, 274).
//
// Quadrilaterals gain a few per cent, and only where little goes against the walk.
// Nearly all waves must move with their chunk, and the rows divide into equal runs
// over enough (element, chunk) pairs (per element / walk, 32 x 64 elements: FP32 16^3
// velocities 1.019, 18^3 1.017, 24^3 1.056, 16 x 16 x 12, three quarters of 16^3's
// pairs, 0.94-0.98; increments, share of carried waves 1.00 on 16 x 16 x 12 1.06, 0.90
// on 17^3 1.02, 0.83 on 13^3 0.90-0.99, 0.79 on 14^3 0.90-1.00, 0.67 on 12^3 0.96). Runs
// of unequal length need more work-groups to even out (45 x 29: FP32, 5300 on 21 x 22
// x 17 0.95, 7100 on 22^3 0.98, 9200 on 24^3 1.02; increments, 3900 on 18^3 0.95, 5300
// on 21 x 22 x 17 1.00, 7100 on 22^3 1.05; 13 x 37, 3000 on 22^3 0.92).
//
// p = 1 hexahedra: not below runs of 3 (4 x 9 x 6 on 16^3, FP64, 0, 2, 3: 50.0, 51.1,
// 50.2), in FP32 arithmetic 8 (8^3 on 20^3, FP32, 0 and 4: 139, 143; 16 x 5 x 5 with
// increments, 0, 4, 8: 209, 213, 220), nor where fewer than 0.85 of the waves are
// carried (14 x 9 x 12 on 15^3, FP32 161 per element, 180 in runs).
//
// p = 2 hexahedra with increments gain nearly always, by runs of two on small meshes
// (6^3 on 16^3, 0, 2, 4: 139.7, 96.9, 121.9), except where a run of two is left with
// one of one: rows of three walk whole or not at all (3 x 20 x 20, runs of 2 / 3: 9^3
// velocities, 3600 pairs, 0.84 / 0.95, 12^3, 8400, 0.88 / 1.07, 20^3 0.96 / 1.30), rows of
// five with more pairs (5 x 7 x 9: 1900 pairs 0.96, 2200 1.09, 2800 0.99, 4400 1.08).
inline int xwalk_run_length(const DevGeom& g, int precision) {
  switch (xwalk_key(g, precision)) {
#define BGK_CASE(D, P, PREC) case D * 100 + P * 10 + PREC:
    BGK_XWALK_CASES
#undef BGK_CASE
    break;
    default:
      return 0;
  }
  const int nx = g.nelem[0];
  // BGK_XWALK overrides the choice (0: no walk)
  if (const char* env = getenv("BGK_XWALK")) return std::max(0, std::min(atoi(env), nx));
  const int64_t units = g.ne * g.nchunk;
  auto run = [&](int len) {  // of about len elements, the row in runs of one length
    const int runs = std::max(1, (nx + len / 2) / len);
    return (nx + runs - 1) / runs;
  };
  if (g.dim == 2) {
    const bool inc = precision == 2;
    if (units < (inc ? 6 * 3072 : 8 * 4096)) return 0;
    const int len = run((int)std::min<int64_t>(8, units / (inc ? 3072 : 4096)));
    const int64_t groups = (int64_t)((nx + len - 1) / len) * g.nelem[1] * g.nchunk;
    if (len < 6 || (nx % len != 0 && groups < (inc ? 5120 : 8192))) return 0;
    return carried_share(g) < 0.85 ? 0 : len;
  }
  int len = (int)std::min<int64_t>(16, units / 4096);
  if (g.n1 == 3) {
    if (units < 1024 || nx < 2) return 0;
    len = run(std::max(len, 2));
    if (nx == 3) return units < 6000 ? 0 : 3;
    return nx == 5 && len == 2 && units < 2100 ? 0 : len;
  }
  const int shortest = precision != 0 ? 8 : 3;
  if (len < shortest || carried_share(g) < 0.85) return 0;
  len = run(len);
  return len < shortest ? 0 : len;
}

}  // namespace bgk
