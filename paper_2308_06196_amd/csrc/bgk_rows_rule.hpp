// bgk_rows_rule.hpp -- which solvers run their stages with several elements of a
// mesh row per work-group (bgk_rows.hpp). Host code without kernels of its own.
#pragma once

#include <cstdlib>

#include "bgk_rows.hpp"

namespace bgk {

#define BGK_ROWS_CASES \
  BGK_CASE(1, 1) BGK_CASE(1, 2) BGK_CASE(1, 3) BGK_CASE(2, 1) BGK_CASE(2, 2)

inline int row_elems_of(const DevGeom& g) {
  switch (g.dim * 10 + (g.n1 - 1)) {
#define BGK_CASE(D, P) \
  case D * 10 + P:     \
    return row_elems<D, P>();
    BGK_ROWS_CASES
#undef BGK_CASE
    default:
      return 0;
  }
}

inline size_t row_tab_bytes(const DevGeom& g, bool collide) {
  return collide ? (size_t)row_elems_of(g) * g.ns * g.tabw * sizeof(double) : 0;
}

// Runs need enough work items to fill the device: from 1024 per-element ones
// (element x velocity chunk) on they measured faster (FP64, us per launch, per
// element / runs: 512-element tube on 8^3 velocities, 1024 items, 13.8 / 12.2;
// 128-element tube on 16^3, 2048 items, 19.6 / 14.6; 32-element tube on 16^3,
// 512 items, 10.2 / 11.7; 16^2 box on 8^3, 512 items, 13.8 / 14.6). On quadrilaterals
// what a row leaves of its last run empty counts: p = 1 (runs of four) gains on rows
// of 3 and 5 but not of one (1 x 60 elements on 20^3, FP64 24.9 / 32.0, FP32 18.0 / 22.6);
// p = 2 (runs of two) in FP64 loses on 3 x 40 (16^3 30.9 / 33.0, 20^3, 3840 items, 54.3 /
// 56.8, but 24^3, 6480, 99.4 / 88.8), and on 5 x 31 and 7 x 7 with few items (1085 21.9 /
// 22.6, 1568 27.3 / 28.3), in FP32 arithmetic
// on 5 x 31 with any number (24^3, 8370 items, 63.3 / 65.3; 7 x 7 equal) and on one or
// two chunks (33 x 33 on 6^3 15.3 / 16.9, on 8^3 22.9 / 23.7, 24 x 24 on 8^3 15.3 / 17.1; 8 x
// 8 on 16^3, 1024 items, 14.0 / 14.6).
inline bool row_runs_pay(const DevGeom& g, int precision, bool collide) {
  const int E = row_elems_of(g), nx = g.nelem[0];
  if (E == 0 || row_tab_bytes(g, collide) > (size_t)kMaxTabBytes) return false;
  // BGK_ROWS overrides the choice (0 or 1)
  if (const char* env = getenv("BGK_ROWS")) return atoi(env) != 0;
  const int64_t units = g.ne * g.nchunk;
  if (units < 1024) return false;
  const double waste = (double)((nx + E - 1) / E * E) / nx;
  if (g.dim == 1) return true;
  if (g.n1 == 2) return waste < 2.0;
  if (precision != 0) return waste <= 1.1 && g.nchunk >= 3 && units >= 1200;
  return waste <= (units < 1600 ? 1.1 : units < 5000 ? 1.2 : 1.34);
}

}  // namespace bgk
