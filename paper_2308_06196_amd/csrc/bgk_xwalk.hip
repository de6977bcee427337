// bgk_xwalk.hip -- instantiations and launcher of the x walk.
#include <cstdlib>
#include <type_traits>

#include "bgk_launch.hpp"
#include "bgk_xwalk.hpp"

namespace bgk {

// (dimension, order, precision) that walk
#define BGK_XWALK_CASES \
  BGK_CASE(2, 3, 1) BGK_CASE(2, 3, 2) BGK_CASE(3, 1, 0) BGK_CASE(3, 1, 1) BGK_CASE(3, 1, 2) \
  BGK_CASE(3, 2, 2)

template <int D, int P, typename ST, int MODE, bool INC>
static void xwalk_one(const StageArgs& A, hipStream_t s) {
  const DevGeom& g = A.g;
  const int64_t runs = (int64_t)((g.nelem[0] + A.walk_tx - 1) / A.walk_tx) * (g.ne / g.nelem[0]);
  hipLaunchKernelGGL((k_stage_xwalk<D, P, ST, MODE, INC>), dim3((unsigned)(g.nchunk * runs)),
                     dim3(kBlock), (XWalk<D, P>::template lds_bytes<ST>(A.walk_ncols)), s, A);
}

template <int D, int P, int PREC>
static void xwalk_case(const StageArgs& A, hipStream_t s) {
  using ST = std::conditional_t<PREC == 0, double, float>;
  constexpr bool kInc = PREC == 2;
  if (kInc ? A.din != nullptr : A.a != 0.0) xwalk_one<D, P, ST, 0, kInc>(A, s);
  else xwalk_one<D, P, ST, 3, kInc>(A, s);
}

static int xwalk_key(const DevGeom& g, int precision) {
  return g.dim * 100 + (g.n1 - 1) * 10 + precision;
}

hipError_t launch_xwalk(int precision, const StageArgs& A, hipStream_t s) {
  switch (xwalk_key(A.g, precision)) {
#define BGK_CASE(D, P, PREC)       \
  case D * 100 + P * 10 + PREC:    \
    xwalk_case<D, P, PREC>(A, s); \
    break;
    BGK_XWALK_CASES
#undef BGK_CASE
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Share of the waves whose velocities all move with their chunk's walk.
static double carried_share(const DevGeom& g) {
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

// Runs of at most 8 elements on quadrilaterals (FP32, 32^2 box, us per launch,
// runs of 4, 8, 16, 32: 551, 541, 549, 556), 16 on hexahedra (p = 1 Taylor-Green
// box, FP64, 8 and 16: 738, 726), and not so long that fewer than about 4096
// work-groups are left (45 x 29 box, 8, 15, 23, 45: 419, 428, 449, 480; 16 x 5 x
// 5 elements on 24^3 velocities, p = 1, FP64, 0 (per element), 4, 8, 16: 314,
// 253, 258, 274). Where that leaves runs too short to pay, one work-group per
// element stays: quadrilaterals below 6 (20^2 box on 16^3, per element and runs
// of 2, 3, 4, 8: 70.2, 73.1, 71.3, 73.3, 78.6), p = 1 hexahedra below 3 (4 x 9 x 6
// on 16^3, FP64, 0, 2, 3: 50.0, 51.1, 50.2), in FP32 arithmetic below 8 (8^3 on
// 20^3, FP32, 0 and 4: 139, 143; 16 x 5 x 5 with increments, 0, 4, 8: 209, 213,
// 220). p = 2 hexahedra with increments always gain (6^3 on
// 16^3, 0, 2, 4: 139.7, 96.9, 121.9). The others also need nearly all waves to
// move with their chunk: on 15^3 velocities, where an octant holds 1.3 to 2
// chunks, most do not (14 x 9 x 12, p = 1, FP32 161 per element, 180 in runs;
// quadrilaterals with increments, share 0.83 on 16 x 16 x 12 as above, 0.63 on
// 13^3 157 and 160, 0.25 on 9^3 141 and 149).
int xwalk_length(const DevGeom& g, int precision) {
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
  const int shortest = g.dim == 2 ? 6 : g.n1 == 3 ? 2 : precision != 0 ? 8 : 3;
  const bool inc2 = g.dim == 2 && precision == 2;
  int len = (int)std::min<int64_t>(g.dim == 2 ? 8 : 16, units / (inc2 ? 3072 : 4096));
  if (g.dim == 3 && g.n1 == 3 && units >= 1024) len = std::max(len, shortest);
  if (len < shortest || (shortest > 2 && carried_share(g) < (inc2 ? 0.7 : 0.85))) return 0;
  const int runs = std::max(1, (nx + len / 2) / len);
  len = (nx + runs - 1) / runs;
  return len < shortest ? 0 : len;
}

}  // namespace bgk
