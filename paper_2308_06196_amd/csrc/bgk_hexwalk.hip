// bgk_hexwalk.hip -- instantiations and launcher of the hexahedral walk.
#include <cmath>
#include <cstdio>
#include <cstdlib>

#include "bgk_hexwalk.hpp"
#include "bgk_launch.hpp"

namespace bgk {

template <typename ST, int MODE, bool INC>
static void walk(const StageArgs& A, hipStream_t s) {
  const DevGeom& g = A.g;
  const int64_t tiles = (int64_t)((g.nelem[0] + A.walk_tx - 1) / A.walk_tx) *
                        ((g.nelem[1] + A.walk_ty - 1) / A.walk_ty) * g.nelem[2];
  hipLaunchKernelGGL((k_stage_walk<ST, MODE, INC>), dim3((unsigned)(g.nchunk * tiles)), dim3(kBlock),
                     HexWalk::lds_bytes<ST>(A.walk_ncols, A.walk_tx), s, A);
}

hipError_t launch_walk(int precision, const StageArgs& A, hipStream_t s) {
  if (precision == 0) {
    if (A.a != 0.0) walk<double, 0, false>(A, s);
    else walk<double, 3, false>(A, s);
  } else {
    if (A.din) walk<float, 0, true>(A, s);
    else walk<float, 3, true>(A, s);
  }
  return hipGetLastError();
}

template <typename K>
static int resident_groups(K k, size_t lds) {
  int dev = 0, cus = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k, kBlock, lds) != hipSuccess)
    n = 0;
  (void)hipGetLastError();
  return n * cus;
}

// Rows of up to five elements: four kept two FP64 (three BF16) work-groups per
// CU, where rows of eight leave one by their LDS (16^3-element Taylor-Green
// box, ms per launch, rows of 2, 4, 8: FP64 5.30, 5.07, 6.44; BF16 3.59, 3.41,
// 3.83). A work-group's start (its operators, and the first loads, which
// nothing covers) costs as much as about 3.5 elements (tiles of 4 x 8 instead
// of 4 x 16: FP64 5.38, BF16 3.56), so a tile takes as many rows as leave
// enough work-groups for the device: the count minimises (1 + 3.5 / elements)
// / eff, eff = R / ceil(R) for R = work-groups / resident work-groups.
void walk_tile(const DevGeom& g, int precision, int ncols, int* tx_out, int* ty_out) {
  const int nx = g.nelem[0], ny = g.nelem[1];
  int tx = (nx + (nx + 4) / 5 - 1) / ((nx + 4) / 5), ty = ny;
  const int resident =
      precision == 0
          ? resident_groups(k_stage_walk<double, 0, false>, HexWalk::lds_bytes<double>(ncols, tx))
          : resident_groups(k_stage_walk<float, 0, true>, HexWalk::lds_bytes<float>(ncols, tx));
  if (resident > 0) {
    const double rows = (double)g.nchunk * g.nelem[2] * ((nx + tx - 1) / tx);
    double best = 0.0;
    for (int n = 1; n <= ny; ++n) {  // n tiles per column of rows
      const int t = (ny + n - 1) / n;
      const double R = rows * ((ny + t - 1) / t) / resident;
      const double cost = (1.0 + 3.5 / (tx * t)) / (R / std::ceil(R)) * ((ny + t - 1) / t * t) / ny;
      if (n == 1 || cost < best) best = cost, ty = t;
    }
  }
  // BGK_WALK_TILE=XxY overrides the choice
  if (const char* env = getenv("BGK_WALK_TILE")) {
    int x = 0, y = 0;
    if (sscanf(env, "%dx%d", &x, &y) == 2 && x > 0 && y > 0) {
      tx = std::min(std::min(x, nx), 16);
      ty = std::min(y, ny);
    }
  }
  *tx_out = tx;
  *ty_out = ty;
}

}  // namespace bgk
