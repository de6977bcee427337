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

static int resident_walks(int precision, int ncols, int tx) {
  return precision == 0
             ? resident_groups(k_stage_walk<double, 0, false>, HexWalk::lds_bytes<double>(ncols, tx))
             : resident_groups(k_stage_walk<float, 0, true>, HexWalk::lds_bytes<float>(ncols, tx));
}

// LDS that one walking work-group may take: a compute unit's 160 KB less its
// line operators.
constexpr int kWalkLds = 160 * 1024 - 4 * (int)sizeof(LineOps);

// Velocity chunks that hold velocities of more than one octant.
static int mixed_chunks(const DevGeom& g) {
  const int vb = HexWalk::VB;
  int mixed = 0;
  for (int c = 0; c < g.nchunk; ++c) {
    bool m = false;
    for (int q = 1; q < 8; ++q)
      m = m || (g.voct[q] > c * vb && g.voct[q] < std::min<int64_t>((c + 1) * vb, g.nv));
    mixed += m;
  }
  return mixed;
}

// Tile of a mesh that gives the device few (element, velocity chunk) pairs per
// resident work-group, fewer than 30, or 2 where no chunk is mixed: a single wave of
// large tiles then ends with its slowest, and small meshes leave the device idle. A
// chunk whose velocities differ in sign (mixed) costs about twice the others' time per
// element (it reads its x and y neighbours, and forms z once per sign); a
// work-group's start costs 1.5 elements, 0.6 where the device is half idle, and
// the last work-groups run half alone. Least of that estimate over tiles of 1 to
// 5 x 1 to ny. Stage launches of 194 problems (1 to 16 elements per axis, 8^3 to
// 20^3 velocities), tiles by the rule for large meshes / by this one / the fastest
// of 16 measured, us: BF16 increments 7 x 9 x 5 on 15 x 14 x 17 466 / 328 / 315, 8 x
// 2 x 2 on 13 x 11 x 9 51 / 25 / 26; FP64 4^3 on 13 x 11 x 9 58 / 52 / 52; 11 % faster
// in the mean, none more than 5 % slower.
static void small_mesh_tile(const DevGeom& g, int precision, int ncols, int mixed, int* tx_out,
                            int* ty_out) {
  const int nx = g.nelem[0], ny = g.nelem[1], nz = g.nelem[2];
  const double start = 1.5, idle = 0.6, top = mixed ? 2.0 : 1.0;
  double best = 0.0;
  for (int tx = 1; tx <= std::min(nx, 5); ++tx) {
    const int resident = resident_walks(precision, ncols, tx);
    if (resident <= 0) continue;
    for (int ty = 1; ty <= ny; ++ty) {
      const double tiles = (double)((nx + tx - 1) / tx) * ((ny + ty - 1) / ty) * nz;
      const double R = g.nchunk * tiles / resident, one = tx * ty * top + start;
      const double all = ((double)(g.nchunk + mixed) * g.ne + start * tiles * g.nchunk) / resident;
      double cost;
      if (R <= 1.0)
        cost = one - (start - idle) * (1.0 - std::max(0.0, 2.0 * R - 1.0));
      else if (mixed == 0 && nx % tx == 0 && ny % ty == 0 && R < 3.0)
        cost = std::ceil(R) * one;
      else
        cost = std::max(one, all + 0.5 * one);
      if (best == 0.0 || cost < best) best = cost, *tx_out = tx, *ty_out = ty;
    }
  }
}

// Large meshes: rows of up to five elements: four kept two FP64 (three BF16)
// work-groups per CU, where rows of eight leave one by their LDS (16^3-element
// Taylor-Green box, ms per launch, rows of 2, 4, 8: FP64 5.22, 5.07, 6.30; BF16
// 3.56, 3.47, 3.84). A work-group's start (its operators, and the first loads,
// which nothing covers) costs as much as about 3.5 elements (tiles of 4 x 8
// instead of 4 x 16: FP64 5.29, BF16 3.52), so a tile takes as many rows as leave
// enough work-groups for the device: the count minimises (1 + 3.5 / elements)
// / eff, eff = R / ceil(R) for R = work-groups / resident work-groups.
void walk_tile(const DevGeom& g, int precision, int ncols, int* tx_out, int* ty_out) {
  const int nx = g.nelem[0], ny = g.nelem[1];
  int tx = (nx + (nx + 4) / 5 - 1) / ((nx + 4) / 5), ty = ny;
  const int resident = resident_walks(precision, ncols, tx);
  const int mixed = mixed_chunks(g);
  if (resident > 0 && (double)g.ne * g.nchunk < (mixed ? 30.0 : 2.0) * resident) {
    small_mesh_tile(g, precision, ncols, mixed, &tx, &ty);
  } else if (resident > 0) {
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
      tx = std::min(x, nx);
      ty = std::min(y, ny);
      // (a row's y traces must fit a compute unit's LDS beside the equilibrium rows,
      // those of up to five elements always do)
      auto lds = [&] {
        return precision == 0 ? HexWalk::lds_bytes<double>(ncols, tx)
                              : HexWalk::lds_bytes<float>(ncols, tx);
      };
      while (tx > 1 && lds() > kWalkLds) --tx;
    }
  }
  *tx_out = tx;
  *ty_out = ty;
}

}  // namespace bgk
