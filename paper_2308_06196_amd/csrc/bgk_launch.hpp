// bgk_launch.hpp -- host-side launch interface between the C-ABI runtime and
// the gfx950 kernels. Internal to libbgk.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "bgk_device.hpp"

namespace bgk {

// Velocities covered by one work-group of the stage kernel (the moment
// partials are per such chunk).
int velocities_per_block(int dim, int order, int precision);
// Hexahedra of this order and storage precision run the one-lane-per-velocity
// stage kernels (else the plane-split ones).
bool hex_one_lane(int order, int precision);

// Elements per work item of the column-sweep stage kernels for this mesh,
// velocity grid and storage precision on the current device (0: no sweep).
int sweep_segment(const DevGeom& g, int precision, bool collide);
// Plane-split hexahedra (p = 3, FP64 storage or BF16 increments): RK stage by
// k_stage_walk, and its tile (elements per row, rows); ncols: most row entries
// per node of any velocity chunk.
hipError_t launch_walk(int precision, const StageArgs& A, hipStream_t s);
void walk_tile(const DevGeom& g, int precision, int ncols, int* tx, int* ty);
// Segments and low-order quadrilaterals: RK stage with several elements of a
// mesh row per work-group (k_stage_rows). rows_pay: whether a solver of this
// mesh uses it; rows_runs: work items per velocity chunk; rows_tab_bytes: LDS
// of the equilibrium rows.
bool rows_pay(const DevGeom& g, int precision, bool collide);
int64_t rows_runs(const DevGeom& g);
size_t rows_tab_bytes(const DevGeom& g, bool collide);
hipError_t launch_rows(int precision, const StageArgs& A, hipStream_t s);
hipError_t launch_rows_batch(int precision, int dim, int order, int stage, const StageArgs* args,
                             const BatchList* list, size_t tab_bytes, unsigned grid,
                             hipStream_t s);
// Some p = 3 quadrilaterals and p <= 2 hexahedra: RK stage by runs of elements
// along x (k_stage_xwalk), and their length (0: not used).
hipError_t launch_xwalk(int precision, const StageArgs& A, hipStream_t s);
int xwalk_length(const DevGeom& g, int precision);
// mode 0: fused RK stage (a variant that does not read f^n when a = 0);
// 1: residual L(f) in FP64; 2: moment partials only; 3, 4: the same two of a
// canonical FP64 array A.fin in lexicographic velocity order (A.g with a single
// octant).
hipError_t launch_stage(int precision, int mode, const StageArgs& A, hipStream_t s);
hipError_t launch_newton(const NewtonArgs& A, hipStream_t s);
// Re-emitted densities of the diffuse-wall flux points of the stage input.
// canonical: W.fin is a canonical FP64 array (W.g with a single octant).
hipError_t launch_wall(int precision, bool canonical, const WallArgs& W, hipStream_t s);
hipError_t launch_reduce_partials(const DevGeom& g, const double* partials, double* Q,
                                  hipStream_t s);
// Moments of the collision term of the stage input A.fin into Cm[nx][5]
// (uses A.partials as scratch).
hipError_t launch_collision_moments(int precision, const StageArgs& A, double* Cm,
                                    hipStream_t s);
// Team size of the equilibrium solve for a mesh of nx nodes.
int newton_team(int64_t nx);
// Whether it sums a velocity grid's axes one after another past the shortest.
bool newton_split(const DevGeom& g);
// Batched launches over descriptor tables in device memory (1-D and 2-D
// members, FP64 or FP32 storage): RK stage `stage` of the members of one
// kernel family, the equilibrium solves of the members of one team size and kind, the
// diffuse-wall fluxes of one family and the wall densities of all members.
// grid: the list's work units (one per work-group); 0 launches nothing.
hipError_t launch_stage_batch(int precision, int dim, int order, int stage, const StageArgs* args,
                              const BatchList* list, size_t tab_bytes, unsigned grid,
                              hipStream_t s);
hipError_t launch_newton_batch(int team, bool split, const NewtonArgs* args,
                               const BatchList* list, unsigned grid, hipStream_t s);
hipError_t launch_wall_flux_batch(int precision, int dim, int order, int stage,
                                  const WallArgs* args, const BatchList* list, unsigned grid,
                                  hipStream_t s);
hipError_t launch_wall_rho_batch(int stage, const WallArgs* args, const BatchList* list,
                                 unsigned grid, hipStream_t s);
hipError_t launch_maxwellian(int precision, const DevGeom& g, const double* prim, void* f,
                             hipStream_t s);
hipError_t launch_to_storage(int precision, const DevGeom& g, const double* in, void* out,
                             int64_t i0, int64_t m, hipStream_t s);
hipError_t launch_from_storage(int precision, const DevGeom& g, const void* in, double* out,
                               int64_t i0, int64_t m, hipStream_t s);

}  // namespace bgk
