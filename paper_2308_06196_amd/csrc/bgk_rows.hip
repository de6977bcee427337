// bgk_rows.hip -- instantiations and launchers of the stage kernels that run
// several elements of a mesh row per work-group.
#include "bgk_launch.hpp"
#include "bgk_rows_rule.hpp"

namespace bgk {

int64_t rows_runs(const DevGeom& g) {
  const int E = row_elems_of(g);
  return (int64_t)((g.nelem[0] + E - 1) / E) * (g.dim == 2 ? g.nelem[1] : 1);
}

size_t rows_tab_bytes(const DevGeom& g, bool collide) { return row_tab_bytes(g, collide); }

bool rows_pay(const DevGeom& g, int precision, bool collide) {
  return row_runs_pay(g, precision, collide);
}

template <int D, int P, typename ST>
static void rows_mode(bool inc, const StageArgs& A, dim3 grid, size_t lds, hipStream_t s) {
  if constexpr (sizeof(ST) == 4) {
    if (inc) {
      if (A.din)
        hipLaunchKernelGGL((k_stage_rows<D, P, ST, 0, true>), grid, dim3(kBlock), lds, s, A);
      else
        hipLaunchKernelGGL((k_stage_rows<D, P, ST, 3, true>), grid, dim3(kBlock), lds, s, A);
      return;
    }
  }
  if (A.a != 0.0)
    hipLaunchKernelGGL((k_stage_rows<D, P, ST, 0>), grid, dim3(kBlock), lds, s, A);
  else
    hipLaunchKernelGGL((k_stage_rows<D, P, ST, 3>), grid, dim3(kBlock), lds, s, A);
}

template <typename ST>
static hipError_t rows_dispatch(bool inc, const StageArgs& A, hipStream_t s) {
  const dim3 grid((unsigned)(A.g.nchunk * rows_runs(A.g)));
  const size_t lds = std::max(rows_tab_bytes(A.g, A.collide), (size_t)mfma_lds_bytes<ST>());
  switch (A.g.dim * 10 + (A.g.n1 - 1)) {
#define BGK_CASE(D, P)                        \
  case D * 10 + P:                            \
    rows_mode<D, P, ST>(inc, A, grid, lds, s); \
    break;
    BGK_ROWS_CASES
#undef BGK_CASE
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_rows(int precision, const StageArgs& A, hipStream_t s) {
  return precision == 0 ? rows_dispatch<double>(false, A, s)
                        : rows_dispatch<float>(precision == 2, A, s);
}

template <int D, int P, typename ST>
static void rows_batch(int stage, const StageArgs* args, const BatchList* list, size_t lds,
                       unsigned grid, hipStream_t s) {
  if (stage == 0)
    hipLaunchKernelGGL((k_stage_rows_batch<D, P, ST, 3>), dim3(grid), dim3(kBlock), lds, s,
                       (table_ptr<StageArgs>)args, (table_ptr<BatchList>)list, stage);
  else
    hipLaunchKernelGGL((k_stage_rows_batch<D, P, ST, 0>), dim3(grid), dim3(kBlock), lds, s,
                       (table_ptr<StageArgs>)args, (table_ptr<BatchList>)list, stage);
}

hipError_t launch_rows_batch(int precision, int dim, int order, int stage, const StageArgs* args,
                             const BatchList* list, size_t tab_bytes, unsigned grid,
                             hipStream_t s) {
  if (grid == 0) return hipSuccess;
  const size_t lds = std::max(tab_bytes, (size_t)(precision == 0 ? mfma_lds_bytes<double>()
                                                                  : mfma_lds_bytes<float>()));
  switch (dim * 10 + order) {
#define BGK_CASE(D, P)                                                      \
  case D * 10 + P:                                                          \
    if (precision == 0) rows_batch<D, P, double>(stage, args, list, lds, grid, s); \
    else rows_batch<D, P, float>(stage, args, list, lds, grid, s);          \
    break;
    BGK_ROWS_CASES
#undef BGK_CASE
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace bgk
