// bgk_xwalk.hip -- instantiations and launcher of the x walk.
#include <type_traits>

#include "bgk_launch.hpp"
#include "bgk_xwalk.hpp"
#include "bgk_xwalk_rule.hpp"

namespace bgk {

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

int xwalk_length(const DevGeom& g, int precision) { return xwalk_run_length(g, precision); }

}  // namespace bgk
