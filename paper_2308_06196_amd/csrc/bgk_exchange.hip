// bgk_exchange.hip -- exchange of states between the canonical and the internal
// layout, and Maxwellian sampling: kernels and launchers.
#include <cmath>

#include <algorithm>

#include "bgk_launch.hpp"

namespace bgk {

// Exchange between the canonical FP64 layout f[elem][node][vel] and the
// internal layout in storage precision (velocity blocks, velocities in slot
// order): entries i0 .. i0+m-1 of the canonical array, held at canon[0 .. m-1]
// (a staging window or the whole array). A lane decodes its velocity once and
// walks NODES consecutive nodes. Lanes follow the written order, so that stores
// are whole lines; the gathered side's partial lines meet in the L2 of the XCD
// that runs the neighbouring chunks. HBM-bound with 16 nodes per lane (one entry
// per lane and iteration, with its two divisions, took 1.00 ms for the FP32 state
// of the 32^2 box, 2.7 TB/s; this 0.52, 5.3 TB/s; FP64 state of the 16^3-element
// Taylor-Green box 4.53 -> 2.89 ms, 5.95 TB/s).
// exchange_shape chooses the nodes per lane and the lanes' order.
// Indices of nodes and lanes fit 32 bits (checked with the footprint), whose
// divisions are short.
struct XShape {
  uint32_t n0;     // first node
  uint32_t lanes;  // per node group, at least nv; whole work-groups unless DENSE
};
struct XItem {
  uint32_t n;      // first node of this lane
  uint32_t first;  // first node of the work-group
  uint32_t j;      // velocity of this lane in the written order
};
// (a uniform quotient is formed on the vector unit: back to a scalar register, so
// that what follows from it stays scalar)
__device__ __forceinline__ uint32_t uniform(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
}
template <int NODES, bool DENSE>
__device__ __forceinline__ XItem exchange_item(const XShape x) {
  const uint32_t tid = threadIdx.x;
  const uint32_t nb = gridDim.x, xcd = blockIdx.x % kNumXCD, per = nb / kNumXCD, rem = nb % kNumXCD;
  const uint32_t w = xcd * per + (xcd < rem ? xcd : rem) + blockIdx.x / kNumXCD;  // xcd_remap
  const uint32_t r = uniform(w * kBlock / x.lanes), t = w * kBlock - r * x.lanes + tid;
  const uint32_t q = DENSE ? t / x.lanes : 0, first = x.n0 + r * NODES;
  return {first + q * NODES, first, t - q * x.lanes};
}
// Consecutive nodes of the mesh from n on: their offsets in the internal layout at
// slot j, with one division for the first.
template <bool UNIFORM>
struct NodeWalk {
  uint32_t e, a;
  __device__ __forceinline__ NodeWalk(const DevGeom& g, uint32_t n) {
    e = n / (uint32_t)g.ns;
    if constexpr (UNIFORM) e = uniform(e);
    a = n - e * (uint32_t)g.ns;
  }
  __device__ __forceinline__ int64_t offset(const DevGeom& g, uint32_t j) const {
    return f_offset(g, e, (int)a, j);
  }
  __device__ __forceinline__ void next(const DevGeom& g) {
    const bool last = a + 1 == (uint32_t)g.ns;
    a = last ? 0 : a + 1;
    e += last ? 1 : 0;
  }
};

template <typename DST, int NODES, bool DENSE>
__global__ void __launch_bounds__(kBlock) k_to_internal(const DevGeom g, const double* canon,
                                                        DST* f, int64_t i0, int64_t m,
                                                        const XShape shape) {
  const XItem x = exchange_item<NODES, DENSE>(shape);
  if (x.j >= (uint32_t)g.nv) return;
  int b[3];
  slot_nodes(g, x.j, b);
  const int jc = b[0] + g.nv1[0] * (b[1] + g.nv1[1] * b[2]);
  double v[NODES];
#pragma unroll
  for (int q = 0; q < NODES; ++q) {
    const int64_t t = (int64_t)(x.n + q) * g.nv + jc - i0;
    v[q] = canon[t < 0 ? 0 : t < m ? t : m - 1];
  }
  NodeWalk<!DENSE> w(g, x.n);
#pragma unroll
  for (int q = 0; q < NODES; ++q, w.next(g)) {
    const int64_t t = (int64_t)(x.n + q) * g.nv + jc - i0;
    if (t >= 0 && t < m) f[w.offset(g, x.j)] = (DST)v[q];
  }
}

template <typename SRC, int NODES, bool DENSE>
__global__ void __launch_bounds__(kBlock) k_to_canonical(const DevGeom g, const SRC* f,
                                                         double* canon, int64_t i0, int64_t m,
                                                         const XShape shape) {
  const XItem x = exchange_item<NODES, DENSE>(shape);
  if (x.j >= (uint32_t)g.nv) return;
  const int slot = vel_slot_of_canonical(g, x.j);
  SRC v[NODES];
  NodeWalk<!DENSE> w(g, min(x.n, (uint32_t)g.nx - 1));
#pragma unroll
  for (int q = 0; q < NODES; ++q) {
    v[q] = f[w.offset(g, slot)];
    if (x.n + q + 1 < (uint32_t)g.nx) w.next(g);
  }
#pragma unroll
  for (int q = 0; q < NODES; ++q) {
    const int64_t t = (int64_t)(x.n + q) * g.nv + x.j - i0;
    if (t >= 0 && t < m) __builtin_nontemporal_store((double)v[q], &canon[t]);
  }
}

// Continuous Maxwellian sampled at every (node, velocity), by the exchange
// kernels' work items; the nodes' normalisations (a power each) are formed
// once per work-group (nv >= 8, so that it covers at most kBlock / 8 + 1 node
// groups).
template <typename ST, int NODES, bool DENSE>
__global__ void __launch_bounds__(kBlock) k_maxwellian(const DevGeom g, const double* prim, ST* f,
                                                       const XShape shape) {
  __shared__ double nrm[(DENSE ? kBlock / 8 + 1 : 1) * NODES];
  const XItem x = exchange_item<NODES, DENSE>(shape);
  const int groups = DENSE ? (kBlock - 2) / (int)shape.lanes + 2 : 1;
  for (int t = threadIdx.x; t < groups * NODES; t += kBlock) {
    const double* q = prim + (int64_t)min(x.first + t, (uint32_t)g.nx - 1) * 5;
    nrm[t] = q[0] / pow(2.0 * M_PI * q[4], 1.5);
  }
  __syncthreads();
  if (x.j >= (uint32_t)g.nv) return;
  const Vel v = velocity_of(g, x.j);
  const double* nr = nrm + (DENSE ? x.n - x.first : 0);
  NodeWalk<!DENSE> w(g, x.n);
#pragma unroll 4
  for (int i = 0; i < NODES; ++i, w.next(g)) {
    const uint32_t n = x.n + i;
    if (n >= (uint32_t)g.nx) break;
    const double* q = prim + (int64_t)n * 5;
    const double dx = v.u[0] - q[1], dy = v.u[1] - q[2], dz = v.u[2] - q[3];
    f[w.offset(g, x.j)] =
        (ST)(nr[i] * exp(-(dx * dx + dy * dy + dz * dz) / (2.0 * q[4])));
  }
}

// Shape of an exchange launch that covers the nodes of entries i0 .. i0 + m - 1:
// nodes per lane (returned), the lanes per node group and the grid. 16 nodes per
// lane need enough entries to fill the device, and work-groups of 256 velocities
// leave lanes idle where those do not nearly divide by 256: the lanes then run on
// into the next nodes, in whole waves unless those are as empty. FP64 state to
// canonical, us, one entry per lane of a strided grid / 16 nodes and 256 velocities
// / now: 120 nodes on 8^3 velocities 24.7 27.6 24.6; 270,000 on 2^3 36 53 33, on 5^3
// 178 127 121, on 6 x 6 x 8 358 330 248. (480 on 12^3, 0.8e6 entries, with 16, 4, 1
// nodes per lane 27.4 26.7 27.9. From 4e6 entries on 16 and 4 differ by 8 % either
// way, and the sampler is up to 30 % faster with 16.)
static int exchange_shape(const DevGeom& g, int64_t i0, int64_t m, XShape* x, dim3* grid) {
  const int64_t n0 = i0 / g.nv, nodes = (i0 + m - 1) / g.nv + 1 - n0;
  const int per = m < 400000 ? 1 : m < 4000000 ? 4 : 16;
  auto padded = [&](int64_t to) { return (g.nv + to - 1) / to * to; };
  auto full = [&](int64_t lanes) { return 20 * g.nv >= 17 * lanes; };
  int64_t lanes = padded(kBlock);
  if (per == 1 || !full(lanes)) lanes = full(padded(64)) ? padded(64) : g.nv;
  x->n0 = (uint32_t)n0;
  x->lanes = (uint32_t)lanes;
  *grid = dim3((unsigned)(((nodes + per - 1) / per * lanes + kBlock - 1) / kBlock));
  return per;
}

#define BGK_EXCHANGE_N(K, T, N, DENSE, ...) \
  hipLaunchKernelGGL((K<T, N, DENSE>), grid, dim3(kBlock), 0, s, g, __VA_ARGS__, x)
#define BGK_EXCHANGE(K, T, ...)                  \
  if (per == 1)                                  \
    BGK_EXCHANGE_N(K, T, 1, true, __VA_ARGS__);  \
  else if (per == 4 && x.lanes % kBlock != 0)    \
    BGK_EXCHANGE_N(K, T, 4, true, __VA_ARGS__);  \
  else if (per == 4)                             \
    BGK_EXCHANGE_N(K, T, 4, false, __VA_ARGS__); \
  else if (x.lanes % kBlock != 0)                \
    BGK_EXCHANGE_N(K, T, 16, true, __VA_ARGS__); \
  else                                           \
    BGK_EXCHANGE_N(K, T, 16, false, __VA_ARGS__)

hipError_t launch_maxwellian(int precision, const DevGeom& g, const double* prim, void* f,
                             hipStream_t s) {
  XShape x;
  dim3 grid;
  const int per = exchange_shape(g, 0, g.nx * g.nv, &x, &grid);
  if (precision == 0) {
    BGK_EXCHANGE(k_maxwellian, double, prim, (double*)f);
  } else {
    BGK_EXCHANGE(k_maxwellian, float, prim, (float*)f);
  }
  return hipGetLastError();
}

hipError_t launch_to_storage(int precision, const DevGeom& g, const double* in, void* out,
                             int64_t i0, int64_t m, hipStream_t s) {
  if (m <= 0) return hipSuccess;
  XShape x;
  dim3 grid;
  const int per = exchange_shape(g, i0, m, &x, &grid);
  if (precision == 0) {
    BGK_EXCHANGE(k_to_internal, double, in, (double*)out, i0, m);
  } else {
    BGK_EXCHANGE(k_to_internal, float, in, (float*)out, i0, m);
  }
  return hipGetLastError();
}

hipError_t launch_from_storage(int precision, const DevGeom& g, const void* in, double* out,
                               int64_t i0, int64_t m, hipStream_t s) {
  if (m <= 0) return hipSuccess;
  XShape x;
  dim3 grid;
  const int per = exchange_shape(g, i0, m, &x, &grid);
  if (precision == 0) {
    BGK_EXCHANGE(k_to_canonical, double, (const double*)in, out, i0, m);
  } else {
    BGK_EXCHANGE(k_to_canonical, float, (const float*)in, out, i0, m);
  }
  return hipGetLastError();
}
#undef BGK_EXCHANGE
#undef BGK_EXCHANGE_N

}  // namespace bgk
