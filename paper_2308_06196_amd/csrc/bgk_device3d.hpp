// bgk_device3d.hpp -- residual and moment kernels of hexahedral (d = 3)
// elements that do not fit one lane's registers, on gfx950 (Dzanic &
// Martinelli, arXiv 2308.06196, Sec. 2.1).
//
// Used at p = 3 with FP64 storage and BF16 increments (the RK stages of these
// solvers are k_stage_walk's, bgk_hexwalk.hpp); the other hexahedra run the
// one-lane-per-velocity kernels of bgk_device.hpp. Here the four lanes of a quad
// share one velocity and lane a_z of the quad owns that z-plane of the element:
// 16 nodes. The x and y operators are lane-local exactly as for quadrilaterals; the
// z-derivative and the z-face traces need the other planes of the same column,
// which come from the other lanes of the quad by DPP permutations (no LDS, no
// barriers). A work-group of 256 lanes covers 64 consecutive velocity slots of one
// element.
#pragma once

#include "bgk_device.hpp"

namespace bgk {

struct Plane3 {
  static constexpr int N1 = 4;
  static constexpr int G = N1;                 // lanes per velocity
  static constexpr int VB = kBlock / G;        // velocities per work-group
  static constexpr int P2 = N1 * N1;           // nodes per plane
  static constexpr int NS = N1 * N1 * N1;
};

// Sum over the lanes of a quad (partners lane ^ 1, lane ^ 2; every lane ends with
// the same bits).
template <typename T>
__device__ __forceinline__ T quad_allsum(T x) {
  x += quad_xor<1>(x);
  x += quad_xor<2>(x);
  return x;
}

// Moment partials of one element on the matrix cores (FP64 MFMA), as in the
// 1-D/2-D kernels: per wave and per plane pl, P[q][m] = sum over the wave's
// 16 velocities v of f[pl][q][v] (w psi_m)(v), a 16 x 16 by 16 x 5 contraction on the matrix cores (wave_moments_4x4, one 16-row tile per
// plane). Every lane stages its plane's values, the first lane of each
// velocity group stages w psi of that velocity; the four waves' results are
// added in a fixed order. `stage` is mfma3_lds_bytes<ST>() bytes, `red`
// 4 x NS x 5 doubles.
template <typename ST>
constexpr int mfma3_lds_bytes() {
  constexpr int G = Plane3::G, K = 64 / G, RS = K + 2;
  return (kBlock / 64) * (K * 5 * (int)sizeof(double) + G * 16 * RS * (int)sizeof(ST));
}

template <typename ST, typename CT>
__device__ __forceinline__ void plane_partials_mfma(const CT (&fv)[Plane3::P2], const Vel& vel,
                                                    double* __restrict__ partials, int64_t node0,
                                                    int64_t nx, int chunk, int lp,
                                                    unsigned char* stage, double* red,
                                                    const int tid) {
  using PL = Plane3;
  constexpr int N1 = PL::N1, G = PL::G, P2 = PL::P2, NS = PL::NS;
  constexpr int K = 64 / G, RS = K + 2;
  static_assert(P2 == 16, "the nodes of a plane fill one 16-row tile");
  const int lane = tid & 63, wave = tid >> 6;
  const int vw = lane / G;  // velocity of this lane inside the wave
  double* ps = reinterpret_cast<double*>(stage) + wave * K * 5;
  ST* gw = reinterpret_cast<ST*>(stage + (kBlock / 64) * K * 5 * sizeof(double)) +
           wave * G * 16 * RS;
#pragma unroll
  for (int q = 0; q < P2; ++q) gw[(lp * 16 + q) * RS + vw] = (ST)fv[q];
  if (lp == 0) {
    const double psi4 = 0.5 * (vel.u[0] * vel.u[0] + vel.u[1] * vel.u[1] + vel.u[2] * vel.u[2]);
    ps[vw * 5 + 0] = vel.w;
    ps[vw * 5 + 1] = vel.w * vel.u[0];
    ps[vw * 5 + 2] = vel.w * vel.u[1];
    ps[vw * 5 + 3] = vel.w * vel.u[2];
    ps[vw * 5 + 4] = vel.w * psi4;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
  wave_moments_4x4<N1, P2, K, ST>(gw, RS, ps, red + wave * NS * 5, tid);
  lds_barrier();
  for (int t = tid; t < NS * 5; t += kBlock) {
    const int node = t / 5, m = t - node * 5;
    double sum = red[node * 5 + m];
#pragma unroll
    for (int w = 1; w < kBlock / 64; ++w) sum += red[(w * NS + node) * 5 + m];
    partials[((int64_t)chunk * nx + node0 + node) * 5 + m] = sum;
  }
}


// One work item (element e x velocity chunk) of the residual L(f) in FP64, of
// the internal state or a canonical array (see Source; the
// RK stages of these elements are k_stage_walk's, bgk_hexwalk.hpp).
template <typename ST, bool CAN>
__device__ __forceinline__ void residual3_item(const StageArgs& A, const int chunk, const int64_t e,
                                               const bool count) {
  using CT = typename Compute<ST>::T;
  using Src = Source<CAN, ST>;
  using FT = typename Src::T;
  using PL = Plane3;
  constexpr bool kMfma = sizeof(CT) == 4;
  constexpr int N1 = PL::N1, G = PL::G, VB = PL::VB, P2 = PL::P2, NS = PL::NS;
  __shared__ FaceRows<CT> frows[kBlock / 64];
  __shared__ LineOps lops[kMfma ? kBlock / 64 : 1];
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  double* tab = reinterpret_cast<double*>(dyn_lds);

  const int tid = (int)threadIdx.x;
  const DevGeom& g = A.g;
  const DevOpsT<CT>& OP = ops_of<CT>(A);
  FaceRows<CT>& fr = frows[tid >> 6];
  face_rows_store<CT, N1, true>(fr, OP, tid);
  LineOps& lo = lops[kMfma ? tid >> 6 : 0];
  if constexpr (kMfma) line_ops_store(lo, A.lops, tid);
  const int64_t nv = g.nv;
  const int S = g.tabw;
  const int64_t node0 = e * NS;

  const int lp = tid % G;  // plane owned by this lane
  const int j = chunk * VB + tid / G;
  const bool act = j < nv;
  const int jj = j < nv ? j : (int)nv - 1;
  const Vel vel = velocity_of(g, jj);

  int ek[3];
  {
    int64_t r = e;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      ek[k] = (int)(r % g.nelem[k]);
      r /= g.nelem[k];
    }
  }
  const int64_t nst = Src::stride(g);
  const FT* __restrict__ fin = (const FT*)A.fin;
  const FT* src[3];
  bool pos[3], use_right[3], wall_in[3][2];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    pos[k] = vel.u[k] * g.scale[k] > 0.0;
    const int nek = sreg(g.nelem[k]);
    const bool wall_lo = sreg(g.bc[k][0]) != 0, wall_hi = sreg(g.bc[k][1]) != 0;
    wall_in[k][1] = ek[k] == 0 && wall_lo;
    wall_in[k][0] = ek[k] == nek - 1 && wall_hi;
    int nk = ek[k] + (pos[k] ? -1 : 1);
    bool wall = false;
    if (nk < 0 || nk >= nek) {
      wall = pos[k] ? wall_lo : wall_hi;
      nk = (nk + nek) % nek;
    }
    int64_t src_e = e;
    int src_j = jj;
    if (wall) {
      int bm[3] = {vel.b[0], vel.b[1], vel.b[2]};
      bm[k] = g.nv1[k] - 1 - bm[k];
      src_j = vel_slot(g, bm);
    } else {
      int64_t stride = 1;
      for (int m = 0; m < k; ++m) stride *= g.nelem[m];
      src_e = e + (int64_t)(nk - ek[k]) * stride;
    }
    use_right[k] = (pos[k] != wall);
    src[k] = fin + Src::offset(g, src_e, lp * P2, src_j);
  }

  // first batch of row loads: 4 x 256 entries for FP32 arithmetic, whose
  // registers are scarcer, 6 x 256 in FP64 (a 64-velocity chunk of the 16^3
  // grid at p = 3 needs 64 x 18 or more)
  constexpr int kU = kMfma ? 4 : 6;
  const RowPick rp = CAN ? row_pick_lexicographic(A, chunk, VB, NS) : row_pick(A, chunk, NS);
  const double* et = A.etab + node0 * S;
  double tv[kU];
  if (A.collide) {
#pragma unroll
    for (int u = 0; u < kU; ++u) {  // clamped, unconditional loads
      const int t = u * kBlock + tid;
      tv[u] = et[rp.offset(t < rp.count ? t : rp.count - 1)];
    }
  }
  const FT* fe = fin + Src::offset(g, e, lp * P2, jj);
  CT f[P2], nb[P2];
#pragma unroll
  for (int q = 0; q < P2; ++q) f[q] = (CT)(ST)fe[q * nst];
#pragma unroll
  for (int q = 0; q < P2; ++q) nb[q] = (CT)(ST)src[0][q * nst];
  if (A.collide) {
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int t = u * kBlock + tid;
      if (t < rp.count) tab[t] = tv[u];
    }
  }

  CT acc[P2];
#pragma unroll
  for (int q = 0; q < P2; ++q) acc[q] = (CT)0;

  // x and y: lines inside the plane, lane-local (FP32 arithmetic on the matrix
  // cores, see line_mfma: a block of four lanes is one velocity's planes). The
  // neighbours' planes are loaded one
  // axis at a time, behind a scheduling barrier.
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    if (k > 0) {
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < P2; ++q) nb[q] = (CT)(ST)src[k][q * nst];
    }
    const int S1 = k == 0 ? 1 : N1;
    const CT a = (CT)(vel.u[k] * g.scale[k]);
    if constexpr (kMfma) {
      const bool uni = quads_agree(pos[k]);
      const int npass = uni ? 1 : 2;
      for (int ps = 0; ps < npass; ++ps) {
        const int sg = uni ? (pos[k] ? 1 : 0) : ps;
        const int ur = sg ? (wall_in[k][1] ? 0 : 1) : (wall_in[k][0] ? 1 : 0);
        float dp[4], ev[4];
        line_ops_row(lo, sg, ur, tid, dp, ev);
        const CT as = (uni || (pos[k] ? 1 : 0) == sg) ? a : (CT)0;
#pragma unroll
        for (int base = 0; base < P2; ++base) {
          if ((base / S1) % N1 != 0) continue;
          float fl[N1], nl[N1];
#pragma unroll
          for (int bb = 0; bb < N1; ++bb) {
            fl[bb] = f[base + bb * S1];
            nl[bb] = nb[base + bb * S1];
          }
          const mfma_f4 c = line_mfma<N1>(dp, ev, fl, nl);
#pragma unroll
          for (int ia = 0; ia < N1; ++ia) acc[base + ia * S1] = fmaf(as, c[ia], acc[base + ia * S1]);
        }
      }
      continue;
    }
    CT lown[N1], lext[N1], Gin[N1];
    {
      const CT* ro = fr.r[pos[k] ? 1 : 0];
      const CT* re = fr.r[use_right[k] ? 0 : 1];
#pragma unroll
      for (int bb = 0; bb < N1; ++bb) {
        lown[bb] = ro[bb];
        Gin[bb] = ro[kMaxN1 + bb];
        lext[bb] = re[bb];
      }
    }
#pragma unroll
    for (int base = 0; base < P2; ++base) {
      if ((base / S1) % N1 != 0) continue;
      CT line[N1];
#pragma unroll
      for (int bb = 0; bb < N1; ++bb) line[bb] = f[base + bb * S1];
      CT own = (CT)0, ext = (CT)0;
#pragma unroll
      for (int bb = 0; bb < N1; ++bb) {
        own += lown[bb] * line[bb];
        ext += lext[bb] * nb[base + bb * S1];
      }
      const CT jump = a * (ext - own);
#pragma unroll
      for (int ia = 0; ia < N1; ++ia) {
        CT df = (CT)0;
#pragma unroll
        for (int bb = 0; bb < N1; ++bb) df += sreg(OP.D[ia][bb]) * line[bb];
        acc[base + ia * S1] += a * df + jump * Gin[ia];
      }
    }
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int q = 0; q < P2; ++q) nb[q] = (CT)(ST)src[2][q * nst];
  // z: the column of node q is spread over the quad's lanes; lane lp holds
  // plane lp and its partners lane ^ r the other planes. The derivative is
  // sum_r D[lp][lp ^ r] f(lp ^ r); the trace difference ext - own is one
  // quad sum of lext(lp) f_nb - lown(lp) f.
  {
    const CT a = (CT)(vel.u[2] * g.scale[2]);
    const CT* ro = fr.r[pos[2] ? 1 : 0];
    const CT* re = fr.r[use_right[2] ? 0 : 1];
    const CT lown_mine = ro[lp], lext_mine = re[lp];
    const CT ag = a * ro[kMaxN1 + lp];
    CT Dr[G];
#pragma unroll
    for (int r = 0; r < G; ++r) Dr[r] = fr.D[lp * kMaxN1 + (lp ^ r)];
#pragma unroll
    for (int q = 0; q < P2; ++q) {
      const CT fq = f[q];
      CT df = Dr[0] * fq;
      df += Dr[1] * quad_xor<1>(fq);
      df += Dr[2] * quad_xor<2>(fq);
      df += Dr[3] * quad_xor<3>(fq);
      const CT jl = quad_allsum(lext_mine * nb[q] - lown_mine * fq);
      acc[q] += a * df + ag * jl;
    }
  }

  // collision term in FP64 from the rows in LDS; the residual C - T goes to
  // the canonical layout
  const int cx = vel.b[0] - rp.x0, oy = rp.nx + vel.b[1] - rp.y0,
            oz = rp.nxy + vel.b[2] - rp.z0;
  const double* tp = tab + lp * P2 * rp.ncols;  // rows of this lane's plane
  const int jc = vel.b[0] + g.nv1[0] * (vel.b[1] + g.nv1[1] * vel.b[2]);
  double* oe1 = (double*)A.out + ((e - A.out_e0) * NS + lp * P2) * nv + jc;
  const bool whole = whole_sectors(g);  // (a wave stores 16 velocities of a node)
  if (A.collide) {  // uniform: rows beyond the first batch, then the relaxation
    table_rest<kU>(tab, et, rp, tid);
    lds_barrier();
#pragma unroll
    for (int q = 0; q < P2; ++q) {
      const double c = collision_term(tp + q * rp.ncols, cx, oy, oz, rp.ncols, (double)f[q]);
      if (act) residual_store(whole, &oe1[(int64_t)q * nv], c - (double)acc[q]);
    }
  } else {
#pragma unroll
    for (int q = 0; q < P2; ++q)
      if (act) residual_store(whole, &oe1[(int64_t)q * nv], -(double)acc[q]);
  }
  if (tid == 0 && count) atomicAdd(&A.diag[4], 1ull);
}

// Three waves per SIMD in FP64, four in FP32 arithmetic (the neighbours'
// planes loaded one axis at a time).
template <typename ST, bool CAN>
__global__ void __launch_bounds__(kBlock)
    __attribute__((amdgpu_waves_per_eu(sizeof(ST) == 8 ? 3 : 4))) k_residual3(const StageArgs A) {
  const int64_t w = xcd_chunk_remap(blockIdx.x, gridDim.x, A.ecount, A.xcd_part);
  residual3_item<ST, CAN>(A, (int)(w / A.ecount), work_element(A.order, A.e0, w, A.ecount), w == 0);
}

template <typename ST, bool CAN>
__global__ void __launch_bounds__(kBlock) k_moments3(const StageArgs A) {
  using CT = typename Compute<ST>::T;
  using Src = Source<CAN, ST>;
  using PL = Plane3;
  constexpr int G = PL::G, VB = PL::VB, P2 = PL::P2, NS = PL::NS;
  __shared__ double red[(kBlock / 64) * NS * 5];
  extern __shared__ __align__(16) unsigned char dyn_lds[];  // MFMA staging
  const DevGeom& g = A.g;
  const int64_t w = xcd_remap(blockIdx.x, gridDim.x);
  const int chunk = (int)(w / A.ecount);
  const int64_t e = work_element(A.order, A.e0, w, A.ecount);
  const int64_t nv = g.nv;
  const int lp = (int)threadIdx.x % G;
  const int j = chunk * VB + (int)threadIdx.x / G;
  const bool valid = j < nv;
  const int jj = valid ? j : (int)nv - 1;
  Vel vel = velocity_of(g, jj);
  if (!valid) vel.w = 0.0;
  const typename Src::T* fe = (const typename Src::T*)A.fin + Src::offset(g, e, lp * P2, jj);
  const int64_t nst = Src::stride(g);
  CT f[P2];
#pragma unroll
  for (int q = 0; q < P2; ++q) f[q] = (CT)(ST)fe[q * nst];
  plane_partials_mfma<ST, CT>(f, vel, A.partials, e * NS, g.nx, chunk, lp, dyn_lds, red,
                                 (int)threadIdx.x);
}

}  // namespace bgk
