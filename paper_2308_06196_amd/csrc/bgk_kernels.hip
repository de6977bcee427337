// bgk_kernels.hip -- kernel instantiations and launchers (gfx950).
//
// Kernels: the fused stage (transport + relaxation + RK + limiter + moment
// partials), the residual, stand-alone moment partials, the per-node Newton
// solve for the discretely conservative equilibrium, and state conversion /
// Maxwellian initialisation. All launched on the caller's stream.
#include <cmath>
#include <cstdlib>

#include "bgk_device.hpp"
#include "bgk_device3d.hpp"
#include "bgk_launch.hpp"

namespace bgk {

// ---------------------------------------------------------------------------
// Discretely conservative equilibrium, one thread per spatial node
// (Sec. 2.1: Maxwellian on a perturbed state whose discrete moments equal
// those of f; Newton's method with the closed-form Jacobian).
//
// g_j = exp(alpha . psi_j) and the trapezoid weights are products over the
// three velocity components, so every sum over the N_v nodes factorises into
// one-dimensional sums S_c^n = sum_b w_c[b] E_c[b] u_b^n (n = 0..4) with
// E_c[b] = exp(alpha_{1+c} u_b + alpha_4 u_b^2 / 2): O(3 N_1d) work per node.
//
// The same product form makes the Newton system an arrow: with m_c^n = S_c^n /
// S_c^0 and A = exp(alpha_0) S_x^0 S_y^0 S_z^0, the Jacobian is A times the
// second moments of psi under g; less the mass row, it is their covariance,
// in which the velocity components are independent. With f = F / A, M = sum_c
// m_c^2 / 2, variances s_c = m_c^2 - (m_c^1)^2, covariances c_c = (m_c^3 - m_c^1
// m_c^2) / 2 with the energy, V = sum_c (m_c^4 - (m_c^2)^2) / 4, and the reduced
// right-hand sides r_c = f_c - m_c^1 f_0, r_4 = f_4 - M f_0:
//   d_4 = (r_4 - sum_c c_c r_c / s_c) / (V - sum_c c_c^2 / s_c),
//   d_c = (r_c - c_c d_4) / s_c,   d_0 = f_0 - sum_c m_c^1 d_c - M d_4.
// (An indefinite pivot marks the node failed.) The solve is bound by its chain
// of dependent FP64 operations on small meshes and by FP64 issue on large ones;
// a 5 x 5 Cholesky factorisation in its place, with five square roots and five
// more divisions in the chain, took 1.6 us longer a launch on 96 nodes (13.1
// against 11.5) and 8.5 on 216,000 (167.6 against 159.0).
// ---------------------------------------------------------------------------
// All-reduce of one FP64 value over the T lanes of a team (T = 16: one DPP
// row, partners lane ^ 8, the mirror inside 8 lanes, lane ^ 2, lane ^ 1;
// T = 4: one quad; T = 2: a lane pair). Each step
// pairs lanes symmetrically, so every lane ends with the same bits.
template <int T>
__device__ __forceinline__ double team_sum(double x) {
  if constexpr (T == 16) x += dpp_partner<8>(x);
  if constexpr (T == 16) x += dpp_partner<4>(x);
  if constexpr (T >= 4) x += dpp_partner<2>(x);
  x += dpp_partner<1>(x);
  return x;
}

// One team of kTeam lanes per spatial node. The lanes split the velocity
// chunks of the moment partials and the nodes of each one-dimensional sum;
// the 5x5 solve is repeated identically in every lane of the team. Large
// meshes use 2- or 4-lane teams (less redundant solve work), small ones
// 16-lane teams (enough waves to fill the device). The one-dimensional sums run
// over the three axes together, up to the longest one; with SPLIT up to the
// shortest one, and each axis' rest alone (newton_split says where).
template <int kTeam, bool SPLIT>
__device__ __forceinline__ void newton_item(const NewtonArgs& A, const int64_t node_raw) {
  const DevGeom& g = A.g;
  const int r = threadIdx.x % kTeam;
  // teams past the last node work on the last node and store nothing, so that
  // every lane reaches the wave-level counter reduction at the end
  const bool active = node_raw < g.nx;
  const int64_t node = active ? node_raw : g.nx - 1;
  const unsigned long long seen =
      __hip_atomic_load(&A.diag[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  double Q[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  const double* pp = A.partials + node * 5;  // chunk c at pp[c * nx * 5]
  constexpr int kH = kTeam >= 16 ? 1 : 2;
  constexpr int kStep = kH * kTeam;
  const int njoint = SPLIT ? (min(g.nv1[0], min(g.nv1[1], g.nv1[2])) + kStep - 1) / kStep * kStep
                           : max(g.nv1[0], max(g.nv1[1], g.nv1[2]));
  // chunk partials: batches of kPB chunks per lane, all loads of a batch in
  // flight (chunks past the last read that one again, with weight 0: a
  // conditional load becomes a branch of its own)
  constexpr int kPB = kTeam >= 16 ? 2 : 8;
  const int64_t pstride = g.nx * 5;
  for (int c0 = r; c0 < g.nchunk; c0 += kPB * kTeam) {
    double v[kPB][5];
#pragma unroll
    for (int u = 0; u < kPB; ++u) {
      const double* p = pp + (int64_t)min(c0 + u * kTeam, g.nchunk - 1) * pstride;
#pragma unroll
      for (int m = 0; m < 5; ++m) v[u][m] = p[m];
    }
#pragma unroll
    for (int u = 0; u < kPB; ++u)
#pragma unroll
      for (int m = 0; m < 5; ++m) Q[m] += c0 + u * kTeam < g.nchunk ? v[u][m] : 0.0;
  }
#pragma unroll
  for (int m = 0; m < 5; ++m) Q[m] = team_sum<kTeam>(Q[m]);
  if (A.Q && r == 0 && active) {
#pragma unroll
    for (int m = 0; m < 5; ++m) A.Q[node * 5 + m] = Q[m];
  }
  double* out = A.params + node * 8;
  if (!A.collide) {  // uniform over the grid
    if (r == 0 && active) {
#pragma unroll
      for (int m = 0; m < 8; ++m) out[m] = 0.0;
    }
    return;
  }
  const double rho = Q[0];
  const double UU = (Q[1] * Q[1] + Q[2] * Q[2] + Q[3] * Q[3]) / (rho * rho);
  const double P = (A.gamma - 1.0) * (Q[4] - 0.5 * rho * UU);
  const double th = P / rho;
  int status = 0, iters = 0;
  double al[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  if (!(rho > 0.0) || !(th > 0.0)) {
    status = 2;
  } else {
    const double tpt = 2.0 * M_PI * th;
    al[0] = log(rho / (tpt * sqrt(tpt))) - UU / (2.0 * th);
    al[1] = Q[1] / rho / th;
    al[2] = Q[2] / rho / th;
    al[3] = Q[3] / rho / th;
    al[4] = -1.0 / th;
    const double sq = rho * sqrt(th);
    const double isq = 1.0 / sq;
    const double isc[5] = {1.0 / rho, isq, isq, isq, 1.0 / Q[4]};
    // the non-conservative model keeps the continuous Maxwellian (no solve)
    for (int it = 0; !A.continuous; ++it) {
      // the three components together (and two nodes each where a lane has
      // several): independent exponentials, whose latency bounds the sums
      double S[3][5];
#pragma unroll
      for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int n = 0; n < 5; ++n) S[c][n] = 0.0;
      for (int b0 = r; b0 < njoint; b0 += kH * kTeam) {
#pragma unroll
        for (int h = 0; h < kH; ++h) {
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            const int b = b0 + h * kTeam, N = g.nv1[c], bb = b < N ? b : N - 1;
            const double u = g.vlo[c] + bb * g.du[c], u2 = u * u;
            const double wc = b >= N ? 0.0 : g.du[c] * (bb == 0 || bb == N - 1 ? 0.5 : 1.0);
            const double t = wc * exp(al[1 + c] * u + al[4] * (0.5 * u2));
            S[c][0] += t;
            S[c][1] += t * u;
            S[c][2] += t * u2;
            S[c][3] += t * u2 * u;
            S[c][4] += t * u2 * u2;
          }
        }
      }
      if constexpr (SPLIT) {  // what is left of the longer axes
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          for (int b = njoint + r; b < g.nv1[c]; b += kTeam) {
            const double u = g.vlo[c] + b * g.du[c], u2 = u * u;
            const double wc = g.du[c] * (b == g.nv1[c] - 1 ? 0.5 : 1.0);
            const double t = wc * exp(al[1 + c] * u + al[4] * (0.5 * u2));
            S[c][0] += t;
            S[c][1] += t * u;
            S[c][2] += t * u2;
            S[c][3] += t * u2 * u;
            S[c][4] += t * u2 * u2;
          }
        }
      }
#pragma unroll
      for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int n = 0; n < 5; ++n) S[c][n] = team_sum<kTeam>(S[c][n]);
      double m[3][5];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const double inv = 1.0 / S[c][0];
        m[c][0] = 1.0;
#pragma unroll
        for (int n = 1; n < 5; ++n) m[c][n] = S[c][n] * inv;
      }
      const double A0 = exp(al[0]) * S[0][0] * S[1][0] * S[2][0];
      const double M = 0.5 * (m[0][2] + m[1][2] + m[2][2]);
      const double G[5] = {A0, A0 * m[0][1], A0 * m[1][1], A0 * m[2][1], A0 * M};
      double F[5], res = 0.0;
#pragma unroll
      for (int a = 0; a < 5; ++a) {
        F[a] = G[a] - Q[a];
        const double ra = fabs(F[a]) * isc[a];
        if (!(ra <= res)) res = ra;
      }
      iters = it + 1;
      const bool conv = res <= A.tol;
      if (!conv && it >= A.maxit) {
        status = 1;
        break;
      }
      const double iA = 1.0 / A0;
      double f[5];
#pragma unroll
      for (int a = 0; a < 5; ++a) f[a] = F[a] * iA;
      double d[5], is[3], cv[3], r[3];
      double r4 = f[4] - M * f[0], V = 0.0;
      bool spd = A0 > 0.0;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const double var = m[c][2] - m[c][1] * m[c][1];
        spd = spd && var > 0.0;
        is[c] = 1.0 / var;
        cv[c] = 0.5 * (m[c][3] - m[c][1] * m[c][2]);
        r[c] = f[1 + c] - m[c][1] * f[0];
        V += 0.25 * (m[c][4] - m[c][2] * m[c][2]) - cv[c] * cv[c] * is[c];
        r4 -= cv[c] * r[c] * is[c];
      }
      // (an energy pivot of rounding size: the energy moment is a multiple of
      // the mass, as with two velocity nodes per component)
      const double e4 = 0.25 * (m[0][4] + m[1][4] + m[2][4]);
      if (!(spd && V > 64.0 * 0x1p-53 * e4)) {
        status = 2;
        break;
      }
      d[4] = r4 / V;
      d[0] = f[0] - M * d[4];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        d[1 + c] = (r[c] - cv[c] * d[4]) * is[c];
        d[0] -= m[c][1] * d[1 + c];
      }
      double an[5];
#pragma unroll
      for (int a = 0; a < 5; ++a) an[a] = al[a] - d[a];
      for (int h = 0; h < 60 && !(an[4] < 0.0); ++h) {
#pragma unroll
        for (int a = 0; a < 5; ++a) {
          d[a] *= 0.5;
          an[a] = al[a] - d[a];
        }
      }
      if (!(an[4] < 0.0)) {
        status = 2;
        break;
      }
#pragma unroll
      for (int a = 0; a < 5; ++a) al[a] = an[a];
      if (conv) break;  // that was the polishing step
    }
  }
  if (status) {
#pragma unroll
    for (int a = 0; a < 5; ++a) al[a] = __builtin_nan("");
  }
  // relaxation time tau = mu / P (Sec. 2) with mu from the temperature law
  const double tr = th / A.theta_ref;
  const double mu = A.sutherland > 0.0
                        ? A.mu_ref * tr * sqrt(tr) * (A.theta_ref + A.sutherland) / (th + A.sutherland)
                        : A.omega != 0.0 ? A.mu_ref * pow(tr, A.omega)
                                         : A.mu_ref;
  const double itau = P / mu;  // 1 / tau
  // one-dimensional factors of the equilibrium in FP64 for every storage
  // precision: exp(alpha_0) and 1/tau folded into x, so that the stage kernels
  // form the collision term as Ex[bx] Ey[by] Ez[bz] - f / tau
  double* row = (double*)A.etab + node * g.tabw;
  const int off1 = g.nv1[0], off2 = off1 + g.nv1[1], off = off2 + g.nv1[2];
  for (int b0 = r; b0 < njoint; b0 += kH * kTeam) {
#pragma unroll
    for (int h = 0; h < kH; ++h) {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const int b = b0 + h * kTeam;
        const double u = g.vlo[c] + b * g.du[c];
        const double v = exp((c == 0 ? al[0] : 0.0) + al[1 + c] * u + al[4] * (0.5 * u * u));
        if (active && b < g.nv1[c]) row[(c == 0 ? 0 : c == 1 ? off1 : off2) + b] = c == 0 ? v * itau : v;
      }
    }
  }
  if constexpr (SPLIT) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      for (int b = njoint + r; b < g.nv1[c]; b += kTeam) {
        const double u = g.vlo[c] + b * g.du[c];
        const double v = exp((c == 0 ? al[0] : 0.0) + al[1 + c] * u + al[4] * (0.5 * u * u));
        if (active) row[(c == 0 ? 0 : c == 1 ? off1 : off2) + b] = c == 0 ? v * itau : v;
      }
    }
  }
  if (r == 0 && active) {
#pragma unroll
    for (int a = 0; a < 5; ++a) out[a] = al[a];
    out[5] = itau;
    out[6] = 1.0 / itau;
    out[7] = (double)status;
    row[off] = itau;  // 1/tau closes the node's row
  }
  // counters: at most one atomic per wave (its teams reduced first). The most
  // iterations rise only in the first launches after a state is installed:
  // waves that do not exceed the value seen at the start leave it alone. (One
  // atomic per wave on one address cost more than the solve: 16,384 nodes with
  // 4, 8, 16 lanes each 34.7, 41.6, 63.3 us, without them 25.6, 28.0, 34.5.)
  int itw = active ? iters : 0;
  for (int o = kTeam; o < 64; o <<= 1) itw = max(itw, __shfl_xor(itw, o, 64));
  const unsigned long long nfail = __popcll(__ballot(active && r == 0 && status != 0));
  if ((threadIdx.x & 63) == 0) {
    if ((unsigned long long)itw > seen) atomicMax(&A.diag[0], (unsigned long long)itw);
    if (nfail) atomicAdd(&A.diag[1], nfail);
  }
}

template <int kTeam, bool SPLIT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4)))
    k_newton(const NewtonArgs A) {
  newton_item<kTeam, SPLIT>(A, ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kTeam);
}

// Equilibrium solves of the batch members of one team size: whole work-groups
// of 256 lanes per member, so that a work-group's arguments are uniform; the
// grid is the list's work-group count.
template <int kTeam, bool SPLIT>
__global__ void __launch_bounds__(256) k_newton_batch(table_ptr<NewtonArgs> args,
                                                      table_ptr<BatchList> list) {
  const int32_t t = blockIdx.x;
  const int m = batch_member(list->newton_off, list->n, t);
  newton_item<kTeam, SPLIT>(table_entry(args, list->slot[m]),
                     ((int64_t)(t - list->newton_off[m]) * 256 + threadIdx.x) / kTeam);
}

// Q[node][5] from the partials (no Newton solve).
__global__ void __launch_bounds__(256) k_reduce_partials(const DevGeom g, const double* partials,
                                                         double* Q) {
  const int64_t node = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (node >= g.nx) return;
  double q[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  const double* pp = partials + node * 5;
  for (int c = 0; c < g.nchunk; ++c)
#pragma unroll
    for (int m = 0; m < 5; ++m) q[m] += pp[(int64_t)c * g.nx * 5 + m];
#pragma unroll
  for (int m = 0; m < 5; ++m) Q[node * 5 + m] = q[m];
}

// Discrete moments of the collision term of a stored state, per node and
// chunk of kBlock velocities: sum_j w_j psi_j C_j with C_j formed by
// collision_term from the FP64 equilibrium rows and the stored values, as in
// the stage kernels. One work-group = one element x one chunk; lanes are
// summed by an xor butterfly and the four waves in a fixed order.
template <typename ST>
__global__ void __launch_bounds__(kBlock) k_collision_moments(const StageArgs A, int nchunk) {
  __shared__ double red[kBlock / 64][5];
  const DevGeom& g = A.g;
  const int64_t e = (int64_t)blockIdx.x / nchunk;
  const int chunk = (int)(blockIdx.x % nchunk);
  const int j = chunk * kBlock + (int)threadIdx.x;
  const bool valid = j < g.nv;
  const int jj = valid ? j : (int)g.nv - 1;
  const Vel vel = velocity_of(g, jj);
  const double wt = valid ? vel.w : 0.0;
  const double psi4 = 0.5 * (vel.u[0] * vel.u[0] + vel.u[1] * vel.u[1] + vel.u[2] * vel.u[2]);
  const int S = g.tabw;
  const int oy = g.nv1[0] + vel.b[1], oz = g.nv1[0] + g.nv1[1] + vel.b[2];
  const ST* fin = (const ST*)A.fin;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int i = 0; i < g.ns; ++i) {
    const int64_t node = e * g.ns + i;
    const double fv = (double)fin[f_offset(g, e, i, jj)];
    const double c = wt * collision_term(A.etab + node * S, vel.b[0], oy, oz, S, fv);
    double m[5] = {c, c * vel.u[0], c * vel.u[1], c * vel.u[2], c * psi4};
#pragma unroll
    for (int q = 0; q < 5; ++q)
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) m[q] += __shfl_xor(m[q], o, 64);
    if (lane == 0) {
#pragma unroll
      for (int q = 0; q < 5; ++q) red[wave][q] = m[q];
    }
    __syncthreads();
    if (threadIdx.x < 5) {
      double sum = 0.0;
#pragma unroll
      for (int w = 0; w < kBlock / 64; ++w) sum += red[w][threadIdx.x];
      A.partials[((int64_t)chunk * g.nx + node) * 5 + threadIdx.x] = sum;
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Diffuse walls. At a flux point of a wall face the gas leaving the domain
// carries the discrete mass flux sum_{outgoing j} w_j |u_k| f_trace; the wall
// re-emits rho_w times the unit wall Maxwellian into the incoming velocities,
// with rho_w = that flux / (incoming flux of the unit wall Maxwellian), so the
// net mass flux through the wall vanishes.
// ---------------------------------------------------------------------------

// Side of a wall work-group or flux point i: the last one that starts at or
// before i, with its entries. All entries are read at once and selected: a loop
// over the sides and indexed entries are a chain of scalar loads from the
// argument memory, which is cold when a kernel starts.
struct WallSide {
  int k, side, off, blk0;
};
template <typename START>
__device__ __forceinline__ WallSide wall_side(const WallArgs& W, const START& start, const int i) {
  WallSide s[4];
  int st[4], n = W.nside;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    s[q] = WallSide{W.side_k[q], W.side_s[q], W.off[q], W.blk0[q]};
    st[q] = start[q];
  }
  // (the values, not the loads, are selected)
#pragma unroll
  for (int q = 0; q < 4; ++q)
    asm volatile("" : "+s"(s[q].k), "+s"(s[q].side), "+s"(s[q].off), "+s"(s[q].blk0), "+s"(st[q]));
  WallSide r = s[0];
#pragma unroll
  for (int q = 1; q < 4; ++q)
    if (q < n && i >= st[q]) r = s[q];
  return r;
}

// One work-group = one wall-face element x one chunk of 256 velocities; the
// flux points' partial sums are reduced in a fixed order (lanes by an xor
// butterfly, then the four waves in LDS). Few work-groups with little work
// each: bound by the chain of latencies in one of them (24 x 40 p = 2 channel on
// 16^3 velocities, 768 work-groups: 19.3 us with eleven dependent scalar loads
// and one vector load before the nodes', 5.4 with three). Waves without an
// outgoing velocity load no nodes.
template <int DIM, int P, typename ST, bool CAN = false>
__device__ __forceinline__ void wall_flux_item(const WallArgs& W, const int b) {
  using Src = Source<CAN, ST>;
  constexpr int N1 = P + 1;
  constexpr int NF = ipow(N1, DIM - 1);
  __shared__ double red[kBlock / 64][NF];
  const DevGeom& g = W.g;
  const WallSide q = wall_side(W, W.blk0, b);
  const bool along_y = DIM == 2 && q.k == 1;
  const int local = b - q.blk0;
  const int face = local / g.nchunk, chunk = local % g.nchunk;
  // element: coordinate k on the wall, the other coordinate (2-D) = face
  const int nx = g.nelem[0], ny = g.nelem[1];
  const int last = (along_y ? ny : nx) - 1, on = q.side == 0 ? 0 : last;
  const int64_t e = DIM == 1 ? on : along_y ? face + (int64_t)nx * on : on + (int64_t)nx * face;
  const int64_t nv = g.nv;
  const int j = chunk * kBlock + (int)threadIdx.x;
  const bool valid = j < nv;
  const int jj = valid ? j : (int)nv - 1;
  const Vel vel = velocity_of(g, jj);
  const double a = along_y ? vel.u[1] : vel.u[0];
  const bool outgoing = valid && (q.side == 0 ? a < 0.0 : a > 0.0);
  const double wt = outgoing ? vel.w * fabs(a) : 0.0;
  double v[NF];
#pragma unroll
  for (int fp = 0; fp < NF; ++fp) v[fp] = 0.0;
  if (__any(outgoing)) {
    const typename Src::T* fe = (const typename Src::T*)W.fin + Src::offset(g, e, 0, jj);
    // nodes of flux point fp's line: base(fp) + bb * along
    const int64_t nst = Src::stride(g), along = along_y ? N1 * nst : nst,
                  across = along_y ? nst : N1 * nst;
    double lam[N1];
#pragma unroll
    for (int bb = 0; bb < N1; ++bb) {
      const double l = W.lamL[bb], r = W.lamR[bb];
      lam[bb] = q.side == 0 ? l : r;
    }
#pragma unroll
    for (int fp = 0; fp < NF; ++fp) {
      double tr = 0.0;
#pragma unroll
      for (int bb = 0; bb < N1; ++bb)
        tr += lam[bb] * (double)(ST)fe[fp * across + bb * along];
      v[fp] = wt * tr;
    }
#pragma unroll
    for (int fp = 0; fp < NF; ++fp) {
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) v[fp] += __shfl_xor(v[fp], o, 64);
    }
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) {
#pragma unroll
    for (int fp = 0; fp < NF; ++fp) red[wave][fp] = v[fp];
  }
  __syncthreads();
  if ((int)threadIdx.x < NF) {
    double sum = 0.0;
#pragma unroll
    for (int w = 0; w < kBlock / 64; ++w) sum += red[w][threadIdx.x];
    W.part[((int64_t)q.off + face * NF + threadIdx.x) * g.nchunk + chunk] = sum;
  }
}

template <int DIM, int P, typename ST, bool CAN>
__global__ void __launch_bounds__(kBlock) k_wall_flux(const WallArgs W) {
  wall_flux_item<DIM, P, ST, CAN>(W, blockIdx.x);
}

template <int DIM, int P, typename ST>
__global__ void __launch_bounds__(kBlock) k_wall_flux_batch(table_ptr<WallArgs> args,
                                                            table_ptr<BatchList> list, int stage) {
  const int32_t t = blockIdx.x;  // grid: the list's wall-flux work-groups
  const int m = batch_member(list->wflux_off, list->n, t);
  wall_flux_item<DIM, P, ST>(table_entry(args, list->slot[m] * 3 + stage),
                             (int)(t - list->wflux_off[m]));
}

// rho_w per wall flux point: the chunk partials summed in order, times the
// inverse incoming flux of the side's unit wall Maxwellian.
__device__ __forceinline__ void wall_rho_item(const WallArgs& W, const int t) {
  if (t >= W.npoints) return;
  const WallSide q = wall_side(W, W.off, t);
  const int n = W.g.nchunk;
  const double inv = W.wallp[(q.k * 2 + q.side) * 8 + 5];
  const double* p = W.part + (int64_t)t * n;
  double sum = 0.0;
  // (batches of loads in flight; those past the last chunk read it again)
  constexpr int kB = 16;
  for (int c0 = 0; c0 < n; c0 += kB) {
    double v[kB];
#pragma unroll
    for (int u = 0; u < kB; ++u) v[u] = p[min(c0 + u, n - 1)];
#pragma unroll
    for (int u = 0; u < kB; ++u) sum += c0 + u < n ? v[u] : 0.0;
  }
  W.rho[t] = sum * inv;
}

__global__ void __launch_bounds__(256) k_wall_rho(const WallArgs W) {
  wall_rho_item(W, blockIdx.x * blockDim.x + threadIdx.x);
}

__global__ void __launch_bounds__(256) k_wall_rho_batch(table_ptr<WallArgs> args,
                                                        table_ptr<BatchList> list, int stage) {
  const int32_t t = blockIdx.x;  // grid: the list's wall-density work-groups
  const int m = batch_member(list->wrho_off, list->n, t);
  wall_rho_item(table_entry(args, list->slot[m] * 3 + stage),
                (int)((t - list->wrho_off[m]) * 256 + threadIdx.x));
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
static inline unsigned grid_of(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

// Hexahedra. The one-lane-per-velocity kernels (k_stage<3, ...>: all
// (p+1)^3 nodes of a velocity in one lane's registers) run FP32 storage at
// every order and FP64 storage and BF16 increments at p <= 2; the plane-split
// kernels (four lanes per velocity, one z-plane each: k_stage_walk, k_residual3,
// k_moments3) run FP64 storage and BF16 increments at p = 3, where one lane
// cannot hold the element (FP64) or the second value per neighbour node (BF16:
// 137 spilled registers, 7.72 ms per stage of the 16^3-element Taylor-Green
// box; k_stage_walk 3.5). At p <= 2 a per-element plane-split stage was slower
// there (ms, plane-split against one-lane): FP64 p = 1 1.18 / 0.82, p = 2 4.95 /
// 2.50 (two waves per SIMD; 6.22 at three, which spill); BF16 p = 1 0.90 /
// 0.51, p = 2 3.31 / 1.62; FP32 p = 3 5.49 / 3.61.
// The choice (hex_one_lane) is per solver, so that all its kernels share one
// velocity-chunk width; it must agree with kHexOneLane below.
template <int P, typename ST>
constexpr bool kHexOneLane(bool inc) {
  return sizeof(ST) == 8 ? P <= 2 : (P <= 2 || !inc);
}

// RK stages over the whole mesh run as column sweeps along the last axis
// (k_stage_sweep) when the solver chose a segment length and the mesh has no
// diffuse wall.
static bool use_sweep(int mode, const StageArgs& A) {
  if (mode != 0 || A.sweep_seg <= 0 || A.g.dim < 2) return false;
  if (A.e0 != 0 || A.ecount != A.g.ne || A.g.nelem[A.g.dim - 1] % A.sweep_seg != 0) return false;
  for (int k = 0; k < 2; ++k)
    if (A.wall_off[k][0] >= 0 || A.wall_off[k][1] >= 0) return false;
  return true;
}

static dim3 sweep_grid(const StageArgs& A) {
  return dim3((unsigned)(A.g.nchunk * (A.g.ne / A.sweep_seg)));
}

template <int D, int P, typename ST, bool kIncBuilt = true>
static void launch_sweep(bool inc, const StageArgs& A, size_t lds, hipStream_t s) {
  const dim3 grid = sweep_grid(A), block(kBlock);
  if constexpr (sizeof(ST) == 4 && kIncBuilt) {
    if (inc) {
      if (A.din)
        hipLaunchKernelGGL((k_stage_sweep<D, P, ST, 0, true>), grid, block, lds, s, A);
      else
        hipLaunchKernelGGL((k_stage_sweep<D, P, ST, 3, true>), grid, block, lds, s, A);
      return;
    }
  }
  if (A.a != 0.0)
    hipLaunchKernelGGL((k_stage_sweep<D, P, ST, 0>), grid, block, lds, s, A);
  else
    hipLaunchKernelGGL((k_stage_sweep<D, P, ST, 3>), grid, block, lds, s, A);
}

template <int P, typename ST>
static hipError_t hex_dispatch(int mode, bool inc, const StageArgs& A, size_t tab, size_t lds,
                               dim3 grid, dim3 block, hipStream_t s) {
  const bool sweep = use_sweep(mode, A);
  if (kHexOneLane<P, ST>(inc)) {
    if constexpr (sizeof(ST) == 8 && P > 2) return hipErrorInvalidValue;  // not built
    else {
      if (sweep) {
        launch_sweep<3, P, ST, (P <= 2)>(inc, A, lds, s);  // one-lane increments: p <= 2
      } else if (mode == 0 && inc) {
        if constexpr (sizeof(ST) == 4 && P <= 2) {
          if (A.din)
            hipLaunchKernelGGL((k_stage<3, P, ST, 0, true>), grid, block, lds, s, A);
          else
            hipLaunchKernelGGL((k_stage<3, P, ST, 3, true>), grid, block, lds, s, A);
        }
      } else if (mode == 0 && A.a != 0.0) {
        hipLaunchKernelGGL((k_stage<3, P, ST, 0>), grid, block, lds, s, A);
      } else if (mode == 0) {
        hipLaunchKernelGGL((k_stage<3, P, ST, 3>), grid, block, lds, s, A);
      } else if (mode == 1) {
        hipLaunchKernelGGL((k_stage<3, P, ST, 1>), grid, block, lds, s, A);
      } else if (mode == 2) {
        hipLaunchKernelGGL((k_moments<3, P, ST>), grid, block, lds, s, A);
      } else if constexpr (P == 3) {  // canonical source: not built (64 nodes spill)
        return hipErrorInvalidValue;
      } else if (mode == 3) {
        hipLaunchKernelGGL((k_residual<3, P, ST>), grid, block, lds, s, A);
      } else {
        hipLaunchKernelGGL((k_moments<3, P, ST, true>), grid, block, lds, s, A);
      }
      return hipGetLastError();
    }
  }
  if constexpr (P == 3) {  // plane-split: FP64 storage, BF16 increments
    if (mode == 0) return launch_walk(sizeof(ST) == 8 ? 0 : 2, A, s);
    if (mode == 1) {
      hipLaunchKernelGGL((k_residual3<ST, false>), grid, block, tab, s, A);
    } else if (mode == 3) {
      hipLaunchKernelGGL((k_residual3<ST, true>), grid, block, tab, s, A);
    } else {
      const size_t lds3 = std::max(tab, (size_t)mfma3_lds_bytes<ST>());
      if (mode == 2) hipLaunchKernelGGL((k_moments3<ST, false>), grid, block, lds3, s, A);
      else hipLaunchKernelGGL((k_moments3<ST, true>), grid, block, lds3, s, A);
    }
    return hipGetLastError();
  }
  return hipErrorInvalidValue;
}

template <typename ST>
static hipError_t stage_dispatch(int mode, bool inc, const StageArgs& A, hipStream_t s) {
  const dim3 grid((unsigned)(A.g.nchunk * A.ecount)), block(kBlock);
  const int key = A.g.dim * 10 + (A.g.n1 - 1);
  // dynamic LDS: equilibrium rows (relaxation), then, in the 1-D/2-D
  // kernels, the MFMA staging of the moment partials in the same bytes
  const size_t tab = A.collide ? (size_t)A.g.ns * A.g.tabw * sizeof(double) : 0;
  const size_t lds = mode != 1 && mode != 3 ? std::max(tab, (size_t)mfma_lds_bytes<ST>()) : tab;
#define BGK_CASE(D, P)                                                     \
  case D * 10 + P:                                                         \
    if (D >= 2 && use_sweep(mode, A)) {                                    \
      launch_sweep<(D >= 2 ? D : 2), P, ST>(inc, A, lds, s);               \
      break;                                                               \
    }                                                                      \
    if constexpr (sizeof(ST) == 4) {                                       \
      if (mode == 0 && inc) {                                              \
        if (A.din)                                                         \
          hipLaunchKernelGGL((k_stage<D, P, ST, 0, true>), grid, block, lds, s, A); \
        else                                                               \
          hipLaunchKernelGGL((k_stage<D, P, ST, 3, true>), grid, block, lds, s, A); \
        break;                                                             \
      }                                                                    \
    }                                                                      \
    if (mode == 0 && A.a != 0.0)                                           \
      hipLaunchKernelGGL((k_stage<D, P, ST, 0>), grid, block, lds, s, A);  \
    else if (mode == 0)                                                    \
      hipLaunchKernelGGL((k_stage<D, P, ST, 3>), grid, block, lds, s, A);  \
    else if (mode == 1)                                                    \
      hipLaunchKernelGGL((k_stage<D, P, ST, 1>), grid, block, lds, s, A);  \
    else if (mode == 2)                                                    \
      hipLaunchKernelGGL((k_moments<D, P, ST>), grid, block, lds, s, A);   \
    else if (mode == 3)                                                    \
      hipLaunchKernelGGL((k_residual<D, P, ST>), grid, block, lds, s, A);  \
    else                                                                   \
      hipLaunchKernelGGL((k_moments<D, P, ST, true>), grid, block, lds, s, A); \
    break;
#define BGK_CASE3(P)                                                       \
  case 30 + P:                                                             \
    return hex_dispatch<P, ST>(mode, inc, A, tab, lds, grid, block, s);
  switch (key) {
    BGK_CASE(1, 1) BGK_CASE(1, 2) BGK_CASE(1, 3)
    BGK_CASE(2, 1) BGK_CASE(2, 2) BGK_CASE(2, 3)
    BGK_CASE3(1) BGK_CASE3(2) BGK_CASE3(3)
    default:
      return hipErrorInvalidValue;
  }
#undef BGK_CASE
#undef BGK_CASE3
  return hipGetLastError();
}

// Work-groups of kernel k (256 lanes, lds bytes of dynamic LDS) that one CU
// holds at once.
template <typename K>
static int groups_per_cu(K k, size_t lds) {
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k, kBlock, lds) != hipSuccess) return 0;
  return n;
}

template <int D, int P, typename ST>
static int sweep_groups_per_cu(bool inc, size_t tab) {
  if constexpr (D == 3) {
    if (!kHexOneLane<P, ST>(inc)) return 0;  // k_stage_walk
    if constexpr (sizeof(ST) == 8 && P > 2) return 0;  // not built
  }
  const size_t lds = std::max(tab, (size_t)mfma_lds_bytes<ST>());
  if constexpr (sizeof(ST) == 4 && (D == 2 || P <= 2)) {
    if (inc) return groups_per_cu(k_stage_sweep<D, P, ST, 0, true>, lds);
  }
  if constexpr (sizeof(ST) == 8 && D == 3 && P > 2) return 0;
  else return groups_per_cu(k_stage_sweep<D, P, ST, 0>, lds);
}

template <typename ST>
static int sweep_groups(int dim, int order, bool inc, size_t tab) {
  switch (dim * 10 + order) {
    case 21: return sweep_groups_per_cu<2, 1, ST>(inc, tab);
    case 22: return sweep_groups_per_cu<2, 2, ST>(inc, tab);
    case 23: return sweep_groups_per_cu<2, 3, ST>(inc, tab);
    case 31: return sweep_groups_per_cu<3, 1, ST>(inc, tab);
    case 32: return sweep_groups_per_cu<3, 2, ST>(inc, tab);
    case 33: return sweep_groups_per_cu<3, 3, ST>(inc, tab);
    default: return 0;
  }
}

// Elements per column-sweep work item (0: no sweep). A work-group walks its
// segment one element after another, so long segments leave the last wave
// of work-groups part of the device idle; each segment's first element reads
// its upwind neighbour's nodes. The choice minimises (1 + 0.2 / seg) / eff,
// eff = R / ceil(R) for R = work items / work-groups resident on the device
// (from the kernel's occupancy), over the divisors seg >= 2 of the number of
// elements along the last axis; seg = 1 (no sweep) when that is cheaper.
// The environment variable BGK_SWEEP_SEG overrides the choice (0: no sweep;
// a length that does not divide the column length means no sweep).
// Sweeps are used where they measured faster than the per-element kernels
// (ms per stage launch, sweep / per element): quadrilaterals in FP64 (32^2
// box, p = 3: 1.021 / 1.039) and p = 3 hexahedra in FP32 (Taylor-Green box,
// one lane per velocity: 3.26 / 3.50; the sweep's last axis loads nothing,
// and without its loads the element fits the registers). Not for FP32 and
// BF16 quadrilaterals (0.626 / 0.588, the loop costs registers at five waves
// per SIMD) or p = 2 hexahedra (Mach-2 box at four waves per SIMD: spills).
// FP64 and BF16 increments at p = 3 walk tiles instead (k_stage_walk).
static bool sweep_pays(const DevGeom& g, int precision) {
  if (g.dim == 2) return precision == 0;
  return g.dim == 3 && g.n1 == 4 && precision == 1;
}

int sweep_segment(const DevGeom& g, int precision, bool collide) {
  if (g.dim < 2) return 0;
  const int nl = g.nelem[g.dim - 1];
  if (const char* env = getenv("BGK_SWEEP_SEG")) {
    const int v = atoi(env);
    return v >= 1 && nl % v == 0 ? v : 0;
  }
  if (!sweep_pays(g, precision)) return 0;
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return 0;
  const size_t tab = collide ? (size_t)g.ns * g.tabw * sizeof(double) : 0;
  const bool inc = precision == 2;
  const int per_cu = precision == 0 ? sweep_groups<double>(g.dim, g.n1 - 1, false, tab)
                                    : sweep_groups<float>(g.dim, g.n1 - 1, inc, tab);
  (void)hipGetLastError();
  if (per_cu <= 0 || cus <= 0) return 0;
  const double resident = (double)per_cu * cus;
  const double cols = (double)(g.ne / nl) * g.nchunk;
  int best = 0;
  double best_cost = 0.0;
  for (int seg = 1; seg <= nl; ++seg) {
    if (nl % seg) continue;
    const double R = cols * (nl / seg) / resident;
    const double eff = R / std::ceil(R);
    const double cost = (1.0 + 0.2 / seg) / eff;
    if (best == 0 || cost < best_cost) {
      best = seg;
      best_cost = cost;
    }
  }
  return best >= 2 ? best : 0;
}

bool hex_one_lane(int order, int precision) {
  return precision != 2 ? (precision == 1 || order <= 2) : order <= 2;
}

int velocities_per_block(int dim, int order, int precision) {
  if (dim < 3 || hex_one_lane(order, precision)) return kBlock;
  return Plane3::VB;
}

hipError_t launch_stage(int precision, int mode, const StageArgs& A, hipStream_t s) {
  if (A.ecount <= 0) return hipSuccess;
  if (mode == 0 && A.rows) return launch_rows(precision, A, s);
  if (mode == 0 && A.walk_tx > 0 && A.walk_ty == 0) return launch_xwalk(precision, A, s);
  // BF16 storage (precision 2): FP32 state with BF16 stage increments; the
  // RK stages use the increment kernels, everything else the FP32 ones
  return precision == 0 ? stage_dispatch<double>(mode, false, A, s)
                        : stage_dispatch<float>(mode, precision == 2, A, s);
}

template <typename ST>
static hipError_t wall_dispatch(bool canonical, const WallArgs& W, hipStream_t s) {
  const dim3 grid((unsigned)W.blk0[W.nside]), block(kBlock);
  switch (W.g.dim * 10 + (W.g.n1 - 1)) {
#define BGK_WALL(D, P)                                                          \
  case D * 10 + P:                                                              \
    if (canonical)                                                              \
      hipLaunchKernelGGL((k_wall_flux<D, P, ST, true>), grid, block, 0, s, W);  \
    else                                                                        \
      hipLaunchKernelGGL((k_wall_flux<D, P, ST, false>), grid, block, 0, s, W); \
    break;
    BGK_WALL(1, 1) BGK_WALL(1, 2) BGK_WALL(1, 3)
    BGK_WALL(2, 1) BGK_WALL(2, 2) BGK_WALL(2, 3)
#undef BGK_WALL
    default:
      return hipErrorInvalidValue;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_wall_rho, dim3(grid_of(W.npoints, 256)), dim3(256), 0, s, W);
  return hipGetLastError();
}

hipError_t launch_wall(int precision, bool canonical, const WallArgs& W, hipStream_t s) {
  if (W.nside == 0) return hipSuccess;
  return precision == 0 ? wall_dispatch<double>(canonical, W, s)
                        : wall_dispatch<float>(canonical, W, s);
}

hipError_t launch_newton(const NewtonArgs& A, hipStream_t s) {
  // teams of 4 lanes per node once there are enough nodes to fill the GPU
  // (16,384 nodes on 24^3 velocities: 26 us against 34 with 16 lanes or 2; 1948
  // nodes on 22 x 23 x 21: 19 against 14.5 with 16), of 2 lanes on large meshes
  // (262,144 nodes on 16^3: 108 us against 124 with 4 and 280 with 16; 216,000
  // nodes on 20^3: 145 against 154)
  const int team = newton_team(A.g.nx);
  const dim3 grid(grid_of(A.g.nx * team, 256)), block(256);
#define BGK_NEWTON(T)                                                   \
  if (newton_split(A.g))                                                \
    hipLaunchKernelGGL((k_newton<T, true>), grid, block, 0, s, A);      \
  else                                                                  \
    hipLaunchKernelGGL((k_newton<T, false>), grid, block, 0, s, A)
  if (team == 2) {
    BGK_NEWTON(2);
  } else if (team == 4) {
    BGK_NEWTON(4);
  } else {
    BGK_NEWTON(16);
  }
#undef BGK_NEWTON
  return hipGetLastError();
}

hipError_t launch_collision_moments(int precision, const StageArgs& A, double* Cm,
                                    hipStream_t s) {
  const int nchunk = (int)((A.g.nv + kBlock - 1) / kBlock);
  const dim3 grid((unsigned)(A.g.ne * nchunk)), block(kBlock);
  if (precision == 0)
    hipLaunchKernelGGL(k_collision_moments<double>, grid, block, 0, s, A, nchunk);
  else
    hipLaunchKernelGGL(k_collision_moments<float>, grid, block, 0, s, A, nchunk);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  DevGeom g = A.g;
  g.nchunk = nchunk;
  return launch_reduce_partials(g, A.partials, Cm, s);
}

hipError_t launch_stage_batch(int precision, int dim, int order, int stage, const StageArgs* args,
                              const BatchList* list, size_t tab_bytes, unsigned grid,
                              hipStream_t s) {
  if (grid == 0) return hipSuccess;
  const size_t lds = std::max(tab_bytes, (size_t)(precision == 0 ? mfma_lds_bytes<double>()
                                                                  : mfma_lds_bytes<float>()));
#define BGK_BATCH(D, P)                                                                       \
  case D * 10 + P:                                                                          \
    if (precision == 0) {                                                                   \
      if (stage == 0)                                                                       \
        hipLaunchKernelGGL((k_stage_batch<D, P, double, 3>), dim3(grid), dim3(kBlock), lds, s, \
                           (table_ptr<StageArgs>)args, (table_ptr<BatchList>)list, stage);                                              \
      else                                                                                  \
        hipLaunchKernelGGL((k_stage_batch<D, P, double, 0>), dim3(grid), dim3(kBlock), lds, s, \
                           (table_ptr<StageArgs>)args, (table_ptr<BatchList>)list, stage);                                              \
    } else {                                                                                \
      if (stage == 0)                                                                       \
        hipLaunchKernelGGL((k_stage_batch<D, P, float, 3>), dim3(grid), dim3(kBlock), lds, s, \
                           (table_ptr<StageArgs>)args, (table_ptr<BatchList>)list, stage);                                              \
      else                                                                                  \
        hipLaunchKernelGGL((k_stage_batch<D, P, float, 0>), dim3(grid), dim3(kBlock), lds, s, \
                           (table_ptr<StageArgs>)args, (table_ptr<BatchList>)list, stage);                                              \
    }                                                                                       \
    break;
  switch (dim * 10 + order) {
    BGK_BATCH(1, 1) BGK_BATCH(1, 2) BGK_BATCH(1, 3)
    BGK_BATCH(2, 1) BGK_BATCH(2, 2) BGK_BATCH(2, 3)
    default:
      return hipErrorInvalidValue;
  }
#undef BGK_BATCH
  return hipGetLastError();
}

hipError_t launch_newton_batch(int team, bool split, const NewtonArgs* args,
                               const BatchList* list, unsigned grid, hipStream_t s) {
  if (grid == 0) return hipSuccess;
#define BGK_NEWTON(T)                                                                    \
  if (split)                                                                             \
    hipLaunchKernelGGL((k_newton_batch<T, true>), dim3(grid), dim3(256), 0, s,           \
                       (table_ptr<NewtonArgs>)args, (table_ptr<BatchList>)list);         \
  else                                                                                   \
    hipLaunchKernelGGL((k_newton_batch<T, false>), dim3(grid), dim3(256), 0, s,          \
                       (table_ptr<NewtonArgs>)args, (table_ptr<BatchList>)list)
  if (team == 16) {
    BGK_NEWTON(16);
  } else if (team == 4) {
    BGK_NEWTON(4);
  } else {
    BGK_NEWTON(2);
  }
#undef BGK_NEWTON
  return hipGetLastError();
}

hipError_t launch_wall_flux_batch(int precision, int dim, int order, int stage,
                                  const WallArgs* args, const BatchList* list, unsigned grid,
                                  hipStream_t s) {
  if (grid == 0) return hipSuccess;
#define BGK_WBATCH(D, P)                                                                        \
  case D * 10 + P:                                                                            \
    if (precision == 0)                                                                       \
      hipLaunchKernelGGL((k_wall_flux_batch<D, P, double>), dim3(grid), dim3(kBlock), 0, s, \
                         (table_ptr<WallArgs>)args, (table_ptr<BatchList>)list, stage);                                                        \
    else                                                                                      \
      hipLaunchKernelGGL((k_wall_flux_batch<D, P, float>), dim3(grid), dim3(kBlock), 0, s, \
                         (table_ptr<WallArgs>)args, (table_ptr<BatchList>)list, stage);                                                        \
    break;
  switch (dim * 10 + order) {
    BGK_WBATCH(1, 1) BGK_WBATCH(1, 2) BGK_WBATCH(1, 3)
    BGK_WBATCH(2, 1) BGK_WBATCH(2, 2) BGK_WBATCH(2, 3)
    default:
      return hipErrorInvalidValue;
  }
#undef BGK_WBATCH
  return hipGetLastError();
}

hipError_t launch_wall_rho_batch(int stage, const WallArgs* args, const BatchList* list,
                                 unsigned grid, hipStream_t s) {
  if (grid == 0) return hipSuccess;
  hipLaunchKernelGGL(k_wall_rho_batch, dim3(grid), dim3(256), 0, s, (table_ptr<WallArgs>)args,
                     (table_ptr<BatchList>)list, stage);
  return hipGetLastError();
}

int newton_team(int64_t nx) { return nx >= 131072 ? 2 : nx >= 8192 ? 4 : 16; }

// The three axes' sums together cost a launch the longest axis three times, but
// their exponentials overlap; so only where the axes together are well below that
// (us a launch, one axis after another / jointly / split: 64 x 8 x 8 velocities on
// 175,616 nodes 189 / 293 / 169, on 16,384 42 / 39 / 29, on 96 19.0 / 18.9 / 16.5; 32 x
// 16 x 8 on 175,616 130 / 142 / 110, on 96, where the joint one stays, 17.7 / 15.2 /
// 16.2; a grid of 16^3 takes 0.6 us more split).
bool newton_split(const DevGeom& g) {
  const int team = newton_team(g.nx), step = team == 16 ? 16 : 2 * team;
  int sum = 0, longest = 0;
  for (int c = 0; c < 3; ++c) {
    const int n = (g.nv1[c] + step - 1) / step * step;
    sum += n;
    longest = std::max(longest, n);
  }
  return sum < (team == 16 ? 0.6 : 0.8) * 3 * longest;
}

hipError_t launch_reduce_partials(const DevGeom& g, const double* partials, double* Q,
                                  hipStream_t s) {
  hipLaunchKernelGGL(k_reduce_partials, dim3(grid_of(g.nx, 256)), dim3(256), 0, s, g, partials,
                     Q);
  return hipGetLastError();
}

}  // namespace bgk
