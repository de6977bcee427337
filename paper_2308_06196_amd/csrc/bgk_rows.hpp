// bgk_rows.hpp -- stage kernels of 1-D and 2-D meshes that run several
// elements of a mesh row per work-group, on gfx950 (Dzanic & Martinelli,
// arXiv 2308.06196, Sec. 2.1).
#pragma once

#include "bgk_device.hpp"

namespace bgk {

// One work-group = E consecutive elements along x x one chunk of 256 velocity
// slots; one lane = one velocity and all nodes of the E elements. A low-order
// element has too few nodes to pay for what a work-group does once (the lane's
// velocity, its operators, the gather of the equilibrium rows, two barriers,
// the matrix products of the moments, which take 16 nodes at a time): E is
// chosen so that the run has about the 16 nodes of a p = 3 quadrilateral. The
// x traces between the elements of the run stay in registers; only the run's
// upwind end reads a neighbour's nodes.
//
// Every sum is the one stage_item forms, in its order, so a run of elements
// gives the bits of E per-element work items.
//
// Measured, us per stage launch, per element against runs (one work-group's
// fixed cost and the latency of its three load batches bound the former, HBM
// the latter): 487-element tube on 22 x 23 x 21 velocities, FP64 p = 1, 2, 3
// 135.5 / 53.4, 148.0 / 75.6, 160.3 / 97.3 (2.8 -> 4.5 TB/s of compulsory
// traffic at p = 3), FP32 95.5 / 32.5, 100.5 / 44.1, 105.2 / 54.6, BF16
// increments 93.1 / 32.1, 98.6 / 43.0, 101.6 / 50.5; 32^2 box on 24^3
// velocities, FP64 p = 1 438.7 / 257.2, p = 2 646.9 / 578.7 (column sweep /
// runs), FP32 300.3 / 139.7 and 390.2 / 341.6; 24 x 40 channel, p = 2, FP64 on
// 16^3 velocities 202.3 / 160.6. Runs twice as long were slower in FP32 (tube
// p = 1 38.5, box p = 2 354.8); p = 3 quadrilaterals already have 16 nodes.
template <int DIM, int P>
constexpr int row_elems() {
  return DIM == 1 ? (P == 1 ? 8 : P == 2 ? 5 : 4) : P == 1 ? 4 : 2;
}

template <int DIM, int P, typename ST, int MODE, bool INC, int E>
__device__ __forceinline__ void row_item(const StageArgs& A, const int chunk, const int ey,
                                         const int ex0, const int cnt, const bool count) {
  static_assert(DIM <= 2, "segments and quadrilaterals");
  static_assert(MODE == 0 || MODE == 3, "RK stages");
  static_assert(!INC || sizeof(ST) == 4, "increment stages: FP32 state");
  using CT = typename Compute<ST>::T;
  constexpr int N1 = P + 1;
  constexpr int NS = ipow(N1, DIM);
  constexpr int NL = ipow(N1, DIM - 1);  // lines per element and axis
  constexpr int R = E * NS;
  __shared__ double red[(kBlock / 64) * part_rows<R>() * 5];
  __shared__ LimiterCounts lim;
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  double* tab = reinterpret_cast<double*>(dyn_lds);

  const int tid = (int)threadIdx.x;
  const DevGeom& g = A.g;
  const DevOpsT<CT>& OP = ops_of<CT>(A);
  const int64_t nv = g.nv;
  const int S = g.tabw;
  const int nx = sreg(g.nelem[0]);
  const int64_t e0 = ex0 + (int64_t)ey * nx;  // first element of the run
  const int64_t node0 = e0 * NS;

  const int j = chunk * kBlock + tid;
  const bool valid = j < nv;
  const int jj = valid ? j : (int)nv - 1;
  Vel vel = velocity_of(g, jj);
  if (!valid) vel.w = 0.0;

  // upwind source per axis (see stage_item): on x the element before or after
  // the run, on y the elements of the row below or above, each for the run's
  // first element; at a specular wall the own elements at the mirrored
  // velocity, at a diffuse wall the own ones (unused)
  const ST* __restrict__ fin = (const ST*)A.fin;
  const int64_t estride = g.nvb * (int64_t)(NS * kVB);
  int64_t src[DIM];
  bool pos[DIM], use_right[DIM], dif[DIM];
#pragma unroll
  for (int k = 0; k < DIM; ++k) {
    pos[k] = vel.u[k] * g.scale[k] > 0.0;
    const int nek = sreg(g.nelem[k]);
    // the run's element whose upwind neighbour on this axis is taken
    const int c = k == 0 ? (pos[0] ? ex0 : ex0 + cnt - 1) : ey;
    int n = c + (pos[k] ? -1 : 1);
    bool wall = false;
    int bc = 0;
    if (n < 0 || n >= nek) {
      bc = pos[k] ? sreg(g.bc[k][0]) : sreg(g.bc[k][1]);
      wall = bc != 0;
      n = n < 0 ? nek - 1 : 0;
    }
    dif[k] = bc == 2;
    int64_t src_e = k == 0 ? e0 + (c - ex0) : e0;
    int src_j = jj;
    if (dif[k]) {
    } else if (wall) {
      int bm[3] = {vel.b[0], vel.b[1], vel.b[2]};
      bm[k] = g.nv1[k] - 1 - bm[k];
      src_j = vel_slot(g, bm);
    } else {
      src_e += (int64_t)(n - c) * (k == 0 ? 1 : nx);
    }
    use_right[k] = pos[k] != wall;
    src[k] = f_offset(g, src_e, 0, src_j);
  }

  // loads in three batches (see stage_item): row entries, own nodes and the
  // x neighbour's; the y neighbours' after the x transport; f^n after the
  // relaxation. Elements past the run's end repeat its last one and store
  // nothing.
  constexpr int kU = 2;
  const RowPick rp = row_pick(A, chunk, cnt * NS);
  const double* et = A.etab + node0 * S;
  double tv[kU];
  if (A.collide) {
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int t = u * kBlock + tid;
      tv[u] = et[rp.offset(t < rp.count ? t : rp.count - 1)];
    }
  }
  constexpr bool kDin = INC && MODE == 0;
  const uint16_t* __restrict__ din = A.din;
  const int64_t own = f_offset(g, e0, 0, jj);
  CT f[R];
  CT fb[INC ? R : 1];
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const ST* fe = fin + own + (i < cnt ? i : cnt - 1) * estride;
#pragma unroll
    for (int q = 0; q < NS; ++q) f[i * NS + q] = (CT)fe[q * kVB];
  }
  CT nbx[NS];
#pragma unroll
  for (int q = 0; q < NS; ++q) nbx[q] = (CT)fin[src[0] + q * kVB];
  if constexpr (INC) {
#pragma unroll
    for (int q = 0; q < R; ++q) fb[q] = f[q];
  }
  if constexpr (kDin) {
#pragma unroll
    for (int i = 0; i < E; ++i) {
      CT v[NS];
#pragma unroll
      for (int q = 0; q < NS; ++q) v[q] = f[i * NS + q];
      add_increments(v, din, own + (i < cnt ? i : cnt - 1) * estride);
#pragma unroll
      for (int q = 0; q < NS; ++q) f[i * NS + q] = v[q];
    }
    add_increments(nbx, din, src[0]);
  }
  if (A.collide) {
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int t = u * kBlock + tid;
      if (t < rp.count) tab[t] = tv[u];
    }
  }

  CT acc[R];
#pragma unroll
  for (int q = 0; q < R; ++q) acc[q] = (CT)0;

  // diffuse walls of axis k at the run's upwind ends (uniform): the re-emitted
  // densities of the side's flux points from element fe on, and the unit wall
  // Maxwellian at this lane's velocity on its inflow side
  const double* rho_lo = nullptr;
  const double* rho_hi = nullptr;
  CT mw = (CT)0;
  auto diffuse = [&](int k) -> bool {
    const int off_lo = sreg(A.wall_off[k][0]), off_hi = sreg(A.wall_off[k][1]);
    const int lo_c = k == 0 ? ex0 : ey, hi_c = k == 0 ? ex0 + cnt - 1 : ey;
    const bool dlo = off_lo >= 0 && lo_c == 0, dhi = off_hi >= 0 && hi_c == sreg(g.nelem[k]) - 1;
    if (!dlo && !dhi) return false;
    const int fe = DIM == 1 ? 0 : k == 0 ? ey : ex0;
    rho_lo = A.wall_rho + (dlo ? off_lo : 0) + fe * NL;
    rho_hi = A.wall_rho + (dhi ? off_hi : 0) + fe * NL;
    const double* wp = A.wallp + (k * 2 + (pos[k] ? 0 : 1)) * 8;
    const double d0 = vel.u[0] - wp[2], d1 = vel.u[1] - wp[3], d2 = vel.u[2] - wp[4];
    mw = (CT)(wp[0] * exp(-(d0 * d0 + d1 * d1 + d2 * d2) * wp[1]));
    return true;
  };

#pragma unroll
  for (int k = 0; k < DIM; ++k) {
    const int S1 = k == 0 ? 1 : N1, SL = k == 0 ? N1 : 1;  // stride in and between lines
    const CT a = (CT)(vel.u[k] * g.scale[k]);
    CT lown[N1], lout[N1], lext[N1], Gin[N1];
#pragma unroll
    for (int b = 0; b < N1; ++b) {
      lown[b] = pos[k] ? OP.lamL[b] : OP.lamR[b];
      lout[b] = pos[k] ? OP.lamR[b] : OP.lamL[b];
      lext[b] = use_right[k] ? OP.lamR[b] : OP.lamL[b];
      Gin[b] = pos[k] ? OP.GL[b] : OP.GR[b];
    }
    const bool dwall = diffuse(k);
    if (k == 1) __builtin_amdgcn_sched_barrier(0);  // batch (2)
    // exterior traces at the run's upwind end (x), from the neighbour element
    CT xend[NL];
    if (k == 0) {
#pragma unroll
      for (int l = 0; l < NL; ++l) {
        CT t = (CT)0;
#pragma unroll
        for (int b = 0; b < N1; ++b) t += lext[b] * nbx[l * SL + b * S1];
        if (dwall) {
          const CT rw = (CT)(pos[0] ? sreg(rho_lo[l]) : sreg(rho_hi[l]));
          t = dif[0] ? rw * mw : t;
        }
        xend[l] = t;
      }
    }
    CT nby[DIM == 2 ? R : 1];
    if constexpr (DIM == 2) {
      if (k == 1) {
#pragma unroll
        for (int i = 0; i < E; ++i) {
          const int64_t so = src[1] + (i < cnt ? i : cnt - 1) * estride;
          CT v[NS];
#pragma unroll
          for (int q = 0; q < NS; ++q) v[q] = (CT)fin[so + q * kVB];
          if constexpr (kDin) add_increments(v, din, so);
#pragma unroll
          for (int q = 0; q < NS; ++q) nby[i * NS + q] = v[q];
        }
      }
    }
    // own inflow traces and, on x, the outflow traces handed to the next
    // element of the run
    CT tout[E][NL];
    if (k == 0) {
#pragma unroll
      for (int i = 0; i < E; ++i)
#pragma unroll
        for (int l = 0; l < NL; ++l) {
          CT t = (CT)0;
#pragma unroll
          for (int b = 0; b < N1; ++b) t += lout[b] * f[i * NS + l * SL + b * S1];
          tout[i][l] = t;
        }
    }
#pragma unroll
    for (int i = 0; i < E; ++i) {
#pragma unroll
      for (int l = 0; l < NL; ++l) {
        const int base = i * NS + l * SL;
        CT line[N1];
#pragma unroll
        for (int b = 0; b < N1; ++b) line[b] = f[base + b * S1];
        CT own_t = (CT)0, ext = (CT)0;
#pragma unroll
        for (int b = 0; b < N1; ++b) own_t += lown[b] * line[b];
        if (k == 0) {
          const CT from_left = i == 0 ? xend[l] : tout[i > 0 ? i - 1 : 0][l];
          const CT from_right = i + 1 >= E || i == cnt - 1 ? xend[l] : tout[i + 1 < E ? i + 1 : i][l];
          ext = pos[0] ? from_left : from_right;
        } else if constexpr (DIM == 2) {
#pragma unroll
          for (int b = 0; b < N1; ++b) ext += lext[b] * nby[base + b * S1];
          if (dwall) {
            const int fp = (i < cnt ? i : cnt - 1) * NL + l;
            const CT rw = (CT)(pos[1] ? sreg(rho_lo[fp]) : sreg(rho_hi[fp]));
            ext = dif[1] ? rw * mw : ext;
          }
        }
        const CT jump = a * (ext - own_t);
#pragma unroll
        for (int ia = 0; ia < N1; ++ia) {
          CT df = (CT)0;
#pragma unroll
          for (int b = 0; b < N1; ++b) df += OP.D[ia][b] * line[b];
          acc[base + ia * S1] += a * df + jump * Gin[ia];
        }
      }
    }
  }

  // relaxation (see stage_item): h = b (f - dt T) + b dt C, formed before f^n
  // is loaded; C in FP64, added in FP64
  const int cx = vel.b[0] - rp.x0, oy = rp.nx + vel.b[1] - rp.y0,
            oz = rp.nxy + vel.b[2] - rp.z0;
  const CT dt = (CT)A.dt, ca = (CT)A.a, cb = (CT)A.b;
  const double wc = A.b * A.dt;
  if (A.collide) {
    table_rest<kU>(tab, et, rp, tid);
    lds_barrier();
#pragma unroll
    for (int q = 0; q < R; ++q) {
      // (rows past the run's end: any row of the table)
      const int row = q / NS < cnt ? q : 0;
      const double c = collision_term(tab + row * rp.ncols, cx, oy, oz, rp.ncols, (double)f[q]);
      if constexpr (sizeof(CT) == 8) {
        acc[q] = fma(wc, c, cb * (f[q] - dt * acc[q]));
      } else {
        acc[q] = (CT)fma(wc, c, (double)(cb * (f[q] - dt * acc[q])));
      }
    }
  } else {
#pragma unroll
    for (int q = 0; q < R; ++q) acc[q] = cb * (f[q] - dt * acc[q]);
  }
  __builtin_amdgcn_sched_barrier(0);
  CT o[R], fnv[R];
  if constexpr (INC) {
#pragma unroll
    for (int q = 0; q < R; ++q) fnv[q] = fb[q];
  } else if constexpr (MODE == 0) {
#pragma unroll
    for (int i = 0; i < E; ++i) {
      const ST* fn = (const ST*)A.fn + own + (i < cnt ? i : cnt - 1) * estride;
#pragma unroll
      for (int q = 0; q < NS; ++q) fnv[i * NS + q] = (CT)__builtin_nontemporal_load(&fn[q * kVB]);
    }
  }
#pragma unroll
  for (int q = 0; q < R; ++q) o[q] = MODE == 0 ? ca * fnv[q] + acc[q] : acc[q];
  if (A.limiter) {
    int hits = 0, bad = 0;
#pragma unroll
    for (int i = 0; i < E; ++i) {
      CT(&oi)[NS] = *reinterpret_cast<CT(*)[NS]>(&o[i * NS]);
      CT fmin = oi[0];
#pragma unroll
      for (int q = 0; q < NS; ++q) fmin = oi[q] < fmin ? oi[q] : fmin;
      const CT mean = tensor_wsum<DIM, N1>(oi, OP.w) / OP.Wsum;
      const bool hit = valid && i < cnt && (fmin < (CT)0);
      if (hit && mean != fmin) {
        CT beta = fabs(mean / (mean - fmin));
        beta = beta > (CT)1 ? (CT)1 : beta;
#pragma unroll
        for (int q = 0; q < NS; ++q) oi[q] = mean + beta * (oi[q] - mean);
      }
      hits += __popcll(__ballot(hit));
      bad += __popcll(__ballot(hit && !(mean > (CT)0)));
    }
    limiter_count(lim, hits, bad, tid);
  }
  if (INC && !A.out_full) {
    if constexpr (INC) {
#pragma unroll
      for (int i = 0; i < E; ++i) {
        const int64_t ooff = own + i * estride;
        const bool live = valid && i < cnt;
        uint32_t* ow = inc_pairs((uint16_t*)A.out, ooff);
        float omin = INFINITY, smin = INFINITY;  // stage values / stored values
        uint32_t wd[NS / 2];
#pragma unroll
        for (int q = 0; q + 1 < NS; q += 2) {
          CT &o0 = o[i * NS + q], &o1 = o[i * NS + q + 1];
          float s0, s1;
          wd[q >> 1] = bf16_increment2(o0, o1, fnv[i * NS + q], fnv[i * NS + q + 1], s0, s1);
          omin = fminf(omin, fminf(o0, o1));
          smin = fminf(smin, fminf(s0, s1));
          o0 = s0;
          o1 = s1;
        }
        if constexpr (NS % 2 != 0) {  // odd last node
          CT& ol = o[i * NS + NS - 1];
          float stored;
          const uint16_t h = bf16_increment(ol, fnv[i * NS + NS - 1], stored);
          if (live) __builtin_nontemporal_store(h, (uint16_t*)A.out + ooff + (NS - 1) * kVB);
          omin = fminf(omin, ol);
          smin = fminf(smin, stored);
          ol = stored;
        }
        if (live) {
#pragma unroll
          for (int m = 0; m < NS / 2; ++m) __builtin_nontemporal_store(wd[m], &ow[m * kVB]);
        }
        const unsigned long long nviol = __popcll(__ballot(live && smin < 0.0f && !(omin < 0.0f)));
        if ((tid & 63) == 0 && nviol) atomicAdd(&A.diag[5], nviol);
      }
    }
  } else if (valid) {
#pragma unroll
    for (int i = 0; i < E; ++i) {
      if (i < cnt) {
        ST* oe = (ST*)A.out + own + i * estride;
#pragma unroll
        for (int q = 0; q < NS; ++q) __builtin_nontemporal_store((ST)o[i * NS + q], &oe[q * kVB]);
      }
    }
  }
  if (A.collide) lds_barrier();
  element_partials_mfma<R, ST, CT>(o, vel, A.partials, node0, g.nx, chunk, dyn_lds, red, tid,
                                   cnt * NS);
  if (A.limiter) limiter_add(lim, A.diag, tid);  // (behind the partials' barrier)
  if (tid == 0 && count) atomicAdd(&A.diag[4], 1ull);
}

// Work items of a mesh: runs of E elements per row, velocity-chunk major.
template <int DIM, int P>
__host__ __device__ __forceinline__ int64_t row_runs(const DevGeom& g) {
  constexpr int E = row_elems<DIM, P>();
  return (int64_t)((g.nelem[0] + E - 1) / E) * (DIM == 2 ? g.nelem[1] : 1);
}

template <int DIM, int P, typename ST, int MODE, bool INC>
__device__ __forceinline__ void row_work(const StageArgs& A, int64_t w) {
  constexpr int E = row_elems<DIM, P>();
  const int64_t per_chunk = row_runs<DIM, P>(A.g);
  const int chunk = (int)(w / per_chunk);
  const int r = (int)(w - chunk * per_chunk);
  const int nr = (A.g.nelem[0] + E - 1) / E;
  const int ey = DIM == 2 ? r / nr : 0;
  const int ex0 = (r - ey * nr) * E;
  row_item<DIM, P, ST, MODE, INC, E>(A, chunk, ey, ex0, min(E, A.g.nelem[0] - ex0), w == 0);
}

template <int DIM, int P, typename ST, int MODE, bool INC = false>
__global__ void __launch_bounds__(kBlock)
    __attribute__((amdgpu_waves_per_eu(sizeof(ST) == 8 ? 3 : 4))) k_stage_rows(const StageArgs A) {
  row_work<DIM, P, ST, MODE, INC>(A, xcd_remap(blockIdx.x, gridDim.x));
}

// Batch members that run rows (see k_stage_batch).
template <int DIM, int P, typename ST, int MODE>
__global__ void __launch_bounds__(kBlock)
    __attribute__((amdgpu_waves_per_eu(sizeof(ST) == 8 ? 3 : 4)))
    k_stage_rows_batch(table_ptr<StageArgs> args, table_ptr<BatchList> list, int stage) {
  const int32_t u = (int32_t)xcd_remap(blockIdx.x, gridDim.x);
  const int m = batch_member(list->stage_off, list->n, u);
  row_work<DIM, P, ST, MODE, false>(table_entry(args, list->slot[m] * 3 + stage),
                                    u - list->stage_off[m]);
}

}  // namespace bgk
