// bgk_xwalk.hpp -- stage kernels that walk runs of elements along x, one lane
// per velocity, on gfx950 (Dzanic & Martinelli, arXiv 2308.06196, Sec. 2.1).
#pragma once

#include "bgk_device.hpp"

namespace bgk {

// One work-group = one chunk of 256 velocity slots walking a run of elements
// of one mesh row in the upwind direction of the chunk; one lane = one velocity
// and all nodes of the element, as in stage_item. Against one work-group per
// element:
//   * what depends on the velocity alone (its decode, the moment functions in
//     LDS, the neighbour offsets, the row entries' positions) is done once per
//     run;
//   * the x traces are handed on in registers, so no x neighbour is read
//     except at the run's entry (and by lanes whose sign differs from the
//     chunk's);
//   * the next element's nodes and rows are loaded once the relaxation has
//     consumed the current ones, so that the limiter, the stores and the
//     moments cover their latency; the y neighbour's are loaded ahead of the x
//     transport, the z neighbour's after the y transport (one neighbour's
//     nodes held at a time);
//   * the operators are scalar operands where a wave's velocities share the
//     sign of u_k (its lanes pick theirs otherwise, in one pass per sign).
// The equilibrium rows have LDS of their own beside the moments' staging, so
// that an element takes two barriers. Every sum is the one stage_item forms,
// in its order: the results have its bits.
//
// Used where it measured faster than one work-group per element (ms per stage
// launch, per element / walk): p = 3 quadrilaterals in FP32 (32^2 box on 24^3
// velocities 0.587 / 0.541, 45 x 29 box on 21 x 22 x 17 0.432 / 0.419) and with
// increments (0.585 / 0.521, 0.428 / 0.406: three waves per SIMD, as with four the
// walk spills and takes 0.635); p = 1 hexahedra (16^3 elements on 16^3, FP64 0.827 /
// 0.726, FP32 0.527 / 0.463, BF16 increments 0.529 / 0.460); p = 2 hexahedra with increments (20^3 elements on
// 20^3 9.72 / 5.85: the element and its increments need more registers than
// the per-element kernel's four waves per SIMD leave). Not for p = 3
// quadrilaterals in FP64 (1.04 / 1.25) and p = 2 hexahedra in FP64 (20^3
// velocities, 14^3 elements 3.29 / 3.88) and FP32 (4.81 / 5.2), whose loop spills or runs at fewer waves.
template <int DIM, int P>
struct XWalk {
  static constexpr int N1 = P + 1, NS = ipow(N1, DIM), NL = ipow(N1, DIM - 1);
  static constexpr int CS = (NS + 1) / 2 * 2 + 2;  // column stride of the rows in LDS
  static constexpr int rows_bytes(int ncols) { return CS * ncols * 8; }
  static constexpr int ps_bytes = kBlock * 5 * 8;
  template <typename ST>
  static constexpr int lds_bytes(int ncols) {
    return rows_bytes(ncols) + ps_bytes + (kBlock / 64) * 16 * kGst * (int)sizeof(ST);
  }
};

// Waves per SIMD: what the registers of a variant allow with at most one spilled
// vector register (p = 1 hexahedra with increments).
template <int DIM, int P, typename ST, bool INC>
constexpr int xwalk_waves() {
  return DIM == 3 && P == 2 ? 2 : sizeof(ST) == 8 || (DIM == 2 && INC) ? 3 : 4;
}

template <int DIM, int P, typename ST, int MODE, bool INC>
__device__ __forceinline__ void xwalk(table_ptr<StageArgs> ap, const int chunk, const int ey,
                                      const int ez, const int x0, const int x1, const bool count) {
  using CT = typename Compute<ST>::T;
  using X = XWalk<DIM, P>;
  constexpr int N1 = X::N1, NS = X::NS, NL = X::NL;
  constexpr bool kDin = INC && MODE == 0;
  static_assert(MODE == 0 || MODE == 3, "RK stages");
  __shared__ double red[(kBlock / 64) * part_rows<NS>() * 5];
  extern __shared__ __align__(16) unsigned char dyn_lds[];

  auto args = [&]() -> const StageArgs& { return table_entry(ap, 0); };
  const StageArgs& A0 = args();
  const DevGeom& g = A0.g;
  const int tid = (int)threadIdx.x, lane = tid & 63, wave = sreg(tid >> 6);
  const int nv = (int)g.nv;
  const int j = chunk * kBlock + tid;
  const bool valid = j < nv;
  const int jj = valid ? j : nv - 1;
  const RowPick rp = row_pick(A0, chunk, NS);
  double* tab = reinterpret_cast<double*>(dyn_lds);
  unsigned char* lw = dyn_lds + X::rows_bytes(rp.ncols);
  double* ps = reinterpret_cast<double*>(lw) + wave * 64 * 5;
  ST* gw = reinterpret_cast<ST*>(lw + X::ps_bytes) + wave * 16 * kGst;
  double* redw = red + wave * part_rows<NS>() * 5;

  CT a[DIM];
  bool pos[DIM];
  int cx, cy, cz;  // this lane's factor columns
  {
    Vel vel = velocity_of(g, jj);
    if (!valid) vel.w = 0.0;
    const double psi4 =
        0.5 * (vel.u[0] * vel.u[0] + vel.u[1] * vel.u[1] + vel.u[2] * vel.u[2]);
    ps[lane * 5 + 0] = vel.w;
    ps[lane * 5 + 1] = vel.w * vel.u[0];
    ps[lane * 5 + 2] = vel.w * vel.u[1];
    ps[lane * 5 + 3] = vel.w * vel.u[2];
    ps[lane * 5 + 4] = vel.w * psi4;
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
      pos[k] = vel.u[k] * g.scale[k] > 0.0;
      a[k] = (CT)(vel.u[k] * g.scale[k]);
    }
    cx = (vel.b[0] - rp.x0) * X::CS;
    cy = (rp.nx + vel.b[1] - rp.y0) * X::CS;
    cz = (rp.nxy + vel.b[2] - rp.z0) * X::CS;
  }
  bool up;  // walk direction: the sign of u_x of the chunk's first slot
  {
    int b0[3];
    slot_nodes(g, chunk * kBlock, b0);
    up = (g.vlo[0] + b0[0] * g.du[0]) * g.scale[0] > 0.0;
  }
  const int64_t estride = g.nvb * (int64_t)(NS * kVB);  // values per element
  const ST* __restrict__ fin = (const ST*)A0.fin;
  const uint16_t* __restrict__ din = A0.din;
  const bool collide = A0.collide;
  auto slot_off = [&](int js) -> int64_t { return (int64_t)(js / kVB) * NS * kVB + js % kVB; };
  const int64_t own_off = slot_off(jj);
  const int64_t e_row = (int64_t)g.nelem[0] * (ey + (int64_t)(DIM == 3 ? g.nelem[1] : 0) * ez);

  // upwind source of axis k for element e with coordinate c on it: offset of
  // its nodes; right: the source's right trace is taken
  auto source = [&](int k, int c, int64_t e, bool& right) -> int64_t {
    const DevGeom& q = args().g;
    const int nk = q.nelem[k];
    const int64_t st = k == 0 ? 1 : k == 1 ? (int64_t)q.nelem[0] : (int64_t)q.nelem[0] * q.nelem[1];
    const bool edge = pos[k] ? c == 0 : c == nk - 1;
    const bool wall = edge && (pos[k] ? q.bc[k][0] : q.bc[k][1]) != 0;
    right = pos[k] != wall;
    if (wall) {  // the own element at the mirrored velocity
      int bm[3];
      slot_nodes(q, jj, bm);
      bm[k] = q.nv1[k] - 1 - bm[k];
      return e * estride + slot_off(vel_slot(q, bm));
    }
    const int d = (pos[k] ? -1 : 1) + (edge ? (pos[k] ? nk : -nk) : 0);
    return (e + d * st) * estride + own_off;
  };
  // the y and z sources stay at the same distance along the row
  bool right[DIM];
  int64_t noff[DIM];
#pragma unroll
  for (int k = 1; k < DIM; ++k) noff[k] = source(k, k == 1 ? ey : ez, 0, right[k]);

  constexpr int kU = 2;
  int rowt[kU];  // offset in the element's rows, LDS index (<< 16)
  auto row_index = [&](int t) -> int {
    const int n = (int)__umulhi((unsigned)t, rp.magic);
    return (t - n * rp.ncols) * X::CS + n;
  };
#pragma unroll
  for (int u = 0; u < kU; ++u) {
    const int t = min(u * kBlock + tid, rp.count - 1);
    rowt[u] = rp.offset(t) | row_index(t) << 16;
  }
  const int row_doubles = NS * rp.S;

  CT f[NS], nb[NS];
  constexpr int NW = kDin ? NS / 2 : 1;
  uint32_t fd[NW], nd[NW];
  uint16_t fd1 = 0, nd1 = 0;  // odd last node's increment
  double tv[kU];
  auto load_nodes = [&](CT(&x)[NS], uint32_t(&d)[NW], uint16_t& d1, int64_t off) {
#pragma unroll
    for (int q = 0; q < NS; ++q) x[q] = (CT)fin[off + q * kVB];
    if constexpr (kDin) {
      const uint32_t* w = inc_pairs(din, off);
#pragma unroll
      for (int m = 0; m < NW; ++m) d[m] = w[m * kVB];
      if constexpr (NS % 2 != 0) d1 = din[off + (NS - 1) * kVB];
    }
  };
  auto add_inc = [&](CT(&x)[NS], const uint32_t(&d)[NW], const uint16_t d1) {
    if constexpr (kDin) {
#pragma unroll
      for (int m = 0; m < NW; ++m) {
        x[2 * m] += bf16_lo(d[m]);
        x[2 * m + 1] += bf16_hi(d[m]);
      }
      if constexpr (NS % 2 != 0) x[NS - 1] += bf16_f32(d1);
    }
  };
  auto load_element = [&](int64_t e) {
    if (collide) {
      const double* et = args().etab + e * row_doubles;
#pragma unroll
      for (int u = 0; u < kU; ++u) tv[u] = et[rowt[u] & 0xFFFF];
    }
    load_nodes(f, fd, fd1, e * estride + own_off);
  };

  const int n = x1 - x0, dx = up ? 1 : -1;
  int ex = up ? x0 : x1 - 1;
  CT trx[NL];  // exterior x traces; at the entry from the neighbour's nodes
  {
    bool rt;
    const int64_t so = source(0, ex, e_row + ex, rt);
    const DevOpsT<CT>& OP = ops_of<CT>(A0);
    load_nodes(nb, nd, nd1, so);
    add_inc(nb, nd, nd1);
#pragma unroll
    for (int l = 0; l < NL; ++l) {
      CT t = (CT)0;
#pragma unroll
      for (int b = 0; b < N1; ++b) t += (rt ? OP.lamR[b] : OP.lamL[b]) * nb[l * N1 + b];
      trx[l] = t;
    }
  }
  load_element(e_row + ex);

  // limiter counters of the wave over the run (shared only behind it: without
  // collisions an element has no barrier between two waves' limiters)
  int hits = 0, bad = 0;
  for (int s = 0; s < n; ++s, ex += dx) {
    asm volatile("" : "+s"(ap));
    const int64_t e = e_row + ex, eoff = e * estride + own_off;
    if (collide) {  // rows -> LDS (every wave is past the last element's reads)
#pragma unroll
      for (int u = 0; u < kU; ++u) tab[rowt[u] >> 16] = tv[u];
      for (int t = kU * kBlock + tid; t < rp.count; t += kBlock)
        tab[row_index(t)] = args().etab[e * row_doubles + rp.offset(t)];
    }
    CT fb[INC ? NS : 1];
    if constexpr (INC) {
#pragma unroll
      for (int q = 0; q < NS; ++q) fb[q] = f[q];
    }
    add_inc(f, fd, fd1);
    load_nodes(nb, nd, nd1, e * estride + noff[1]);
    CT acc[NS];
#pragma unroll
    for (int q = 0; q < NS; ++q) acc[q] = (CT)0;
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
      if (k > 0) asm volatile("" : "+s"(ap));
      const DevOpsT<CT>& OP = ops_of<CT>(args());
      const int S1 = k == 0 ? 1 : k == 1 ? N1 : N1 * N1;  // stride in a line
      bool rt = k > 0 ? right[k] : false;
      if constexpr (DIM == 3) {
        if (k == 2) {
          __builtin_amdgcn_sched_barrier(0);
          load_nodes(nb, nd, nd1, e * estride + noff[2]);
        }
      }
      if (k > 0) add_inc(nb, nd, nd1);
      // exterior traces of the lines
      CT ext[NL];
      if (k == 0) {
#pragma unroll
        for (int l = 0; l < NL; ++l) ext[l] = trx[l];
        // lanes whose sign is not the walk's read their own neighbour, line by
        // line (only waves in which the velocity octants change)
        const bool lane_carry = s == 0 || pos[0] == up;
        if (__ballot(!lane_carry) != 0) {
          const int64_t so = source(0, ex, e, rt);
#pragma unroll
          for (int l = 0; l < NL; ++l) {
            CT t = (CT)0;
#pragma unroll
            for (int b = 0; b < N1; ++b) {
              CT x = (CT)fin[so + (l * N1 + b) * kVB];
              if constexpr (kDin) x += increment_of<NS>(din, so, l * N1 + b);
              t += (rt ? OP.lamR[b] : OP.lamL[b]) * x;
            }
            ext[l] = lane_carry ? ext[l] : t;
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      } else {
        const CT(&x)[NS] = nb;
        const bool mixed = __ballot(rt) != 0 && __ballot(!rt) != 0;
        auto traces = [&](auto&& lam) {
#pragma unroll
          for (int l = 0; l < NL; ++l) {
            const int base = (l / S1) * S1 * N1 + l % S1;
            CT t = (CT)0;
#pragma unroll
            for (int b = 0; b < N1; ++b) t += lam(b) * x[base + b * S1];
            ext[l] = t;
          }
        };
        if (mixed) {
          traces([&](int b) { return rt ? OP.lamR[b] : OP.lamL[b]; });
        } else {
          const bool ur = __ballot(rt) != 0;
          traces([&](int b) { return ur ? OP.lamR[b] : OP.lamL[b]; });
        }
      }
      // own traces, jumps and derivatives, once per sign of u_k in the wave
      const int s_lo = __ballot(!pos[k]) == 0 ? 1 : 0, s_hi = __ballot(pos[k]) == 0 ? 0 : 1;
#pragma unroll 1
      for (int sg = s_lo; sg <= s_hi; ++sg) {
        const bool mine = s_lo == s_hi || (pos[k] ? 1 : 0) == sg;
        CT lin[N1], gin[N1];
#pragma unroll
        for (int b = 0; b < N1; ++b) {
          lin[b] = sg ? OP.lamL[b] : OP.lamR[b];
          gin[b] = sg ? OP.GL[b] : OP.GR[b];
        }
#pragma unroll
        for (int l = 0; l < NL; ++l) {
          const int base = (l / S1) * S1 * N1 + l % S1;
          CT line[N1];
#pragma unroll
          for (int b = 0; b < N1; ++b) line[b] = f[base + b * S1];
          CT own = (CT)0;
#pragma unroll
          for (int b = 0; b < N1; ++b) own += lin[b] * line[b];
          const CT jump = mine ? a[k] * (ext[l] - own) : (CT)0;
          const CT as = mine ? a[k] : (CT)0;
#pragma unroll
          for (int ia = 0; ia < N1; ++ia) {
            CT df = (CT)0;
#pragma unroll
            for (int b = 0; b < N1; ++b) df += OP.D[ia][b] * line[b];
            acc[base + ia * S1] += as * df + jump * gin[ia];
          }
        }
      }
      if (k == 0) {  // outflow traces: the next element's exterior traces
#pragma unroll
        for (int l = 0; l < NL; ++l) {
          CT t = (CT)0;
#pragma unroll
          for (int b = 0; b < N1; ++b) t += (up ? OP.lamR[b] : OP.lamL[b]) * f[l * N1 + b];
          trx[l] = t;
        }
      }
    }
    asm volatile("" : "+s"(ap));
    const StageArgs& A = args();
    const CT dt = (CT)A.dt, ca = (CT)A.a, cb = (CT)A.b;
    const double wc = A.b * A.dt;
    // relaxation (see stage_item)
    if (collide) {
      lds_barrier();
      asm volatile("" : "+v"(cx), "+v"(cy), "+v"(cz));
      const double *tx = tab + cx, *ty = tab + cy, *tz = tab + cz,
                   *tt = tab + (rp.ncols - 1) * X::CS;
#pragma unroll
      for (int q = 0; q < NS; ++q) {
        const double c = collision_term(tx[q], ty[q], tz[q], tt[q], (double)f[q]);
        if constexpr (sizeof(CT) == 8) acc[q] = fma(wc, c, cb * (f[q] - dt * acc[q]));
        else acc[q] = (CT)fma(wc, c, (double)(cb * (f[q] - dt * acc[q])));
      }
    } else {
#pragma unroll
      for (int q = 0; q < NS; ++q) acc[q] = cb * (f[q] - dt * acc[q]);
    }
    __builtin_amdgcn_sched_barrier(0);
    CT fnv[MODE == 0 && !INC ? NS : 1];
    if constexpr (MODE == 0 && !INC) {
      const ST* fn = (const ST*)A.fn + eoff;
#pragma unroll
      for (int q = 0; q < NS; ++q) fnv[q] = (CT)__builtin_nontemporal_load(&fn[q * kVB]);
    }
    if (s + 1 < n) load_element(e + dx);
    __builtin_amdgcn_sched_barrier(0);
    CT o[NS];
#pragma unroll
    for (int q = 0; q < NS; ++q) {
      if constexpr (MODE != 0) o[q] = acc[q];
      else if constexpr (INC) o[q] = ca * fb[q] + acc[q];
      else o[q] = ca * fnv[q] + acc[q];
    }
    const DevOpsT<CT>& OP = ops_of<CT>(A);
    if (A.limiter) {
      CT fmin = o[0];
#pragma unroll
      for (int q = 0; q < NS; ++q) fmin = o[q] < fmin ? o[q] : fmin;
      const CT mean = tensor_wsum<DIM, N1>(o, OP.w) / OP.Wsum;
      const bool hit = valid && (fmin < (CT)0);
      if (hit && mean != fmin) {
        CT beta = fabs(mean / (mean - fmin));
        beta = beta > (CT)1 ? (CT)1 : beta;
#pragma unroll
        for (int q = 0; q < NS; ++q) o[q] = mean + beta * (o[q] - mean);
      }
      hits += __popcll(__ballot(hit));
      bad += __popcll(__ballot(hit && !(mean > (CT)0)));
    }
    if (INC && !A.out_full) {
      if constexpr (INC) {
        uint32_t* ow = inc_pairs((uint16_t*)A.out, eoff);
        float omin = INFINITY, smin = INFINITY;  // stage values / stored values
        uint32_t wd[NS / 2];
#pragma unroll
        for (int q = 0; q + 1 < NS; q += 2) {
          float s0, s1;
          wd[q >> 1] = bf16_increment2(o[q], o[q + 1], fb[q], fb[q + 1], s0, s1);
          omin = fminf(omin, fminf(o[q], o[q + 1]));
          smin = fminf(smin, fminf(s0, s1));
          o[q] = s0;
          o[q + 1] = s1;
        }
        uint16_t last = 0;
        if constexpr (NS % 2 != 0) {
          float stored;
          last = bf16_increment(o[NS - 1], fb[NS - 1], stored);
          omin = fminf(omin, o[NS - 1]);
          smin = fminf(smin, stored);
          o[NS - 1] = stored;
        }
        if (valid) {
#pragma unroll
          for (int m = 0; m < NS / 2; ++m) __builtin_nontemporal_store(wd[m], &ow[m * kVB]);
          if constexpr (NS % 2 != 0)
            __builtin_nontemporal_store(last, (uint16_t*)A.out + eoff + (NS - 1) * kVB);
        }
        const unsigned long long nviol = __popcll(__ballot(valid && smin < 0.0f && !(omin < 0.0f)));
        if (lane == 0 && nviol) atomicAdd(&A.diag[5], nviol);
      }
    } else if (valid) {
      ST* oe = (ST*)A.out + eoff;
#pragma unroll
      for (int q = 0; q < NS; ++q) __builtin_nontemporal_store((ST)o[q], &oe[q * kVB]);
    }
    // moment partials of what was stored (the previous element's sums were
    // read before the relaxation's barrier; without collisions before this one)
    if (!collide) lds_barrier();
    element_tiles<0, NS, ST, CT>(o, gw, ps, redw, tid);
    lds_barrier();
    for (int t = tid; t < 5 * NS; t += kBlock) {
      double sum = red[t];
#pragma unroll
      for (int w = 1; w < kBlock / 64; ++w) sum += red[w * part_rows<NS>() * 5 + t];
      A.partials[((int64_t)chunk * A.g.nx + e * NS) * 5 + t] = sum;
    }
  }
  __shared__ LimiterCounts lim;
  if (args().limiter) {
    limiter_count(lim, hits, bad, tid);
    lds_barrier();
    limiter_add(lim, args().diag, tid);
  }
  if (tid == 0 && count) atomicAdd(&args().diag[4], 1ull);
}

template <int DIM, int P, typename ST, int MODE, bool INC = false>
__global__ void __launch_bounds__(kBlock)
    __attribute__((amdgpu_waves_per_eu(xwalk_waves<DIM, P, ST, INC>())))
    k_stage_xwalk(const StageArgs A) {
  const DevGeom& g = A.g;
  const int len = A.walk_tx, nx = g.nelem[0];
  const int nr = (nx + len - 1) / len, rows = DIM == 3 ? g.nelem[1] * g.nelem[2] : g.nelem[1];
  const int64_t per_chunk = (int64_t)nr * rows;
  const int64_t w = xcd_chunk_remap(blockIdx.x, gridDim.x, per_chunk, A.xcd_part);
  const int chunk = (int)(w / per_chunk);
  const int r = (int)(w - chunk * per_chunk);
  const int seg = r / rows, row = r - seg * rows;  // neighbouring rows in flight together
  const int ez = DIM == 3 ? row / g.nelem[1] : 0, ey = DIM == 3 ? row - ez * g.nelem[1] : row;
  xwalk<DIM, P, ST, MODE, INC>((table_ptr<StageArgs>)__builtin_amdgcn_kernarg_segment_ptr(), chunk,
                               ey, ez, seg * len, min(seg * len + len, nx), w == 0);
}

}  // namespace bgk
