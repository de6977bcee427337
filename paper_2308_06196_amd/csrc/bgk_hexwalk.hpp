// bgk_hexwalk.hpp -- RK stage of p = 3 hexahedra whose element does not fit
// one lane's registers (FP64 storage, BF16 increments) on gfx950 (Dzanic &
// Martinelli, arXiv 2308.06196, Sec. 2.1).
#pragma once

#include "bgk_device3d.hpp"

namespace bgk {

// Sum and minimum over the four 16-lane rows of a wave (lanes v, 16 + v,
// 32 + v, 48 + v): v_permlane16_swap of a value with itself leaves the even
// and the odd rows' values in two registers, v_permlane32_swap the lower and
// the upper halves'. Every lane ends with the same bits.
__device__ __forceinline__ void rows_split16(uint32_t x, uint32_t& even, uint32_t& odd) {
  const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  even = r[0], odd = r[1];
}
__device__ __forceinline__ void rows_split32(uint32_t x, uint32_t& lo, uint32_t& hi) {
  const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  lo = r[0], hi = r[1];
}
template <bool HALVES>
__device__ __forceinline__ void rows_split(float x, float& a, float& b) {
  uint32_t p, q;
  if constexpr (HALVES) rows_split32(__float_as_uint(x), p, q);
  else rows_split16(__float_as_uint(x), p, q);
  a = __uint_as_float(p), b = __uint_as_float(q);
}
template <bool HALVES>
__device__ __forceinline__ void rows_split(double x, double& a, double& b) {
  uint32_t p0, q0, p1, q1;
  const uint32_t l = (uint32_t)__double2loint(x), h = (uint32_t)__double2hiint(x);
  if constexpr (HALVES) {
    rows_split32(l, p0, q0);
    rows_split32(h, p1, q1);
  } else {
    rows_split16(l, p0, q0);
    rows_split16(h, p1, q1);
  }
  a = __hiloint2double((int)p1, (int)p0), b = __hiloint2double((int)q1, (int)q0);
}
template <typename T>
__device__ __forceinline__ T rows_allsum(T x) {
  T a, b;
  rows_split<false>(x, a, b);
  x = a + b;
  rows_split<true>(x, a, b);
  return a + b;
}
template <typename T>
__device__ __forceinline__ T rows_allmin(T x) {
  T a, b;
  rows_split<false>(x, a, b);
  x = b < a ? b : a;
  rows_split<true>(x, a, b);
  return b < a ? b : a;
}

// Thread mapping. A wave holds 16 velocities of one element: lane 16 a_z + v
// owns the z-plane a_z (16 nodes) of velocity v, so that every load or store
// of a wave covers whole 64 (FP32) or 128 (FP64) byte runs of four node rows
// (with the planes of one velocity in adjacent lanes, as before, each quarter
// of a wave touched four cache lines). A work-group of four waves holds the
// 64 velocities of one velocity block. x and y lines are lane-local; the z
// contraction runs over the lane rows and is one matrix product per node of
// the plane: lane row = K index and result row of v_mfma_f64_4x4x4_4b (blocks
// of four velocities) and of v_mfma_f32_16x16x4 (operator row i at matrix row
// 4 i, so that lane row i receives it in the first result register).
//
// Walk. The work-group visits a tile of tx x ty elements of one z-layer row
// by row, in the upwind directions of its velocity chunk, and hands on the
// outflow traces: along x in registers (four lines per lane), along y in LDS
// (four lines per lane and element of the row). Lanes whose sign differs from
// the chunk's, and all lanes at the tile's entry faces, form the trace from
// the neighbour's nodes by the same sum, so results do not depend on the tile.
// Only the z-neighbour's nodes are read for every element. Walking at fixed z
// keeps every per-velocity quantity (operators, z-neighbour offset, row
// positions) constant over the tile. The next element's own and z-neighbour
// nodes are loaded as soon as the relaxation has consumed the current ones,
// so that their latency is covered by the limiter, the stores and the moments.
//
// Measured on the 16^3-element Taylor-Green box with 16^3 velocities (1.07e9
// values), ms per stage launch averaged over a step, against the per-element
// kernel this replaces (planes of one velocity in adjacent lanes, all three
// neighbours' nodes read, five dependent load batches): FP64 5.06 against 9.77
// (4.5 TB/s of compulsory traffic; stages 2-3 move 33.5 GB, the z-neighbours
// that miss L2 among them, at 6.4 TB/s: bound by HBM); BF16 increments 3.47-3.65
// by box against 5.27 (19.6 and 22.8 GB in stages 2 and 3; vector issue 40 % busy).
// Waves per SIMD: two in FP64 (237 registers; three spill and take 10.6 ms),
// three with increments (two 3.64 ms, four 5.06 ms).
struct HexWalk {
  static constexpr int N1 = 4, P2 = 16, NS = 64, VB = 64;
  static constexpr int RS = 18;                    // row stride of the staged values
  static constexpr int kRed = NS * 5;              // doubles of one wave's moment sums
  static constexpr int kWaveBytes = kRed * 8;      // per wave: staged rows, then its sums
  static constexpr int kPsBytes = 16 * 5 * 8;      // per wave: weighted moment functions
  // dynamic LDS: rows | staging and sums | moment functions | y traces. Rows are
  // kept column by column, so that a lane's factors of successive nodes are
  // contiguous (immediate offsets from one address per factor); the column
  // stride puts the columns that the lanes of a wave read on different banks.
  static constexpr int CS = NS + 2;
  static constexpr int rows_bytes(int ncols) { return CS * ncols * 8; }
  template <typename ST>
  static constexpr int lds_bytes(int ncols, int tx) {
    return rows_bytes(ncols) + 4 * (kWaveBytes + kPsBytes) + tx * 4 * kBlock * (int)sizeof(ST);
  }
};

// z contraction of one node of the plane: c + Op applied over the lane rows.
__device__ __forceinline__ double rows_mfma(double op, double x, double c) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(op, x, c, 0, 0, 0);
}
__device__ __forceinline__ mfma_f4 rows_mfma(float op, float x, mfma_f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(op, x, c, 0, 0, 0);
}

template <typename ST, int MODE, bool INC>
__device__ __forceinline__ void hex_walk(table_ptr<StageArgs> ap, const int chunk, const int ez,
                                         const int x0, const int x1, const int y0, const int y1,
                                         const bool count) {
  using CT = typename Compute<ST>::T;
  using H = HexWalk;
  constexpr int N1 = H::N1, P2 = H::P2, NS = H::NS;
  constexpr bool kF32 = sizeof(CT) == 4;
  constexpr bool kDin = INC && MODE == 0;
  static_assert(MODE == 0 || MODE == 3, "RK stages");
  extern __shared__ __align__(16) unsigned char dyn_lds[];

  // arguments, read again (scalar loads) where they are used instead of being
  // held across the walk: ap is opaque to the compiler for every element
  auto args = [&]() -> const StageArgs& { return table_entry(ap, 0); };
  const StageArgs& A0 = args();
  const DevGeom& g = A0.g;
  const int tid = (int)threadIdx.x, lane = tid & 63, wave = sreg(tid >> 6);
  const int az = lane >> 4, v = lane & 15;
  const int nv = (int)g.nv;
  const int j = chunk * H::VB + wave * 16 + v;
  const bool valid = j < nv;
  const int jj = valid ? j : nv - 1;
  Vel vel = velocity_of<false>(g, jj);
  if (!valid) vel.w = 0.0;

  const RowPick rp = row_pick(A0, chunk, NS);
  double* tab = reinterpret_cast<double*>(dyn_lds);
  unsigned char* lw = dyn_lds + H::rows_bytes(rp.ncols);
  ST* gw = reinterpret_cast<ST*>(lw + wave * H::kWaveBytes);
  const double* red = reinterpret_cast<const double*>(lw);  // wave w's sums at w * kRed
  double* redw = reinterpret_cast<double*>(lw + wave * H::kWaveBytes);
  double* ps = reinterpret_cast<double*>(lw + 4 * H::kWaveBytes + wave * H::kPsBytes);
  CT* try_ = reinterpret_cast<CT*>(lw + 4 * (H::kWaveBytes + H::kPsBytes));

  __shared__ LineOps line_ops[kF32 ? 4 : 1];  // per wave
  LineOps* lops = &line_ops[kF32 ? wave : 0];
  if constexpr (kF32) line_ops_store(*lops, A0.lops, tid);

  // moment functions of the wave's velocities, constant over the walk
  if (az == 0) {
    ps[v * 5 + 0] = vel.w;
    ps[v * 5 + 1] = vel.w * vel.u[0];
    ps[v * 5 + 2] = vel.w * vel.u[1];
    ps[v * 5 + 3] = vel.w * vel.u[2];
    ps[v * 5 + 4] =
        vel.w * (0.5 * (vel.u[0] * vel.u[0] + vel.u[1] * vel.u[1] + vel.u[2] * vel.u[2]));
  }

  bool up[2], pos[3];
  {
    int b0[3];
    slot_nodes<false>(g, chunk * H::VB < nv ? chunk * H::VB : nv - 1, b0);
#pragma unroll
    for (int k = 0; k < 2; ++k) up[k] = (g.vlo[k] + b0[k] * g.du[k]) * g.scale[k] > 0.0;
  }
  CT a[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    pos[k] = vel.u[k] * g.scale[k] > 0.0;
    a[k] = (CT)(vel.u[k] * g.scale[k]);
  }
  const int64_t estride = g.nvb * (int64_t)(NS * kVB);  // values per element
  const ST* __restrict__ fin = (const ST*)A0.fin;
  const uint16_t* __restrict__ din = A0.din;
  const bool collide = A0.collide;
  // offset of this lane's plane inside an element, at velocity slot js
  auto lane_off = [&](int js) -> int64_t {
    return ((int64_t)(js / kVB) * NS + az * P2) * kVB + js % kVB;
  };
  const int64_t own_off = lane_off(jj);

  // upwind source of axis k for the element e with coordinate c on it: offset
  // of its planes, and whether the source's right trace is taken
  auto source = [&](int k, int c, int64_t e, bool& right) -> int64_t {
    const DevGeom& g = args().g;
    const int nk = g.nelem[k];
    const int64_t st = k == 0 ? 1 : k == 1 ? (int64_t)g.nelem[0] : (int64_t)g.nelem[0] * g.nelem[1];
    const bool edge = pos[k] ? c == 0 : c == nk - 1;
    const bool wall = edge && (pos[k] ? g.bc[k][0] : g.bc[k][1]) != 0;
    right = pos[k] != wall;
    if (wall) {  // the own element at the mirrored velocity
      int bm[3];
      slot_nodes<false>(g, jj, bm);
      bm[k] = g.nv1[k] - 1 - bm[k];
      return e * estride + lane_off(vel_slot(g, bm));
    }
    const int d = (pos[k] ? -1 : 1) + (edge ? (pos[k] ? nk : -nk) : 0);
    return (e + d * st) * estride + own_off;
  };

  // z operators of this lane: Dp = D - G_in lam_own^T on the own planes, E =
  // G_in lam_ext^T on the upwind neighbour's (or the mirrored own planes at a
  // specular wall). One pass with the lane's own sign where the velocities
  // sharing an operator agree (four in FP64, the wave's 16 in FP32), else one
  // pass per sign, each applied to its lanes only.
  bool right_z;
  const int64_t zoff = source(2, ez, 0, right_z);  // relative to the element
  const bool uni_z = kF32 ? (__ballot(pos[2]) == 0 || __ballot(!pos[2]) == 0) : quads_agree(pos[2]);
  auto z_ops = [&](bool sg, CT& dp, CT& ev) {
    const DevOpsT<CT>& OP = ops_of<CT>(args());
    const DevGeom& g = args().g;
    const bool wall = sg ? ez == 0 && g.bc[2][0] != 0 : ez == g.nelem[2] - 1 && g.bc[2][1] != 0;
    const int i = kF32 ? v >> 2 : v & 3;
    const bool row = !kF32 || (v & 3) == 0;
    CT d = (CT)0, l = (CT)0, r = (CT)0, gi = (CT)0;
#pragma unroll
    for (int b = 0; b < N1; ++b) {
      if (b == az) l = OP.lamL[b], r = OP.lamR[b];
      if (b == i) gi = sg ? OP.GL[b] : OP.GR[b];
#pragma unroll
      for (int c = 0; c < N1; ++c)
        if (b == i && c == az) d = OP.D[b][c];
    }
    dp = row ? d - gi * (sg ? l : r) : (CT)0;
    ev = row ? gi * ((sg != wall) ? r : l) : (CT)0;
  };
  CT zdp, zev;
  z_ops(pos[2], zdp, zev);

  // this lane's factor columns (first node of its plane)
  int cx = (vel.b[0] - rp.x0) * H::CS + az * P2, cy = (rp.nx + vel.b[1] - rp.y0) * H::CS + az * P2,
      cz = (rp.nxy + vel.b[2] - rp.z0) * H::CS + az * P2;

  auto load_planes16 = [&](CT(&x)[P2], int64_t off) {
#pragma unroll
    for (int q = 0; q < P2; ++q) x[q] = (CT)fin[off + q * kVB];
  };

  const int nxt = x1 - x0, nyt = y1 - y0;
  // the walk: element coordinates of position (ix, iy) of the tile
  const int dx = up[0] ? 1 : -1, dy = up[1] ? 1 : -1;
  const int ex0 = up[0] ? x0 : x1 - 1, ey0 = up[1] ? y0 : y1 - 1;
  const int64_t ezb = (int64_t)g.nelem[1] * ez;

  CT f[P2], nb[P2], trx[N1];
  constexpr int NW = kDin ? P2 / 2 : 1;
  uint32_t fd[NW], nd[NW];
  constexpr int kU = 5;  // covers 64 x 20 entries (64 velocities of an 8 x 8 x 1 octant slab: 18)
  double tv[kU];
  // row entry t: its offset in the element's rows and its LDS index; those of
  // the first batch are kept for the walk (14 bits each: at most 128 columns)
  auto row_index = [&](int t) -> int {
    const int n = (int)__umulhi((unsigned)t, rp.magic);
    return (t - n * rp.ncols) * H::CS + n;
  };
  int rowt[kU];
#pragma unroll
  for (int u = 0; u < kU; ++u) {
    const int t = min(u * kBlock + tid, rp.count - 1);
    rowt[u] = rp.offset(t) | row_index(t) << 16;
  }
  const int row_doubles = NS * rp.S;
  auto load_rows = [&](int64_t e) {
    if (!collide) return;
    const double* et = args().etab + e * row_doubles;
#pragma unroll
    for (int u = 0; u < kU; ++u) tv[u] = et[rowt[u] & 0xFFFF];
  };
  auto load_element = [&](int64_t e) {
    const int64_t o = e * estride + own_off, z = e * estride + zoff;
    load_planes16(f, o);
    if constexpr (kDin) {
#pragma unroll
      for (int m = 0; m < NW; ++m) fd[m] = inc_pairs(din, o)[m * kVB];
    }
    load_planes16(nb, z);
    if constexpr (kDin) {
#pragma unroll
      for (int m = 0; m < NW; ++m) nd[m] = inc_pairs(din, z)[m * kVB];
    }
  };
  int64_t e = ex0 + (int64_t)g.nelem[0] * (ey0 + ezb);
  load_rows(e);
  load_element(e);
#pragma unroll
  for (int l = 0; l < N1; ++l) trx[l] = (CT)0;

  int hits = 0, bad = 0;  // limiter counters of the wave over the walk
  for (int ix = 0, iy = 0; iy < nyt;) {
    asm volatile("" : "+s"(ap));
    const int64_t eoff = e * estride + own_off;
    // rows of this element -> LDS (every wave has passed the previous
    // element's second barrier, and with it its last read of the rows)
    if (collide) {
      // (entries past the count repeat the last one)
#pragma unroll
      for (int u = 0; u < kU; ++u) tab[rowt[u] >> 16] = tv[u];
      for (int t = kU * kBlock + tid; t < rp.count; t += kBlock)
        tab[row_index(t)] = args().etab[e * row_doubles + rp.offset(t)];
    }
    CT fb[INC ? P2 : 1];  // the FP32 state F that increments are taken against
    if constexpr (INC) {
#pragma unroll
      for (int q = 0; q < P2; ++q) fb[q] = f[q];
    }
    if constexpr (kDin) {
#pragma unroll
      for (int m = 0; m < NW; ++m) {
        f[2 * m] += bf16_lo(fd[m]);
        f[2 * m + 1] += bf16_hi(fd[m]);
        nb[2 * m] += bf16_lo(nd[m]);
        nb[2 * m + 1] += bf16_hi(nd[m]);
      }
    }
    CT acc[P2];
    // z: over the lane rows, on the matrix cores
#pragma unroll
    for (int q = 0; q < P2; ++q) {
      if constexpr (kF32) {
        mfma_f4 c = {0.0f, 0.0f, 0.0f, 0.0f};
        c = rows_mfma(zdp, f[q], c);
        c = rows_mfma(zev, nb[q], c);
        acc[q] = a[2] * c[0];
      } else {
        acc[q] = a[2] * rows_mfma(zev, nb[q], rows_mfma(zdp, f[q], 0.0));
      }
    }
    if (!uni_z) {
      // lanes of the other sign than their operator group's: once per sign
#pragma unroll 1
      for (int sg = 0; sg < 2; ++sg) {
        CT dp, ev;
        z_ops(sg != 0, dp, ev);
        const bool mine = (pos[2] ? 1 : 0) == sg;
#pragma unroll
        for (int q = 0; q < P2; ++q) {
          if constexpr (kF32) {
            mfma_f4 c = {0.0f, 0.0f, 0.0f, 0.0f};
            c = rows_mfma(dp, f[q], c);
            c = rows_mfma(ev, nb[q], c);
            acc[q] = mine ? a[2] * c[0] : acc[q];
          } else {
            const CT c = rows_mfma(ev, nb[q], rows_mfma(dp, f[q], 0.0));
            acc[q] = mine ? a[2] * c : acc[q];
          }
        }
      }
    }
    // x, then y: lines inside the plane
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      asm volatile("" : "+s"(ap));
      const DevOpsT<CT>& OP = ops_of<CT>(args());
      const int S1 = k == 0 ? 1 : N1, SL = k == 0 ? N1 : 1;  // stride in and between lines
      const bool carried = k == 0 ? ix > 0 : iy > 0;
      const bool lane_carry = carried && pos[k] == up[k];
      CT ext[N1];
      if (k == 0) {
#pragma unroll
        for (int l = 0; l < N1; ++l) ext[l] = trx[l];
      } else {
#pragma unroll
        for (int l = 0; l < N1; ++l) ext[l] = try_[(ix * N1 + l) * kBlock + tid];
      }
      const bool read_nb = __ballot(!lane_carry) != 0;
      if (read_nb) {  // lanes without a carried trace read the neighbour's nodes
        bool right;
        const int64_t so = source(k, k == 0 ? ex0 + dx * ix : ey0 + dy * iy, e, right);
        CT x[P2];
        load_planes16(x, so);
        if constexpr (kDin) {
#pragma unroll
          for (int m = 0; m < NW; ++m) {
            const uint32_t w = inc_pairs(din, so)[m * kVB];
            x[2 * m] += bf16_lo(w);
            x[2 * m + 1] += bf16_hi(w);
          }
        }
#pragma unroll
        for (int l = 0; l < N1; ++l) {
          CT tl = (CT)0, tr = (CT)0;
#pragma unroll
          for (int b = 0; b < N1; ++b) {
            tl += OP.lamL[b] * x[l * SL + b * S1];
            tr += OP.lamR[b] * x[l * SL + b * S1];
          }
          ext[l] = lane_carry ? ext[l] : right ? tr : tl;
        }
      }
      if constexpr (kF32) {
        // lines on the matrix cores (line_mfma_own, and G_in times the exterior
        // trace): with each lane's own operators where every four velocities
        // share the sign of u_k, otherwise once per sign
        const bool uni = quads_agree(pos[k]);
#pragma unroll 1
        for (int p = 0; p < (uni ? 1 : 2); ++p) {
          const int sg = uni ? (pos[k] ? 1 : 0) : p;
          const CT as = (pos[k] ? 1 : 0) == sg ? a[k] : (CT)0;
          const float4 d4 = *reinterpret_cast<const float4*>(&lops->Dp[sg][tid & 3][0]);
          const float dp[4] = {d4.x, d4.y, d4.z, d4.w}, gin = lops->G[sg][tid & 3];
#pragma unroll
          for (int l = 0; l < N1; ++l) {
            float fl[N1];
#pragma unroll
            for (int b = 0; b < N1; ++b) fl[b] = f[l * SL + b * S1];
            mfma_f4 c = line_mfma_own<N1>(dp, fl);
            c = __builtin_amdgcn_mfma_f32_4x4x1f32(gin, ext[l], c, 0, 0, 0);
#pragma unroll
            for (int i = 0; i < N1; ++i)
              acc[l * SL + i * S1] = fmaf(as, c[i], acc[l * SL + i * S1]);
          }
        }
      } else {
        // once per sign of u_k among the wave's lanes (one, unless the velocity
        // octants change inside it): the operators are then uniform
        const int s_lo = __ballot(!pos[k]) == 0 ? 1 : 0, s_hi = __ballot(pos[k]) == 0 ? 0 : 1;
#pragma unroll 1
        for (int sg = s_lo; sg <= s_hi; ++sg) {
          const CT as = (pos[k] ? 1 : 0) == sg ? a[k] : (CT)0;
          CT lin[N1], gin[N1];
#pragma unroll
          for (int b = 0; b < N1; ++b) {
            lin[b] = sg ? OP.lamL[b] : OP.lamR[b];
            gin[b] = sg ? OP.GL[b] : OP.GR[b];
          }
#pragma unroll
          for (int l = 0; l < N1; ++l) {
            CT line[N1];  // a f
#pragma unroll
            for (int b = 0; b < N1; ++b) line[b] = as * f[l * SL + b * S1];
            CT jump = as * ext[l];
#pragma unroll
            for (int b = 0; b < N1; ++b) jump -= lin[b] * line[b];
#pragma unroll
            for (int i = 0; i < N1; ++i) {
              CT d = acc[l * SL + i * S1] + gin[i] * jump;
#pragma unroll
              for (int b = 0; b < N1; ++b) d += OP.D[i][b] * line[b];
              acc[l * SL + i * S1] = d;
            }
          }
        }
      }
      // outflow traces: the next element's exterior traces
#pragma unroll
      for (int l = 0; l < N1; ++l) {
        CT t = (CT)0;
#pragma unroll
        for (int b = 0; b < N1; ++b) t += (up[k] ? OP.lamR[b] : OP.lamL[b]) * f[l * SL + b * S1];
        if (k == 0) trx[l] = t;
        else try_[(ix * N1 + l) * kBlock + tid] = t;
      }
    }
    asm volatile("" : "+s"(ap));
    const StageArgs& A = args();
    const CT dt = (CT)A.dt, ca = (CT)A.a, cb = (CT)A.b;
    const double wc = A.b * A.dt;
    // f^n: a stream no other work-group reads (MODE 0)
    CT fnv[MODE == 0 && !INC ? P2 : 1];
    if constexpr (MODE == 0 && !INC) {
      const ST* fn = (const ST*)A.fn + eoff;
#pragma unroll
      for (int q = 0; q < P2; ++q) fnv[q] = (CT)__builtin_nontemporal_load(&fn[q * kVB]);
    }
    // relaxation folded with the transport: h = b (f - dt T) + b dt C, C in FP64
    if (collide) {
      lds_barrier();
      asm volatile("" : "+v"(cx), "+v"(cy), "+v"(cz));
      const double *tx_ = tab + cx, *ty_ = tab + cy, *tz_ = tab + cz,
                   *tt_ = tab + (rp.ncols - 1) * H::CS + az * P2;
#pragma unroll
      for (int q = 0; q < P2; ++q) {
        const double c = collision_term(tx_[q], ty_[q], tz_[q], tt_[q], (double)f[q]);
        acc[q] = (CT)fma(wc, c, (double)(cb * (f[q] - dt * acc[q])));
      }
    } else {
#pragma unroll
      for (int q = 0; q < P2; ++q) acc[q] = cb * (f[q] - dt * acc[q]);
    }
    // the next element's loads, covered by the rest of this one
    int jx = ix + 1, jy = iy;
    if (jx == nxt) jx = 0, ++jy;
    const int64_t e_next =
        jy < nyt ? ex0 + dx * jx + (int64_t)A.g.nelem[0] * (ey0 + dy * jy + ezb) : e;
    __builtin_amdgcn_sched_barrier(0);
    load_rows(e_next);
    load_element(e_next);
    __builtin_amdgcn_sched_barrier(0);

    CT o[P2];
#pragma unroll
    for (int q = 0; q < P2; ++q) {
      if constexpr (MODE != 0) o[q] = acc[q];
      else if constexpr (INC) o[q] = ca * fb[q] + acc[q];
      else o[q] = ca * fnv[q] + acc[q];
    }
    const DevOpsT<CT>& OP = ops_of<CT>(A);
    if (A.limiter) {
      CT wz = (CT)0;
#pragma unroll
      for (int b = 0; b < N1; ++b) wz = b == az ? OP.w[b] : wz;
      CT fmin = o[0];
#pragma unroll
      for (int q = 0; q < P2; ++q) fmin = o[q] < fmin ? o[q] : fmin;
      const CT mean = rows_allsum(wz * tensor_wsum<2, N1>(o, OP.w)) / OP.Wsum;
      fmin = rows_allmin(fmin);
      const bool hit = valid && (fmin < (CT)0);
      if (hit && mean != fmin) {
        CT beta = fabs(mean / (mean - fmin));
        beta = beta > (CT)1 ? (CT)1 : beta;
#pragma unroll
        for (int q = 0; q < P2; ++q) o[q] = mean + beta * (o[q] - mean);
      }
      hits += __popcll(__ballot(hit && az == 0));
      bad += __popcll(__ballot(hit && az == 0 && !(mean > (CT)0)));
    }
    if (INC && !A.out_full) {
      if constexpr (INC) {
        // the increment o - F in BF16, and the stored state F + increment for
        // the moments
        uint32_t* ow = inc_pairs((uint16_t*)A.out, eoff);
        float omin = INFINITY, smin = INFINITY;  // stage values / stored values
        uint32_t w[P2 / 2];
#pragma unroll
        for (int q = 0; q < P2; q += 2) {
          float s0, s1;
          w[q >> 1] = bf16_increment2(o[q], o[q + 1], fb[q], fb[q + 1], s0, s1);
          omin = fminf(omin, fminf(o[q], o[q + 1]));
          smin = fminf(smin, fminf(s0, s1));
          o[q] = s0;
          o[q + 1] = s1;
        }
        if (valid) {
#pragma unroll
          for (int m = 0; m < P2 / 2; ++m) __builtin_nontemporal_store(w[m], &ow[m * kVB]);
        }
        // (velocity, plane) pairs whose stored stage is negative where the
        // stage itself is not
        const unsigned long long nviol = __popcll(__ballot(valid && smin < 0.0f && !(omin < 0.0f)));
        if (lane == 0 && nviol) atomicAdd(&A.diag[5], nviol);
      }
    } else if (valid) {
      ST* oe = (ST*)A.out + eoff;
#pragma unroll
      for (int q = 0; q < P2; ++q) __builtin_nontemporal_store((ST)o[q], &oe[q * kVB]);
    }
    // moment partials of what was stored (wave_moments_4x4's scheme): four
    // tiles of 16 rows, row 4 a_z + q % 4 of tile q / 4, the wave's 16
    // velocities in four K steps
    {
      const int k4 = lane >> 4, blk = (lane >> 2) & 3, jm = lane & 3, ra = lane & 15;
      double b0[4], b1[4], d0[4], d1[4];
#pragma unroll
      for (int st = 0; st < 4; ++st) {
        b0[st] = ps[(4 * st + k4) * 5 + jm];
        b1[st] = jm == 0 ? ps[(4 * st + k4) * 5 + 4] : 0.0;
      }
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        d0[t] = d1[t] = 0.0;
        // the lanes of a wave read what the others wrote; the previous
        // element's sums (the same LDS) were read before this element's
        // first barrier, without collisions before the one below
        if (t == 0 && !collide) lds_barrier();
#pragma unroll
        for (int i = 0; i < 4; ++i) gw[(az * 4 + i) * H::RS + v] = (ST)o[4 * t + i];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
        double av[4];
#pragma unroll
        for (int st = 0; st < 4; ++st) av[st] = (double)gw[ra * H::RS + 4 * st + k4];
#pragma unroll
        for (int st = 0; st < 4; ++st) {
          d0[t] = __builtin_amdgcn_mfma_f64_4x4x4f64(av[st], b0[st], d0[t], 0, 0, 0);
          d1[t] = __builtin_amdgcn_mfma_f64_4x4x4f64(av[st], b1[st], d1[t], 0, 0, 0);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
      }
      // result row 4 blk + k4 of tile t: plane blk, node 4 t + k4 of the plane
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        double* r = redw + (blk * P2 + 4 * t + k4) * 5;
        r[jm] = d0[t];
        if (jm == 0) r[4] = d1[t];
      }
    }
    lds_barrier();
    const int64_t node0 = e * NS;
    for (int t = tid; t < H::kRed; t += kBlock) {
      double sum = red[t];
#pragma unroll
      for (int w = 1; w < 4; ++w) sum += red[w * H::kRed + t];
      A.partials[((int64_t)chunk * A.g.nx + node0) * 5 + t] = sum;
    }
    e = e_next;
    ix = jx;
    iy = jy;
  }
  if (lane == 0) {
    if (hits) atomicAdd(&args().diag[2], (unsigned long long)hits);
    if (bad) atomicAdd(&args().diag[3], (unsigned long long)bad);
  }
  if (tid == 0 && count) atomicAdd(&args().diag[4], 1ull);
}

template <typename ST, int MODE, bool INC>
__global__ void __launch_bounds__(kBlock)
    __attribute__((amdgpu_waves_per_eu(sizeof(ST) == 8 ? 2 : 3)))
    k_stage_walk(const StageArgs A) {
  const DevGeom& g = A.g;
  const int tx = A.walk_tx, ty = A.walk_ty;
  const int ntx = (g.nelem[0] + tx - 1) / tx, nty = (g.nelem[1] + ty - 1) / ty, nz = g.nelem[2];
  const int64_t per_chunk = (int64_t)ntx * nty * nz;
  const int64_t w = xcd_chunk_remap(blockIdx.x, gridDim.x, per_chunk, A.xcd_part);
  const int chunk = (int)(w / per_chunk);
  const int r = (int)(w - chunk * per_chunk);
  const int t = r / nz, ez = r - t * nz;  // z fastest: neighbouring layers in flight together
  const int iy = t / ntx, ix = t - iy * ntx;
  const int x0 = ix * tx, y0 = iy * ty;
  hex_walk<ST, MODE, INC>((table_ptr<StageArgs>)__builtin_amdgcn_kernarg_segment_ptr(), chunk, ez, x0, min(x0 + tx, g.nelem[0]), y0,
                          min(y0 + ty, g.nelem[1]), w == 0);
}

}  // namespace bgk
