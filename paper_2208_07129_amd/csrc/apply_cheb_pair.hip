// Fused Chebyshev filter step, Out = a D A (D Y) + b Y + c Xp, for axis-aligned
// cells in the register-resident form (pair_body.h): one wavefront per (segment
// of a line of cells along y, tile of 16 columns).
//
// The cell's D goes through LDS (one load per node instead of one per node and
// column).  Rows of several contributors get a D V by addition (Out holds b Y +
// c Xp there); the others are stored, and their Y and Xp are loaded into the
// registers that the contractions have left free before the next cell's values
// take them: the loads must not stand behind the additions, which they would
// wait for, so the stores come first, then the next cell's loads, then the
// additions.  Bound as the apply, plus the two more reads of the stored rows; a
// step with its initialisation at p = 6, 16^3 cells, 64 columns: 801 (box kernel)
// -> 557 us; p = 4, 24^3: 898 -> 677; p = 2, 32^3: 499 -> 323.
#include "pair_body.h"

#ifndef MF_P
#error "compile with -DMF_P=<degree>"
#endif

namespace mf {
namespace {

template <int NP, int NQ, bool HASX>
__global__ void __attribute__((amdgpu_flat_work_group_size(64, 64),
                               amdgpu_waves_per_eu(pair_waves(NQ), pair_waves(NQ))))
apply_cheb_pair_kernel(const GridDesc grid, const double* __restrict__ geo,
                       const double* __restrict__ vq, const double* __restrict__ Y, double* Out,
                       uint32_t ld, int nvec, const PairPlan plan, uint32_t bytes,
                       const ChebArgs ca) {
  using PC = PairCell<NP, NQ>;
  constexpr int P = PC::P, HP = PC::HP, MP = PC::MP, HQ = PC::HQ, MQ = PC::MQ, NQ2 = PC::NQ2;
  constexpr int NPM = PC::NPM, NP3 = NP * NP * NP, ND = (NP3 + 63) / 64;
  __shared__ double2 pms[NQ2 * 4];
  __shared__ double sd[NP3];
  __shared__ double carry[2][NP][64];
  const int item = (int)xcd_item(blockIdx.x, plan.chunk);
  if (item >= plan.items) return;
  int it = item / plan.ntiles;
  const int v0 = (item - it * plan.ntiles) * kPairCols;
  const int cx = it % plan.nxg;
  it /= plan.nxg;
  const int seg = it % plan.nseg, cz = it / plan.nseg;
  const int cya = seg * plan.len, cyb = min(grid.n[1], cya + plan.len);
  const uint32_t plane = (uint32_t)(grid.N[0] * grid.N[1]), N0 = (uint32_t)grid.N[0];
  const BufF64 by(Y, bytes), bo(Out, bytes), bx(ca.Xp, HASX ? bytes : 0);
  const BufF64 bd(ca.D, plane * (uint32_t)grid.N[2] * 8u);
  const double g0 = geo[0], g1 = geo[3], g2 = geo[5];
  PC c;

  // Byte offsets of the lane's node (0, 0, z) of plane h and column, for the x
  // nodes 0, 1 .. P-1 (mid) and P (the wrapped node).
  struct Lane {
    uint32_t lo[2], mid[2], hi[2];
  };
  auto locate = [&](Lane& q, int l, bool on) {
    const int k = l >> 4, v = v0 + (l & (kPairCols - 1));
    const bool live = on && v < nvec;
    const int gx = cx * grid.p;
    const int gxp = gx + P == grid.N[0] ? 0 : gx + P;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      int gz = cz * grid.p + (h ? P - k : k);
      if (gz >= grid.N[2]) gz = 0;  // the wrapped layer (k past the pairs: not used)
      const bool ok = live && k < (h ? HP : HP + MP) &&
                      !(grid.dirichlet && (gz == 0 || gz == grid.N[2] - 1));
      const uint32_t zr = (uint32_t)gz * plane;
      q.mid[h] = ok ? ((zr + (uint32_t)gx) * ld + (uint32_t)v) * 8u : kOob;
      q.hi[h] = ok && !(grid.dirichlet && cx == grid.n[0] - 1)
                    ? ((zr + (uint32_t)gxp) * ld + (uint32_t)v) * 8u : kOob;
      q.lo[h] = grid.dirichlet && cx == 0 ? kOob : q.mid[h];
    }
  };
  double2 pq[NPM];
  double dq[ND];
  // D of local node idx = i + NP (j + NP k) of cell cy, 0 on constrained rows
  auto scaling = [&](int cy, int idx) {
    idx = min(idx, NP3 - 1);
    int gx = cx * grid.p + idx % NP, gy = cy * grid.p + idx / NP % NP;
    int gz = cz * grid.p + idx / (NP * NP);
    if (gx == grid.N[0]) gx = 0;
    if (gy == grid.N[1]) gy = 0;
    if (gz == grid.N[2]) gz = 0;
    const bool dead = grid.dirichlet && (gx == 0 || gx == grid.N[0] - 1 || gy == 0 ||
                                         gy == grid.N[1] - 1 || gz == 0 || gz == grid.N[2] - 1);
    return bd.load(dead ? kOob : ((uint32_t)gz * plane + (uint32_t)gy * N0 + (uint32_t)gx) * 8u, 0);
  };
  auto potential = [&](int cy, int idx) {  // the two potential values of (p, m) entry idx
    idx = min(idx, NQ2 * 4 - 1);
    const int xy = idx >> 2, kk = idx & 3, ka = kk < HQ + MQ ? kk : 0;
    const double* vs = vq + (int64_t)(cx + grid.n[0] * (cy + grid.n[1] * cz)) * (NQ2 * NQ);
    return make_double2(vs[xy + NQ2 * ka], vs[xy + NQ2 * (NQ - 1 - ka)]);
  };
  auto fetch = [&](int cy, bool on) {
    const int l = fresh_lane();
    Lane q;
    locate(q, l, on);
    uint32_t lb = ld * 8u;
    asm volatile("" : "+s"(lb));  // the node offsets are formed here, not once for the segment
    const bool ylo = grid.dirichlet && cy == 0, yhi = grid.dirichlet && cy == grid.n[1] - 1;
    const bool wrapy = cy * grid.p + P == grid.N[1];
    const uint32_t row0 = (uint32_t)(cy * grid.p) * N0 * lb;
#pragma unroll
    for (int j = 0; j < NP; ++j) {
      const bool dead = (j == 0 && ylo) || (j == P && yhi);
      const uint32_t row = j == P && wrapy ? 0u : row0 + (uint32_t)j * N0 * lb;
#pragma unroll
      for (int i = 0; i < NP; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          uint32_t v = i == 0 ? q.lo[h] : (i == P ? q.hi[h] : q.mid[h]);
          if (j == 0 || j == P) v = dead ? kOob : v;
          c.T[h][j][i] = by.load(v, i == P ? row : row + (uint32_t)i * lb);
        }
    }
#pragma unroll
    for (int r = 0; r < NPM; ++r) pq[r] = potential(cy, l + 64 * r);
#pragma unroll
    for (int r = 0; r < ND; ++r) dq[r] = scaling(cy, l + 64 * r);
  };

  fetch(cya, true);
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int i = 0; i < NP; ++i) carry[h][i][threadIdx.x] = 0.0;

  for (int cy = cya; cy < cyb; ++cy) {
    const bool first = cy == cya, last = cy + 1 == cyb;
    {
      const int l = fresh_lane();
      lds_handover();
#pragma unroll
      for (int r = 0; r < NPM; ++r)
        if (l + 64 * r < NQ2 * 4)
          pms[l + 64 * r] = make_double2(0.5 * (pq[r].x + pq[r].y), 0.5 * (pq[r].x - pq[r].y));
#pragma unroll
      for (int r = 0; r < ND; ++r)
        if (l + 64 * r < NP3) sd[l + 64 * r] = dq[r];
      lds_handover();
      const int k = l >> 4, kz = min(k, P);
      const double* d0 = sd + kz * (NP * NP);
      const double* d1 = sd + (P - kz) * (NP * NP);
#pragma unroll
      for (int j = 0; j < NP; ++j)
#pragma unroll
        for (int i = 0; i < NP; ++i) {
          c.T[0][j][i] *= d0[j * NP + i];
          c.T[1][j][i] *= d1[j * NP + i];
        }
      c.contract(&pms[k], g0, g1, g2);
    }
    const int l = fresh_lane();
    Lane q;
    locate(q, l, true);
    const bool zin = (l >> 4) > 0;  // nodes off the z faces: one contributor unless on an x face
    uint32_t vin[2], vfc[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      vin[h] = zin ? q.mid[h] : kOob;
      vfc[h] = zin ? kOob : q.mid[h];
    }
    uint32_t lb = ld * 8u;
    asm volatile("" : "+s"(lb));
    const bool ylo = grid.dirichlet && cy == 0, yhi = grid.dirichlet && cy == grid.n[1] - 1;
    const uint32_t row0 = (uint32_t)(cy * grid.p) * N0 * lb;
    auto row_of = [&](int j) { return row0 + (uint32_t)j * N0 * lb; };

    // Y and Xp of the stored rows j, RB rows at a time, one group ahead
    constexpr int RB = P >= 3 ? 2 : 1, NG = (P + RB - 1) / RB, NI = P > 1 ? P - 1 : 1;
    double ya[2][RB][NI][2], xa[2][RB][NI][2];
    auto rows_load = [&](int gr) {
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        const int j = gr * RB + r;
        if (j >= P) break;
        const bool off = j == 0 && first;
#pragma unroll
        for (int i = 1; i < P; ++i)
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const uint32_t v = off ? kOob : vin[h], s = row_of(j) + (uint32_t)i * lb;
            ya[gr & 1][r][i - 1][h] = by.load(v, s);
            if constexpr (HASX) xa[gr & 1][r][i - 1][h] = bx.load(v, s);
          }
      }
    };
    rows_load(0);
    stage_end();
#pragma unroll
    for (int j = 0; j < NP; ++j) {
      c.back_x(j);
      stage_end();
    }
    const double t0 = kPairTab<NP, NQ>.t[0][l], t1 = kPairTab<NP, NQ>.t[1][l];
    const int kz = min(l >> 4, P);
    const double* d0 = sd + kz * (NP * NP);
    const double* d1 = sd + (P - kz) * (NP * NP);
    // N^T along z and a D, in place
    auto back_z = [&](int j) {
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        const double e = mfma_z(t0, c.U[0][j][i], 0.0), o = mfma_z(t1, c.U[1][j][i], 0.0);
        c.U[0][j][i] = (e + o) * (ca.a * d0[j * NP + i]);
        c.U[1][j][i] = (e - o) * (ca.a * d1[j * NP + i]);
      }
    };
#pragma unroll
    for (int i = 0; i < NP; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        c.U[h][0][i] += carry[h][i][l];
        carry[h][i][l] = c.U[h][P][i];
      }
#pragma unroll
    for (int gr = 0; gr < NG; ++gr) {
      if (gr + 1 < NG) rows_load(gr + 1);
      stage_end();
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        const int j = gr * RB + r;
        if (j >= P) break;
        back_z(j);
        const bool off = j == 0 && first;
#pragma unroll
        for (int i = 1; i < P; ++i)
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            double o = fma(ca.b, ya[gr & 1][r][i - 1][h], c.U[h][j][i]);
            if constexpr (HASX) o = fma(ca.c, xa[gr & 1][r][i - 1][h], o);
            bo.store(o, off ? kOob : vin[h], row_of(j) + (uint32_t)i * lb);
          }
      }
      stage_end();
    }
    if (last) back_z(P);
    pin(c.U);
    stage_end();
    fetch(last ? cy : cy + 1, !last);  // the next cell's values, in flight during the additions
    stage_end();
#pragma unroll
    for (int j = 0; j < P; ++j) {
      const bool dead = j == 0 && ylo, part = j == 0 && first;
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        const uint32_t s = i == P ? row_of(j) : row_of(j) + (uint32_t)i * lb;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          uint32_t v = i == 0 ? q.lo[h] : i == P ? q.hi[h] : part ? q.mid[h] : vfc[h];
          if (j == 0) v = dead ? kOob : v;
          bo.add(c.U[h][j][i], v, s);
        }
      }
    }
    if (last) {
      const uint32_t row = cy * grid.p + P == grid.N[1] ? 0u : row_of(P);
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        const uint32_t s = i == P ? row : row + (uint32_t)i * lb;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const uint32_t v = i == 0 ? q.lo[h] : (i == P ? q.hi[h] : q.mid[h]);
          bo.add(c.U[h][P][i], yhi ? kOob : v, s);
        }
      }
    }
  }
}

template <int NP, int NQ>
hipError_t launch_pq(const Operator& op, const double* Y, double* Out, int64_t ld, int nvec,
                     const ChebArgs& ca, const PairPlan& plan, hipStream_t s) {
  if constexpr (NQ <= kPairMaxN) {
    const uint32_t bytes = (uint32_t)(((op.ndofs - 1) * ld + nvec) * 8);
    auto k = ca.Xp ? apply_cheb_pair_kernel<NP, NQ, true> : apply_cheb_pair_kernel<NP, NQ, false>;
    hipLaunchKernelGGL(k, dim3((unsigned)(plan.chunk * kXcds)), dim3(64), 0, s, op.grid, op.d_geo,
                       op.d_vq, Y, Out, (uint32_t)ld, nvec, plan, bytes, ca);
    return hipGetLastError();
  }
  return hipErrorInvalidValue;
}

}  // namespace

template <>
hipError_t launch_cheb_pair_p<MF_P>(const Operator& op, const double* Y, double* Out, int64_t ld,
                                    int nvec, const ChebArgs& ca, const PairPlan& plan,
                                    hipStream_t s) {
  switch (op.q - MF_P) {
    case 1: return launch_pq<MF_P + 1, MF_P + 1>(op, Y, Out, ld, nvec, ca, plan, s);
    case 2: return launch_pq<MF_P + 1, MF_P + 2>(op, Y, Out, ld, nvec, ca, plan, s);
    case 3: return launch_pq<MF_P + 1, MF_P + 3>(op, Y, Out, ld, nvec, ca, plan, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace mf
