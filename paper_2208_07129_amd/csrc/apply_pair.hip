// FP64 fused apply of axis-aligned cells, register-resident form (pair_body.h):
// one wavefront per (segment of a line of cells along y, column tile).
#include "pair_body.h"

#ifndef MF_P
#error "compile with -DMF_P=<degree>"
#endif

namespace mf {
namespace {

// B columns of pair_cells(B) cells adjacent in x per wavefront (B = 16: one
// cell); slots past them idle.
template <int NP, int NQ, int B, bool ACCUM>
__global__ void __attribute__((amdgpu_flat_work_group_size(64, 64),
                               amdgpu_waves_per_eu(pair_waves(NQ), pair_waves(NQ))))
apply_pair_kernel(const GridDesc grid, const double* __restrict__ geo,
                  const double* __restrict__ vq, const double* __restrict__ X,
                  double* __restrict__ Y, uint32_t ldx, uint32_t ldy, int nvec,
                  const PairPlan plan, uint32_t xbytes, uint32_t ybytes) {
  using PC = PairCell<NP, NQ>;
  constexpr int P = PC::P, HP = PC::HP, MP = PC::MP, HQ = PC::HQ, MQ = PC::MQ, NQ2 = PC::NQ2;
  constexpr int LX = pair_cells(B), NPM = (LX * NQ2 * 4 + 63) / 64;
  __shared__ double2 pms[LX][NQ2 * 4];
  __shared__ double carry[2][NP][64];
  const int item = (int)xcd_item(blockIdx.x, plan.chunk);
  if (item >= plan.items) return;
  int it = item / plan.ntiles;
  const int v0 = (item - it * plan.ntiles) * B;
  const int xg = it % plan.nxg;
  it /= plan.nxg;
  const int seg = it % plan.nseg, cz = it / plan.nseg;
  const int cya = seg * plan.len, cyb = min(grid.n[1], cya + plan.len);
  const uint32_t plane = (uint32_t)(grid.N[0] * grid.N[1]), N0 = (uint32_t)grid.N[0];
  const BufF64 bx(X, xbytes), by(Y, ybytes);
  const double g0 = geo[0], g1 = geo[3], g2 = geo[5];
  PC c;

  // Byte offsets of the lane's node (0, 0, z) of plane h and column, for the x
  // nodes 0, 1 .. P-1 (mid) and P (the wrapped node; the uniform offset of a
  // node adds i ld for i < P and the row's y part).
  struct Lane {
    uint32_t lo[2], mid[2], hi[2];
  };
  auto locate = [&](Lane& q, int l, uint32_t ld, bool on) {
    const int k = l >> 4, slot = l & (kPairCols - 1);
    const int v = v0 + slot % B, cx = xg * LX + slot / B;
    const bool live = on && v < nvec && (LX == 1 || (slot < B * LX && cx < grid.n[0]));
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
  auto potential = [&](int cy, int idx) {  // the two potential values of (p, m) entry idx
    idx = min(idx, LX * NQ2 * 4 - 1);
    const int lx = idx / (NQ2 * 4), xy = (idx >> 2) % NQ2, kk = idx & 3;
    const int ka = kk < HQ + MQ ? kk : 0;
    const int cx = min(xg * LX + lx, grid.n[0] - 1);
    const double* vs = vq + (int64_t)(cx + grid.n[0] * (cy + grid.n[1] * cz)) * (NQ2 * NQ);
    return make_double2(vs[xy + NQ2 * ka], vs[xy + NQ2 * (NQ - 1 - ka)]);
  };
  auto put_pm = [&](double2 v, int idx) {
    if (idx < LX * NQ2 * 4) (&pms[0][0])[idx] = make_double2(0.5 * (v.x + v.y), 0.5 * (v.x - v.y));
  };
  auto fetch = [&](int cy, bool on) {
    const int l = fresh_lane();
    Lane q;
    locate(q, l, ldx, on);
    uint32_t lb = ldx * 8u;
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
          c.T[h][j][i] = bx.load(v, i == P ? row : row + (uint32_t)i * lb);
        }
    }
#pragma unroll
    for (int r = 0; r < NPM; ++r) pq[r] = potential(cy, l + 64 * r);
  };

  fetch(cya, true);
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int i = 0; i < NP; ++i) carry[h][i][threadIdx.x] = 0.0;

  for (int cy = cya; cy < cyb; ++cy) {
    {
      const int l = fresh_lane();
      lds_handover();
#pragma unroll
      for (int r = 0; r < NPM; ++r) put_pm(pq[r], l + 64 * r);
      lds_handover();
      const int slot = l & (kPairCols - 1);
      c.contract(&pms[min(slot / B, LX - 1)][l >> 4], g0, g1, g2);
    }
    const bool first = cy == cya, last = cy + 1 == cyb;
    fetch(last ? cy : cy + 1, !last);  // the next cell's values, in flight during the assembly
    stage_end();
#pragma unroll
    for (int j = 0; j < NP; ++j) {
      c.back_x(j);
      stage_end();
    }
    const int l = fresh_lane();
    Lane q;
    locate(q, l, ldy, true);
    const double t0 = kPairTab<NP, NQ>.t[0][l], t1 = kPairTab<NP, NQ>.t[1][l];
    const bool zin = (l >> 4) > 0;  // nodes off the z faces: one contributor unless on an x face
    uint32_t vin[2], vfc[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      vin[h] = zin ? q.mid[h] : kOob;
      vfc[h] = zin ? kOob : q.mid[h];
    }
    uint32_t lb = ldy * 8u;
    asm volatile("" : "+s"(lb));
    const bool ylo = grid.dirichlet && cy == 0, yhi = grid.dirichlet && cy == grid.n[1] - 1;
    const uint32_t row0 = (uint32_t)(cy * grid.p) * N0 * lb;
#pragma unroll
    for (int j = 0; j < P; ++j) {
      const uint32_t row = row0 + (uint32_t)j * N0 * lb;
      const bool dead = j == 0 && ylo, part = j == 0 && first;
      double d[2][NP];
#pragma unroll
      for (int i = 0; i < NP; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          d[h][i] = mfma_z(h ? t1 : t0, j == 0 ? c.U[h][0][i] + carry[h][i][l] : c.U[h][j][i], 0.0);
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        const double y[2] = {d[0][i] + d[1][i], d[0][i] - d[1][i]};
        const uint32_t s = i == P ? row : row + (uint32_t)i * lb;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          if (i == 0 || i == P) {
            uint32_t v = i == 0 ? q.lo[h] : q.hi[h];
            if (j == 0) v = dead ? kOob : v;
            by.add(y[h], v, s);
          } else if (part) {
            by.add(y[h], dead ? kOob : q.mid[h], s);
          } else {
            by.add(y[h], vfc[h], s);
            by.store(ACCUM ? y[h] + by.load(vin[h], s) : y[h], vin[h], s);
          }
        }
      }
    }
    if (!last) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < NP; ++i) carry[h][i][l] = c.U[h][P][i];
    } else {
      const uint32_t row = cy * grid.p + P == grid.N[1] ? 0u : row0 + (uint32_t)P * N0 * lb;
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        const double d0 = mfma_z(t0, c.U[0][P][i], 0.0), d1 = mfma_z(t1, c.U[1][P][i], 0.0);
        const double y[2] = {d0 + d1, d0 - d1};
        const uint32_t s = i == P ? row : row + (uint32_t)i * lb;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const uint32_t v = i == 0 ? q.lo[h] : (i == P ? q.hi[h] : q.mid[h]);
          by.add(y[h], yhi ? kOob : v, s);
        }
      }
    }
  }
}

template <int NP, int NQ, int B>
hipError_t launch_pair(const ApplyLaunch& a, const PairPlan& plan, hipStream_t s) {
  const auto span = [&](int64_t ld) { return (uint32_t)((((int64_t)a.grid.N[0] * a.grid.N[1] * a.grid.N[2] - 1) * ld + a.nvec) * 8); };
  auto k = apply_pair_kernel<NP, NQ, B, false>;
  if (a.accumulate) {
    if constexpr (NQ <= kPairAccumMaxQ) k = apply_pair_kernel<NP, NQ, B, true>;
    else return hipErrorInvalidValue;
  }
  hipLaunchKernelGGL(k, dim3((unsigned)(plan.chunk * kXcds)), dim3(64), 0, s, a.grid, a.geo, a.vq,
                     a.X, a.Y, (uint32_t)a.ldx, (uint32_t)a.ldy, a.nvec, plan, span(a.ldx),
                     span(a.ldy));
  return hipGetLastError();
}

template <int NP, int NQ>
hipError_t launch_pq(const ApplyLaunch& a, const PairPlan& plan, hipStream_t s) {
  if constexpr (NQ <= kPairMaxN) {
    switch (plan.cols) {
      case 16: return launch_pair<NP, NQ, 16>(a, plan, s);
      case 8: return launch_pair<NP, NQ, 8>(a, plan, s);
      case 4: return launch_pair<NP, NQ, 4>(a, plan, s);
      case 2: return launch_pair<NP, NQ, 2>(a, plan, s);
      case 1: return launch_pair<NP, NQ, 1>(a, plan, s);
    }
  }
  return hipErrorInvalidValue;
}

}  // namespace

template <>
hipError_t launch_apply_pair_p<MF_P>(const Operator& op, const ApplyLaunch& a,
                                     const PairPlan& plan, hipStream_t s) {
  switch (op.q - MF_P) {
    case 1: return launch_pq<MF_P + 1, MF_P + 1>(a, plan, s);
    case 2: return launch_pq<MF_P + 1, MF_P + 2>(a, plan, s);
    case 3: return launch_pq<MF_P + 1, MF_P + 3>(a, plan, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace mf
