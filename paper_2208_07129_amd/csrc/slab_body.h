// Slab form of the FP64 fused apply for axis-aligned cells (the arithmetic of
// box_body.h: T = (N x N x N) U, T <- det J (V + sigma) o T + sum_s g_s Lf_s T,
// V = (N x N x N)^T T, every 1D contraction in even-odd form).
#pragma once

#include "mf_internal.h"
#include "sf_common.h"
#include "sf_tables.h"

namespace mf {

template <int NP, int NQ, int B, int G>
struct Slab {
  static constexpr int SY = NQ | 1;
  static constexpr int SZ = (SY * (NQ - 1) + NQ) | 1;
  static constexpr int CELL = SZ * (NQ - 1) + SY * (NQ - 1) + NQ;
  static constexpr int LANES = NQ * B * G;
  static constexpr int NT = (LANES + 63) / 64 * 64;
  static constexpr size_t LDS = (size_t)CELL * B * G * sizeof(double);
};

template <int NP, int NQ, int B, int G, bool ACCUM, typename Off>
__device__ __forceinline__ void slab_item(double* __restrict__ lds, const GridDesc& grid, int64_t e,
                                          const double* __restrict__ geo,
                                          const double* __restrict__ vq,
                                          const double* __restrict__ X, double* __restrict__ Y,
                                          Off ldx, Off ldy, int nvec, int v0, int tid) {
  using S = Slab<NP, NQ, B, G>;
  using Nf = MatN<NP, NQ>;
  using Lf = MatL<NP, NQ>;
  constexpr int SY = S::SY, SZ = S::SZ, P = NP - 1;
  const int col = tid % B, s = (tid / B) % NQ;
  const int cx = (int)e % grid.n[0], cyz = (int)e / grid.n[0];
  const int cy = cyz % grid.n[1], cz = cyz / grid.n[1];
  const int v = v0 + col;
  const bool vok = v < nvec;
  auto at = [&](int x, int y, int z) { return (x + SY * y + SZ * z) * B; };
  double* __restrict__ zs = lds + s * SZ * B + col;  // (x, y) at z = s
  double* __restrict__ ys = lds + s * SY * B + col;  // (x, z) at y = s
  // A
  int gz = cz * grid.p + s;
  if (gz >= grid.N[2]) gz = s < NP ? 0 : 0;
  if (s < NP) {
    const Off zo = (Off)gz * (Off)grid.N[0] * (Off)grid.N[1] * ldx + (Off)(vok ? v : nvec - 1);
    double x[NP][NP];
#pragma unroll
    for (int j = 0; j < NP; ++j) {
      int gy = cy * grid.p + j;
      if (j == P && gy == grid.N[1]) gy = 0;
      const Off yo = (Off)gy * (Off)grid.N[0] * ldx;
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        int gx = cx * grid.p + i;
        if (i == P && gx == grid.N[0]) gx = 0;
        x[i][j] = X[zo + (yo + (Off)gx * ldx)];
      }
    }
    if (grid.dirichlet) {
      const bool zc = gz == 0 || gz == grid.N[2] - 1;
#pragma unroll
      for (int j = 0; j < NP; ++j) {
        const bool yc = zc || (j == 0 && cy == 0) || (j == P && cy == grid.n[1] - 1);
#pragma unroll
        for (int i = 0; i < NP; ++i)
          if (yc || (i == 0 && cx == 0) || (i == P && cx == grid.n[0] - 1)) x[i][j] = 0.0;
      }
    }
    double o[NP][NQ];
    eo_matvec<Nf, NQ, NP, false, NP, NP>(x, o);
#pragma unroll
    for (int i = 0; i < NP; ++i)
#pragma unroll
      for (int a = 0; a < NQ; ++a) zs[at(i, a, 0)] = o[i][a];
  }
  __syncthreads();
  // B
  const double g0 = geo[e * 6 + 0], g1 = geo[e * 6 + 3], g2 = geo[e * 6 + 5];
  double u[NQ][NQ];  // [x][z]
  {
    double t[NP][NQ];  // [z][x]
    {
      double r[NP][NP];
#pragma unroll
      for (int k = 0; k < NP; ++k)
#pragma unroll
        for (int i = 0; i < NP; ++i) r[k][i] = ys[at(i, 0, k)];
      eo_matvec<Nf, NQ, NP, false, NP, NP>(r, t);
    }
    const double* vs = vq + e * (NQ * NQ * NQ) + s * NQ;
#pragma unroll
    for (int a = 0; a < NQ; ++a) {
      double in[1][NP], T[1][NQ], l[1][NQ], m[NQ];
#pragma unroll
      for (int k = 0; k < NP; ++k) in[0][k] = t[k][a];
      eo_matvec<Nf, NQ, NP, false, NP, 1>(in, T);
#pragma unroll
      for (int c = 0; c < NQ; ++c) {
        ys[at(a, 0, c)] = T[0][c];
        m[c] = vs[a + c * NQ * NQ] * T[0][c];
      }
      eo_matvec<Lf, NQ, NQ, false, NQ, 1>(T, l);
#pragma unroll
      for (int c = 0; c < NQ; ++c) u[a][c] = fma(g2, l[0][c], m[c]);
    }
#pragma unroll
    for (int c = 0; c < NQ; ++c) {
      double T[1][NQ], l[1][NQ];
#pragma unroll
      for (int a = 0; a < NQ; ++a) T[0][a] = ys[at(a, 0, c)];
      eo_matvec<Lf, NQ, NQ, false, NQ, 1>(T, l);
#pragma unroll
      for (int a = 0; a < NQ; ++a) u[a][c] = fma(g0, l[0][a], u[a][c]);
    }
  }
  __syncthreads();
  // C
#pragma unroll
  for (int a = 0; a < NQ; ++a) {
    double T[1][NQ], l[1][NQ];
#pragma unroll
    for (int b = 0; b < NQ; ++b) T[0][b] = zs[at(a, b, 0)];
    eo_matvec<Lf, NQ, NQ, false, NQ, 1>(T, l);
#pragma unroll
    for (int b = 0; b < NQ; ++b) zs[at(a, b, 0)] = g1 * l[0][b];
  }
  __syncthreads();
  // D
  {
    double w[NP][NQ];  // [z][x]
#pragma unroll
    for (int a = 0; a < NQ; ++a) {
      double o[1][NP], in[1][NQ];
#pragma unroll
      for (int c = 0; c < NQ; ++c) in[0][c] = u[a][c] + ys[at(a, 0, c)];
      eo_matvec<Nf, NP, NQ, true, NP, 1>(in, o);
#pragma unroll
      for (int k = 0; k < NP; ++k) w[k][a] = o[0][k];
    }
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      double o[1][NP], in[1][NQ];
#pragma unroll
      for (int a = 0; a < NQ; ++a) in[0][a] = w[k][a];
      eo_matvec<Nf, NP, NQ, true, NP, 1>(in, o);
#pragma unroll
      for (int i = 0; i < NP; ++i) ys[at(i, 0, k)] = o[0][i];
    }
  }
  __syncthreads();
  // E
  const bool zc = grid.dirichlet && (gz == 0 || gz == grid.N[2] - 1);
  if (s >= NP || !vok || zc) return;
  const bool zin = s > 0 && s < P;
  const Off zo = (Off)gz * (Off)grid.N[0] * (Off)grid.N[1] * ldy + (Off)v;
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    double in[1][NQ], o[1][NP];
#pragma unroll
    for (int b = 0; b < NQ; ++b) in[0][b] = zs[at(i, b, 0)];
    eo_matvec<Nf, NP, NQ, true, NP, 1>(in, o);
    int gx = cx * grid.p + i;
    if (i == P && gx == grid.N[0]) gx = 0;
    if (grid.dirichlet && ((i == 0 && cx == 0) || (i == P && cx == grid.n[0] - 1))) continue;
    const Off xo = (Off)gx * ldy;
#pragma unroll
    for (int j = 0; j < NP; ++j) {
      int gy = cy * grid.p + j;
      if (j == P && gy == grid.N[1]) gy = 0;
      if (grid.dirichlet && ((j == 0 && cy == 0) || (j == P && cy == grid.n[1] - 1))) continue;
      double* dst = Y + (zo + ((Off)gy * (Off)grid.N[0] * ldy + xo));
      if (i > 0 && i < P && j > 0 && j < P) {
        if (zin) {
          if (ACCUM) *dst += o[0][j];
          else *dst = o[0][j];
        } else {
          unsafeAtomicAdd(dst, o[0][j]);
        }
      } else {
        unsafeAtomicAdd(dst, o[0][j]);
      }
    }
  }
}

}  // namespace mf
