// Register-resident body of the FP64 fused apply for axis-aligned cells with at
// most seven points per direction (the arithmetic of box_body.h:
// T = (N x N x N) U, T <- det J (V + sigma) o T + sum_s g_s Lf_s T,
// V = (N x N x N)^T T).
//
// One wavefront holds a whole cell of 16 columns in registers.  Lane l owns the
// column slot l mod 16 and the z pair k = l / 16: the points k and N-1-k (for
// odd N the middle point belongs to the last pair), for every (x, y).  The
// even-odd split along z is then an addition and a subtraction inside a lane,
// and the even and odd halves of a contraction along z are 4 x 4 matrices
// acting across the four lane groups: one v_mfma_f64_4x4x4_4b each, with
// operand and result in the same lanes (B[k][j] and D[i][j] of block b in lane
// j + 4 b + 16 k).  The contractions along x and y run on the vector ALUs, on
// the even and the odd plane separately.  No cell array passes through LDS and
// no barrier separates the stages.
//
// The potential couples the two planes at each (x, y): with the values v, v' at
// the points of the pair, p = (v + v') / 2 and m = (v - v') / 2 give
// u_e += p e + m o, u_o += m e + p o; (p, m) are formed once per cell in LDS.
//
// The wavefront marches along y over a segment of a line of cells: the row of
// nodes shared by consecutive cells is carried in LDS before the last z
// contraction, so only rows on x and z cell faces and at the ends of a segment
// have several contributors.
//
// What bounds it (p = 6, 16^3 cells, 64 columns): the FP64 additions to shared
// rows run at 186 G/s whatever their locality (218 of a cell's 343 nodes, added
// by the box kernel's every cell, take 307 us by themselves; the march leaves 144
// + 74 per segment), and 128-byte rows (16 columns) halve the requests of
// 64-byte ones.  Without any memory access the contractions take 280 us: 4850
// vector instructions per cell at one wavefront per SIMD, whose two planes
// before and after the derivative stage fill 480 registers.  Eight columns at
// two wavefronts per SIMD contract in 231 us but run at 450 us (64-byte rows); the
// next cell's loads are issued before the assembly, because loads issued after
// it wait for its additions.  Apply with zero fill: 506 (box kernel) -> 418 us;
// p = 4, 24^3: 585 -> 460; p = 2, 32^3: 455 -> 247; p = 6, 20^3, 128 columns:
// 1.90 -> 1.50 ms.
// By the counters the one wavefront per SIMD issues an instruction in 43% of its
// cycles, waits for a result or an issue slot in 40% and for memory in 17%.
#pragma once

#include "mf_internal.h"
#include "sf_common.h"
#include "sf_tables.h"

namespace mf {

constexpr int kPairCols = 16;   // column slots of a wavefront
constexpr int kPairMaxN = 7;    // points per direction: a pair index below four

// FP64 atomic addition through a buffer descriptor, without a result.
extern "C" __device__ double mf_buffer_fadd(double, __amdgpu_buffer_rsrc_t, int, int, int) __asm(
    "llvm.amdgcn.raw.ptr.buffer.atomic.fadd.f64");

// Offsets from kOob on are outside every descriptor (the host admits spans below
// kPairMaxSpan bytes): a load there gives zero, a store or an addition is dropped.
constexpr uint32_t kOob = 0xFFFF0000u;

struct BufF64 {
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ BufF64(const double* p, uint32_t bytes)
      : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(p), 0, bytes, 0x00027000)) {}
  __device__ __forceinline__ double load(uint32_t lane, uint32_t uniform) const {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, lane, uniform, 0));
  }
  __device__ __forceinline__ void store(double x, uint32_t lane, uint32_t uniform) const {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, x), r, lane, uniform, 0);
  }
  __device__ __forceinline__ void add(double x, uint32_t lane, uint32_t uniform) const {
    (void)mf_buffer_fadd(x, r, lane, uniform, 0);
  }
};

// Operand A of the z contractions, one double per lane: A[i][k] of every block
// in lane i + 4 b + 16 k.  n: N, l: 2 L on pairs (input the unfolded pair
// values), t: N^T with the fold's factor two on pairs; [0] even, [1] odd.
template <int NP, int NQ>
struct PairTab {
  double n[2][64], l[2][64], t[2][64];
};
template <int NP, int NQ>
constexpr PairTab<NP, NQ> make_pair_tab() {
  static_assert(NQ <= kPairMaxN && NP <= NQ, "pair indices below four");
  using EN = EoMat<MatN<NP, NQ>, NQ, NP, false, NP>;
  using EL = EoMat<MatL<NP, NQ>, NQ, NQ, false, NQ>;
  using ET = EoMat<MatN<NP, NQ>, NP, NQ, true, NP>;
  constexpr int HP = NP / 2, MP = NP % 2, HQ = NQ / 2, MQ = NQ % 2;
  PairTab<NP, NQ> r{};
  for (int lane = 0; lane < 64; ++lane) {
    const int i = lane & 3, k = lane >> 4;
    if (i < HQ + MQ && k < HP + MP) r.n[0][lane] = EN::e(i, k);
    if (i < HQ + MQ && k < HQ + MQ) r.l[0][lane] = EL::e(i, k) * (k < HQ ? 2.0 : 1.0);
    if (i < HP + MP && k < HQ + MQ) r.t[0][lane] = ET::e(i, k) * (k < HQ ? 2.0 : 1.0);
    if (i < HQ && k < HP) r.n[1][lane] = EN::d(i, k);
    if (i < HQ && k < HQ) r.l[1][lane] = 2.0 * EL::d(i, k);
    if (i < HP && k < HQ) r.t[1][lane] = 2.0 * ET::d(i, k);
  }
  return r;
}
template <int NP, int NQ>
__device__ constexpr PairTab<NP, NQ> kPairTab = make_pair_tab<NP, NQ>();

__device__ __forceinline__ double mfma_z(double a, double b, double c) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}

// Keeps the computation of a block of values where it stands: without it the
// compiler sinks a stage past the next cell's loads, whose registers then
// overlap with the stage's inputs.
template <int N>
__device__ __forceinline__ void pin(double (&v)[2][N][N]) {
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int j = 0; j < N; ++j)
#pragma unroll
      for (int i = 0; i < N; ++i) asm volatile("" : "+v"(v[h][j][i]));
}
__device__ __forceinline__ void stage_end() { __builtin_amdgcn_sched_barrier(0); }

// Between LDS accesses of different lanes of the wavefront to the same places: keeps the
// stores before it in front of the reads behind it and the reads before it in front of
// the stores behind it.  Nothing is emitted, as a wavefront's LDS accesses execute in order.
__device__ __forceinline__ void lds_handover() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// The lane number, recomputed where it is used: what depends on it is not held
// in registers across the cells of a segment.
__device__ __forceinline__ int fresh_lane() {
  int l = threadIdx.x & 63;
  asm volatile("" : "+v"(l));
  return l;
}

// y[r] = M x[r] as eo_matvec, with the odd part accumulated onto the even one:
// y_o = e + d, then y_{m-1-o} = 2 e - y_o, one operation less per pair of
// outputs than two separate sums.
template <class M, int NOUT, int NIN, bool TR, int LD, int RN>
__device__ __forceinline__ void eo_apply(double (&x)[RN][NIN], double (&y)[RN][NOUT]) {
  using E = EoMat<M, NOUT, NIN, TR, LD>;
  static_assert(centrosymmetric<M, NOUT, NIN, TR, LD>(), "matrix is not centrosymmetric");
#pragma unroll
  for (int r = 0; r < RN; ++r)
#pragma unroll
    for (int i = 0; i < E::HI; ++i) {
      const double a = x[r][i], b = x[r][NIN - 1 - i];
      x[r][i] = a + b;
      x[r][NIN - 1 - i] = a - b;
    }
  double ev[E::HO + E::MO][RN];
  sfor<E::HO + E::MO>([&](auto O) {
    constexpr int o = decltype(O)::value;
    constexpr int fe = E::first_e(o);
    sfor<E::HI + E::MI>([&](auto I) {
      constexpr int i = decltype(I)::value;
      constexpr double c = E::e(o, i);
#pragma unroll
      for (int r = 0; r < RN; ++r) {
        if constexpr (fe < 0) ev[o][r] = 0.0;
        else if constexpr (i == fe) ev[o][r] = c * x[r][i];
        else if constexpr (i > fe && c != 0.0) ev[o][r] = fma(c, x[r][i], ev[o][r]);
      }
    });
  });
  sfor<E::HO>([&](auto O) {
    constexpr int o = decltype(O)::value;
#pragma unroll
    for (int r = 0; r < RN; ++r) y[r][o] = ev[o][r];
    sfor<E::HI>([&](auto I) {
      constexpr int i = decltype(I)::value;
      constexpr double c = E::d(o, i);
      if constexpr (c != 0.0) {
#pragma unroll
        for (int r = 0; r < RN; ++r) y[r][o] = fma(c, x[r][NIN - 1 - i], y[r][o]);
      }
    });
#pragma unroll
    for (int r = 0; r < RN; ++r) y[r][NOUT - 1 - o] = fma(2.0, ev[o][r], -y[r][o]);
  });
  if constexpr (E::MO == 1) {
#pragma unroll
    for (int r = 0; r < RN; ++r) y[r][E::HO] = ev[E::HO][r];
  }
}

template <int NP, int NQ>
struct PairCell {
  static constexpr int P = NP - 1, HP = NP / 2, MP = NP % 2, HQ = NQ / 2, MQ = NQ % 2;
  static constexpr int NQ2 = NQ * NQ;
  static constexpr int NPM = (NQ2 * 4 + 63) / 64;  // (p, m) entries per lane and cell
  using Nf = MatN<NP, NQ>;
  using Lf = MatL<NP, NQ>;
  double T[2][NQ][NQ], U[2][NQ][NQ];  // [plane][y][x]

  // T: node values at (k, NP-1-k) -> T at the quadrature points, U: all but
  // the y derivative, then U <- N^T along y of the whole sum.  pm: this lane's
  // (p, m) of point (x, y) at pm[4 (x + NQ y)].
  __device__ __forceinline__ void contract(const double2* pm, double g0, double g1, double g2) {
    const int l = fresh_lane();
    {
      const double a0 = kPairTab<NP, NQ>.n[0][l], a1 = kPairTab<NP, NQ>.n[1][l];
#pragma unroll
      for (int j = 0; j < NP; ++j)
#pragma unroll
        for (int i = 0; i < NP; ++i) {
          const double a = T[0][j][i], b = T[1][j][i];
          T[0][j][i] = mfma_z(a0, a + b, 0.0);
          T[1][j][i] = mfma_z(a1, a - b, 0.0);
        }
    }
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      double in[2][NP], o[2][NQ];
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < NP; ++j) in[h][j] = T[h][j][i];
      eo_apply<Nf, NQ, NP, false, NP, 2>(in, o);
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int b = 0; b < NQ; ++b) T[h][b][i] = o[h][b];
    }
    const double l0 = kPairTab<NP, NQ>.l[0][l] * g2, l1 = kPairTab<NP, NQ>.l[1][l] * g2;
#pragma unroll
    for (int b = 0; b < NQ; ++b) {
      double in[2][NP], o[2][NQ], lx[2][NQ];
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < NP; ++i) in[h][i] = T[h][b][i];
      eo_apply<Nf, NQ, NP, false, NP, 2>(in, o);
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int a = 0; a < NQ; ++a) T[h][b][a] = o[h][a];
      eo_apply<Lf, NQ, NQ, false, NQ, 2>(o, lx);
#pragma unroll
      for (int a = 0; a < NQ; ++a) {
        const double2 c = pm[(b * NQ + a) * 4];
        const double t0 = T[0][b][a], t1 = T[1][b][a];
        U[0][b][a] = mfma_z(l0, t0, fma(g0, lx[0][a], fma(c.y, t1, c.x * t0)));
        U[1][b][a] = mfma_z(l1, t1, fma(g0, lx[1][a], fma(c.y, t0, c.x * t1)));
      }
      stage_end();
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int a = 0; a < NQ; ++a) {
        double in[1][NQ], o[1][NQ], w[1][NP];
#pragma unroll
        for (int b = 0; b < NQ; ++b) in[0][b] = T[h][b][a];
        eo_apply<Lf, NQ, NQ, false, NQ, 1>(in, o);
#pragma unroll
        for (int b = 0; b < NQ; ++b) o[0][b] = fma(g1, o[0][b], U[h][b][a]);
        eo_apply<Nf, NP, NQ, true, NP, 1>(o, w);
#pragma unroll
        for (int j = 0; j < NP; ++j) U[h][j][a] = w[0][j];
        stage_end();
      }
    pin(U);
    stage_end();
  }

  // N^T along x of row j, in place.
  __device__ __forceinline__ void back_x(int j) {
    double in[2][NQ], o[2][NP];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int a = 0; a < NQ; ++a) in[h][a] = U[h][j][a];
    eo_apply<Nf, NP, NQ, true, NP, 2>(in, o);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < NP; ++i) U[h][j][i] = o[h][i];
  }
};

}  // namespace mf
