// Symmetric eigen-decomposition of k x k blocks with 64 < k <= 2048 (the
// orthogonalisation and Rayleigh-Ritz steps of Alg. ChFSi at block sizes of
// hundreds to a thousand vectors) by the two-sided block Jacobi method.
//
// The indices are cut into blocks of 32 (k padded to a multiple of 64 with
// decoupled zero rows and columns).  One sweep pairs every two blocks once
// (round-robin pairing of the nb blocks, nb - 1 rounds).  In a round, each of
// the nb/2 disjoint block pairs gets one cyclic Jacobi sweep over its 64
// indices (one workgroup, the 64 x 64 sub-block in LDS), whose accumulated
// rotation J_i (64 x 64, orthogonal) is then applied to the whole matrix,
// A := J^T A J with J = diag(J_i) in the pairs' index sets, and to the
// accumulated eigenvectors, V := V J: one workgroup per 64 x 64 piece of A
// (two small products each) or of V.  Every pair of indices is rotated at
// least once per sweep, so this is a cyclic Jacobi ordering and converges
// quadratically.  After each sweep the off-diagonal Frobenius norm is
// measured; once it is at most 1e-14 of the block's, a device flag stops the
// remaining launches (they return at once), so the host never waits.
#include <algorithm>

#include "mf_internal.h"

namespace mf {
namespace {

constexpr int kBj = 32, kBjPair = 2 * kBj, kBjLd = kBjPair + 1;
constexpr int kBjMaxK = 2048, kBjMaxSweeps = 40, kBjNormThreads = 256;

struct BjState {  // at the start of the work array
  double nrm2;    // squared Frobenius norm of the block
  double off2;    // squared off-diagonal norm after the last sweep
  double done;    // 1 once off2 <= 1e-28 nrm2
  double sweeps;  // sweeps taken
  unsigned arrived;  // workgroups of the norm that have written their part
};
constexpr int64_t kBjHead = 8;  // doubles reserved for BjState (keeps the arrays 64-byte aligned)

__host__ __device__ inline int bj_padded(int k) { return (k + kBjPair - 1) / kBjPair * kBjPair; }

// Pair t of round r of the round-robin pairing of n items (n even): position
// 0 holds item 0, position i > 0 item 1 + (i - 1 + r) mod (n - 1), and
// positions t and n - 1 - t meet.
__device__ inline void round_robin(int n, int r, int t, int& p, int& q) {
  const int m = n - 1, i1 = n - 1 - t;
  const int x0 = t == 0 ? 0 : 1 + (t - 1 + r) % m;
  const int x1 = 1 + (i1 - 1 + r) % m;
  p = x0 < x1 ? x0 : x1;
  q = x0 < x1 ? x1 : x0;
}

// Global index of position i (< 64) of the block pair (P, Q).
__device__ inline int pair_index(int P, int Q, int i) {
  return i < kBj ? P * kBj + i : Q * kBj + (i - kBj);
}

__global__ void bj_init_kernel(int k, int K, const double* __restrict__ A, int64_t lda,
                               double* __restrict__ Aw, double* __restrict__ Vw, BjState* st) {
  const int64_t total = (int64_t)K * K;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int i = (int)(idx / K), j = (int)(idx - (int64_t)i * K);
    Aw[idx] = (i < k && j < k) ? A[(int64_t)i * lda + j] : 0.0;
    Vw[idx] = i == j ? 1.0 : 0.0;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) st->arrived = 0;
}

// first = true: the block's norm and whether it is diagonal already;
// otherwise (after a sweep, unless done): one more sweep counted, and done
// when the off-diagonal norm is small enough.  Every workgroup sums its rows
// into part[2 b], part[2 b + 1] (free between sweeps: the rotations' array);
// the last one to arrive adds the parts in order, so the result does not depend
// on which that is.  One workgroup for the whole block took 75 us at K = 256, this 8.
constexpr int kBjNormRows = 8;  // rows per workgroup
__global__ void __launch_bounds__(kBjNormThreads)
bj_norm_kernel(int K, const double* __restrict__ Aw, double* __restrict__ part, BjState* st,
               int first) {
  if (!first && st->done != 0.0) return;
  __shared__ double ra[kBjNormThreads], ro[kBjNormThreads];
  __shared__ int last;
  const int t = threadIdx.x, r0 = blockIdx.x * kBjNormRows;
  double all = 0.0, off = 0.0;
  for (int e = t; e < kBjNormRows * K; e += kBjNormThreads) {
    const int i = r0 + e / K, j = e % K;
    const double x = Aw[(int64_t)i * K + j];
    all = fma(x, x, all);
    if (i != j) off = fma(x, x, off);
  }
  auto reduce = [&]() {
    ra[t] = all;
    ro[t] = off;
    __syncthreads();
    for (int s = kBjNormThreads / 2; s > 0; s >>= 1) {
      if (t < s) {
        ra[t] += ra[t + s];
        ro[t] += ro[t + s];
      }
      __syncthreads();
    }
  };
  reduce();
  if (t == 0) {
    part[2 * blockIdx.x] = ra[0];
    part[2 * blockIdx.x + 1] = ro[0];
    __threadfence();
    last = atomicAdd(&st->arrived, 1u) == gridDim.x - 1;
  }
  __syncthreads();
  if (!last) return;
  __threadfence();
  all = off = 0.0;
  if (t < (int)gridDim.x) {  // at most kBjMaxK / kBjNormRows = 256 parts
    all = __hip_atomic_load(part + 2 * t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    off = __hip_atomic_load(part + 2 * t + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  reduce();
  if (t == 0) {
    st->arrived = 0;
    if (first) {
      st->nrm2 = ra[0];
      st->sweeps = 0.0;
    } else {
      st->sweeps += 1.0;
    }
    st->off2 = ro[0];
    st->done = ro[0] <= 1e-28 * st->nrm2 ? 1.0 : 0.0;
  }
}

// One cyclic Jacobi sweep over the 64 indices of block pair blockIdx.x of
// round r; writes the accumulated rotation to J + 64^2 blockIdx.x (row-major,
// column j = the new basis vector j in the pair's old coordinates).
//
// A serial chain of 63 rounds on one CU: what counts is the length of a round.
// The 64 indices sit in 32 slot pairs (position t above position 63 - t) and
// move one position per round, so every round reads and writes the same places:
// the 2 x 2 block of slot pairs (i < j) takes the row rotation of pair i and the
// column rotation of pair j at once and is stored at its place of the next
// round (two LDS copies; four planes [slot][slot] of 32 x 32, of which the blocks
// i < j are kept up: the matrix is symmetric).  The 13 wavefronts work side by
// side with one barrier per round: wavefront 0 has the diagonal blocks in
// registers and forms the next round's angles, for which it takes the two
// elements that meet through this round's rotations by itself; eight rotate the
// off-diagonal blocks, one per lane; four hold the rotation V in registers (lane =
// row, a wavefront = eight slot pairs) and pass two columns each to their
// neighbours.  The angle needs two chains of reciprocal square roots.  155 us a
// launch with division, separate row and column passes and three barriers; 63
// with the angles, the blocks and V one after the other; 35 so.
constexpr int kBjP2 = kBjPair / 2;  // slot pairs
constexpr int kBjPlane = kBjP2 * kBjP2;
constexpr int kBjAWaves = 8, kBjVWaves = 4;  // wavefronts on the blocks, on V
constexpr int kBjSweepThreads = 64 * (1 + kBjAWaves + kBjVWaves);
constexpr size_t kBjSweepLds = 2 * 4 * (size_t)kBjPlane * sizeof(double);
static_assert(kBjP2 * (kBjP2 - 1) / 2 <= 64 * kBjAWaves, "one off-diagonal block per lane");
static_assert(2 * 4 * kBjPlane >= kBjPair * kBjLd, "V is written out through the blocks' LDS");

// x^{-1/2} for x in [1/8, 4]: the hardware estimate and two Newton steps.
__device__ __forceinline__ double rsqrt_unit(double x) {
  double y = __builtin_amdgcn_rsq(x);
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    const double e = fma(-x * y, y, 1.0);
    y = fma(0.5 * y, e, y);
  }
  return y;
}

// The rotation that zeroes apq, |angle| <= pi/4: with d = aqq - app and
// b = 2 apq, cos 2t = |d| / sqrt(d^2 + b^2) and sin 2t = sign(d) b / sqrt(d^2 + b^2)
// (d = 0: the positive angle); d and b are scaled by a power of two first.
__device__ __forceinline__ void jacobi_angle(double app, double aqq, double apq, double& c,
                                             double& s) {
  c = 1.0;
  s = 0.0;
  if (!(fabs(apq) > 1e-300)) return;
  double d = aqq - app, b = 2.0 * apq;
  const double m = fmax(fabs(d), fabs(b));
  if (!(m < 1.7e308)) {  // infinite or not a number: as the quotient form would have it
    const double th = d / b, at = fabs(th);
    const double tn = (th >= 0.0 ? 1.0 : -1.0) / (at + sqrt(th * th + 1.0));
    c = 1.0 / sqrt(tn * tn + 1.0);
    s = tn * c;
    return;
  }
  const int ex = -__builtin_amdgcn_frexp_exp(m);
  d = __builtin_amdgcn_ldexp(d, ex);
  b = __builtin_amdgcn_ldexp(b, ex);
  const double rh = rsqrt_unit(fma(d, d, b * b));
  const double c2 = fma(0.5 * fabs(d), rh, 0.5);
  const double rc = rsqrt_unit(c2);
  c = c2 * rc;
  s = (d == 0.0 ? 0.5 * fabs(b) : (d < 0.0 ? -0.5 : 0.5) * b) * rh * rc;
}

// Where the member of slot pair pr in slot (0 above, 1 below) goes next round.
__device__ __forceinline__ void bj_next(int slot, int pr, int& ns, int& np) {
  if (slot == 0) {
    ns = pr == 1;  // position 1 -> 63
    np = pr <= 1 ? 0 : pr - 1;
  } else {
    ns = pr < kBjP2 - 1;  // position 32 -> 31
    np = pr < kBjP2 - 1 ? pr + 1 : kBjP2 - 1;
  }
}

__global__ void __launch_bounds__(kBjSweepThreads)
bj_pair_kernel(int K, int r, const double* __restrict__ Aw, double* __restrict__ J,
               const BjState* __restrict__ st) {
  if (st->done != 0.0) return;
  extern __shared__ double sh[];
  double* a = sh;  // 2 copies of 4 planes
  __shared__ double2 cs[2][kBjP2];
  __shared__ double dg[2][2][kBjP2];              // rotated diagonal, [round][slot][pair]
  __shared__ double xch[2][kBjVWaves][2][64];     // V's columns on their way to a neighbour
  const int t = threadIdx.x, nb = K / kBj, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  constexpr int kRounds = kBjPair - 1;
  int P, Q;
  round_robin(nb, r, blockIdx.x, P, Q);
  for (int i = t; i < kBjPair * kBjPair; i += kBjSweepThreads) {
    const int row = i / kBjPair, col = i % kBjPair;
    const int si = row >= kBjP2, sj = col >= kBjP2;
    const int pi = si ? kBjPair - 1 - row : row, pj = sj ? kBjPair - 1 - col : col;
    a[(si * 2 + sj) * kBjPlane + pi * kBjP2 + pj] =
        Aw[(int64_t)pair_index(P, Q, row) * K + pair_index(P, Q, col)];
  }
  __syncthreads();
  if (wave == 0) {
    const int p = lane & (kBjP2 - 1);
    double d0 = a[p * (kBjP2 + 1)], d1 = a[3 * kBjPlane + p * (kBjP2 + 1)];
    double x = a[kBjPlane + p * (kBjP2 + 1)], c, s;
    // items at the two positions; the angle is that of the smaller one first
    int i0 = p == 0 ? 0 : p, i1 = kBjPair - 1 - p;
    auto angle = [&]() {
      const bool up = i0 < i1;
      jacobi_angle(up ? d0 : d1, up ? d1 : d0, x, c, s);
      s = up ? s : -s;
    };
    angle();
    if (lane < kBjP2) cs[0][p] = make_double2(c, s);
    __syncthreads();
    // the members of slot pair p next round sit in (u, pu) and (w, pw) now
    const int u = p == kBjP2 - 1 ? 1 : 0, pu = p == kBjP2 - 1 ? p : (p == 0 ? 0 : p + 1);
    const int w = p == 0 ? 0 : 1, pw = p == 0 ? 1 : p - 1;
    const bool sw = pu > pw;  // the blocks above the diagonal are kept
    const int lo = sw ? pw : pu, hi = sw ? pu : pw;
    const int m01 = sw ? 2 : 1, m10 = 3 - m01;  // plane of (slot of pu, slot of pw)
    const double* blk = a + lo * kBjP2 + hi;
    // the pair's own off-diagonal element, 0 now, goes to a block of the next round
    int is, ip, js, jp;
    bj_next(0, p, is, ip);
    bj_next(1, p, js, jp);
    double* zero = a + (is * 2 + js) * kBjPlane + ip * kBjP2 + jp;  // ip < jp
    for (int rr = 0; rr + 1 < kRounds; ++rr) {
      const double* ac = blk + (rr & 1) * 4 * kBjPlane;
      const double m00 = ac[0], v01 = ac[m01 * kBjPlane], v10 = ac[m10 * kBjPlane],
                   m11 = ac[3 * kBjPlane];
      const double2 ru = cs[rr & 1][pu], rw = cs[rr & 1][pw];
      // this round's rotation of the diagonal, handed on to the next places
      const double cx = c * x, sx = s * x;
      const double y0 = c * d0 - sx, y1 = s * d0 + cx;  // rows, first column
      const double z0 = cx - s * d1, z1 = sx + c * d1;  // rows, second column
      if (lane < kBjP2) {
        dg[rr & 1][0][p] = c * y0 - s * z0;
        dg[rr & 1][1][p] = s * y1 + c * z1;
        zero[((rr + 1) & 1) * 4 * kBjPlane] = 0.0;
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      const double a0 = u ? ru.y : ru.x, a1 = u ? ru.x : -ru.y;
      const double b0 = w ? rw.y : rw.x, b1 = w ? rw.x : -rw.y;
      const double e0 = fma(a0, m00, a1 * v10), e1 = fma(a0, v01, a1 * m11);
      x = fma(b0, e0, b1 * e1);
      d0 = dg[rr & 1][u][pu];
      d1 = dg[rr & 1][w][pw];
      i0 = p == 0 ? 0 : (i0 == kRounds ? 1 : i0 + 1);
      i1 = i1 == kRounds ? 1 : i1 + 1;
      angle();
      if (lane < kBjP2) cs[(rr + 1) & 1][p] = make_double2(c, s);
      __syncthreads();
    }
    __syncthreads();
    __syncthreads();
  } else if (wave <= kBjAWaves) {
    // off-diagonal block (pi, pj): rows r and 30 - r of the triangle fill 32 lanes
    const int e = t - 64, fr = e / kBjP2, fk = e % kBjP2;
    const bool upper = fk < kBjP2 - 1 - fr;
    const int pi = upper ? fr : kBjP2 - 2 - fr, pj = upper ? fr + 1 + fk : fk;
    const bool on = fr < kBjP2 / 2 - 1 || upper;
    int to[2][2];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        int is, ip, js, jp;
        bj_next(u, pi, is, ip);
        bj_next(w, pj, js, jp);
        to[u][w] = ip <= jp ? (is * 2 + js) * kBjPlane + ip * kBjP2 + jp
                            : (js * 2 + is) * kBjPlane + jp * kBjP2 + ip;
      }
    __syncthreads();
    for (int rr = 0; rr + 1 < kRounds; ++rr) {
      const double* ac = a + (rr & 1) * 4 * kBjPlane + pi * kBjP2 + pj;
      double* an = a + ((rr + 1) & 1) * 4 * kBjPlane;
      if (on) {
        const double2 ri = cs[rr & 1][pi], rj = cs[rr & 1][pj];
        const double tt = ac[0], tb = ac[kBjPlane], bt = ac[2 * kBjPlane], bb = ac[3 * kBjPlane];
        // rows: (top, bottom) <- (c top - s bottom, s top + c bottom), then columns
        const double x0 = ri.x * tt - ri.y * bt, y0 = ri.x * tb - ri.y * bb;
        const double x1 = ri.y * tt + ri.x * bt, y1 = ri.y * tb + ri.x * bb;
        an[to[0][0]] = rj.x * x0 - rj.y * y0;
        an[to[0][1]] = rj.y * x0 + rj.x * y0;
        an[to[1][0]] = rj.x * x1 - rj.y * y1;
        an[to[1][1]] = rj.y * x1 + rj.x * y1;
      }
      __syncthreads();
    }
    __syncthreads();
    __syncthreads();
  } else {
    constexpr int G = kBjP2 / kBjVWaves;  // slot pairs of a wavefront
    const int g = wave - 1 - kBjAWaves;
    double top[G], bot[G];
#pragma unroll
    for (int k = 0; k < G; ++k) {
      top[k] = lane == G * g + k ? 1.0 : 0.0;
      bot[k] = lane == kBjPair - 1 - (G * g + k) ? 1.0 : 0.0;
    }
    __syncthreads();
    for (int rr = 0; rr < kRounds; ++rr) {
#pragma unroll
      for (int k = 0; k < G; ++k) {
        const double2 q = cs[rr & 1][G * g + k];
        const double x = top[k], y = bot[k];
        top[k] = q.x * x - q.y * y;
        bot[k] = q.y * x + q.x * y;
      }
      xch[rr & 1][g][0][lane] = top[0];
      xch[rr & 1][g][1][lane] = bot[G - 1];
      __syncthreads();
      // one position on: tops to the left, bottoms to the right
      const double t0 = top[0], t1 = top[1], bl = bot[G - 1];
#pragma unroll
      for (int k = 0; k + 1 < G; ++k) top[k] = top[k + 1];
#pragma unroll
      for (int k = G - 1; k > 0; --k) bot[k] = bot[k - 1];
      if (g == kBjVWaves - 1) top[G - 1] = bl;
      else top[G - 1] = xch[rr & 1][g + 1][0][lane];
      if (g == 0) {
        top[0] = t0;
        bot[0] = t1;
      } else {
        bot[0] = xch[rr & 1][g - 1][1][lane];
      }
    }
    // after 63 rounds every index is back at its own position
#pragma unroll
    for (int k = 0; k < G; ++k) {
      a[lane * kBjLd + G * g + k] = top[k];
      a[lane * kBjLd + kBjPair - 1 - (G * g + k)] = bot[k];
    }
    __syncthreads();
  }
  double* out = J + (int64_t)blockIdx.x * kBjPair * kBjPair;
  for (int i = t; i < kBjPair * kBjPair; i += kBjSweepThreads)
    out[i] = a[(i / kBjPair) * kBjLd + i % kBjPair];
}

// The round's rotation applied to the matrix and to the eigenvectors.
// Workgroups [0, np^2): the piece of A in the rows of pair i and the columns
// of pair j, replaced by J_i^T piece J_j.  Workgroups [np^2, np^2 + np K/64):
// rows 64 rb .. 64 rb + 63 of V in the columns of pair j, replaced by
// piece J_j.  The pieces are disjoint, so the update is in place.
//
// Matrix cores (v_mfma_f64_16x16x4f64: A[i][c] in lane i + 16 c, B[c][j] in lane
// j + 16 c, D[i][j] in lane j + 16 (i mod 4), register i / 4).  A wavefront forms
// 16 columns of the result: first of piece J_j, whose registers are then the
// operand B of J_i^T times it, so nothing but the piece (transposed) and the
// rotations passes through LDS.  Bound by the two products at the matrix cores'
// rate on as many CUs as there are pieces: K = 256, 24 us with 256 threads on the
// vector ALUs (6 bytes of LDS per multiply-add), 16.5 with 512, 14.8 so.
constexpr int kBjUpdThreads = 256;
typedef double v4d __attribute__((ext_vector_type(4)));
__global__ void __launch_bounds__(kBjUpdThreads)
bj_update_kernel(int K, int r, double* __restrict__ Aw, double* __restrict__ Vw,
                 const double* __restrict__ J, const BjState* __restrict__ st) {
  if (st->done != 0.0) return;
  extern __shared__ double sh[];
  double* Bt = sh;                      // the piece, transposed
  double* Ji = sh + kBjPair * kBjLd;
  double* Jj = sh + 2 * kBjPair * kBjLd;
  const int t = threadIdx.x, nb = K / kBj, np = nb / 2;
  int wg = blockIdx.x;
  const bool on_a = wg < np * np;
  int i = 0, j, rb = 0;
  if (on_a) {
    i = wg / np;
    j = wg % np;
  } else {
    wg -= np * np;
    rb = wg / np;
    j = wg % np;
  }
  int Pj, Qj, Pi = 0, Qi = 0;
  round_robin(nb, r, j, Pj, Qj);
  if (on_a) round_robin(nb, r, i, Pi, Qi);
  const double* jj = J + (int64_t)j * kBjPair * kBjPair;
  const double* ji = J + (int64_t)i * kBjPair * kBjPair;
  double* base = on_a ? Aw : Vw;
#pragma unroll
  for (int e0 = 0; e0 < kBjPair * kBjPair; e0 += kBjUpdThreads) {
    const int e = e0 + t;
    const int row = e / kBjPair, col = e % kBjPair;
    const int grow = on_a ? pair_index(Pi, Qi, row) : rb * kBjPair + row;
    Bt[col * kBjLd + row] = base[(int64_t)grow * K + pair_index(Pj, Qj, col)];
    Jj[row * kBjLd + col] = jj[e];
    if (on_a) Ji[row * kBjLd + col] = ji[e];
  }
  __syncthreads();
  const int lane = t & 63, l16 = lane & 15, c4 = lane >> 4, n0 = (t >> 6) * 16;
  // M^T (16 columns of N): tile m of rows, operands M[b][row], N[b][column]
  v4d p[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) p[m] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
  for (int b = 0; b < kBjPair; b += 4) {
    const double y = Jj[(b + c4) * kBjLd + n0 + l16];
#pragma unroll
    for (int m = 0; m < 4; ++m)
      p[m] = __builtin_amdgcn_mfma_f64_16x16x4f64(Bt[(b + c4) * kBjLd + 16 * m + l16], y, p[m], 0,
                                                  0, 0);
  }
  if (on_a) {
    v4d q[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) q[m] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int b = 0; b < kBjPair; b += 4) {  // rows b .. b + 3 of the first product
      const double y = p[b / 16][(b / 4) % 4];
#pragma unroll
      for (int m = 0; m < 4; ++m)
        q[m] = __builtin_amdgcn_mfma_f64_16x16x4f64(Ji[(b + c4) * kBjLd + 16 * m + l16], y, q[m],
                                                    0, 0, 0);
    }
#pragma unroll
    for (int m = 0; m < 4; ++m) p[m] = q[m];
  }
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int row = 16 * m + 4 * u + c4;
      const int grow = on_a ? pair_index(Pi, Qi, row) : rb * kBjPair + row;
      base[(int64_t)grow * K + pair_index(Pj, Qj, n0 + l16)] = p[m][u];
    }
}

// Eigenvalues ascending by rank (ties by index), eigenvector columns moved to
// their rank and scaled by w^vpow.  Workgroup (x, y): 64 columns, rows
// y kBjOutRows ..; four threads count a column's rank.  (One thread per column
// for rank and all rows: 109 us at k = 256; this: 8 us.)
constexpr int kBjOutRows = 16;
__global__ void __launch_bounds__(256)
bj_output_kernel(int k, int K, const double* __restrict__ Aw, const double* __restrict__ Vw,
                 double* __restrict__ w, double* __restrict__ V, int64_t ldv, double vpow) {
  __shared__ double diag[kBjMaxK];
  __shared__ int cnt[256];
  const int t = threadIdx.x, c = t & 63, g = t >> 6;
  const int j = blockIdx.x * 64 + c;
  for (int i = t; i < k; i += 256) diag[i] = Aw[(int64_t)i * K + i];
  __syncthreads();
  const double lj = diag[j < k ? j : 0];
  int rank = 0;
  for (int i = g; i < k; i += 4) {
    const double li = diag[i];
    rank += (li < lj) || (li == lj && i < j);
  }
  cnt[t] = rank;
  __syncthreads();
  if (j >= k) return;
  rank = cnt[c] + cnt[c + 64] + cnt[c + 128] + cnt[c + 192];
  if (blockIdx.y == 0 && g == 0) w[rank] = lj;
  const double f = (vpow != 0.0 && lj > 0.0) ? pow(lj, vpow) : 1.0;
  const int r1 = min(k, (int)(blockIdx.y + 1) * kBjOutRows);
  for (int i = blockIdx.y * kBjOutRows + g; i < r1; i += 4)
    V[(int64_t)i * ldv + rank] = Vw[(int64_t)i * K + j] * f;
}

// status: 2 if vpow != 0 and some eigenvalue <= 0, else 0 converged / 1 not.
__global__ void bj_status_kernel(int k, int K, const double* __restrict__ Aw, double vpow,
                                 const BjState* __restrict__ st, int* __restrict__ status) {
  __shared__ int bad;
  if (threadIdx.x == 0) bad = 0;
  __syncthreads();
  if (vpow != 0.0)
    for (int j = threadIdx.x; j < k; j += blockDim.x)
      if (!(Aw[(int64_t)j * K + j] > 0.0)) atomicOr(&bad, 1);
  __syncthreads();
  if (threadIdx.x == 0) *status = bad ? 2 : (st->done != 0.0 ? 0 : 1);
}

}  // namespace

int eig_blocked_max_k() { return kBjMaxK; }

int64_t sym_eig_blocked_work(int k) {
  const int64_t K = bj_padded(k), np = K / kBjPair;
  return kBjHead + 2 * K * K + np * kBjPair * kBjPair;
}

hipError_t launch_sym_eig_blocked(int k, const double* A, int64_t lda, double* w, double* V,
                                  int64_t ldv, double vpow, int* status, double* work,
                                  hipStream_t s) {
  const int K = bj_padded(k), nb = K / kBj, np = nb / 2;
  BjState* st = reinterpret_cast<BjState*>(work);
  double* Aw = work + kBjHead;
  double* Vw = Aw + (int64_t)K * K;
  double* J = Vw + (int64_t)K * K;
  const size_t lds_upd = 3 * (size_t)kBjPair * kBjLd * sizeof(double);
  KernelFacts f;  // raise the dynamic LDS limits on this device
  hipError_t err = kernel_facts(reinterpret_cast<const void*>(bj_pair_kernel), kBjSweepThreads,
                                kBjSweepLds, f);
  if (err == hipSuccess)
    err = kernel_facts(reinterpret_cast<const void*>(bj_update_kernel), kBjUpdThreads, lds_upd, f);
  if (err != hipSuccess) return err;
  const int64_t total = (int64_t)K * K;
  const unsigned init_blocks = (unsigned)std::min<int64_t>((total + 255) / 256, 4096);
  hipLaunchKernelGGL(bj_init_kernel, dim3(init_blocks), dim3(256), 0, s, k, K, A, lda, Aw, Vw,
                     st);
  const dim3 norm_grid((unsigned)(K / kBjNormRows));
  hipLaunchKernelGGL(bj_norm_kernel, norm_grid, dim3(kBjNormThreads), 0, s, K, Aw, J, st, 1);
  const unsigned upd_blocks = (unsigned)(np * np + (K / kBjPair) * np);
  for (int sweep = 0; sweep < kBjMaxSweeps; ++sweep) {
    for (int r = 0; r < nb - 1; ++r) {
      hipLaunchKernelGGL(bj_pair_kernel, dim3(np), dim3(kBjSweepThreads), kBjSweepLds, s, K, r, Aw,
                         J, st);
      hipLaunchKernelGGL(bj_update_kernel, dim3(upd_blocks), dim3(kBjUpdThreads), lds_upd, s, K, r,
                         Aw, Vw, J, st);
    }
    hipLaunchKernelGGL(bj_norm_kernel, norm_grid, dim3(kBjNormThreads), 0, s, K, Aw, J, st, 0);
  }
  hipLaunchKernelGGL(bj_output_kernel,
                     dim3((k + 63) / 64, (k + kBjOutRows - 1) / kBjOutRows), dim3(256), 0, s, k, K,
                     Aw, Vw, w, V, ldv, vpow);
  hipLaunchKernelGGL(bj_status_kernel, dim3(1), dim3(256), 0, s, k, K, Aw, vpow, st, status);
  return hipGetLastError();
}

}  // namespace mf
