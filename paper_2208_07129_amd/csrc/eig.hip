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
// the 2 x 2 block of slot pairs (i, j) takes the row rotation of pair i and the
// column rotation of pair j at once and is stored at its place of the next
// round (two LDS copies, four planes [slot][slot] of 32 x 32, so consecutive
// lanes touch consecutive words).  Wavefront 0 forms a round's angles while the
// others apply the round before to the rotation V.  Per round two barriers, one
// pass over the block and two chains of reciprocal square roots (a division, two
// square roots and two divisions, three barriers and separate row and column
// passes before): 155 -> 63 us a launch.
constexpr int kBjSweepThreads = 512;
constexpr int kBjP2 = kBjPair / 2;                       // slot pairs
constexpr int kBjPlane = kBjP2 * kBjP2;
constexpr size_t kBjSweepLds =
    (2 * 4 * (size_t)kBjPlane + 2 * 2 * (size_t)kBjPair * kBjP2) * sizeof(double);

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

__global__ void __launch_bounds__(kBjSweepThreads)
bj_pair_kernel(int K, int r, const double* __restrict__ Aw, double* __restrict__ J,
               const BjState* __restrict__ st) {
  if (st->done != 0.0) return;
  extern __shared__ double sh[];
  double* a = sh;                        // 2 copies of 4 planes
  double* v = sh + 2 * 4 * kBjPlane;     // 2 copies of [slot][row][pair]
  constexpr int VC = 2 * kBjPair * kBjP2, VS = kBjPair * kBjP2;
  __shared__ double2 cs[2][kBjP2];
  const int t = threadIdx.x, nb = K / kBj;
  int P, Q;
  round_robin(nb, r, blockIdx.x, P, Q);
  for (int i = t; i < kBjPair * kBjPair; i += kBjSweepThreads) {
    const int row = i / kBjPair, col = i % kBjPair;
    const int si = row >= kBjP2, sj = col >= kBjP2;
    const int pi = si ? kBjPair - 1 - row : row, pj = sj ? kBjPair - 1 - col : col;
    a[(si * 2 + sj) * kBjPlane + pi * kBjP2 + pj] =
        Aw[(int64_t)pair_index(P, Q, row) * K + pair_index(P, Q, col)];
    v[sj * VS + row * kBjP2 + pj] = row == col ? 1.0 : 0.0;
  }
  __syncthreads();
  // where slot pair t's members go next round: above (0, t) and below (1, t)
  auto next = [](int slot, int pr, int& ns, int& np) {
    if (slot == 0) {
      ns = pr == 1;                       // position 1 -> 63
      np = pr == 0 ? 0 : (pr == 1 ? 0 : pr - 1);
    } else {
      ns = pr < kBjP2 - 1;                // position 32 -> 31
      np = pr < kBjP2 - 1 ? pr + 1 : kBjP2 - 1;
    }
  };
  for (int rr = 0; rr < kBjPair; ++rr) {
    if (t < 64) {
      if (t < kBjP2 && rr < kBjPair - 1) {
        const double* ac = a + (rr & 1) * 4 * kBjPlane + t * (kBjP2 + 1);
        const double top = ac[0], bot = ac[3 * kBjPlane];
        // the items at the two positions this round; p is the smaller one
        const int x0 = t == 0 ? 0 : 1 + (t - 1 + rr) % (kBjPair - 1);
        const int x1 = 1 + (kBjPair - 2 - t + rr) % (kBjPair - 1);
        double c, s;
        jacobi_angle(x0 < x1 ? top : bot, x0 < x1 ? bot : top,
                     ac[(x0 < x1 ? 1 : 2) * kBjPlane], c, s);
        cs[rr & 1][t] = make_double2(c, x0 < x1 ? s : -s);
      }
    } else if (rr > 0) {
      const double* vc = v + ((rr - 1) & 1) * VC;
      double* vn = v + (rr & 1) * VC;
      for (int i = t - 64; i < kBjPair * kBjP2; i += kBjSweepThreads - 64) {
        const int row = i / kBjP2, pj = i % kBjP2;
        const double2 r2 = cs[(rr - 1) & 1][pj];
        const double x = vc[i], y = vc[VS + i];
        int s0, p0, s1, p1;
        next(0, pj, s0, p0);
        next(1, pj, s1, p1);
        vn[s0 * VS + row * kBjP2 + p0] = r2.x * x - r2.y * y;
        vn[s1 * VS + row * kBjP2 + p1] = r2.y * x + r2.x * y;
      }
    }
    __syncthreads();
    if (rr < kBjPair - 1) {
      const double* ac = a + (rr & 1) * 4 * kBjPlane;
      double* an = a + ((rr + 1) & 1) * 4 * kBjPlane;
#pragma unroll
      for (int i = t; i < kBjPlane; i += kBjSweepThreads) {
        const int pi = i / kBjP2, pj = i % kBjP2;
        const double2 ri = cs[rr & 1][pi], rj = cs[rr & 1][pj];
        const double tt = ac[i], tb = ac[kBjPlane + i], bt = ac[2 * kBjPlane + i],
                     bb = ac[3 * kBjPlane + i];
        // rows: (top, bottom) <- (c top - s bottom, s top + c bottom), then columns
        const double x0 = ri.x * tt - ri.y * bt, y0 = ri.x * tb - ri.y * bb;
        const double x1 = ri.y * tt + ri.x * bt, y1 = ri.y * tb + ri.x * bb;
        int is[2], ip[2], js[2], jp[2];
        next(0, pi, is[0], ip[0]);
        next(1, pi, is[1], ip[1]);
        next(0, pj, js[0], jp[0]);
        next(1, pj, js[1], jp[1]);
        auto put = [&](int u, int w, double x) {
          an[(is[u] * 2 + js[w]) * kBjPlane + ip[u] * kBjP2 + jp[w]] = x;
        };
        put(0, 0, rj.x * x0 - rj.y * y0);
        put(0, 1, rj.y * x0 + rj.x * y0);
        put(1, 0, rj.x * x1 - rj.y * y1);
        put(1, 1, rj.y * x1 + rj.x * y1);
      }
    }
    __syncthreads();
  }
  // after 63 rounds every index is back at its own position
  const double* vf = v + ((kBjPair - 1) & 1) * VC;
  double* out = J + (int64_t)blockIdx.x * kBjPair * kBjPair;
  for (int i = t; i < kBjPair * kBjPair; i += kBjSweepThreads) {
    const int row = i / kBjPair, col = i % kBjPair;
    out[i] = col < kBjP2 ? vf[row * kBjP2 + col] : vf[VS + row * kBjP2 + kBjPair - 1 - col];
  }
}

// The round's rotation applied to the matrix and to the eigenvectors.
// Workgroups [0, np^2): the piece of A in the rows of pair i and the columns
// of pair j, replaced by J_i^T piece J_j.  Workgroups [np^2, np^2 + np K/64):
// rows 64 rb .. 64 rb + 63 of V in the columns of pair j, replaced by
// piece J_j.  The pieces are disjoint, so the update is in place.
// Bound by the LDS reads of the products (6 bytes per multiply-add); 512 threads
// instead of 256 hide more of the loads: 24 -> 16.5 us at K = 256.
constexpr int kBjUpdThreads = 512;
__global__ void __launch_bounds__(kBjUpdThreads)
bj_update_kernel(int K, int r, double* __restrict__ Aw, double* __restrict__ Vw,
                 const double* __restrict__ J, const BjState* __restrict__ st) {
  if (st->done != 0.0) return;
  extern __shared__ double sh[];
  double* B = sh;                       // the piece (then J_i^T piece)
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
    B[row * kBjLd + col] = base[(int64_t)grow * K + pair_index(Pj, Qj, col)];
    Jj[row * kBjLd + col] = jj[e];
    if (on_a) Ji[row * kBjLd + col] = ji[e];
  }
  __syncthreads();
  // thread (ty, tx): rows ty + 32 u, columns tx + 16 w of the 64 x 64 result
  const int ty = t / 16, tx = t % 16;
  double acc[2][4];
  if (on_a) {  // B := J_i^T B
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int w = 0; w < 4; ++w) acc[u][w] = 0.0;
    for (int b = 0; b < kBjPair; ++b) {
      double x[2], y[4];
#pragma unroll
      for (int u = 0; u < 2; ++u) x[u] = Ji[b * kBjLd + ty + 32 * u];
#pragma unroll
      for (int w = 0; w < 4; ++w) y[w] = B[b * kBjLd + tx + 16 * w];
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int w = 0; w < 4; ++w) acc[u][w] = fma(x[u], y[w], acc[u][w]);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int w = 0; w < 4; ++w) B[(ty + 32 * u) * kBjLd + tx + 16 * w] = acc[u][w];
    __syncthreads();
  }
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int w = 0; w < 4; ++w) acc[u][w] = 0.0;
  for (int b = 0; b < kBjPair; ++b) {  // B J_j
    double x[2], y[4];
#pragma unroll
    for (int u = 0; u < 2; ++u) x[u] = B[(ty + 32 * u) * kBjLd + b];
#pragma unroll
    for (int w = 0; w < 4; ++w) y[w] = Jj[b * kBjLd + tx + 16 * w];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int w = 0; w < 4; ++w) acc[u][w] = fma(x[u], y[w], acc[u][w]);
  }
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int row = ty + 32 * u;
    const int grow = on_a ? pair_index(Pi, Qi, row) : rb * kBjPair + row;
#pragma unroll
    for (int w = 0; w < 4; ++w)
      base[(int64_t)grow * K + pair_index(Pj, Qj, tx + 16 * w)] = acc[u][w];
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
  hipError_t err = kernel_facts(reinterpret_cast<const void*>(bj_pair_kernel), kBjSweepThreads, kBjSweepLds, f);
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
      hipLaunchKernelGGL(bj_pair_kernel, dim3(np), dim3(kBjSweepThreads), kBjSweepLds, s, K, r, Aw, J,
                         st);
      hipLaunchKernelGGL(bj_update_kernel, dim3(upd_blocks), dim3(kBjUpdThreads), lds_upd, s, K, r, Aw,
                         Vw, J, st);
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
