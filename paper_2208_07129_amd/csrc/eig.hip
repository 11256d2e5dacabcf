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
// round (two LDS copies of four planes [slot][slot] of 32 x 33).  The 13
// wavefronts work side by side with one barrier per round: wavefront 0 has the
// diagonal blocks in registers and forms the next round's angles, for which it
// takes the elements that meet through this round's rotations by itself; eight
// rotate the off-diagonal blocks, (i, j) and (j, i) per lane; four hold the
// rotation V in registers (lane = row, a wavefront = eight slot pairs) and pass
// two columns each to their neighbours.  155 us a launch with separate row and
// column passes and three barriers, 64.6 so with the 13 next to each other.
//
// What a round then waits for is instruction issue: wavefronts go to the four SIMDs in
// turn, which put the angles (by instruction count 800 of a round's 2400 cycles), two of
// the blocks (370 each) and one of V (420) on the first.  With three empty wavefronts in
// between, the first SIMD has the angles and one of V only, the others two or three of
// blocks and one of V: 53.9 us a launch.
//
// The arithmetic is that of the plain cyclic sweep, element by element: rows, then
// columns, p the smaller index of a pair, ap' = fma(c, ap, -(s aq)) and aq' =
// fma(s, ap, c aq), nothing taken from symmetry.  Jacobi's path is sensitive enough
// to roundings that other orders, or a shorter formula for the angle (two reciprocal
// square roots, 35 us a launch with half of the blocks), end with the signs of some
// eigenvectors changed; the same holds for the order of the update's sums.
constexpr int kBjP2 = kBjPair / 2;  // slot pairs
constexpr int kBjRow = kBjP2 + 1, kBjPlane = kBjP2 * kBjRow;
constexpr int kBjAWaves = 8, kBjVWaves = 4;  // wavefronts on the blocks, on V
constexpr int kBjSweepThreads = 1024;       // with the empty ones
constexpr size_t kBjSweepLds = 2 * 4 * (size_t)kBjPlane * sizeof(double);
static_assert(kBjAWaves + kBjVWaves <= 12, "three of every four wavefronts, and the fifth");
static_assert(kBjP2 * (kBjP2 - 1) / 2 <= 64 * kBjAWaves, "two off-diagonal blocks per lane");
static_assert(2 * 4 * kBjPlane >= kBjPair * kBjLd, "V is written out through the blocks' LDS");

// The rotation that zeroes apq, |angle| <= pi/4.
__device__ __forceinline__ void jacobi_angle(double app, double aqq, double apq, double& c,
                                             double& s) {
  c = 1.0;
  s = 0.0;
  if (fabs(apq) > 1e-300) {
    const double th = (aqq - app) / (2.0 * apq);
    const double at = fabs(th);
    const double tn =
        (th >= 0.0 ? 1.0 : -1.0) / (at + (at < 1e150 ? sqrt(fma(th, th, 1.0)) : at));
    c = 1.0 / sqrt(fma(tn, tn, 1.0));
    s = tn * c;
  }
}
// The rotated pair (p, q).
__device__ __forceinline__ double rot_p(double c, double s, double p, double q) {
  return fma(c, p, -(s * q));
}
__device__ __forceinline__ double rot_q(double c, double s, double p, double q) {
  return fma(s, p, c * q);
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
// The place next round of element (member u of pair pi, member w of pair pj).
__device__ __forceinline__ int bj_place(int u, int pi, int w, int pj) {
  int is, ip, js, jp;
  bj_next(u, pi, is, ip);
  bj_next(w, pj, js, jp);
  return (is * 2 + js) * kBjPlane + ip * kBjRow + jp;
}

__global__ void __launch_bounds__(kBjSweepThreads)
bj_pair_kernel(int K, int r, const double* __restrict__ Aw, double* __restrict__ J,
               const BjState* __restrict__ st) {
  if (st->done != 0.0) return;
  extern __shared__ double sh[];
  double* a = sh;  // 2 copies of 4 planes
  constexpr int kCopy = 4 * kBjPlane;
  __shared__ double2 cs[2][kBjP2];             // (c, s); -c where the lower member is p
  __shared__ double dg[2][2][kBjP2];           // rotated diagonal, [round][slot][pair]
  __shared__ double xch[2][kBjVWaves][2][64];  // V's columns on their way to a neighbour
  const int t = threadIdx.x, nb = K / kBj, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  constexpr int kRounds = kBjPair - 1;
  // the angles, blocks 1 .., V, or (above) nothing to do
  int role = 1 + kBjAWaves + kBjVWaves;
  if ((wave & 3) == 0) {
    if (wave == 0) role = 0;
    if (wave == 4) role = kBjAWaves + kBjVWaves;
  } else {
    const int n = (wave >> 2) * 3 + (wave & 3);  // 1..12
    if (n < kBjAWaves + kBjVWaves) role = n;
  }
  int P, Q;
  round_robin(nb, r, blockIdx.x, P, Q);
  for (int i = t; i < kBjPair * kBjPair; i += kBjSweepThreads) {
    const int row = i / kBjPair, col = i % kBjPair;
    const int si = row >= kBjP2, sj = col >= kBjP2;
    const int pi = si ? kBjPair - 1 - row : row, pj = sj ? kBjPair - 1 - col : col;
    a[(si * 2 + sj) * kBjPlane + pi * kBjRow + pj] =
        Aw[(int64_t)pair_index(P, Q, row) * K + pair_index(P, Q, col)];
  }
  __syncthreads();
  if (role == 0) {
    __builtin_amdgcn_s_setprio(3);  // the chain that every round waits for
    const int p = lane & (kBjP2 - 1), dia = p * kBjRow + p;
    // the pair's block, [slot][slot]
    double dtt = a[dia], dtb = a[kBjPlane + dia], dbt = a[2 * kBjPlane + dia],
           dbb = a[3 * kBjPlane + dia], c, s;
    int i0 = p, i1 = kBjPair - 1 - p;  // the items at the two positions
    auto angle = [&]() {
      const bool up = i0 < i1;
      jacobi_angle(up ? dtt : dbb, up ? dbb : dtt, up ? dtb : dbt, c, s);
    };
    angle();
    if (lane < kBjP2) cs[0][p] = make_double2(i0 < i1 ? c : -c, s);
    __syncthreads();
    // the members of slot pair p next round sit in (u, pu) and (w, pw) now
    const int u = p == kBjP2 - 1 ? 1 : 0, pu = p == kBjP2 - 1 ? p : (p == 0 ? 0 : p + 1);
    const int w = p == 0 ? 0 : 1, pw = p == 0 ? 1 : p - 1;
    const int to_tb = bj_place(0, p, 1, p), to_bt = bj_place(1, p, 0, p);
    for (int rr = 0; rr + 1 < kRounds; ++rr) {
      const double* ac = a + (rr & 1) * kCopy;
      double* an = a + ((rr + 1) & 1) * kCopy;
      const double2 ru = cs[rr & 1][pu], rw = cs[rr & 1][pw];
      const double cu = fabs(ru.x), su = ru.y, cw = fabs(rw.x), sw = rw.y;
      const int fu = __double2hiint(ru.x) < 0, fw = __double2hiint(rw.x) < 0;  // slot of p
      // element (member m of pair x, member n of pair y) after this round
      auto meet = [&](int x, int m, int fx, double cx, double sx, int y, int n, int fy, double cy,
                      double sy) {
        const double* e = ac + x * kBjRow + y;
        const double pp = e[(fx * 2 + fy) * kBjPlane], pq = e[(fx * 2 + 1 - fy) * kBjPlane];
        const double qp = e[((1 - fx) * 2 + fy) * kBjPlane],
                     qq = e[((1 - fx) * 2 + 1 - fy) * kBjPlane];
        const bool rp = m == fx, cp = n == fy;
        const double ra = rp ? cx : sx, rb = rp ? -sx : cx;
        const double ca = cp ? cy : sy, cb = cp ? -sy : cy;
        const double yp = fma(ra, pp, rb * qp), yq = fma(ra, pq, rb * qq);
        return fma(ca, yp, cb * yq);
      };
      const double ntb = meet(pu, u, fu, cu, su, pw, w, fw, cw, sw);
      const double nbt = meet(pw, w, fw, cw, sw, pu, u, fu, cu, su);
      // this round's rotation of the pair's own block, handed on to the next places
      {
        const bool up = i0 < i1;
        const double pp = up ? dtt : dbb, pq = up ? dtb : dbt, qp = up ? dbt : dtb,
                     qq = up ? dbb : dtt;
        const double yp = rot_p(c, s, pp, qp), yq = rot_p(c, s, pq, qq);
        const double zp = rot_q(c, s, pp, qp), zq = rot_q(c, s, pq, qq);
        const double npp = rot_p(c, s, yp, yq), npq = rot_q(c, s, yp, yq);
        const double nqp = rot_p(c, s, zp, zq), nqq = rot_q(c, s, zp, zq);
        if (lane < kBjP2) {
          dg[rr & 1][0][p] = up ? npp : nqq;
          dg[rr & 1][1][p] = up ? nqq : npp;
          an[to_tb] = up ? npq : nqp;
          an[to_bt] = up ? nqp : npq;
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      dtt = dg[rr & 1][u][pu];
      dbb = dg[rr & 1][w][pw];
      dtb = ntb;
      dbt = nbt;
      i0 = p == 0 ? 0 : (i0 == kRounds ? 1 : i0 + 1);
      i1 = i1 == kRounds ? 1 : i1 + 1;
      angle();
      if (lane < kBjP2) cs[(rr + 1) & 1][p] = make_double2(i0 < i1 ? c : -c, s);
      __syncthreads();
    }
    __syncthreads();
    __syncthreads();
  } else if (role <= kBjAWaves) {
    // off-diagonal blocks (pi, pj) and (pj, pi), pi < pj: rows fr and 30 - fr of the
    // triangle fill 32 lanes
    const int e = (role - 1) * 64 + lane, fr = e / kBjP2, fk = e % kBjP2;
    const bool upper = fk < kBjP2 - 1 - fr;
    const int pi = upper ? fr : kBjP2 - 2 - fr, pj = upper ? fr + 1 + fk : fk;
    const bool on = fr < kBjP2 / 2 - 1 || upper;
    int to[2][2][2];  // [block][member][member]
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        to[0][m][n] = bj_place(m, pi, n, pj);
        to[1][m][n] = bj_place(m, pj, n, pi);
      }
    __syncthreads();
    for (int rr = 0; rr + 1 < kRounds; ++rr) {
      const double* ac = a + (rr & 1) * kCopy;
      double* an = a + ((rr + 1) & 1) * kCopy;
      if (on) {
        const double2 r0 = cs[rr & 1][pi], r1 = cs[rr & 1][pj];
        const int f0 = __double2hiint(r0.x) < 0, f1 = __double2hiint(r1.x) < 0;
        auto block = [&](int x, int y, int fx, int fy, double cx, double sx, double cy, double sy,
                         const int (&dst)[2][2]) {
          const double* b = ac + x * kBjRow + y;
          const int px = fx * 2 * kBjPlane, qx = 2 * kBjPlane - px, py = fy * kBjPlane,
                    qy = kBjPlane - py;
          const double pp = b[px + py], pq = b[px + qy], qp = b[qx + py], qq = b[qx + qy];
          const double yp = rot_p(cx, sx, pp, qp), yq = rot_p(cx, sx, pq, qq);
          const double zp = rot_q(cx, sx, pp, qp), zq = rot_q(cx, sx, pq, qq);
          const int d0p = fy ? dst[0][1] : dst[0][0], d0q = fy ? dst[0][0] : dst[0][1];
          const int d1p = fy ? dst[1][1] : dst[1][0], d1q = fy ? dst[1][0] : dst[1][1];
          an[fx ? d1p : d0p] = rot_p(cy, sy, yp, yq);
          an[fx ? d1q : d0q] = rot_q(cy, sy, yp, yq);
          an[fx ? d0p : d1p] = rot_p(cy, sy, zp, zq);
          an[fx ? d0q : d1q] = rot_q(cy, sy, zp, zq);
        };
        block(pi, pj, f0, f1, fabs(r0.x), r0.y, fabs(r1.x), r1.y, to[0]);
        block(pj, pi, f1, f0, fabs(r1.x), r1.y, fabs(r0.x), r0.y, to[1]);
      }
      __syncthreads();
    }
    __syncthreads();
    __syncthreads();
  } else if (role > kBjAWaves + kBjVWaves) {  // as many barriers as the others
    for (int rr = 0; rr < kRounds + 2; ++rr) __syncthreads();
  } else {
    constexpr int G = kBjP2 / kBjVWaves;  // slot pairs of a wavefront
    const int g = role - 1 - kBjAWaves;
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
        const double2 q2 = cs[rr & 1][G * g + k];
        const double c = fabs(q2.x), s = q2.y;
        const bool up = __double2hiint(q2.x) >= 0;
        const double x = up ? top[k] : bot[k], y = up ? bot[k] : top[k];
        const double xr = rot_p(c, s, x, y), yr = rot_q(c, s, x, y);
        top[k] = up ? xr : yr;
        bot[k] = up ? yr : xr;
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
// Bound by the LDS reads of the products (6 bytes per multiply-add); 512 threads
// instead of 256 hide more of the loads: 24 -> 18 us at K = 256.
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
