// Dispatch of the fused apply by polynomial degree, and the zero-fill kernel.
#include <algorithm>

#include "mf_internal.h"
#include "sf_common.h"

namespace mf {

namespace {

// Y rows [0, nrows) x columns [0, ncols) := 0.  A kernel rather than a memset
// so that it also clears strided (ld > ncols) outputs and can be captured in a
// graph.
__global__ void zero_rows_kernel(double* __restrict__ Y, int64_t nrows, int ncols, int64_t ld) {
  const int64_t total = nrows * ncols;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = i / ncols, c = i % ncols;
    Y[r * ld + c] = 0.0;
  }
}

// X[i] := a fixed pseudo-random value in [-1, 1) (an integer hash of i): the
// input the launch-shape tuner times the kernels on.
__global__ void fill_pattern_kernel(double* __restrict__ X, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    uint64_t h = (uint64_t)i * 0x9E3779B97F4A7C15ull;
    h ^= h >> 29;
    X[i] = (double)(h >> 44) * (1.0 / (1 << 19)) - 1.0;
  }
}

// FP64 FMA issue-rate probe: every thread runs `iters` rounds of 8
// independent FMA chains (no loads), then writes their sum so nothing is
// dropped.  8 iters x 2 flops per thread and round.
__global__ void __launch_bounds__(256) fma_probe_kernel(int64_t iters, double seed, double* out) {
  double v[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) v[c] = seed + c + threadIdx.x * 1e-3;
  const double a = 0.999999, b = 1e-7;
#pragma unroll 4
  for (int64_t i = 0; i < iters; ++i)
#pragma unroll
    for (int c = 0; c < 8; ++c) v[c] = fma(v[c], a, b);
  double s = 0.0;
#pragma unroll
  for (int c = 0; c < 8; ++c) s += v[c];
  out[(int64_t)blockIdx.x * blockDim.x + threadIdx.x] = s;
}

// Node lines (gy, gz) of the Nx x Ny x Nz grid, each taken whole by `team`
// threads, a workgroup or one of its wavefronts (a grid-stride loop when there are
// fewer teams than lines).
// A line on a shared plane (gz a multiple of p, gy a multiple of py or equal to
// ylast) is zeroed whole; otherwise only the rows gx = 0, p, 2p, ... are.  Threads form (row, column)
// pairs, the columns of a row on cw = 2^cw_log2 consecutive lanes (the next
// power of two >= ncols, at most 64), so narrow multivectors keep every lane
// busy and wide ones store 64 contiguous columns at a time.  Rows of
// cell-interior nodes are skipped: the box kernel writes them.
__global__ void zero_shared_rows_kernel(double* __restrict__ Y, int Nx, int Ny, int p, int py,
                                        int ylast, int ncols, int64_t ld, int64_t lines,
                                        int cw_log2, int team) {
  const int cw = 1 << cw_log2;
  const int t = threadIdx.x & (team - 1), teams = blockDim.x / team;
  const int c0 = t & (cw - 1);
  const int r0 = t >> cw_log2, rstep = team >> cw_log2;
  for (int64_t line = (int64_t)blockIdx.x * teams + threadIdx.x / team; line < lines;
       line += (int64_t)gridDim.x * teams) {
    const int gz = (int)((uint32_t)line / (uint32_t)Ny), gy = (int)line - gz * Ny;
    const bool full = (gy % py == 0) || gy == ylast || (gz % p == 0);
    const int step = full ? 1 : p;
    const int nrows = full ? Nx : (Nx + p - 1) / p;
    double* base = Y + line * Nx * ld;
    for (int r = r0; r < nrows; r += rstep) {
      double* row = base + (int64_t)r * step * ld;
      for (int c = c0; c < ncols; c += cw) row[c] = 0.0;
    }
  }
}

// Chebyshev step initialisation: the face rows of the zero fill's line walk
// (cell-interior rows are written by the fused kernel) get b Y + c Xp, and
// constrained rows (the boundary of a zero-Dirichlet mesh) 0.
__global__ void cheb_init_kernel(const double* __restrict__ Y, const double* Xp, double* Out,
                                 int Nx, int Ny, int Nz, int p, int py, int ylast, int dirichlet,
                                 int ncols, int64_t ld, double b, double c) {
  const int line = blockIdx.x;
  const int gy = line % Ny, gz = line / Ny;
  const bool full = (gy % py == 0) || gy == ylast || (gz % p == 0);
  const bool yz_bnd = dirichlet && (gy == 0 || gy == Ny - 1 || gz == 0 || gz == Nz - 1);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const int step = full ? 1 : p;
  for (int gx = wave * step; gx < Nx; gx += nw * step) {
    const int64_t row = ((int64_t)line * Nx + gx) * ld;
    const bool cons = yz_bnd || (dirichlet && (gx == 0 || gx == Nx - 1));
    for (int j = lane; j < ncols; j += 64) {
      double v = 0.0;
      if (!cons) {
        v = b * Y[row + j];
        if (Xp) v = fma(c, Xp[row + j], v);
      }
      Out[row + j] = v;
    }
  }
}

// GLL-lumped mass: per cell and local node, w_a w_b w_c det J added to the
// node's row (the GLL rule of the element's own nodes makes the mass
// diagonal).
struct GllWeights {
  double w[kMaxP + 1];
};
__global__ void gll_mass_kernel(GridDesc g, int np, GllWeights wt, double detj,
                                double* __restrict__ m) {
  const int e = blockIdx.x;
  const int cx = e % g.n[0], cy = (e / g.n[0]) % g.n[1], cz = e / (g.n[0] * g.n[1]);
  const int F = np * np * np;
  for (int i = threadIdx.x; i < F; i += blockDim.x) {
    const int i1 = i % np, i2 = (i / np) % np, i3 = i / (np * np);
    const int node = grid_node(g, cx, cy, cz, i1, i2, i3);
    if (node >= 0) unsafeAtomicAdd(m + node, wt.w[i1] * wt.w[i2] * wt.w[i3] * detj);
  }
}
__global__ void inv_sqrt_kernel(double* __restrict__ m, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    m[i] = m[i] > 0.0 ? 1.0 / sqrt(m[i]) : 0.0;
}

// Batched form: kBatchZeroSplit workgroups per node plane gz of any operator of
// the batch, each taking a contiguous share of the plane's face rows
// (per-line workgroups are too small for the batch's small meshes and column
// counts).  A plane on a cell face (gz a multiple of p) is zeroed whole;
// otherwise its face rows are enumerated as k = 0 .. n-1: first the lines
// gy = 0, p, 2p, ... whole, then the rows gx = 0, p, 2p, ... of the other
// lines.  Lanes take columns in groups of the next power of two >= ncols (up
// to 64), so a wavefront stores 64 / group rows at a time.
constexpr int kBatchZeroSplit = 16;

__global__ void batch_zero_kernel(const BatchOp* __restrict__ ops,
                                  const uint8_t* __restrict__ plane_op, BatchPtrs ptrs,
                                  int64_t first) {
  const int64_t g = first + blockIdx.x;
  const int o = plane_op[g];
  const BatchOp& op = ops[o];
  const int gz = (int)(g - op.plane_begin);
  const int Nx = op.nodes[0], Ny = op.nodes[1], p = op.p;
  const int64_t ld = ptrs.ldy[o];
  const int ncols = ptrs.nvec[o];
  double* base = ptrs.Y[o] + (int64_t)gz * Nx * Ny * ld;
  const bool full = p == 1 || gz % p == 0;
  const int nyf = (Ny + p - 1) / p, nxf = (Nx + p - 1) / p;
  const int64_t nrows = full ? (int64_t)Nx * Ny : (int64_t)nyf * Nx + (int64_t)(Ny - nyf) * nxf;
  int lpr = 1;
  while (lpr < ncols && lpr < 64) lpr *= 2;
  const int rpw = 64 / lpr;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const int sub = lane / lpr, c0 = lane % lpr;
  // a plane has fewer than 2^31 nodes: the row numbers in 32 bits (their divisions in
  // 64 bits: 64 small meshes 25 us, so 23)
  const uint32_t k0 = (uint32_t)(nrows * blockIdx.y / gridDim.y),
                 k1 = (uint32_t)(nrows * (blockIdx.y + 1) / gridDim.y);
  const uint32_t nx = Nx, face = (uint32_t)nyf * nx, nf = nxf, pm = p > 1 ? p - 1 : 1;
  for (uint32_t k = k0 + wave * rpw + sub; k < k1; k += nw * rpw) {
    uint32_t row;
    if (full) {
      row = k;
    } else if (k < face) {
      const uint32_t y = k / nx;
      row = y * p * nx + (k - y * nx);
    } else {
      const uint32_t kk = k - face, j = kk / nf;
      row = (j + j / pm + 1) * nx + (kk - j * nf) * p;
    }
    double* dst = base + (int64_t)row * ld;
    for (int c = c0; c < ncols; c += lpr) dst[c] = 0.0;
  }
}

}  // namespace

hipError_t launch_batch_zero(const BatchOp* ops, const uint8_t* plane_op, const BatchPtrs& ptrs,
                             int64_t first, int64_t planes, hipStream_t s) {
  if (planes < 1) return hipSuccess;
  hipLaunchKernelGGL(batch_zero_kernel, dim3((unsigned)planes, kBatchZeroSplit), dim3(256), 0, s,
                     ops, plane_op, ptrs, first);
  return hipGetLastError();
}

hipError_t launch_batched(int prec, int bcfg, const BatchOp* ops, const uint8_t* item_op,
                          const int64_t* bounds, const BatchPtrs& ptrs, int grid, hipStream_t s) {
#define MF_BATCH_CASE(P, C)                                                                  \
  if (prec == P && bcfg == C)                                                                \
    return launch_batched_kernel<P, C>(ops, item_op, bounds, ptrs, grid, s);
  MF_BATCH_CASE(MF_FP64, 0) MF_BATCH_CASE(MF_FP64, 1) MF_BATCH_CASE(MF_FP64, 2)
  MF_BATCH_CASE(MF_FP32, 0) MF_BATCH_CASE(MF_FP32, 1) MF_BATCH_CASE(MF_FP32, 2)
  MF_BATCH_CASE(MF_BF16, 0) MF_BATCH_CASE(MF_BF16, 1) MF_BATCH_CASE(MF_BF16, 2)
#undef MF_BATCH_CASE
  return hipErrorInvalidValue;
}

hipError_t launch_batched_kind_any(int prec, int p, bool loop, const BatchOp* ops,
                                   const uint8_t* item_op,
                                   const int64_t* bounds, const BatchPtrs& ptrs, int grid,
                                   hipStream_t s) {
  if (prec == MF_FP64)
    return launch_batched_kind<MF_FP64>(p, loop, ops, item_op, bounds, ptrs, grid, s);
  if (prec == MF_FP32)
    return launch_batched_kind<MF_FP32>(p, loop, ops, item_op, bounds, ptrs, grid, s);
  if (prec == MF_BF16)
    return launch_batched_kind<MF_BF16>(p, loop, ops, item_op, bounds, ptrs, grid, s);
  return hipErrorInvalidValue;
}

int batched_kind_blocks_per_cu(int prec, int p) {
  if (prec == MF_FP64) return batched_kind_occupancy<MF_FP64>(p);
  if (prec == MF_FP32) return batched_kind_occupancy<MF_FP32>(p);
  if (prec == MF_BF16) return batched_kind_occupancy<MF_BF16>(p);
  return 0;
}

int batched_blocks_per_cu(int prec, int bcfg) {
#define MF_BATCH_CASE(P, C) \
  if (prec == P && bcfg == C) return batched_occupancy<P, C>();
  MF_BATCH_CASE(MF_FP64, 0) MF_BATCH_CASE(MF_FP64, 1) MF_BATCH_CASE(MF_FP64, 2)
  MF_BATCH_CASE(MF_FP32, 0) MF_BATCH_CASE(MF_FP32, 1) MF_BATCH_CASE(MF_FP32, 2)
  MF_BATCH_CASE(MF_BF16, 0) MF_BATCH_CASE(MF_BF16, 1) MF_BATCH_CASE(MF_BF16, 2)
#undef MF_BATCH_CASE
  return 0;
}

// The last plane of nodes in y where it is a cell face of its own (free direction).
static int last_face_y(const int64_t* nodes, int p) {
  return nodes[1] % p == 1 || p == 1 ? (int)nodes[1] - 1 : -1;
}

constexpr int64_t kNarrowLine = 512;  // rows times columns of a line
hipError_t launch_zero_shared_rows(double* Y, const int64_t nodes[3], int p, int py, int ncols,
                                   int64_t ld, hipStream_t s) {
  const int64_t lines = nodes[1] * nodes[2];
  if (lines < 1 || ncols < 1) return hipSuccess;
  int cw_log2 = 0;
  while (cw_log2 < 6 && (1 << cw_log2) < ncols) ++cw_log2;
  // about 2048 grid elements per workgroup (some 7 KB of face rows), at least
  // one workgroup per CU, at most one per line
  int64_t wgs = nodes[0] * lines * ncols / 2048;
  if (wgs < 256) wgs = 256;
  if (wgs > lines) wgs = lines;
  // Lines of few elements go to single wavefronts, a line or a few each: with a
  // workgroup per line most of its threads have no row (one column, between events: p = 6,
  // 16^3 12.9 -> 7.2 us, 30^3 23 -> 13; four columns, 16^3 10.8 -> 8.0; but lines of 8 rows and
  // 200 columns 11.3, with single wavefronts 12.0).
  const bool narrow = nodes[0] * std::max(ncols, 1 << cw_log2) <= kNarrowLine;
  if (narrow) wgs = std::min<int64_t>((lines + 3) / 4, 4096);
  hipLaunchKernelGGL(zero_shared_rows_kernel, dim3((unsigned)wgs), dim3(256), 0, s, Y,
                     (int)nodes[0], (int)nodes[1], p, py, last_face_y(nodes, p), ncols, ld, lines,
                     cw_log2, narrow ? 64 : 256);
  return hipGetLastError();
}

hipError_t launch_cheb_init(const Operator& op, const double* Y, const double* Xp, double* Out,
                            int64_t ld, int nvec, double b, double c, int py, hipStream_t s) {
  const int64_t lines = op.nodes[1] * op.nodes[2];
  if (lines < 1) return hipSuccess;
  hipLaunchKernelGGL(cheb_init_kernel, dim3((unsigned)lines), dim3(256), 0, s, Y, Xp, Out,
                     (int)op.nodes[0], (int)op.nodes[1], (int)op.nodes[2], op.p, py,
                     last_face_y(op.nodes, op.p), op.grid.dirichlet, nvec, ld, b, c);
  return hipGetLastError();
}

// The same over an explicit map with a det J per cell (refined meshes).
__global__ void gll_mass_map_kernel(const int32_t* __restrict__ map,
                                    const double* __restrict__ detj, int np, GllWeights wt,
                                    double* __restrict__ m) {
  const int64_t e = blockIdx.x;
  const int F = np * np * np;
  const double dj = detj[e];
  for (int i = threadIdx.x; i < F; i += blockDim.x) {
    const int i1 = i % np, i2 = (i / np) % np, i3 = i / (np * np);
    const int node = map[e * F + i];
    if (node >= 0) unsafeAtomicAdd(m + node, wt.w[i1] * wt.w[i2] * wt.w[i3] * dj);
  }
}

// Row-major elementwise passes over n rows x nvec columns: one row per
// wavefront step, lane = column (no per-element division).
__global__ void scale_rows_kernel(int64_t n, int nvec, const double* __restrict__ D,
                                  const double* __restrict__ Y, int64_t ld,
                                  double* __restrict__ W) {
  const int lane = threadIdx.x % 64;
  const int64_t waves = (int64_t)gridDim.x * (blockDim.x / 64);
  for (int64_t r = (int64_t)blockIdx.x * (blockDim.x / 64) + threadIdx.x / 64; r < n; r += waves) {
    const double d = D[r];
    for (int j = lane; j < nvec; j += 64) W[r * nvec + j] = d * Y[r * ld + j];
  }
}

// Xp may alias Out: each element is read before it is written, by one thread.
__global__ void cheb_combine_kernel(int64_t n, int nvec, const double* __restrict__ D,
                                    const double* __restrict__ V, const double* __restrict__ Y,
                                    const double* Xp, double* Out, int64_t ld, double a, double b,
                                    double c) {
  const int lane = threadIdx.x % 64;
  const int64_t waves = (int64_t)gridDim.x * (blockDim.x / 64);
  for (int64_t r = (int64_t)blockIdx.x * (blockDim.x / 64) + threadIdx.x / 64; r < n; r += waves) {
    const double d = D[r];
    for (int j = lane; j < nvec; j += 64) {
      const int64_t at = r * ld + j;
      double v = 0.0;
      if (d != 0.0) {
        v = a * d * V[r * nvec + j] + b * Y[at];
        if (Xp) v += c * Xp[at];
      }
      Out[at] = v;
    }
  }
}

static unsigned grid_1d(int64_t total) {
  int64_t blocks = (total + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  return (unsigned)(blocks < 1 ? 1 : blocks);
}

hipError_t launch_gll_mass_map(const Operator& op, double* out, hipStream_t s) {
  hipLaunchKernelGGL(zero_rows_kernel, dim3(grid_1d(op.ndofs)), dim3(256), 0, s, out, op.ndofs, 1,
                     (int64_t)1);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  GllWeights wt{};
  for (int i = 0; i < op.np && i <= kMaxP; ++i) wt.w[i] = op.wgll[i];
  hipLaunchKernelGGL(gll_mass_map_kernel, dim3((unsigned)op.ncells), dim3(256), 0, s, op.d_map,
                     op.d_detj, op.np, wt, out);
  return hipGetLastError();
}

hipError_t launch_inv_sqrt(double* m, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(inv_sqrt_kernel, dim3(grid_1d(n)), dim3(256), 0, s, m, n);
  return hipGetLastError();
}

// four rows per 256-thread workgroup step, at most 65536 workgroups
static unsigned grid_rows(int64_t n) {
  int64_t blocks = (n + 3) / 4;
  if (blocks > 65536) blocks = 65536;
  return (unsigned)(blocks < 1 ? 1 : blocks);
}

hipError_t launch_scale_rows(int64_t n, int nvec, const double* D, const double* Y, int64_t ld,
                             double* W, hipStream_t s) {
  hipLaunchKernelGGL(scale_rows_kernel, dim3(grid_rows(n)), dim3(256), 0, s, n, nvec, D, Y, ld, W);
  return hipGetLastError();
}

hipError_t launch_cheb_combine(int64_t n, int nvec, const double* D, const double* V,
                               const double* Y, const double* Xp, double* Out, int64_t ld,
                               double a, double b, double c, hipStream_t s) {
  hipLaunchKernelGGL(cheb_combine_kernel, dim3(grid_rows(n)), dim3(256), 0, s, n, nvec, D, V, Y,
                     Xp, Out, ld, a, b, c);
  return hipGetLastError();
}

hipError_t launch_gll_mass(const Operator& op, int inv_sqrt, double* out, hipStream_t s) {
  const int64_t n = op.ndofs;
  unsigned blocks = (unsigned)((n + 255) / 256 > 65536 ? 65536 : (n + 255) / 256);
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(zero_rows_kernel, dim3(blocks), dim3(256), 0, s, out, n, 1, (int64_t)1);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  GllWeights wt{};
  for (int i = 0; i < op.np && i <= kMaxP; ++i) wt.w[i] = op.wgll[i];
  hipLaunchKernelGGL(gll_mass_kernel, dim3((unsigned)op.ncells), dim3(256), 0, s, op.grid, op.np,
                     wt, op.detj, out);
  err = hipGetLastError();
  if (err != hipSuccess || !inv_sqrt) return err;
  hipLaunchKernelGGL(inv_sqrt_kernel, dim3(blocks), dim3(256), 0, s, out, n);
  return hipGetLastError();
}

hipError_t launch_apply_cheb(const Operator& op, const double* Y, double* Out, int64_t ld,
                             int nvec, const ChebArgs& ca, hipStream_t s) {
  switch (op.p) {
    case 1: return launch_cheb_p<1>(op, Y, Out, ld, nvec, ca, s);
    case 2: return launch_cheb_p<2>(op, Y, Out, ld, nvec, ca, s);
    case 3: return launch_cheb_p<3>(op, Y, Out, ld, nvec, ca, s);
    case 4: return launch_cheb_p<4>(op, Y, Out, ld, nvec, ca, s);
    case 5: return launch_cheb_p<5>(op, Y, Out, ld, nvec, ca, s);
    case 6: return launch_cheb_p<6>(op, Y, Out, ld, nvec, ca, s);
    case 7: return launch_cheb_p<7>(op, Y, Out, ld, nvec, ca, s);
    case 8: return launch_cheb_p<8>(op, Y, Out, ld, nvec, ca, s);
    case 9: return launch_cheb_p<9>(op, Y, Out, ld, nvec, ca, s);
    case 10: return launch_cheb_p<10>(op, Y, Out, ld, nvec, ca, s);
    default: return hipErrorInvalidValue;
  }
}

bool apply_box_supported(int p, int q, int cfg) {
  if (p < 1 || p > kMaxP || q < p + 1 || q > p + kMaxQExtra || cfg < 0 || cfg >= kBoxCfgs)
    return false;
  if (cfg == kBoxMfmaCfg) return q == p + 1 && q <= kMfmaMaxN;
  return box_cfg(p + 1, q, cfg).B > 0;
}

int choose_cfg_box(int np, int nq, int nvec) {
  // the default shape, unless the columns fill a smaller tile better
  const int b0 = box_cfg(np, nq, 0).B;
  if (nvec >= b0) return 0;
  int best = 0, bestB = b0;
  for (int c = 1; c < kBoxCfgs; ++c) {
    if (c == kBoxMfmaCfg) continue;
    const int b = box_cfg(np, nq, c).B;
    if (b >= nvec && b < bestB) {
      best = c;
      bestB = b;
    }
  }
  return best;
}

bool apply_mixed_supported(int p, int q, int cfg) {
  if (p < 1 || p > kMaxP || q < p + 1 || q > p + kMaxQExtra || cfg < 0 || cfg >= kMixedCfgs)
    return false;
  if (cfg >= kMixedMfmaCfgs) return vec32_cfg(p + 1, q, cfg).B > 0;
  return mixed_cfg(p + 1, q, cfg).B > 0;
}

int choose_cfg_mixed(int np, int nq, int nvec, int prec) {
  if (prec == MF_FP32) {
    // FP32: the vector shapes measured fastest (p = 6: 0.42 vs 0.50 ms for the
    // matrix-core shape at nvec 64; p = 8: 0.42 vs 0.61 ms): 16 columns, one per
    // thread, where the workgroup fits, else 8; 8 for narrow multivectors.
    if (nvec > 8 && vec32_cfg(np, nq, 6).B > 0) return 6;
    if (vec32_cfg(np, nq, 5).B > 0) return 5;
  }
  const int b0 = mixed_cfg(np, nq, 0).B;
  if (nvec >= b0) return 0;
  int best = 0, bestB = b0;
  for (int c = 1; c < kMixedMfmaCfgs; ++c) {
    const int b = mixed_cfg(np, nq, c).B;
    if (b >= nvec && b < bestB) {
      best = c;
      bestB = b;
    }
  }
  return best;
}

hipError_t launch_apply_mixed(const Operator& op, const ApplyLaunch& a, int prec, hipStream_t s) {
  switch (op.p) {
    case 1: return launch_apply_mixed_p<1>(op, a, prec, s);
    case 2: return launch_apply_mixed_p<2>(op, a, prec, s);
    case 3: return launch_apply_mixed_p<3>(op, a, prec, s);
    case 4: return launch_apply_mixed_p<4>(op, a, prec, s);
    case 5: return launch_apply_mixed_p<5>(op, a, prec, s);
    case 6: return launch_apply_mixed_p<6>(op, a, prec, s);
    case 7: return launch_apply_mixed_p<7>(op, a, prec, s);
    case 8: return launch_apply_mixed_p<8>(op, a, prec, s);
    case 9: return launch_apply_mixed_p<9>(op, a, prec, s);
    case 10: return launch_apply_mixed_p<10>(op, a, prec, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_apply_box(const Operator& op, const ApplyLaunch& a, hipStream_t s) {
  switch (op.p) {
    case 1: return launch_apply_box_p<1>(op, a, s);
    case 2: return launch_apply_box_p<2>(op, a, s);
    case 3: return launch_apply_box_p<3>(op, a, s);
    case 4: return launch_apply_box_p<4>(op, a, s);
    case 5: return launch_apply_box_p<5>(op, a, s);
    case 6: return launch_apply_box_p<6>(op, a, s);
    case 7: return launch_apply_box_p<7>(op, a, s);
    case 8: return launch_apply_box_p<8>(op, a, s);
    case 9: return launch_apply_box_p<9>(op, a, s);
    case 10: return launch_apply_box_p<10>(op, a, s);
    default: return hipErrorInvalidValue;
  }
}

// The accumulating form is built for at most three points per direction: its read of
// a stored row waits for the additions issued before it, which more points cost more
// than the form gains (box kernel against this, us: p = 6, 16^3, 64 columns 563 / 768,
// 16 columns 112 / 152; p = 4, 24^3, 64 columns 550 / 698; p = 3, 20^3, 24 columns -25 %;
// p = 2, 32^3, 64 columns 405 / 252, one column 41 / 27; p = 1, 40^3, 16 columns 66 / 56).
bool pair_built(int q, bool accumulate) { return q <= (accumulate ? kPairAccumMaxQ : 7); }

// Work of the register-resident form: cells (groups of cells in x) times column tiles per
// resident wavefront.
static double pair_steps(const Operator& op, int nvec, int cols) {
  const int lx = pair_cells(cols);
  return (double)((op.grid.n[0] + lx - 1) / lx) * op.grid.n[1] * op.grid.n[2] *
         ((nvec + cols - 1) / cols) / (1024.0 * pair_waves(op.nq));
}

// The steps (pair_steps) from which the register-resident apply is the faster one, < 0 where
// it never is.  A cell takes a wavefront some 15 us, so small multivectors need the box
// kernel's many short workgroups, and a tile of 16 columns costs the same when half of it
// is idle, where the box kernel has tiles of 8.  Box kernel against this, us or the ratio
// of the two, at the steps given:
//  1, 2 columns: the box kernel assembles along rows there; p = 2, 32^3 (2.0) 1.44 and 1.09, p = 1,
//    40^3 (3.9) 1.58; more than three points 0.5 to 0.87 at up to 16 steps.
//  3, 4: three points 1.4 to 2; four 0.95 (3.5), 1.06 to 1.17 (7.8); five 0.92 to 0.97 (p = 2 1.6);
//    seven 0.85 to 0.94.
//  5 to 7: four and more points 1.04 to 1.36 from 6 steps on.  8, no idle slots in the box
//    kernel: three points 0.98 (1.7), 1.05 (4.0), 1.35 (13.5); five, p < 4, 1.08 to 1.23; else 0.89 to
//    1.05.
//  More, the last tile filled (k mod 16 = 9 to 15): from 2 steps on at up to three points, 4
//    above.  k mod 16 = 0: three points from 2; four and five 6 (p = 4, 24^3, 6.8 158 / 132, p = 3,
//    20^3, 32 columns, 7.8 1.10); seven 7 (p = 6, 12^3, 6.8 0.99; 16^3, 16 columns, 4 117 / 122, 32, 8 1.15).
//  The last tile at most half filled: 24 columns 0.92 to 0.99 with four, with five at p = 3 and with
//    seven points, 1.0 to 1.2 with three and with five else; 17 to 23 not for seven points (p =
//    4 0.93, p = 6, 20 columns 0.94); 40, 56 and so on 1.05 to 1.3 from 7 steps on, seven points from
//    14 (p = 6: 0.94 at 6.8, 0.99 at 12, 1.06 at 16).
//  Two points (p = 1): whole tiles from 12 steps (1.06 to 1.17; 0.98 at 6), half tiles of 40 and
//    more columns from 30 (1.06 to 1.17; 0.84 at 6, 0.97 at 21), 8 and 24 columns 0.79 to 1.06; on
//    meshes of few cells in x none of these (7 x 64 x 64: 16 columns 0.93, 20 0.94, 56 0.89; the
//    others there 1.2 to 1.4).
//  Four points at p < 3: with idle slots in the box kernel (p = 2, 40^3: 9 columns 1.45; 24 0.81),
//    whole tiles from 60 steps (1.04 to 1.11; 28^3, 16 columns, 10.7 0.91, 64, 43 0.98); p = 1: 3 and 4
//    columns 2.4, others 0.75 to 1.02.
//  Six points: three pairs for four lane groups, 0.9 to 1.1.
static double pair_least_steps(const Operator& op, int nvec) {
  const int p = op.p, nq = op.nq, rem = nvec % 16;
  if (nq > 7 || nq == 6) return -1.0;
  if (nvec <= 2) return nq <= 3 ? 2.0 : -1.0;
  if (nvec <= 4) return nq <= 3 ? 2.0 : nq == 4 || (nq == 5 && p == 2) ? 6.0 : -1.0;
  if (nq == 4 && p == 1) return -1.0;
  if (nvec < 8) return nq <= 3 ? 2.0 : 6.0;
  if (nvec == 8) return nq == 3 ? 4.0 : nq == 5 && p < 4 ? 6.0 : -1.0;
  const bool half = rem >= 1 && rem <= 8;  // idle half of the last tile
  if (nq == 2) {
    if ((nvec % 8 == 0 || (half && nvec % 4 == 0)) && op.grid.n[0] < 16) return -1.0;
    if (nvec % 8 == 0) return rem == 0 ? 12.0 : nvec >= 40 ? 30.0 : -1.0;
    return 2.0;
  }
  if (nq == 4 && p == 2)
    return rem == 0 ? 60.0 : nvec % 8 == 0 || (half && nvec < 32) ? -1.0 : 6.0;
  if (rem == 8) {
    if (nvec == 24) return nq == 3 || (nq == 5 && p != 3) ? 6.0 : -1.0;
    return nq == 3 ? 4.0 : nq == 7 ? 14.0 : 7.0;
  }
  if (half && nvec % 4 == 0)
    return nq == 7 && nvec < 32 ? -1.0 : nq <= 3 || (nq == 5 && p == 4) ? 4.0 : 7.0;
  if (half) return nq == 7 && p == 4 && nvec < 32 ? -1.0 : nq <= 3 ? 2.0 : 4.0;
  if (rem == 0) return nq == 3 ? 2.0 : nq == 7 ? 7.0 : 6.0;
  return nq <= 3 ? 2.0 : 4.0;
}

// Whether the register-resident apply is the built-in choice.  Accumulating, whole and half
// tiles gain less (p = 2: 8 columns 0.97 at 4 steps, 1.16 at 13.5; 24 columns 0.95 at 6.8, 1.03 at 16; 40
// 1.18 at 24), and a mesh with fewer cells in x than share a wavefront loses (p = 2, 1 x 30000
// x 1, one column 42 / 81 us).
bool pair_chosen(const Operator& op, int nvec, bool accumulate) {
  if (!pair_built(op.nq, accumulate)) return false;
  double least = pair_least_steps(op, nvec);
  if (least < 0.0) return false;
  const int cols = pair_columns(nvec);
  if (accumulate && op.grid.n[0] < pair_cells(cols)) return false;
  if (accumulate && nvec % 16 == 8) least = std::max(least, 12.0);
  return pair_steps(op, nvec, cols) >= least;
}

// The columns per wavefront and the segment length of the register-resident
// apply.  Segments: shorter ones give more wavefronts, longer ones share more
// rows between consecutive cells, and a wavefront's first cell has nothing to
// hide its loads behind; the estimate is rounds of resident wavefronts times
// (cells of a segment + that start).  Only the fewest segments of each length are
// looked at, some 2 sqrt(ny) of them: the plan is made on every call.
PairPlan pair_plan(const Operator& op, int nvec, int cols) {
  PairPlan b{};
  b.cols = cols > 0 ? cols : pair_columns(nvec);
  b.ntiles = (nvec + b.cols - 1) / b.cols;
  const int lx = pair_cells(b.cols);
  b.nxg = (op.grid.n[0] + lx - 1) / lx;
  const int64_t lines = (int64_t)b.nxg * op.grid.n[2] * b.ntiles, ny = op.grid.n[1];
  const double slots = 1024.0 * pair_waves(op.nq);
  double best = 0.0;
  for (int64_t nseg = 1, len = ny;; nseg = (ny + len - 2) / (len - 1)) {
    len = (ny + nseg - 1) / nseg;
    const double r = (double)(lines * nseg) / slots;
    const double rounds = r < 4.0 ? (double)(int64_t)(r + 0.999999) : r + 0.5;
    const double cost = rounds * ((double)len + 0.5);  // p = 6, 16^3, 64 columns: 406 us in one
                                                       // segment of 16, 422 in two, 453 in four
    if (b.len == 0 || cost < best) {
      best = cost;
      b.len = (int)len;
      b.nseg = (int)nseg;
    }
    if (len == 1) break;
  }
  const int64_t items = lines * b.nseg;
  b.items = items < (1LL << 30) ? (int)items : 0;
  b.chunk = (items + 7) / 8;
  return b;
}

// The steps from which the Chebyshev step is faster in the register-resident form, < 0 where
// it never is.  Measured with the initialisation, time of the box kernel over this one's, at the
// steps given:
//  k <= 8: half of the 16 columns idle, not taken.  k mod 16 = 9 to 15 and whole tiles: three
//    points from 2 (p = 2, 16^3, 32 columns, 2 1.19); seven from 4 (p = 6, 16^3, 16, 4 1.15; 12^3, 1.7
//    0.98); five from 6 (p = 4, 24^3, 16, 6.8 1.08; 16^3, 2 0.86); four at p = 3 from 10, with idle
//    slots in the box kernel's tiles from 6 (16^3, 48 columns, 6 0.92, 20^3, 11.7 1.04; 36, 6 1.09); six from
//    10 (p = 5, 20^3, 16, 7.8 1.05; 14^3, 2.7 0.92); two from 12 (p = 1, 40^3 1.08; 20^3, 7.8 0.98).
//  24 columns (a quarter of two tiles idle): three and five points from 12 (p = 2, 24^3, 6.8 0.98; p =
//    3, q = 5, 28^3, 21 1.06, 20^3, 7.8 0.91), seven from 8 (p = 6, 16^3 1.07; p = 4, 14^3, 5.4 0.92); others
//    0.76 to 0.93.  17 to 23: not with six points (p = 3 0.90 to 0.92, p = 4 0.91), seven from 8.
//  40, 56 and so on: three points from 2, five from 7 (p = 4, 16^3, 6 0.88, 8 1.08), seven from 8 (p = 5, 12^3,
//    5.1 0.98), four at p = 3 from 15 (20^3, 11.7 0.95, 15.6 1.00), six from 12 (p = 4, 14^3, 10.7 0.88); two
//    points 0.78 to 1.17, not taken.
//  Four points at p < 3: p = 2 with idle slots in the box kernel's tiles from 10 (28^3, 9 columns 1.13),
//    whole tiles of 48 and more columns from 30 (48, 32 1.01; 64, 43 1.05; 32, 21 0.94); p = 1 0.78 to 1.05.
static double cheb_least_steps(int p, int nq, int nvec) {
  const int rem = nvec % 16;
  const bool half = rem >= 1 && rem <= 8;
  if (nvec <= 8 || nq > 7 || (nq == 4 && p == 1)) return -1.0;
  if (nq == 4 && p == 2) {
    if (rem == 0) return nvec >= 48 ? 30.0 : -1.0;
    return nvec % 8 == 0 || (half && nvec < 32) ? -1.0 : 10.0;
  }
  if (half && nvec <= 24) {
    if (nq == 6 || (nvec == 24 && (nq == 2 || nq == 4))) return -1.0;
    if (nq == 7) return 8.0;
    if (nvec == 24) return 12.0;
  }
  if (nq == 2) return rem == 8 ? -1.0 : 12.0;
  if (nq == 3) return 2.0;
  if (nq == 7) return half && nvec % 4 == 0 ? 8.0 : 4.0;
  if (nq == 6) return half ? 12.0 : 10.0;
  if (nq == 5) return rem == 8 ? 7.0 : 6.0;
  return rem == 8 ? 15.0 : rem == 0 ? 10.0 : 6.0;
}
PairPlan cheb_pair_plan(const Operator& op, int nvec, int64_t span) {
  if (op.nq > 7 || op.deterministic || op.cfg > 0 || span >= kPairMaxSpan ||
      op.ndofs * 8 >= kPairMaxSpan)
    return PairPlan{};
  const double least = cheb_least_steps(op.p, op.nq, nvec);
  const bool chosen = op.cfg == 0 || (least > 0.0 && pair_steps(op, nvec, 16) >= least);
  return chosen ? pair_plan(op, nvec, 16) : PairPlan{};
}

hipError_t launch_cheb_pair(const Operator& op, const double* Y, double* Out, int64_t ld, int nvec,
                            const ChebArgs& ca, const PairPlan& plan, hipStream_t s) {
  switch (op.p) {
    case 1: return launch_cheb_pair_p<1>(op, Y, Out, ld, nvec, ca, plan, s);
    case 2: return launch_cheb_pair_p<2>(op, Y, Out, ld, nvec, ca, plan, s);
    case 3: return launch_cheb_pair_p<3>(op, Y, Out, ld, nvec, ca, plan, s);
    case 4: return launch_cheb_pair_p<4>(op, Y, Out, ld, nvec, ca, plan, s);
    case 5: return launch_cheb_pair_p<5>(op, Y, Out, ld, nvec, ca, plan, s);
    case 6: return launch_cheb_pair_p<6>(op, Y, Out, ld, nvec, ca, plan, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_apply_pair(const Operator& op, const ApplyLaunch& a, const PairPlan& plan,
                             hipStream_t s) {
  switch (op.p) {
    case 1: return launch_apply_pair_p<1>(op, a, plan, s);
    case 2: return launch_apply_pair_p<2>(op, a, plan, s);
    case 3: return launch_apply_pair_p<3>(op, a, plan, s);
    case 4: return launch_apply_pair_p<4>(op, a, plan, s);
    case 5: return launch_apply_pair_p<5>(op, a, plan, s);
    case 6: return launch_apply_pair_p<6>(op, a, plan, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_apply_mfma(const Operator& op, const ApplyLaunch& a, hipStream_t s) {
  switch (op.p) {
    case 1: return launch_apply_mfma_p<1>(op, a, s);
    case 2: return launch_apply_mfma_p<2>(op, a, s);
    case 3: return launch_apply_mfma_p<3>(op, a, s);
    case 4: return launch_apply_mfma_p<4>(op, a, s);
    case 5: return launch_apply_mfma_p<5>(op, a, s);
    case 6: return launch_apply_mfma_p<6>(op, a, s);
    case 7: return launch_apply_mfma_p<7>(op, a, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_apply_box_map(const Operator& op, const ApplyLaunch& a, hipStream_t s) {
  switch (op.p) {
    case 1: return launch_apply_box_map_p<1>(op, a, s);
    case 2: return launch_apply_box_map_p<2>(op, a, s);
    case 3: return launch_apply_box_map_p<3>(op, a, s);
    case 4: return launch_apply_box_map_p<4>(op, a, s);
    case 5: return launch_apply_box_map_p<5>(op, a, s);
    case 6: return launch_apply_box_map_p<6>(op, a, s);
    case 7: return launch_apply_box_map_p<7>(op, a, s);
    case 8: return launch_apply_box_map_p<8>(op, a, s);
    case 9: return launch_apply_box_map_p<9>(op, a, s);
    case 10: return launch_apply_box_map_p<10>(op, a, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_apply_box_map32(const Operator& op, const ApplyLaunch& a, hipStream_t s) {
  switch (op.p) {
    case 1: return launch_apply_box_map32_p<1>(op, a, s);
    case 2: return launch_apply_box_map32_p<2>(op, a, s);
    case 3: return launch_apply_box_map32_p<3>(op, a, s);
    case 4: return launch_apply_box_map32_p<4>(op, a, s);
    case 5: return launch_apply_box_map32_p<5>(op, a, s);
    case 6: return launch_apply_box_map32_p<6>(op, a, s);
    case 7: return launch_apply_box_map32_p<7>(op, a, s);
    case 8: return launch_apply_box_map32_p<8>(op, a, s);
    case 9: return launch_apply_box_map32_p<9>(op, a, s);
    case 10: return launch_apply_box_map32_p<10>(op, a, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_zero_rows(double* Y, int64_t nrows, int ncols, int64_t ld, hipStream_t s) {
  const int64_t total = nrows * ncols;
  int64_t blocks = (total + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(zero_rows_kernel, dim3((unsigned)blocks), dim3(256), 0, s, Y, nrows, ncols, ld);
  return hipGetLastError();
}

hipError_t launch_fma_probe(int blocks, int64_t iters, double* out, hipStream_t s) {
  hipLaunchKernelGGL(fma_probe_kernel, dim3((unsigned)blocks), dim3(256), 0, s, iters, 1.0, out);
  return hipGetLastError();
}

hipError_t launch_fill_pattern(double* X, int64_t n, hipStream_t s) {
  int64_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(fill_pattern_kernel, dim3((unsigned)blocks), dim3(256), 0, s, X, n);
  return hipGetLastError();
}

bool apply_f64_supported(int p, int q) {
  if (p < 1 || p > kMaxP || q < p + 1 || q > p + kMaxQExtra) return false;
  return f64_bmax(p + 1, q) >= 1;
}

int choose_vtile_f64(int np, int nq, int nvec) {
  // the default tile, or for fewer columns the smallest built tile covering them
  const int bd = f64_bdef(np, nq);
  if (nvec >= bd) return bd;
  for (int b = 1; b <= bd; ++b)
    if (b >= nvec && f64_tile_built(np, nq, b)) return b;
  return bd;
}

hipError_t launch_apply_f64(const Operator& op, const ApplyLaunch& a, hipStream_t s) {
  switch (op.p) {
    case 1: return launch_apply_f64_p<1>(op, a, s);
    case 2: return launch_apply_f64_p<2>(op, a, s);
    case 3: return launch_apply_f64_p<3>(op, a, s);
    case 4: return launch_apply_f64_p<4>(op, a, s);
    case 5: return launch_apply_f64_p<5>(op, a, s);
    case 6: return launch_apply_f64_p<6>(op, a, s);
    case 7: return launch_apply_f64_p<7>(op, a, s);
    case 8: return launch_apply_f64_p<8>(op, a, s);
    case 9: return launch_apply_f64_p<9>(op, a, s);
    case 10: return launch_apply_f64_p<10>(op, a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace mf
