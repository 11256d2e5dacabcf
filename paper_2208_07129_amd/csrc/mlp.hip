// Kernels of the learned cell-local preconditioner: a small MLP applied to
// every (cell, column) of a residual block, trained on the GPU.
//
// Batch layout is feature-major: an activation block is [features][rows],
// row = e * k + j for cell e and column j, so a layer is C = W^T X with the
// long batch dimension as the GEMM's N and the weights as the row-major A
// operand.  The cell-blocked variant stores each cell's features x columns
// block contiguously (element (i, e k + j) at e * ld + i * k + j): the cell
// gather and the node assembly then stream whole cells instead of 256-byte
// pieces a batch row apart.  The GEMM runs on the gfx950 matrix cores
// (v_mfma_f32_16x16x32_bf16: BF16 operands, FP32 accumulation, k in order): one
// kernel walks down M with its columns of a long batch in registers, the other
// takes 128 x 128 or 64 x 64 output tiles per 256-thread workgroup with K staged
// through LDS in steps of 32.  Epilogues fuse bias, ReLU, the ReLU mask of the
// backward pass and the BF16 conversion; weight gradients split the batch
// dimension across workgroups and add FP32 partial tiles atomically.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "mf_internal.h"
#include "sf_common.h"

namespace mf {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ inline uint16_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);  // round to nearest even (finite inputs)
  return (uint16_t)(u >> 16);
}
__device__ inline float bf16_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

namespace {

constexpr int kKStep = 32, kPad = 40;  // LDS rows of 80 bytes

// C (M x N) = op(A) (M x K) * op(B) (K x N).  A: row-major M x K (lda), or,
// with TA, stored K x M.  B: row-major K x N (ldb), or, with TB, stored N x K.
// M, N, K multiples of 8.  The K range is cut into pieces of kchunk.  Output
// tiles (T x T) are numbered with the M tile fastest, then N, then the K piece,
// and workgroup b takes tile (b mod 8) c + b / 8 (c = gridDim.x / 8):
// consecutive workgroups go to different XCDs, so this gives each XCD a
// contiguous range of tiles, and the tiles that share an N slice of B (the long
// batch operand), or a K piece of both operands, run on one XCD, which reads
// them from HBM once into its L2.
//
// 2 x 2 wavefronts of T/2 x T/2.  What bounds it is LDS and staging work per
// matrix instruction, so T = 128 (16 matrix instructions per 8 fragment reads;
// T = 64: 4 per 4) wherever the tiles fill the chip.  Two wavefronts stage A,
// two stage B.  An operand stored with k running slowest is transposed in
// registers: a thread loads 8 k rows of T/32 columns and permutes them to
// 16-byte runs of k (one byte permute per two elements; storing single elements
// into LDS took eight stores a chunk).  Run c of LDS row r sits at place
// c ^ (r / 16 mod 4): with 80-byte rows neither those stores nor the fragment
// reads meet on a bank.  Without TB the matrix instruction takes B as its first
// operand, so a lane holds four consecutive columns of C and stores 16 bytes.
//
// 344 x 600 x 128000 (TB, 16 pieces of K): 124 us, 426 TFLOP/s (64 x 64 tiles with
// element-wise transposing stores and loads selected after they arrive: 250).
struct GemmVec {  // whether the tiled kernel's outputs take 4-element stores and its mask 4-element loads
  int f32, bf16, mask;
};

// Staging of one operand: T rows (of m or n) by 32 k, by 128 threads.  Loads go
// through a buffer whose base moves by a step's k (uniform 64-bit address) with
// 32-bit offsets per lane; what lies outside the operand takes an offset past
// the buffer's end and reads 0 (a select on the loaded value would have to wait
// for it).  FAR: the offsets of one step exceed 32 bits; addresses are formed in
// 64 bits and the values selected.
constexpr uint32_t kGemmBuffer = 0xFFFF0000u;  // bytes; also the offset that reads 0
template <int T, bool TR, bool FAR>
struct GemmStage {
  static constexpr int NV = T / 32;  // columns per thread (TR), row passes otherwise
  const uint16_t* base;  // uniform: element (first row or column of the tile, k = kb)
  int64_t kstep;         // elements from one step's base to the next
  int64_t rs;            // TR: stride of k rows; otherwise of 32 rows
  uint32_t off[TR ? 1 : NV];
  int64_t far;           // FAR: this thread's first element from base
  int kk, row;           // first k of this thread in a step, first row or column
  int left;              // rows or columns of the operand from this thread's first on
};

// Thread u's part of the rows [r0, r0 + T) of R from k = kb on (TR, blk > 0:
// columns in blocks of blk, ld the block stride, k rows blk apart).
template <int T, bool TR, bool FAR>
__device__ __forceinline__ GemmStage<T, TR, FAR> gemm_stage(const uint16_t* X, int64_t ld, int r0,
                                                            int R, int kb, int blk, int u) {
  GemmStage<T, TR, FAR> s;
  s.kk = TR ? (u >> 5) * 8 : (u & 3) * 8;
  s.row = TR ? (u & 31) * s.NV : u >> 2;
  s.left = R - r0 - s.row;
  if constexpr (TR) {
    s.rs = blk > 0 ? blk : ld;
    s.kstep = kKStep * s.rs;
    const int b0 = blk > 0 ? r0 / blk : 0, r = s.left > 0 ? r0 + s.row : r0;
    s.base = X + (blk > 0 ? (int64_t)b0 * ld : r0) + kb * s.rs;
    s.far = blk > 0 ? (int64_t)(r / blk - b0) * ld + r % blk : r - r0;
    s.off[0] = s.left > 0 ? (uint32_t)(2 * (s.far + s.kk * s.rs)) : kGemmBuffer;
  } else {
    s.rs = 32 * ld;
    s.kstep = kKStep;
    s.base = X + (int64_t)r0 * ld + kb;
    s.far = s.left > 0 ? s.row * ld : 0;
#pragma unroll
    for (int i = 0; i < s.NV; ++i)
      s.off[i] = 32 * i < s.left ? (uint32_t)(2 * ((s.row + 32 * i) * ld + s.kk)) : kGemmBuffer;
  }
  return s;
}

// The step's loads (step: its number, rem: how many of its 32 k there are).
template <int T, bool TR, bool FAR>
__device__ __forceinline__ void gemm_load(const GemmStage<T, TR, FAR>& s, uint32_t* v, int step,
                                          int rem) {
  constexpr int NV = T / 32;
  const bool kin = s.kk < rem;
  const uint16_t* base = s.base + step * s.kstep;
  if constexpr (FAR) {
    if constexpr (TR) {
      const bool in = kin && s.left > 0;
      const uint16_t* q = base + s.far + (kin ? s.kk * s.rs : 0);
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int n = 0; n < NV / 2; ++n) {
          const uint32_t x = *reinterpret_cast<const uint32_t*>(q + i * s.rs + 2 * n);
          v[i * (NV / 2) + n] = in ? x : 0u;
        }
    } else {
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const bool in = kin && 32 * i < s.left;
        const uint4 x = *reinterpret_cast<const uint4*>(base + s.far + (kin ? s.kk : 0) +
                                                        (in ? i * s.rs : 0));
        v[4 * i] = in ? x.x : 0u;
        v[4 * i + 1] = in ? x.y : 0u;
        v[4 * i + 2] = in ? x.z : 0u;
        v[4 * i + 3] = in ? x.w : 0u;
      }
    }
  } else {
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(base), 0,
                                                        (int)kGemmBuffer, 0x00020000);
    if constexpr (TR) {
      const int o = kin ? (int)s.off[0] : (int)kGemmBuffer;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int so = (int)(2 * i * s.rs);
        if constexpr (NV == 4) {
          const auto x = __builtin_amdgcn_raw_buffer_load_b64(rsrc, o, so, 0);
          v[2 * i] = x[0];
          v[2 * i + 1] = x[1];
        } else {
          v[i] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, o, so, 0);
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const int o = kin ? (int)s.off[i] : (int)kGemmBuffer;
        const auto x = __builtin_amdgcn_raw_buffer_load_b128(rsrc, o, 0, 0);
#pragma unroll
        for (int w = 0; w < 4; ++w) v[4 * i + w] = x[w];
      }
    }
  }
}

template <int T, bool TR, bool FAR>
__device__ __forceinline__ void gemm_store(const GemmStage<T, TR, FAR>& s, const uint32_t* v,
                                           uint16_t (*sh)[kPad]) {
  constexpr int NV = T / 32;
  auto put = [&](int r, uint4 x) {
    *reinterpret_cast<uint4*>(&sh[r][((s.kk >> 3) ^ ((r >> 4) & 3)) * 8]) = x;
  };
#pragma unroll
  for (int n = 0; n < NV; ++n) {
    if constexpr (TR) {
      const uint32_t sel = n & 1 ? 0x07060302u : 0x05040100u;
      uint32_t w[4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        w[i] = __builtin_amdgcn_perm(v[(2 * i + 1) * (NV / 2) + n / 2],
                                     v[(2 * i) * (NV / 2) + n / 2], sel);
      put(s.row + n, uint4{w[0], w[1], w[2], w[3]});
    } else {
      put(s.row + 32 * n, uint4{v[4 * n], v[4 * n + 1], v[4 * n + 2], v[4 * n + 3]});
    }
  }
}

template <int T, bool TA, bool TB, bool FAR>
__global__ void __launch_bounds__(256)
gemm_bf16_kernel(int M, int N, int K, const uint16_t* __restrict__ A, int64_t lda,
                 const uint16_t* __restrict__ B, int64_t ldb, int kchunk, GemmEpi ep,
                 GemmVec vec) {
  // two LDS buffers: step s is staged into buffer s mod 2 while its global
  // loads for step s + 1 are already in flight (one barrier per step)
  __shared__ __attribute__((aligned(16))) uint16_t As[2][T][kPad];  // [m][k]
  __shared__ __attribute__((aligned(16))) uint16_t Bs[2][T][kPad];  // [n][k]
  constexpr int W = T / 32;  // 16 x 16 tiles per direction of a wavefront
  const int mtiles = (M + T - 1) / T, ntiles = (N + T - 1) / T;
  const int64_t tiles = (int64_t)mtiles * ntiles;
  const int64_t lt = (int64_t)(blockIdx.x % kXcds) * (gridDim.x / kXcds) + blockIdx.x / kXcds;
  const int kz = (K + kchunk - 1) / kchunk;
  if (lt >= tiles * kz) return;  // the few padding workgroups of the last XCD range
  const int64_t mn = lt % tiles;
  const int m0 = (int)(mn % mtiles) * T, n0 = (int)(mn / mtiles) * T;
  const int kb = (int)(lt / tiles) * kchunk;
  const int ke = min(K, kb + kchunk);
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = (wave >> 1) * (T / 2), wn = (wave & 1) * (T / 2);
  f32x4 acc[W][W];
#pragma unroll
  for (int i = 0; i < W; ++i)
#pragma unroll
    for (int j = 0; j < W; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  auto product = [&](int buf) {
    bf16x8 a[W], b[W];
#pragma unroll
    for (int i = 0; i < W; ++i) {
      const int ra = wm + i * 16 + (lane & 15), rb = wn + i * 16 + (lane & 15);
      a[i] = *reinterpret_cast<const bf16x8*>(&As[buf][ra][((lane >> 4) ^ ((ra >> 4) & 3)) * 8]);
      b[i] = *reinterpret_cast<const bf16x8*>(&Bs[buf][rb][((lane >> 4) ^ ((rb >> 4) & 3)) * 8]);
    }
#pragma unroll
    for (int i = 0; i < W; ++i)
#pragma unroll
      for (int j = 0; j < W; ++j)
        acc[i][j] = TB ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0)
                       : __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j], a[i], acc[i][j], 0, 0, 0);
  };
  const bool on_a = wave < 2;
  const auto sa = gemm_stage<T, TA, FAR>(A, lda, m0, M, kb, 0, t & 127);
  const auto sb = gemm_stage<T, !TB, FAR>(B, ldb, n0, N, kb, ep.kb, t & 127);
  uint32_t v[2][T / 8];  // the next two steps' operands
  const int nsteps = (ke - kb + kKStep - 1) / kKStep;
  auto load = [&](int step, uint32_t* w) {
    const int rem = ke - kb - step * kKStep;
    if (on_a) gemm_load(sa, w, step, rem);
    else gemm_load(sb, w, step, rem);
  };
  auto one = [&](int step, int buf) {
    if (on_a) gemm_store(sa, v[buf], As[buf]);
    else gemm_store(sb, v[buf], Bs[buf]);
    __syncthreads();
    if (step + 2 < nsteps) load(step + 2, v[buf]);
    product(buf);
  };
  load(0, v[0]);
  if (nsteps > 1) load(1, v[1]);
  for (int step = 0; step < nsteps; step += 2) {
    one(step, 0);
    if (step + 1 < nsteps) one(step + 1, 1);
  }

  // D layout of the 16 x 16 tile: lane -> column lane % 16, rows 4 (lane / 16) + r;
  // rows are m with TB, n otherwise.  The bias is loaded and added inside its branch: a load
  // whose value is chosen behind the branch puts its wait there, and with it one for
  // every store and addition so far, also where there is no bias (344 x 65536 x 32 with B
  // transposed 22.1 -> 19.7 us, 1024 x 131072 x 128 303 -> 265).
  if constexpr (TB) {
#pragma unroll
    for (int i = 0; i < W; ++i)
#pragma unroll
      for (int j = 0; j < W; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int m = m0 + wm + i * 16 + (lane >> 4) * 4 + r;
          const int n = n0 + wn + j * 16 + (lane & 15);
          if (m >= M || n >= N) continue;
          float x = acc[i][j][r];
          if (ep.bias) x += ep.bias[m];
          if (ep.relu) x = x > 0.f ? x : 0.f;
          if (ep.mask && !(bf16_to_f32(ep.mask[(int64_t)m * ep.ldmask + n]) > 0.f)) x = 0.f;
          if (ep.out_f32) {
            float* o = ep.out_f32 + (int64_t)m * ep.ld_f32 + n;
            if (ep.atomic) unsafeAtomicAdd(o, x);
            else *o = x;
          }
          if (ep.out_bf16) ep.out_bf16[(int64_t)m * ep.ld_bf16 + n] = f32_to_bf16(x);
        }
  } else {
#pragma unroll
    for (int j = 0; j < W; ++j) {
      const int n = n0 + wn + j * 16 + (lane >> 4) * 4;  // four columns, inside one block
      if (n >= N) continue;
      const int64_t nb = ep.kb > 0 ? n / ep.kb : 0, nr = ep.kb > 0 ? n % ep.kb : n;
      const int64_t of = ep.kb > 0 ? nb * ep.ld_f32 + nr : nr, sf = ep.kb > 0 ? ep.kb : ep.ld_f32;
      const int64_t ob = ep.kb > 0 ? nb * ep.ld_bf16 + nr : nr,
                    sb = ep.kb > 0 ? ep.kb : ep.ld_bf16;
#pragma unroll
      for (int i = 0; i < W; ++i) {
        const int m = m0 + wm + i * 16 + (lane & 15);
        if (m >= M) continue;
        f32x4 x = acc[i][j];
        if (ep.bias) {
          const float bias = ep.bias[m];
#pragma unroll
          for (int r = 0; r < 4; ++r) x[r] += bias;
        }
        if (ep.relu) {
#pragma unroll
          for (int r = 0; r < 4; ++r) x[r] = x[r] > 0.f ? x[r] : 0.f;
        }
        if (ep.mask) {
          const uint16_t* q = ep.mask + (int64_t)m * ep.ldmask + n;
          ushort4 h;
          if (vec.mask) h = *reinterpret_cast<const ushort4*>(q);
          else h = ushort4{q[0], q[1], q[2], q[3]};
          if (!(bf16_to_f32(h.x) > 0.f)) x[0] = 0.f;
          if (!(bf16_to_f32(h.y) > 0.f)) x[1] = 0.f;
          if (!(bf16_to_f32(h.z) > 0.f)) x[2] = 0.f;
          if (!(bf16_to_f32(h.w) > 0.f)) x[3] = 0.f;
        }
        if (ep.out_f32) {
          float* o = ep.out_f32 + of + m * sf;
          if (ep.atomic) {
#pragma unroll
            for (int r = 0; r < 4; ++r) unsafeAtomicAdd(o + r, x[r]);
          } else if (vec.f32) {
            *reinterpret_cast<f32x4*>(o) = x;
          } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) o[r] = x[r];
          }
        }
        if (ep.out_bf16) {
          uint16_t* o = ep.out_bf16 + ob + m * sb;
          const ushort4 h{f32_to_bf16(x[0]), f32_to_bf16(x[1]), f32_to_bf16(x[2]),
                          f32_to_bf16(x[3])};
          if (vec.bf16) {
            *reinterpret_cast<ushort4*>(o) = h;
          } else {
            o[0] = h.x;
            o[1] = h.y;
            o[2] = h.z;
            o[3] = h.w;
          }
        }
      }
    }
  }
}

// Partition-of-unity weight of a free node: 1 / (number of (cell, local
// node) occurrences), per direction 2 on a shared cell face, 1 otherwise.
__device__ inline double pou_weight(const GridDesc& g, int i1, int i2, int i3, int cx, int cy,
                                    int cz) {
  const int li[3] = {i1, i2, i3}, c[3] = {cx, cy, cz};
  double w = 1.0;
  for (int d = 0; d < 3; ++d) {
    const bool periodic = g.N[d] == g.n[d] * g.p;
    const bool lo = li[d] == 0, hi = li[d] == g.p;
    if (!(lo || hi)) continue;
    const bool outer = !periodic && ((lo && c[d] == 0) || (hi && c[d] == g.n[d] - 1));
    if (!outer) w *= 0.5;
  }
  return w;
}

// The node number of a local node of cell (cx, cy, cz) (-1: constrained) and its
// input factor sqrt(w)^[pou_sqrt] / sqrt(d) (d = dsc[node], 1 without dsc).
__device__ inline int cell_node_factor(const GridDesc& g, int np, int cx, int cy, int cz, int i,
                                       int pou_sqrt, const double* __restrict__ dsc, double& fin,
                                       double* dhalf = nullptr) {
  const int i1 = i % np, i2 = (i / np) % np, i3 = i / (np * np);
  const int node = grid_node(g, cx, cy, cz, i1, i2, i3);
  double dh = 1.0;
  fin = 0.0;
  if (node >= 0) {
    const double ws = pou_sqrt ? sqrt(pou_weight(g, i1, i2, i3, cx, cy, cz)) : 1.0;
    dh = dsc ? sqrt(dsc[node]) : 1.0;
    fin = ws / dh;
  }
  if (dhalf) *dhalf = dh;
  return node;
}

// The same product for op(B) = B (a long batch N), K <= 32 KS and no split.  A
// wavefront keeps its 16 NB columns of B in registers for the whole K range and
// the workgroup walks down M, 16 rows at a time, so B is read from memory once
// (the tiled kernel reads it once per 128 rows of C) and only A (the weights)
// goes through LDS, laid out as the matrix instruction's operands (every LDS
// access is contiguous), two steps deep.  A lane loads NB neighbouring columns
// of 8 k rows of B and permutes them to runs of k, which leaves it with columns
// NB c .. NB c + NB - 1 of C (c = lane % 16): one store per row, 64 NB bytes of
// FP32 in a run.  Bound by memory; 344 x 1024000 x 344, FP32 out, cell-blocked
// (2.1 GB): 500 us, 4.2 TB/s; the tiled kernel above takes 980.
// 256 x 128000 x 344, bias, ReLU, BF16 out: 45 us (72 tiled).
// The epilogue is a template parameter and its stores are dropped past the edge
// by the buffer's bound: with a branch the count of stores in flight is unknown
// and every step waited for the last one's (2.3 us a step).
constexpr int kWideMaxM = 4096;   // rows of C, for the bias in LDS
constexpr int kWideMinN = 32768;  // 128 columns on each of 256 CUs
constexpr int wide_buffer(int ks, bool ta) { return ta ? 1024 : (ks * 64 + 255) / 256 * 256; }
enum WideEpi { kWideF32, kWideF32Bias, kWideReluBf16, kWideMaskBf16, kWideMse };
//
// CELLS: B is not read but formed, the scaled cell values of an FP64 multivector
// (column e k + j of B: column j of cell e, row i its local node i, times the
// node's factor, rounded to BF16 by way of FP32 as the cell gather does), so the
// gathered block is neither written nor read (8000 cells, p = 6, 128 columns: with
// the assembly 1848 -> 1662 us).
struct WideCells {
  GridDesc g;
  int np, k, cells;  // cells: table entries per workgroup
  const double* R;
  int64_t ldr;
  int pou_sqrt;
  const double* dsc;
};
template <int KS, int NB, bool TA, int EPI, bool CELLS>
__global__ void __launch_bounds__(256, 2)
gemm_wide_kernel(int M, int N, int K, const uint16_t* __restrict__ A, int64_t lda,
                 const uint16_t* __restrict__ B, int64_t ldb, GemmEpi ep, WideCells wc) {
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  constexpr int kOob = (int)kGemmBuffer;
  extern __shared__ __attribute__((aligned(16))) char wide_sh[];
  constexpr int kBuf = wide_buffer(KS, TA);
  u32x4* sa = reinterpret_cast<u32x4*>(wide_sh);       // [2][KS][64], padded to kBuf
  float* sbias = reinterpret_cast<float*>(sa + 2 * kBuf);  // [M rounded up to 16]
  const int t = threadIdx.x, lane = t & 63, c = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int64_t lt = (int64_t)(blockIdx.x % kXcds) * (gridDim.x / kXcds) + blockIdx.x / kXcds;
  if (lt * 64 * NB >= N) return;
  const int64_t n0 = (lt * 4 + wave) * (16 * NB);
  const int64_t n = n0 + NB * c;
  const bool nok = n < N;
  auto rsrc_of = [](const uint16_t* p) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p), 0, kOob, 0x00020000);
  };
  // 8 k rows (rs2 bytes apart) of W neighbouring elements, and their W runs of k
  auto columns = [](auto rsrc, int o, int rs2, auto wc, uint32_t* v) {
    constexpr int W = decltype(wc)::value;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if constexpr (W == 4) {
        const auto x = __builtin_amdgcn_raw_buffer_load_b64(rsrc, o, i * rs2, 0);
        v[2 * i] = x[0];
        v[2 * i + 1] = x[1];
      } else {
        v[i] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, o, i * rs2, 0);
      }
    }
  };
  auto runs = [](const uint32_t* v, auto wc, u32x4* out) {
    constexpr int W = decltype(wc)::value;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const uint32_t sel = w & 1 ? 0x07060302u : 0x05040100u;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        out[w][i] = __builtin_amdgcn_perm(v[(2 * i + 1) * (W / 2) + w / 2],
                                          v[2 * i * (W / 2) + w / 2], sel);
    }
  };
  using WB = std::integral_constant<int, NB>;
  using W4 = std::integral_constant<int, 4>;
  u32x4 b[KS][NB];
  if constexpr (CELLS) {
    // node numbers and factors of the workgroup's cells, rows past F with factor 0
    constexpr int RT = KS * 32;
    double* sf = reinterpret_cast<double*>(sbias);
    int* sn = reinterpret_cast<int*>(sf + wc.cells * RT);
    const int ncells = wc.g.n[0] * wc.g.n[1] * wc.g.n[2];
    const int e0 = (int)(lt * 64 * NB / wc.k);
    for (int q = t; q < wc.cells * RT; q += 256) {
      const int ce = q / RT, i = q - ce * RT, e = min(e0 + ce, ncells - 1);
      double f;
      int node = cell_node_factor(wc.g, wc.np, e % wc.g.n[0], e / wc.g.n[0] % wc.g.n[1],
                                  e / (wc.g.n[0] * wc.g.n[1]), min(i, wc.np * wc.np * wc.np - 1),
                                  wc.pou_sqrt, wc.dsc, f);
      sf[q] = i < wc.np * wc.np * wc.np && node >= 0 ? f : 0.0;
      sn[q] = node >= 0 ? node : 0;
    }
    __syncthreads();
    const int64_t nl = nok ? n : 0;
    const int e = nok ? (int)(nl / wc.k) : e0;
    const double* Rj = wc.R + (nl - (int64_t)(nl / wc.k) * wc.k);
    const int at = (e - e0) * RT + 8 * g;
    // a step's rows are asked for while the step before is rounded and packed
    double2 x[2][8][NB / 2];
    auto ask = [&](int ks) {
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int w = 0; w < NB / 2; ++w)
          x[ks & 1][i][w] = *reinterpret_cast<const double2*>(
              Rj + (int64_t)sn[at + 32 * ks + i] * wc.ldr + 2 * w);
    };
    ask(0);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if (ks + 1 < KS) ask(ks + 1);
      __builtin_amdgcn_sched_barrier(0);
      uint32_t h[8][NB];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const double f = sf[at + 32 * ks + i];
#pragma unroll
        for (int w = 0; w < NB; ++w) {
          const double y = w & 1 ? x[ks & 1][i][w / 2].y : x[ks & 1][i][w / 2].x;
          h[i][w] = f32_to_bf16((float)(f != 0.0 ? y * f : 0.0));
        }
      }
#pragma unroll
      for (int w = 0; w < NB; ++w)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          uint32_t r = h[2 * i][w] | h[2 * i + 1][w] << 16;
          asm volatile("" : "+v"(r));  // packed here, not where it is used
          b[ks][w][i] = r;
        }
      __builtin_amdgcn_sched_barrier(0);
    }
  } else {
    const int64_t rs = ep.kb > 0 ? ep.kb : ldb;
    const int64_t nc = n0 < N ? n0 : 0;  // past the end: nothing is read
    const int64_t b0 = ep.kb > 0 ? nc / ep.kb : 0;
    const uint16_t* base = B + (ep.kb > 0 ? b0 * ldb : nc);
    const int64_t far = ep.kb > 0 ? (n / ep.kb - b0) * ldb + n % ep.kb : n - nc;
    const int vo = nok ? (int)(uint32_t)(2 * (far + 8 * g * rs)) : kOob;
    uint32_t v[KS][4 * NB];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      columns(rsrc_of(base + ks * 32 * rs), 32 * ks + 8 * g < K ? vo : kOob, (int)(2 * rs), WB{},
              v[ks]);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) runs(v[ks], WB{}, b[ks]);
  }
  // staging of 16 rows of A: TA one item (8 k rows, 4 columns) per thread,
  // otherwise PT runs of 8 k; the operand of (ks, g, row r) at sa[ks][16 g + r]
  constexpr int PT = TA ? 1 : (KS * 64 + 255) / 256;
  static_assert(!TA || KS * 16 <= 256, "one item per thread");
  uint32_t st[TA ? 16 : 4 * PT];
  auto stage_load = [&](int m0) {
    if constexpr (TA) {
      const int m = m0 + (t & 3) * 4, k = (t >> 2) * 8;
      const int o = m < M && k < K ? (int)(uint32_t)(2 * (k * lda + m)) : kOob;
      columns(rsrc_of(A), o, (int)(2 * lda), W4{}, st);
    } else {
#pragma unroll
      for (int i = 0; i < PT; ++i) {
        const int e = t + 256 * i, m = m0 + (e & 15), k = (e >> 4) * 8;
        const int o = m < M && k < K ? (int)(uint32_t)(2 * ((e & 15) * lda + k)) : kOob;
        const auto x = __builtin_amdgcn_raw_buffer_load_b128(rsrc_of(A + (int64_t)m0 * lda), o, 0, 0);
#pragma unroll
        for (int w = 0; w < 4; ++w) st[4 * i + w] = x[w];
      }
    }
  };
  auto stage_store = [&](u32x4* dst) {
    if constexpr (TA) {
      u32x4 x[4];
      runs(st, W4{}, x);
#pragma unroll
      for (int j = 0; j < 4; ++j) dst[(t >> 2) * 16 + (t & 3) * 4 + j] = x[j];
    } else {
#pragma unroll
      for (int i = 0; i < PT; ++i)
        dst[t + 256 * i] = u32x4{st[4 * i], st[4 * i + 1], st[4 * i + 2], st[4 * i + 3]};
    }
  };
  // this lane's place in C (rows 4 g .. 4 g + 3 of a step) and the mask, in bytes
  // from a uniform base that moves 16 rows a step
  constexpr bool kF32 = EPI == kWideF32 || EPI == kWideF32Bias;
  constexpr bool kBias = EPI == kWideF32Bias || EPI == kWideReluBf16 || EPI == kWideMse;
  constexpr int SZ = kF32 ? 4 : 2;
  const int64_t ldc = kF32 ? ep.ld_f32 : ep.ld_bf16;
  const int64_t sc = ep.kb > 0 ? ep.kb : ldc;
  const int64_t nc = n0 < N ? n0 : 0, b0 = ep.kb > 0 ? nc / ep.kb : 0;
  char* cbase = (kF32 ? reinterpret_cast<char*>(ep.out_f32) : reinterpret_cast<char*>(ep.out_bf16)) +
                SZ * (ep.kb > 0 ? b0 * ldc : nc);
  const int co = nok ? (int)(uint32_t)(SZ * ((ep.kb > 0 ? (n / ep.kb - b0) * ldc + n % ep.kb
                                                        : n - nc) + 4 * g * sc))
                     : kOob;
  const uint16_t* mbase = EPI == kWideMaskBf16 ? ep.mask + nc : nullptr;
  const int mo = nok ? (int)(uint32_t)(2 * (n - nc + 4 * g * ep.ldmask)) : kOob;
  // kWideMse: targets in the same way, the row weights (0 past the rows), the loss
  const float* tbase = EPI == kWideMse ? ep.target + nc : nullptr;
  const int to = nok ? (int)(uint32_t)(4 * (n - nc + 4 * g * ep.ldt)) : kOob;
  float rw[NB];
  double lsum = 0.0;
  if constexpr (EPI == kWideMse) {
#pragma unroll
    for (int j = 0; j < NB; ++j)
      rw[j] = n + j < ep.nrows ? (ep.roww ? ep.roww[n + j] : 1.f) : 0.f;
  }
  stage_load(0);
  if constexpr (kBias)
    for (int i = t; i < (M + 15) / 16 * 16; i += 256) sbias[i] = ep.bias && i < M ? ep.bias[i] : 0.f;
  stage_store(sa);
  stage_load(16);
  __syncthreads();
  for (int m0 = 0, buf = 0; m0 < M; m0 += 16, buf ^= 1) {
    stage_store(sa + (buf ^ 1) * kBuf);
    stage_load(m0 + 32);
    const bool in = m0 + 4 * g < M;  // M is a multiple of 8
    uint32_t hm[4][NB / 2];
    if constexpr (EPI == kWideMaskBf16) {
      const auto rm = rsrc_of(mbase + (int64_t)m0 * ep.ldmask);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if constexpr (NB == 4) {
          const auto d = __builtin_amdgcn_raw_buffer_load_b64(rm, in ? mo : kOob,
                                                              (int)(2 * r * ep.ldmask), 0);
          hm[r][0] = d[0];
          hm[r][1] = d[1];
        } else {
          hm[r][0] = __builtin_amdgcn_raw_buffer_load_b32(rm, in ? mo : kOob,
                                                          (int)(2 * r * ep.ldmask), 0);
        }
      }
    }
    float tv[4][NB];
    if constexpr (EPI == kWideMse) {
      const auto rt = rsrc_of(reinterpret_cast<const uint16_t*>(tbase + (int64_t)m0 * ep.ldt));
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int o = in && m0 + 4 * g + r < ep.feat ? to : kOob;
        if constexpr (NB == 4) {
          const auto d = __builtin_amdgcn_raw_buffer_load_b128(rt, o, (int)(4 * r * ep.ldt), 0);
#pragma unroll
          for (int j = 0; j < 4; ++j) tv[r][j] = __uint_as_float(d[j]);
        } else {
          const auto d = __builtin_amdgcn_raw_buffer_load_b64(rt, o, (int)(4 * r * ep.ldt), 0);
          tv[r][0] = __uint_as_float(d[0]);
          tv[r][1] = __uint_as_float(d[1]);
        }
      }
    }
    f32x4 acc[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const u32x4* a = sa + buf * kBuf + lane;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8 x = __builtin_bit_cast(bf16x8, a[ks * 64]);
#pragma unroll
      for (int j = 0; j < NB; ++j)
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, __builtin_bit_cast(bf16x8, b[ks][j]),
                                                         acc[j], 0, 0, 0);
    }
    f32x4 bias;
    if constexpr (kBias)
      bias = *reinterpret_cast<const f32x4*>(&sbias[m0 + 4 * g]);
    const auto rc =
        __builtin_amdgcn_make_buffer_rsrc(cbase + (int64_t)SZ * m0 * sc, 0, kOob, 0x00020000);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float x[NB];
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        x[j] = acc[j][r];
        if constexpr (kBias) x[j] += bias[r];
        if constexpr (EPI == kWideReluBf16) x[j] = x[j] > 0.f ? x[j] : 0.f;
        if constexpr (EPI == kWideMaskBf16)
          x[j] = bf16_to_f32((uint16_t)(hm[r][j / 2] >> (16 * (j & 1)))) > 0.f ? x[j] : 0.f;
        if constexpr (EPI == kWideMse) {
          const bool live = m0 + 4 * g + r < ep.feat && n + j < ep.nrows;
          const float d = live ? x[j] - tv[r][j] : 0.f;
          lsum += (double)rw[j] * d * d;
          x[j] = 2.0f * ep.scale * rw[j] * d;
        }
      }
      uint32_t d[kF32 ? NB : NB / 2];
      if constexpr (kF32) {
#pragma unroll
        for (int j = 0; j < NB; ++j) d[j] = __float_as_uint(x[j]);
      } else {
#pragma unroll
        for (int j = 0; j < NB / 2; ++j)
          d[j] = f32_to_bf16(x[2 * j]) | (uint32_t)f32_to_bf16(x[2 * j + 1]) << 16;
      }
      typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
      const int o = in ? co : kOob, so = (int)(SZ * r * sc);
      if constexpr (sizeof(d) == 16)
        __builtin_amdgcn_raw_buffer_store_b128(u32x4{d[0], d[1], d[2], d[3]}, rc, o, so, 0);
      else if constexpr (sizeof(d) == 8)
        __builtin_amdgcn_raw_buffer_store_b64(u32x2{d[0], d[1]}, rc, o, so, 0);
      else
        __builtin_amdgcn_raw_buffer_store_b32(d[0], rc, o, so, 0);
    }
    __syncthreads();
  }
  if constexpr (EPI == kWideMse) {  // one addition to the loss per workgroup
    double* part = reinterpret_cast<double*>(wide_sh);
    part[t] = lsum;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
      if (t < s) part[t] += part[t + s];
      __syncthreads();
    }
    if (t == 0) unsafeAtomicAdd(ep.loss, part[0] * (double)ep.scale);
  }
}

// One workgroup per (C cells, chunk of 64 columns); lane l of a wavefront: cell
// l / k and column l % k of the C k <= 64 (cell, column) rows (C = 1: column l of
// the chunk), wavefront ph: nodes i = ph, ph + 4, ...  rho = RMS of the cell's
// residual column (over the cell's F = np^3 node values, constrained nodes as
// 0); X0t[i][row] = R[node_i][j] / rho as BF16 (rows i in [F, Fp) zero),
// Tt[i][row] = E[node_i][j] / rho in FP32 when E is given (training targets).
// The node numbers and the per-node input and target factors of the cells are
// formed once per workgroup in LDS, so the column loops only load, scale and
// store.  Bound by memory; several cells per workgroup for few columns because
// one cell's columns leave the other lanes idle and write X0t and Tt in pieces
// (k = 16, p = 6, 8000 cells, with E: 470 -> 190 us).
constexpr int kCols = 64;
constexpr int kGatherNodeBytes = 2 * sizeof(double) + sizeof(int);  // LDS per (cell, node)

// Per local node of a cell: the node number, the input factor and sqrt(d).
__device__ inline void cell_node_factors(const GridDesc& g, int np, int cx, int cy, int cz,
                                         int pou_sqrt, const double* __restrict__ dsc, int* snode,
                                         double* sfin, double* sdh) {
  const int F = np * np * np;
  for (int i = threadIdx.x; i < F; i += blockDim.x)
    snode[i] = cell_node_factor(g, np, cx, cy, cz, i, pou_sqrt, dsc, sfin[i],
                                sdh ? sdh + i : nullptr);
}

template <bool MULTI>
__global__ void __launch_bounds__(256)
cell_gather_kernel(GridDesc g, int np, int k, int C_, const double* __restrict__ R, int64_t ldr,
                   const double* __restrict__ E, int64_t lde, int Fp, uint16_t* __restrict__ X0t,
                   float* __restrict__ Tt, int64_t ldx, float* __restrict__ rho, int pou_sqrt,
                   const double* __restrict__ dsc, int blocked) {
  extern __shared__ double gather_sh[];
  __shared__ double part[256];
  const int F = np * np * np, ncells = g.n[0] * g.n[1] * g.n[2];
  const int t = threadIdx.x, jj = t % kCols, ph = t / kCols;
  const int C = MULTI ? C_ : 1;
  const int e0 = blockIdx.x * C, cells = MULTI ? min(C, ncells - e0) : 1;
  // lanes past the last row take the first cell and the last column and store nothing
  const bool jok = MULTI ? jj < cells * k : (int)(blockIdx.y * kCols) + jj < k;
  const int c = MULTI && jok ? jj / k : 0, e = e0 + c;
  const int j = jok ? (MULTI ? jj - c * k : (int)(blockIdx.y * kCols) + jj) : k - 1;
  for (int u = 0; u < cells; ++u) {
    const int cx = (e0 + u) % g.n[0], cy = ((e0 + u) / g.n[0]) % g.n[1],
              cz = (e0 + u) / (g.n[0] * g.n[1]);
    cell_node_factors(g, np, cx, cy, cz, pou_sqrt, dsc,
                      reinterpret_cast<int*>(gather_sh + 2 * C * F) + u * F, gather_sh + u * F,
                      gather_sh + (C + u) * F);
  }
  const double* sfin = gather_sh + c * F;
  const double* sdh = gather_sh + (C + c) * F;
  const int* snode = reinterpret_cast<const int*>(gather_sh + 2 * C * F) + c * F;
  __syncthreads();
  // Loads never sit behind a branch: constrained nodes and the padding rows
  // read a valid element (clamped index) whose value a select then drops;
  // batches of kGatherBatch rows are loaded before they are used.
  constexpr int kGatherBatch = 8;
  const int nrows = (Fp - ph + 3) / 4;  // rows i = ph, ph + 4, ... < Fp of this wavefront
  auto node_of = [&](int i) { return snode[i < F ? i : F - 1]; };
  double s = 1.0;  // without rho: no normalisation
  if (rho) {
    double ss = 0.0;
    for (int r0 = 0; r0 < nrows; r0 += kGatherBatch) {
      double xv[kGatherBatch];
#pragma unroll
      for (int u = 0; u < kGatherBatch; ++u) {
        const int node = node_of(ph + 4 * (r0 + u));
        xv[u] = R[(int64_t)(node >= 0 ? node : 0) * ldr + j];
      }
#pragma unroll
      for (int u = 0; u < kGatherBatch; ++u) {
        const int i = ph + 4 * (r0 + u);
        const double f = i < F ? sfin[i] : 0.0;  // 0 for constrained nodes and padding
        const double x = f != 0.0 ? xv[u] * f : 0.0;
        ss = fma(x, x, ss);
      }
    }
    part[t] = ss;
    __syncthreads();
    double tot = part[jj] + part[jj + 64] + part[jj + 128] + part[jj + 192];
    const double r = sqrt(tot / F);
    s = r > 0.0 ? 1.0 / r : 0.0;
    if (jok && ph == 0) rho[(int64_t)e * k + j] = (float)r;
  }
  if (!jok) return;
  const int64_t row = (int64_t)e * k + j;
  // element (i, row) at i * istep + base
  const int64_t base = blocked ? (int64_t)e * ldx + j : row, istep = blocked ? k : ldx;
  auto rows = [&](auto with_e) {
    constexpr bool WE = decltype(with_e)::value;
    for (int r0 = 0; r0 < nrows; r0 += kGatherBatch) {
      double xv[kGatherBatch], yv[kGatherBatch];
#pragma unroll
      for (int u = 0; u < kGatherBatch; ++u) {
        const int node = node_of(ph + 4 * (r0 + u));
        const int64_t nc = node >= 0 ? node : 0;
        xv[u] = R[nc * ldr + j];
        if constexpr (WE) yv[u] = E[nc * lde + j];
      }
#pragma unroll
      for (int u = 0; u < kGatherBatch; ++u) {
        if (r0 + u >= nrows) break;  // uniform across the wavefront
        const int i = ph + 4 * (r0 + u);
        const double f = i < F ? sfin[i] : 0.0;
        const double x = f != 0.0 ? xv[u] * s * f : 0.0;
        X0t[i * istep + base] = f32_to_bf16((float)x);
        if constexpr (WE) Tt[i * istep + base] = f != 0.0 ? (float)(yv[u] * s * sdh[i]) : 0.0f;
      }
    }
  };
  if (E) rows(std::true_type{});
  else rows(std::false_type{});
}

// The incidences of grid node g (0 <= g < N) along one direction: the cells
// c[0..cnt) holding it and its local index l[] there, with the
// partition-of-unity factor of the direction (1/2 when two cells share the
// node, 1 otherwise, as pou_weight).  Periodic directions have N = n p (node
// n p is node 0); with n = 1 a vertex node meets the one cell twice.
__device__ inline int node_incidences(int g, int n, int N, int p, int* c, int* l, double* w) {
  const bool periodic = N == n * p;
  const int cq = g / p, r = g - cq * p;
  if (r != 0) {
    c[0] = cq;
    l[0] = r;
    *w = 1.0;
    return 1;
  }
  int cnt = 0;
  if (cq < n) {  // the cell starting at the node
    c[cnt] = cq;
    l[cnt++] = 0;
  }
  if (cq > 0 || periodic) {  // the cell ending at the node
    c[cnt] = cq > 0 ? cq - 1 : n - 1;
    l[cnt++] = p;
  }
  *w = cnt == 2 ? 0.5 : 1.0;
  return cnt;
}

// Z[node][j] = (R[node][j] / diag[node] or 0) + sum over the node's
// incidences (cell e, local node i) of w^[1/2] rho[e k + j] Yt(i, e k + j)
// (divided by sqrt(dsc[node])): the partition-of-unity assembly taken node by
// node, so every Z element is written once by one lane, with a fixed order of
// its up to eight terms (no atomics; bitwise reproducible).  Constrained nodes
// get only the Jacobi term, as the scattered form never adds to them.
//
// One wavefront per (x-line of a cell, 64 columns): the nodes gx = cx p + l,
// l = 0 .. p - 1 (and l = p in the last cell of a non-periodic direction), at
// fixed (gy, gz), lanes over the columns.  Along the line only l = 0 can have
// a second x-incidence, and the y, z incidences are the same for every node,
// so with p and their counts as template parameters all the line's loads are
// independent and in flight together (one node per wavefront left the kernel
// bound by memory latency).
constexpr int kAsmLines = 4;  // lines (wavefronts) per workgroup

struct AsmArgs {
  GridDesc g;
  int k;
  const float* Yt;
  int64_t ldy;
  const float* rho;
  const double* diag;
  const double* R;
  int64_t ldr;
  double* Z;
  int64_t ldz;
  int pou_sqrt;
  const double* dsc;
  int blocked;
};

// lane l's value of v, as a wave-uniform value
__device__ __forceinline__ double wave_bcast(double v, int l) {
  const int2 h = __builtin_bit_cast(int2, v);
  const int2 r{__builtin_amdgcn_readlane(h.x, l), __builtin_amdgcn_readlane(h.y, l)};
  return __builtin_bit_cast(double, r);
}

template <int P, int NY, int NZ, bool BLK, bool RHO, bool DIAG>
__device__ __forceinline__ void assemble_line(const AsmArgs& a, int cx, int gy, int gz,
                                              const int* cy, const int* ly, double wy,
                                              const int* cz, const int* lz, double wz, int j,
                                              bool jok) {
  constexpr int NP = P + 1;
  const GridDesc& g = a.g;
  const int n0 = g.n[0], N0 = g.N[0];
  const bool periodic_x = N0 == n0 * P;
  const bool has_left = periodic_x || cx > 0;   // a cell ends at gx = cx p
  const bool extra = !periodic_x && cx == n0 - 1;  // node l = p is this line's too
  const int cxl = cx > 0 ? cx - 1 : n0 - 1;
  const bool line_constrained =
      g.dirichlet && (gy == 0 || gy == g.N[1] - 1 || gz == 0 || gz == g.N[2] - 1);
  int64_t eyz[NY * NZ];
  int iyz[NY * NZ];
#pragma unroll
  for (int c = 0; c < NZ; ++c)
#pragma unroll
    for (int b = 0; b < NY; ++b) {
      eyz[c * NY + b] = (int64_t)n0 * (cy[b] + (int64_t)g.n[1] * cz[c]);
      iyz[c * NY + b] = NP * (ly[b] + NP * lz[c]);
    }
  auto yload = [&](int64_t e, int i) -> float {
    return BLK ? a.Yt[e * a.ldy + (int64_t)i * a.k + j] : a.Yt[(int64_t)i * a.ldy + e * a.k + j];
  };
  auto rload = [&](int64_t e) -> float {
    if constexpr (RHO) return a.rho[e * a.k + j];
    return 1.0f;
  };
  // all the line's loads first (independent, in flight together), then the sums
  constexpr int Q = NY * NZ;
  float yv[P + 2][Q], rv[3][Q];  // rows: l = 0 .. p - 1, the left cell's p, this cell's p
#pragma unroll
  for (int q = 0; q < Q; ++q) {
#pragma unroll
    for (int l = 0; l < P; ++l) yv[l][q] = yload(cx + eyz[q], l + iyz[q]);
    yv[P][q] = yload(cxl + eyz[q], P + iyz[q]);
    yv[P + 1][q] = yload(cx + eyz[q], P + iyz[q]);
    rv[0][q] = rload(cx + eyz[q]);
    rv[1][q] = rload(cxl + eyz[q]);
  }
  double acc[P + 1];
#pragma unroll
  for (int l = 0; l < P; ++l) {
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < Q; ++q) s += (double)rv[0][q] * (double)yv[l][q];
    if (l == 0) {  // the cell to the left, local node p (added if it exists)
      double t = 0.0;
#pragma unroll
      for (int q = 0; q < Q; ++q) t += (double)rv[1][q] * (double)yv[P][q];
      s += has_left ? t : 0.0;
    }
    acc[l] = s;
  }
  acc[P] = 0.0;
#pragma unroll
  for (int q = 0; q < Q; ++q) acc[P] += (double)rv[0][q] * (double)yv[P + 1][q];
  if (!extra) acc[P] = 0.0;
  // per-node factors of the line, one node per lane (lanes 0 .. p), then read
  // back as wave-uniform values: 1 / diag and w^[1/2] / sqrt(dsc)
  const double wyz = wy * wz;
  const int64_t row0 = (int64_t)N0 * (gy + (int64_t)g.N[1] * gz);
  const int lane = threadIdx.x & 63;
  double invd = 0.0, fac = 0.0;
  if (lane <= P) {
    const int gx = cx * P + (lane < P || extra ? lane : 0);
    const int64_t node = row0 + gx;
    if constexpr (DIAG) invd = 1.0 / a.diag[node];
    const double pw = ((lane == 0 && has_left) ? 0.5 : 1.0) * wyz;
    fac = a.pou_sqrt ? sqrt(pw) : pw;
    if (a.dsc) fac /= sqrt(a.dsc[node]);
  }
  double rj[P + 1];  // the Jacobi term's R values (l = p: a valid node when not this line's)
  if constexpr (DIAG) {
#pragma unroll
    for (int l = 0; l <= P; ++l) {
      const int gx = cx * P + (l < P || extra ? l : 0);
      rj[l] = a.R[(row0 + gx) * a.ldr + j];
    }
  }
#pragma unroll
  for (int l = 0; l <= P; ++l) {
    if (l == P && !extra) break;
    const int gx = cx * P + l;
    const int64_t node = row0 + gx;
    const double il = wave_bcast(invd, l), fl = wave_bcast(fac, l);
    double z = 0.0;
    if constexpr (DIAG) z = rj[l] * il;
    const bool constrained = line_constrained || (g.dirichlet && (gx == 0 || gx == N0 - 1));
    if (!constrained) z = fma(fl, acc[l], z);
    if (jok) a.Z[node * a.ldz + j] = z;
  }
}

// BLK: cell-blocked Yt; RHO: rho given; DIAG: the Jacobi term (compile-time,
// so that no load sits behind a branch and the line's loads issue together)
template <int P, bool BLK, bool RHO, bool DIAG>
__global__ void __attribute__((amdgpu_flat_work_group_size(1, 64 * kAsmLines),
                               amdgpu_waves_per_eu(1, 4)))
node_assemble_kernel(AsmArgs a, int nlines, int nchunks) {
  // the column chunk varies fastest, so the halves of a Z row (and of an R
  // row) are written and read together
  const int chunk = (int)(blockIdx.x % nchunks);
  const int line = (int)(blockIdx.x / nchunks) * kAsmLines + (int)(threadIdx.x >> 6);  // < 2^31
  // every lane stays (lanes 0 .. p form the line's node factors); lanes past
  // the last column read column k - 1 and store nothing
  const int jl = chunk * 64 + (threadIdx.x & 63);
  const bool jok = jl < a.k;
  const int j = jok ? jl : a.k - 1;
  if (line >= nlines) return;
  const GridDesc& g = a.g;
  const int cx = line % g.n[0];
  const int rest = line / g.n[0];
  const int gy = rest % g.N[1], gz = rest / g.N[1];
  int cy[2], cz[2], ly[2], lz[2];
  double wy, wz;
  const int ny = node_incidences(gy, g.n[1], g.N[1], P, cy, ly, &wy);
  const int nz = node_incidences(gz, g.n[2], g.N[2], P, cz, lz, &wz);
  if (ny == 1 && nz == 1) assemble_line<P, 1, 1, BLK, RHO, DIAG>(a, cx, gy, gz, cy, ly, wy, cz, lz, wz, j, jok);
  else if (ny == 2 && nz == 1) assemble_line<P, 2, 1, BLK, RHO, DIAG>(a, cx, gy, gz, cy, ly, wy, cz, lz, wz, j, jok);
  else if (ny == 1) assemble_line<P, 1, 2, BLK, RHO, DIAG>(a, cx, gy, gz, cy, ly, wy, cz, lz, wz, j, jok);
  else assemble_line<P, 2, 2, BLK, RHO, DIAG>(a, cx, gy, gz, cy, ly, wy, cz, lz, wz, j, jok);
}

// dYt = 2 scale w[n] (Yt - Tt) for features < F (0 for the padding features and in
// the columns from nrows to ncols), as BF16; loss += scale sum w[n] (Yt - Tt)^2 (w = 1 when the row weights are
// null).  Pieces of one feature by 4 x 256 batch rows, 16-byte loads and 8-byte
// stores where VEC says that every row starts on such a boundary.  Bound by
// memory (344 x 128000: 92 us, 4.8 TB/s).
template <bool VEC>
__global__ void __launch_bounds__(256)
mse_grad_kernel(int F, int Fp, int64_t nrows, int64_t ncols, const float* __restrict__ Yt,
                const float* __restrict__ Tt, int64_t ld, const float* __restrict__ roww,
                float scale, uint16_t* __restrict__ dYt, double* __restrict__ loss) {
  __shared__ double part[256];
  double acc = 0.0;
  const int64_t chunks = (ncols + 1023) / 1024, pieces = chunks * Fp;
  for (int64_t u = blockIdx.x; u < pieces; u += gridDim.x) {
    const int i = (int)(u / chunks);
    const int64_t n = (u - i * chunks) * 1024 + 4 * threadIdx.x;
    const int64_t o = (int64_t)i * ld + n;
    if (VEC && n + 4 <= nrows) {
      f32x4 w = {1.f, 1.f, 1.f, 1.f}, d = {0.f, 0.f, 0.f, 0.f};
      if (roww) w = *reinterpret_cast<const f32x4*>(roww + n);
      if (i < F) {
        const f32x4 y = *reinterpret_cast<const f32x4*>(Yt + o);
        const f32x4 x = *reinterpret_cast<const f32x4*>(Tt + o);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          d[r] = y[r] - x[r];
          acc += (double)w[r] * d[r] * d[r];
        }
      }
      ushort4 h;
      h.x = f32_to_bf16(2.0f * scale * w[0] * d[0]);
      h.y = f32_to_bf16(2.0f * scale * w[1] * d[1]);
      h.z = f32_to_bf16(2.0f * scale * w[2] * d[2]);
      h.w = f32_to_bf16(2.0f * scale * w[3] * d[3]);
      *reinterpret_cast<ushort4*>(dYt + o) = h;
    } else {
      for (int r = 0; r < 4 && n + r < ncols; ++r) {
        const bool live = n + r < nrows;
        const float w = roww && live ? roww[n + r] : 1.0f;
        float d = 0.f;
        if (i < F && live) {
          d = Yt[o + r] - Tt[o + r];
          acc += (double)w * d * d;
        }
        dYt[o + r] = f32_to_bf16(2.0f * scale * w * d);
      }
    }
  }
  part[threadIdx.x] = acc;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) part[threadIdx.x] += part[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) unsafeAtomicAdd(loss, part[0] * (double)scale);
}

// out[m] (+)= sum_n X[m][n] (BF16 rows): bias gradients.  The order of the sum is
// fixed: 256 partial sums, number r over the n = r mod 256 in order, then a tree (the
// optimiser divides a gradient by its own size, so another order of the FP32 sums
// would show in the weights).  One workgroup per row, a thread for two neighbouring
// partial sums where VEC says that rows start on 4 bytes, kAhead loads in flight, which
// is what it takes to cover the latency of a few wavefronts per CU.  256 x 128000:
// 19 us (256 threads, one element in flight each, 120).
constexpr int kRowParts = 256;
template <bool VEC>
__global__ void __launch_bounds__(kRowParts / (VEC ? 2 : 1))
row_sums_kernel(int64_t N, const uint16_t* __restrict__ X, int64_t ld, float* __restrict__ out,
                int accumulate) {
  constexpr int W = VEC ? 2 : 1, kAhead = 32;
  __shared__ float part[kRowParts];
  const int m = blockIdx.x;
  const uint16_t* row = X + (int64_t)m * ld;
  float acc[W];
#pragma unroll
  for (int w = 0; w < W; ++w) acc[w] = 0.f;
  int64_t n = W * (int64_t)threadIdx.x;
  for (; n + (kAhead - 1) * kRowParts + W <= N; n += kAhead * kRowParts) {
    uint32_t x[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      if constexpr (VEC) x[u] = *reinterpret_cast<const uint32_t*>(row + n + u * kRowParts);
      else x[u] = row[n + u * kRowParts];
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      acc[0] += __uint_as_float(x[u] << 16);
      if constexpr (VEC) acc[1] += __uint_as_float(x[u] & 0xffff0000u);
    }
  }
  for (; n < N; n += kRowParts)
#pragma unroll
    for (int w = 0; w < W; ++w)
      if (n + w < N) acc[w] += bf16_to_f32(row[n + w]);
#pragma unroll
  for (int w = 0; w < W; ++w) part[W * threadIdx.x + w] = acc[w];
  __syncthreads();
  for (int s = kRowParts / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) part[threadIdx.x] += part[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[m] = (accumulate ? out[m] : 0.f) + part[0];
}

// Adam on FP32 master parameters; writes the BF16 copy when given.
__global__ void adam_kernel(int64_t n, float* __restrict__ w, const float* __restrict__ grad,
                            float* __restrict__ m1, float* __restrict__ m2,
                            uint16_t* __restrict__ wbf, float lr, float b1, float b2, float eps,
                            float c1, float c2) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const float gi = grad[i];
    const float a = b1 * m1[i] + (1.f - b1) * gi;
    const float b = b2 * m2[i] + (1.f - b2) * gi * gi;
    m1[i] = a;
    m2[i] = b;
    const float wi = w[i] - lr * (a / c1) / (sqrtf(b / c2) + eps);
    w[i] = wi;
    if (wbf) wbf[i] = f32_to_bf16(wi);
  }
}

// S <- (S + S^T) / 2 on the leading n x n block of a row-major matrix (ld),
// with its BF16 copy (same layout) refreshed.
__global__ void symmetrize_kernel(int n, float* __restrict__ S, int64_t ld, uint16_t* __restrict__ Sbf) {
  const int64_t total = (int64_t)n * n;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int i = (int)(idx / n), j = (int)(idx % n);
    if (j < i) continue;
    const float v = 0.5f * (S[(int64_t)i * ld + j] + S[(int64_t)j * ld + i]);
    S[(int64_t)i * ld + j] = v;
    S[(int64_t)j * ld + i] = v;
    if (Sbf) {
      const uint16_t b = f32_to_bf16(v);
      Sbf[(int64_t)i * ld + j] = b;
      Sbf[(int64_t)j * ld + i] = b;
    }
  }
}

__global__ void to_bf16_kernel(int64_t n, const float* __restrict__ src, uint16_t* __restrict__ dst) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    dst[i] = f32_to_bf16(src[i]);
}

__global__ void fill_f32_kernel(float* __restrict__ v, int64_t n, float x) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    v[i] = x;
}

// A[i][j] = (S[i][j] + S[j][i]) / 2 in FP64.
__global__ void skip_sym_kernel(int F, const float* __restrict__ S, int64_t lds,
                                double* __restrict__ A) {
  const int64_t total = (int64_t)F * F;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int i = (int)(idx / F), j = (int)(idx - (int64_t)i * F);
    A[idx] = 0.5 * ((double)S[(int64_t)i * lds + j] + (double)S[(int64_t)j * lds + i]);
  }
}

// S[i][j] = sum_r V[i][r] max(w_r, floor) V[j][r], written to S (FP32) and
// Sbf (BF16), floor = -1 + margin + 2^-8 (||w||_2 + sqrt(F)) (every thread
// forms it in the same order).  The product V[i][r] V[j][r] is formed first,
// so (i, j) and (j, i) take identical operations: exactly symmetric.
__global__ void skip_rebuild_kernel(int F, const double* __restrict__ V,
                                    const double* __restrict__ w, double margin,
                                    float* __restrict__ S, int64_t lds, uint16_t* __restrict__ Sbf,
                                    int64_t ldsb) {
  double n2 = 0.0;
  for (int r = 0; r < F; ++r) n2 = fma(w[r], w[r], n2);
  const double floor = -1.0 + margin + 0.00390625 * (sqrt(n2) + sqrt((double)F));
  const int64_t total = (int64_t)F * F;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int i = (int)(idx / F), j = (int)(idx - (int64_t)i * F);
    double acc = 0.0;
    for (int r = 0; r < F; ++r) {
      const double lam = w[r] > floor ? w[r] : floor;
      acc = fma(V[(int64_t)i * F + r] * V[(int64_t)j * F + r], lam, acc);
    }
    S[(int64_t)i * lds + j] = (float)acc;
    Sbf[(int64_t)i * ldsb + j] = f32_to_bf16((float)acc);
  }
}

unsigned blocks_for(int64_t total) {
  int64_t b = (total + 255) / 256;
  if (b > 65536) b = 65536;
  return (unsigned)(b < 1 ? 1 : b);
}

// Whether stores of four elements (and loads of the mask) are aligned.
bool aligned4(const void* p, int64_t ld, int kb, size_t n) {
  return reinterpret_cast<uintptr_t>(p) % n == 0 && ld % 4 == 0 && kb % 4 == 0;
}
GemmVec gemm_vec(const GemmEpi& ep) {
  return {aligned4(ep.out_f32, ep.ld_f32, ep.kb, 16), aligned4(ep.out_bf16, ep.ld_bf16, ep.kb, 8),
          aligned4(ep.mask, ep.ldmask, 0, 8)};
}
// The operands' offsets of one tiled step in 32 bits: T rows of an operand with k
// along the rows, 32 k rows otherwise (in blocks: 32 rows of a block and the tile's
// later blocks).
bool gemm_far(bool ta, bool tb, int64_t lda, int64_t ldb, int kb) {
  const int64_t span_a = (ta ? 32 : 128) * lda;
  const int64_t span_b =
      tb ? 128 * ldb : kb > 0 ? (int64_t)32 * kb + (128 / kb + 1) * ldb : 32 * ldb;
  return 2 * (span_a > span_b ? span_a : span_b) + 1024 >= (int64_t)1 << 31;
}

// The epilogue with which the one-pass kernel can take a product (-1: it cannot): the one
// place where its limits stand, for the dispatch and for the callers that need it (the
// tiled kernel knows no targets).  K: the operands of the networks up to degree 6 (344
// and, with 256 hidden values, 600), 11 x 4 or 19 x 2 runs of k in a lane's registers;
// longer ones were not built.
int wide_epi(int M, int N, int K, bool ta, bool tb, int64_t lda, int64_t ldb, const GemmEpi& ep) {
  const GemmVec vec = gemm_vec(ep);
  if (tb || ep.atomic || N < kWideMinN || M > kWideMaxM || K > (ta ? 352 : 608)) return -1;
  if (ep.out_f32 ? ep.out_bf16 || !vec.f32 : !vec.bf16) return -1;
  const int64_t kbn = ep.kb > 0 ? 256 / ep.kb + 1 : 0;  // blocks that a wavefront may touch
  const int64_t ldc = ep.out_f32 ? ep.ld_f32 : ep.ld_bf16;
  const int64_t far_wide = 4 * (16 * (ep.kb > 0 ? ep.kb : ldc) + kbn * (ldc + ldb) + 256 +
                                (ta ? (int64_t)K : 16) * lda + K + M + 16 * ep.ldmask +
                                (ep.target ? 16 * ep.ldt : 0));
  if (gemm_far(ta, tb, lda, ldb, ep.kb) || far_wide >= (int64_t)1 << 31) return -1;
  if (ep.target)
    return !ta && !ep.kb && !ep.mask && !ep.relu && ep.out_bf16 && aligned4(ep.target, ep.ldt, 0, 16)
               ? kWideMse : -1;
  if (ta) return ep.mask && !ep.bias && !ep.relu && ep.out_bf16 && vec.mask ? kWideMaskBf16 : -1;
  if (ep.mask) return -1;
  if (ep.relu) return ep.out_bf16 ? kWideReluBf16 : -1;
  return ep.out_f32 ? (ep.bias ? kWideF32Bias : kWideF32) : -1;
}

}  // namespace

hipError_t launch_gemm_bf16(int M, int N, int K, bool ta, bool tb, const uint16_t* A, int64_t lda,
                            const uint16_t* B, int64_t ldb, int kchunk, const GemmEpi& ep,
                            hipStream_t s) {
  const bool split = kchunk > 0;
  if (kchunk <= 0 || kchunk > K) kchunk = K;
  kchunk = (kchunk + kKStep - 1) / kKStep * kKStep;
  const int kz = (K + kchunk - 1) / kchunk;
  auto tiles_of = [&](int t) { return ((int64_t)N + t - 1) / t * (((int64_t)M + t - 1) / t); };
  // Tiles of 128 halve the LDS reads of a product, tiles of 64 give four times the
  // workgroups, which is what counts while K is short or the tiles are few.  Measured, us
  // with 64 and with 128, at 512 and more tiles of 128: plain FP32 out, K = 256 20.9 / 19.1 (344 x
  // 31000) and 16.2 / 15.1 (256 x 32768), K = 128 15.8 / 17.5; 64 over 128, BF16 out: 0.98 to 1.08 at
  // K = 416 and 1.03 to 1.16 at 512 (344 x 31000: 1.26); B transposed: 0.95 to 1.15 at 512 and 1.07
  // to 1.28 at 600; the mask: 0.88 to 1.10 at 512, 0.89 to 1.14 at 600 and 1.06 to 1.33 at 1024.
  // Some 350 tiles are enough for a longer K (344 x 16384, 384 tiles: FP32 out, K = 512 20.6 / 19.2;
  // K = 2048, mask 1.20, B transposed 1.10).  Half a tile is idle below 65 rows or columns (64 x 131072:
  // K = 600 with B transposed 40.8 / 45.9, 1024 70 / 75).
  // Long pieces of a split K range: once the pieces fill most of the CUs, as one round of
  // 128-row tiles (114 us with pieces of 8192) then takes less than the several of the
  // others (344 x 600 x 128000, 240 tiles of 128: 145 / 124; 512 x 768 x 65536, 192: 105 / 116; 256 x
  // 256 x 128000, 64: 66 / 113).  The pieces are the caller's: each adds its FP32 sum once, so
  // another cut would round the results differently.
  constexpr int kFill = 480, kFillLong = 350, kFillSplit = 224, kLongPiece = 4096;
  const bool far = gemm_far(ta, tb, lda, ldb, ep.kb);
  const bool plain = !ta && !tb && !ep.out_bf16;
  const int64_t tiles = tiles_of(128) * kz;
  const bool big =
      !far && M > 64 && N > 64 &&
      (split && kchunk >= kLongPiece
           ? tiles >= kFillSplit
           : tiles >= (kchunk >= (plain ? 512 : 1024) ? kFillLong : kFill) &&
                 kchunk >= (ta || tb ? 576 : plain ? 256 : 448));
  const int64_t total = tiles_of(big ? 128 : 64) * kz;
  const dim3 grid((unsigned)((total + kXcds - 1) / kXcds * kXcds));
  // A long batch takes the one-pass kernel, with 128 columns per workgroup as soon
  // as that gives every CU one (256 x 32768 x 344: 26 us, tiled 30; 16384 columns:
  // 22.6 and 21.8), with 256 from twice as many on (128000 columns: 45 us, 48 with
  // 128; 65536: 35 and 34).  Where its 16-row steps hold too little work for their
  // barrier and loads, the tiled kernel stays ahead: few rows at a short K (32 x 65536,
  // K = 32: tiled 6.3, one-pass 7.0; K = 128 7.5 and 6.4), 512 to 1024 rows of 32768 columns
  // at K <= 64 (ReLU 27 and 30), with BF16 out 2048 too (52 and 61; FP32 69 and 55), and
  // the mask, which a step loads just before it needs it (256 x 32768, K = 32 12 and 17,
  // K = 256 19 and 22, K = 344 even; 65536 columns, K = 64 22 and 24, with 1024 rows 112 and 93).
  const int epi = wide_epi(M, N, K, ta, tb, lda, ldb, ep);
  if (ep.target && epi < 0) return hipErrorInvalidValue;
  const bool few = M <= 32 && K <= 96 && N < 4 * kWideMinN;
  const bool thin = ta ? (N < 2 * kWideMinN && K <= 256) || (N < 4 * kWideMinN && K < 128 && M <= 512)
                       : N < 2 * kWideMinN && M >= 512 && M <= (ep.out_bf16 ? 2048 : 1024) && K <= 64;
  if (epi >= 0 && (ep.target || !(few || thin))) {
    auto wide = [&](auto ksc, auto nbc, auto tac) {
      constexpr int KS = decltype(ksc)::value, NB = decltype(nbc)::value;
      constexpr bool TA = decltype(tac)::value;
      const int64_t wgs = ((int64_t)N + 64 * NB - 1) / (64 * NB);
      const dim3 wgrid((unsigned)((wgs + kXcds - 1) / kXcds * kXcds));
      const size_t lds = 2 * 16 * wide_buffer(KS, TA) + ((size_t)M + 15) / 16 * 64;  // <= 56 KiB
      auto run = [&](auto ec) {
        hipLaunchKernelGGL((gemm_wide_kernel<KS, NB, TA, decltype(ec)::value, false>), wgrid,
                           dim3(256), lds, s, M, N, K, A, lda, B, ldb, ep, WideCells{});
      };
      if constexpr (TA) run(std::integral_constant<int, kWideMaskBf16>{});
      else if (epi == kWideMse) run(std::integral_constant<int, kWideMse>{});
      else if (epi == kWideF32) run(std::integral_constant<int, kWideF32>{});
      else if (epi == kWideF32Bias) run(std::integral_constant<int, kWideF32Bias>{});
      else run(std::integral_constant<int, kWideReluBf16>{});
    };
    auto by_k = [&](auto nbc, auto tac) {
      if (K <= 128) wide(std::integral_constant<int, 4>{}, nbc, tac);
      else if (K <= 256) wide(std::integral_constant<int, 8>{}, nbc, tac);
      else wide(std::integral_constant<int, 11>{}, nbc, tac);
    };
    using I2 = std::integral_constant<int, 2>;
    using I4 = std::integral_constant<int, 4>;
    if (K > 352) wide(std::integral_constant<int, 19>{}, I2{}, std::false_type{});
    else if (ta && N >= 2 * kWideMinN) by_k(I4{}, std::true_type{});
    else if (ta) by_k(I2{}, std::true_type{});
    else if (N >= 2 * kWideMinN) by_k(I4{}, std::false_type{});
    else by_k(I2{}, std::false_type{});
    return hipGetLastError();
  }
  auto go = [&](auto tc, auto fa, auto fb, auto fr) {
    hipLaunchKernelGGL((gemm_bf16_kernel<decltype(tc)::value, decltype(fa)::value,
                                         decltype(fb)::value, decltype(fr)::value>),
                       grid, dim3(256), 0, s, M, N, K, A, lda, B, ldb, kchunk, ep, gemm_vec(ep));
  };
  auto form = [&](auto tc, auto fr) {
    if (!ta && !tb) go(tc, std::false_type{}, std::false_type{}, fr);
    else if (ta && !tb) go(tc, std::true_type{}, std::false_type{}, fr);
    else if (!ta) go(tc, std::false_type{}, std::true_type{}, fr);
    else go(tc, std::true_type{}, std::true_type{}, fr);
  };
  if (far) form(std::integral_constant<int, 64>{}, std::true_type{});
  else if (big) form(std::integral_constant<int, 128>{}, std::false_type{});
  else form(std::integral_constant<int, 64>{}, std::false_type{});
  return hipGetLastError();
}

hipError_t launch_gemm_mse(int M, int N, int K, const uint16_t* A, int64_t lda, const uint16_t* B,
                           int64_t ldb, const GemmEpi& ep, float* Y, int64_t ldy, hipStream_t s) {
  // Fused where the one-pass kernel takes the product with its targets: the output is
  // neither written nor read back (a training step of 8000 cells, p = 6, 16 columns: 947
  // -> 880 us).
  if (wide_epi(M, N, K, false, false, lda, ldb, ep) == kWideMse)
    return launch_gemm_bf16(M, N, K, false, false, A, lda, B, ldb, 0, ep, s);
  GemmEpi out{};
  out.bias = ep.bias;
  out.out_f32 = Y;
  out.ld_f32 = ldy;
  hipError_t err = launch_gemm_bf16(M, N, K, false, false, A, lda, B, ldb, 0, out, s);
  if (err != hipSuccess) return err;
  return launch_mse_grad(ep.feat, M, ep.nrows, N, Y, ep.target, ldy, ep.roww, ep.scale, ep.out_bf16,
                         ep.loss, s);
}

// Y = S X0 cell by cell, X0 the gathered block (not normalised), in the cell-blocked
// layout (block stride ldy).  Fused where the batch is long, a cell's rows fit the
// one-pass kernel and a workgroup's cells their table, else the gather
// into X0 and the product.  With the assembly, gather and product against this:
// p = 6, 12^3 cells, 24 columns 120 / 103 us, 64 225 / 189, 256 825 / 740; p = 4, 14^3,
// 16 66 / 56, 64 110 / 86; p = 2, 24^3, 8 78 / 71, 128 271 / 244.
hipError_t launch_cell_linear(const Operator& op, int k, const double* R, int64_t ldr, int Fp,
                              const uint16_t* S, int64_t lds, uint16_t* X0, float* Y, int64_t ldy,
                              int pou_sqrt, const double* dsc, hipStream_t s) {
  const int64_t n = op.ncells * k;
  const int ks = Fp <= 128 ? 4 : Fp <= 256 ? 8 : 11;
  constexpr int NB = 2, kCols = 64 * NB;
  const int cells = kCols % k == 0 ? kCols / k : k % kCols == 0 ? 1 : (kCols - 1) / k + 2;
  const size_t table = (size_t)cells * ks * 32 * (sizeof(double) + sizeof(int));
  const bool aligned = ldr % 2 == 0 && reinterpret_cast<uintptr_t>(R) % 16 == 0 &&
                       reinterpret_cast<uintptr_t>(Y) % 16 == 0 && ldy % 4 == 0;
  const int64_t far = 4 * (16 * (int64_t)k + (kCols / k + 2) * ldy + 16 * lds + Fp);
  GemmEpi ep{};
  ep.out_f32 = Y;
  ep.ld_f32 = ldy;
  ep.kb = k;
  if (k % 8 || n < kWideMinN || Fp > 352 || table > 32 * 1024 || !aligned ||
      far >= (int64_t)1 << 31) {
    hipError_t err = launch_cell_gather(op, k, R, ldr, nullptr, 0, Fp, X0, nullptr,
                                        (int64_t)Fp * k, nullptr, pou_sqrt, dsc, 1, s);
    if (err != hipSuccess) return err;
    return launch_gemm_bf16(Fp, (int)n, Fp, false, false, S, lds, X0, (int64_t)Fp * k, 0, ep, s);
  }
  const WideCells wc{op.grid, op.np, k, cells, R, ldr, pou_sqrt, dsc};
  const int64_t wgs = (n + kCols - 1) / kCols;
  const dim3 grid((unsigned)((wgs + kXcds - 1) / kXcds * kXcds));
  auto go = [&](auto ksc) {
    constexpr int KS = decltype(ksc)::value;
    hipLaunchKernelGGL((gemm_wide_kernel<KS, NB, false, kWideF32, true>), grid, dim3(256),
                       2 * 16 * wide_buffer(KS, false) + table, s, Fp, (int)n, Fp, S, lds, nullptr,
                       (int64_t)0, ep, wc);
  };
  if (ks == 4) go(std::integral_constant<int, 4>{});
  else if (ks == 8) go(std::integral_constant<int, 8>{});
  else go(std::integral_constant<int, 11>{});
  return hipGetLastError();
}

hipError_t launch_cell_gather(const Operator& op, int k, const double* R, int64_t ldr,
                              const double* E, int64_t lde, int Fp, uint16_t* X0t, float* Tt,
                              int64_t ldx, float* rho, int pou_sqrt, const double* dsc,
                              int blocked, hipStream_t s) {
  // Few columns: several cells fill the 64 lanes, up to 8 and to 64 KiB of LDS (p = 6, 4096
  // cells, with E: k = 1 173 -> 55 us, k = 8 167 -> 62, k = 32 260 -> 196; p = 10, one or two
  // cells: k = 1 298 -> 245).  Every cell more lengthens a workgroup, so no more than leave
  // the chip two workgroups per CU (k = 1, one cell and eight: p = 6, 512 cells 36.9 and 40.1,
  // p = 2, 27 cells 6.2 and 9.1; 1000 cells, two and eight: 37.9 and 40.7); but 16 rows, which
  // gathers of fewer pay for with their stores, where a cell has enough to store (p = 6,
  // 512 cells: k = 4 36.8 alone, 26.1 four at a time, k = 2 37.2 and 30.5 by eight; p = 2, 27
  // cells, k = 4 6.2 and 6.9).
  const int F = op.np * op.np * op.np;
  int most = k < kCols ? kCols / k : 1;
  most = std::max(1, std::min({most, 8, 65536 / (F * kGatherNodeBytes)}));
  int C = (int)std::min<int64_t>((op.ncells + 511) / 512, most);
  const int full = (16 + k - 1) / k;  // cells of 16 rows
  if (full <= most && F * k >= 500) C = std::max(C, full);
  dim3 grid((unsigned)((op.ncells + C - 1) / C), C > 1 ? 1 : (k + kCols - 1) / kCols);
  // One cell: LDS as if for the largest cell, six workgroups on a CU (eight of them
  // take 95 instead of 91 us at p = 2, k = 64, 13824 cells).
  const size_t lds = std::max<size_t>((size_t)C * F * kGatherNodeBytes, C > 1 ? 0 : 26640);
  auto go = [&](auto multi) {
    hipLaunchKernelGGL((cell_gather_kernel<decltype(multi)::value>), grid, dim3(256),
                       lds, s, op.grid, op.np, k, C, R, ldr, E, lde,
                       Fp, X0t, Tt, ldx, rho, pou_sqrt, dsc, blocked);
  };
  if (C > 1) go(std::true_type{});
  else go(std::false_type{});
  return hipGetLastError();
}

hipError_t launch_skip_sym(int F, const float* S, int64_t lds, double* A, hipStream_t s) {
  hipLaunchKernelGGL(skip_sym_kernel, dim3(blocks_for((int64_t)F * F)), dim3(256), 0, s, F, S, lds,
                     A);
  return hipGetLastError();
}

hipError_t launch_skip_rebuild(int F, const double* V, const double* w, double margin, float* S,
                               int64_t lds, uint16_t* Sbf, int64_t ldsb, hipStream_t s) {
  hipLaunchKernelGGL(skip_rebuild_kernel, dim3(blocks_for((int64_t)F * F)), dim3(256), 0, s, F, V,
                     w, margin, S, lds, Sbf, ldsb);
  return hipGetLastError();
}

hipError_t launch_cell_scatter(const Operator& op, int k, const float* Yt, int64_t ldy,
                               const float* rho, const double* diag, const double* R, int64_t ldr,
                               double* Z, int64_t ldz, int pou_sqrt, const double* dsc,
                               int blocked, hipStream_t s) {
  const AsmArgs a{op.grid, k, Yt, ldy, rho, diag, R, ldr, Z, ldz, pou_sqrt, dsc, blocked};
  const int nlines = (int)((int64_t)op.grid.n[0] * op.grid.N[1] * op.grid.N[2]);  // <= ndofs
  const int nch = (k + 63) / 64;
  dim3 grid((unsigned)(((int64_t)nlines + kAsmLines - 1) / kAsmLines * nch));
  dim3 block(64 * kAsmLines);
  auto go = [&](auto pc) {
    constexpr int P = decltype(pc)::value;
    const int v = (blocked ? 4 : 0) + (rho ? 2 : 0) + (diag ? 1 : 0);
#define MF_ASM(B, Rh, D) \
  hipLaunchKernelGGL((node_assemble_kernel<P, B, Rh, D>), grid, block, 0, s, a, nlines, nch)
    switch (v) {
      case 0: MF_ASM(false, false, false); break;
      case 1: MF_ASM(false, false, true); break;
      case 2: MF_ASM(false, true, false); break;
      case 3: MF_ASM(false, true, true); break;
      case 4: MF_ASM(true, false, false); break;
      case 5: MF_ASM(true, false, true); break;
      case 6: MF_ASM(true, true, false); break;
      default: MF_ASM(true, true, true); break;
    }
#undef MF_ASM
  };
  switch (op.p) {
    case 1: go(std::integral_constant<int, 1>{}); break;
    case 2: go(std::integral_constant<int, 2>{}); break;
    case 3: go(std::integral_constant<int, 3>{}); break;
    case 4: go(std::integral_constant<int, 4>{}); break;
    case 5: go(std::integral_constant<int, 5>{}); break;
    case 6: go(std::integral_constant<int, 6>{}); break;
    case 7: go(std::integral_constant<int, 7>{}); break;
    case 8: go(std::integral_constant<int, 8>{}); break;
    case 9: go(std::integral_constant<int, 9>{}); break;
    case 10: go(std::integral_constant<int, 10>{}); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_mse_grad(int F, int Fp, int64_t nrows, int64_t ncols, const float* Yt,
                           const float* Tt, int64_t ld, const float* roww, float scale,
                           uint16_t* dYt, double* loss, hipStream_t s) {
  auto at = [](const void* p, size_t n) { return reinterpret_cast<uintptr_t>(p) % n == 0; };
  const int64_t pieces = (ncols + 1023) / 1024 * Fp;
  const dim3 grid((unsigned)std::min<int64_t>(pieces, 2048));  // one addition to loss each
  if (ld % 4 == 0 && at(Yt, 16) && at(Tt, 16) && at(roww, 16) && at(dYt, 8))
    hipLaunchKernelGGL((mse_grad_kernel<true>), grid, dim3(256), 0, s, F, Fp, nrows, ncols, Yt, Tt, ld,
                       roww, scale, dYt, loss);
  else
    hipLaunchKernelGGL((mse_grad_kernel<false>), grid, dim3(256), 0, s, F, Fp, nrows, ncols, Yt, Tt, ld,
                       roww, scale, dYt, loss);
  return hipGetLastError();
}

hipError_t launch_row_sums(int M, int64_t N, const uint16_t* X, int64_t ld, float* out,
                           bool accumulate, hipStream_t s) {
  const bool vec = ld % 2 == 0 && reinterpret_cast<uintptr_t>(X) % 4 == 0;
  if (vec)
    hipLaunchKernelGGL((row_sums_kernel<true>), dim3(M), dim3(kRowParts / 2), 0, s, N, X, ld, out,
                       accumulate ? 1 : 0);
  else
    hipLaunchKernelGGL((row_sums_kernel<false>), dim3(M), dim3(kRowParts), 0, s, N, X, ld, out,
                       accumulate ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_adam(int64_t n, float* w, const float* g, float* m1, float* m2, uint16_t* wbf,
                       float lr, float b1, float b2, float eps, int step, hipStream_t s) {
  const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
  hipLaunchKernelGGL(adam_kernel, dim3(blocks_for(n)), dim3(256), 0, s, n, w, g, m1, m2, wbf, lr,
                     b1, b2, eps, c1, c2);
  return hipGetLastError();
}

hipError_t launch_symmetrize(int n, float* S, int64_t ld, uint16_t* Sbf, hipStream_t s) {
  hipLaunchKernelGGL(symmetrize_kernel, dim3(blocks_for((int64_t)n * n)), dim3(256), 0, s, n, S, ld,
                     Sbf);
  return hipGetLastError();
}

hipError_t launch_to_bf16(int64_t n, const float* src, uint16_t* dst, hipStream_t s) {
  hipLaunchKernelGGL(to_bf16_kernel, dim3(blocks_for(n)), dim3(256), 0, s, n, src, dst);
  return hipGetLastError();
}

hipError_t launch_fill_f32(float* v, int64_t n, float x, hipStream_t s) {
  hipLaunchKernelGGL(fill_f32_kernel, dim3(blocks_for(n)), dim3(256), 0, s, v, n, x);
  return hipGetLastError();
}

}  // namespace mf
