// Device kernels of the SIS hot path for gfx950 (CDNA4, 64-wide wavefronts).
//
//  assemble      plan-time: dense matrix of h -> L+(h) from the fast-spectral
//                real-space kernels (one 32x32 output tile per workgroup,
//                direction tables staged through LDS)
//  class_rows    the cells' sums over the reflections that commute with the operator (FP64,
//                FP32 or bf16 pairs): the contraction then runs on one small matrix per class
//  gemm          collision contraction acc = X * op^T on MFMA
//                (FP64 v_mfma_f64_16x16x4; FP32 / 3xBF16 variants)
//  finish        per-cell epilogue: correction of eq. guided, delta scaling,
//                source, L, moments A1/A2, invariant projection
//  sweep1d       upwind transport sweep per velocity pair (+v1, -v1),
//                moments of h^{k+1/2} as per-wave partial sums
//  diffusion1d   per-case march of the SIS velocity equation, flow rates,
//                convergence test
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "kernels.h"

namespace sis {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(1))) void gbl_void_t;

__device__ inline double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// num / den where inv = 1 / den is known: the quotient by inv corrected by its own remainder
// (rounded as a division is, but for the last bit now and then), so that a chain of divisions
// by denominators known beforehand waits for three multiply-adds each.  Where the remainder has
// no value (infinities, den = 0) the plain product stands, which is then what a division gives.
__device__ __forceinline__ double div_known(double num, double den, double inv) {
  const double q = num * inv;
  const double r = __builtin_fma(__builtin_fma(-den, q, num), inv, q);
  return r == r ? r : q;
}

// Block-wide sum of K values per thread, fixed order.  Result in out[] for all threads.
// NT: the workgroup's threads where they are known (0: not): the reads of the waves' sums are then in flight
// together (a finish step of 17 rows of 512 with the projection: 15.8 -> 14.4 us with its contraction).
template <int K, int NT = 0>
__device__ inline void block_sum(double (&v)[K], double* sh /* >= 4*K */) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int nw = NT ? NT / 64 : (blockDim.x + 63) >> 6;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const double s = wave_sum(v[k]);
    if (lane == 0) sh[wave * K + k] = s;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < K; ++k) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < nw; ++w) s += sh[w * K + k];
    v[k] = s;
  }
  __syncthreads();
}

// ------------------------------------------------------------------ assemble
constexpr int kAsmPB = 8;      // terms staged per LDS round
constexpr int kAsmOuts = 7;    // outputs per thread (n^2 <= 256 * 7)

// One workgroup per (i0 i1, j0 j1) pair of velocity rows: the n x n outputs
// (i2, j2) share the difference row (d0, d1) of every kernel table.
__global__ __launch_bounds__(256) void assemble_kernel(int n, int T, const double* __restrict__ X,
                                                       const double* __restrict__ Y,
                                                       const double* __restrict__ feq, double lossc,
                                                       const double* __restrict__ beta_r,
                                                       double* __restrict__ op, int64_t ldo, int accumulate) {
  const int nd = 2 * n - 1;
  const int n3 = n * n * n;
  const int bi = blockIdx.x, bj = blockIdx.y;
  const int i0 = bi / n, i1 = bi % n, j0 = bj / n, j1 = bj % n;
  const int d0 = i0 - j0 + n - 1, d1 = i1 - j1 + n - 1;
  extern __shared__ double sm[];
  double* sY = sm;
  double* sX = sm + kAsmPB * nd;
  const int nout = n * n;
  double acc[kAsmOuts];
#pragma unroll
  for (int k = 0; k < kAsmOuts; ++k) acc[k] = 0.0;
  const size_t row = (static_cast<size_t>(d0) * nd + d1) * nd;
  const size_t nd3 = static_cast<size_t>(nd) * nd * nd;
  for (int t0 = 0; t0 < T; t0 += kAsmPB) {
    const int tb = min(kAsmPB, T - t0);
    for (int q = threadIdx.x; q < tb * nd; q += blockDim.x) {
      const int tt = q / nd, r = q % nd;
      sY[tt * nd + r] = Y[static_cast<size_t>(t0 + tt) * nd3 + row + r];
    }
    for (int q = threadIdx.x; q < tb * n; q += blockDim.x) {
      const int tt = q / n, r = q % n;
      sX[tt * n + r] = X[static_cast<size_t>(t0 + tt) * n3 + static_cast<size_t>(bi) * n + r];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kAsmOuts; ++k) {
      const int o = threadIdx.x + k * blockDim.x;
      if (o < nout) {
        const int i2 = o / n, j2 = o % n, dd = i2 - j2 + n - 1;
        double a = acc[k];
        for (int tt = 0; tt < tb; ++tt) a += sX[tt * n + i2] * sY[tt * nd + dd];
        acc[k] = a;
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int k = 0; k < kAsmOuts; ++k) {
    const int o = threadIdx.x + k * blockDim.x;
    if (o < nout) {
      const int i2 = o / n, j2 = o % n, dd = i2 - j2 + n - 1;
      const int ii = bi * n + i2, jj = bj * n + j2;
      double v = acc[k];
      if (feq) v -= lossc * feq[ii] * beta_r[row + dd];
      double* dst = op + static_cast<size_t>(ii) * ldo + jj;
      *dst = accumulate ? *dst + v : v;
    }
  }
}

// Restriction of the operator to distributions odd in v3 (and even in v2):
// red[i][j] = sum over the mirror images s(j) of j of sign(s) op[i][s(j)],
// rows and columns over the stored half (quarter) grid of every species.
__global__ void reduce_operator_kernel(const double* __restrict__ op, int64_t ld, double* __restrict__ red,
                                       int nsp, int n, int parity) {
  const int d2 = parity == 2 ? n / 2 : n, d3 = n / 2;
  const int nv = n * d2 * d3, n3 = n * n * n;
  const int64_t ldr = static_cast<int64_t>(nsp) * nv;
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (idx >= ldr * ldr) return;
  const int64_t ri = idx / ldr, rj = idx % ldr;
  auto full = [&](int64_t r) {  // full-grid index of a stored (species, velocity) row
    const int s = static_cast<int>(r / nv), v = static_cast<int>(r % nv);
    const int j1 = v / (d2 * d3), j2 = (v / d3) % d2 + (n - d2), j3 = v % d3 + n / 2;
    return static_cast<int64_t>(s) * n3 + (static_cast<int64_t>(j1) * n + j2) * n + j3;
  };
  const int64_t fi = full(ri), fj = full(rj);
  const int j3 = static_cast<int>(fj % n), j2 = static_cast<int>((fj / n) % n);
  const int64_t m3 = fj + (n - 1 - 2 * j3);            // v3 -> -v3
  const double* row = op + fi * ld;
  double s = row[fj] - row[m3];
  if (parity == 2) {
    const int64_t dm2 = static_cast<int64_t>(n - 1 - 2 * j2) * n;  // v2 -> -v2
    s += row[fj + dm2] - row[m3 + dm2];
  }
  red[idx] = s;
}

__global__ void convert_f32_kernel(const double* __restrict__ in, float* __restrict__ out, int64_t count) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < count) out[i] = static_cast<float>(in[i]);
}

// ------------------------------------------------------------------ reflection classes
// Images of orbit k of a row (see SymMap): off[g], bit a of g reflecting the a-th reflected axis.
// With PAIR the images of orbit k + 1 follow at off[g] + 1, or at off[g] - 1 where the third axis
// (LOGB = 3, top bit of g) is reflected.
template <int LOGB>
__device__ __forceinline__ void orbit_images(const SymMap& m, int k, int (&off)[1 << LOGB]) {
  // k / d with the multiplier ceil(2^32 / d): exact while k d < 2^32
  const int j1 = m.d23r == 1 ? k : static_cast<int>(__umulhi(static_cast<unsigned>(k), m.mul23));
  const int r = k - j1 * m.d23r;
  const int j2 = m.d3r == 1 ? r : static_cast<int>(__umulhi(static_cast<unsigned>(r), m.mul3));
  const int j3 = r - j2 * m.d3r;
  const int base = (m.lo1 + j1) * m.s1 + (m.lo2 + j2) * m.s2 + m.lo3 + j3;
  int e[3];
  if constexpr (LOGB == 1) {
    e[0] = m.lo1 ? (2 * j1 + 1) * m.s1 : (2 * j2 + 1) * m.s2;
  } else {
    e[0] = (2 * j1 + 1) * m.s1;
    e[1] = (2 * j2 + 1) * m.s2;
    e[2] = 2 * j3 + 1;
  }
#pragma unroll
  for (int g = 0; g < (1 << LOGB); ++g) {
    int o = base;
#pragma unroll
    for (int a = 0; a < LOGB; ++a)
      if (g & (1 << a)) o -= e[a];
    off[g] = o;
  }
}

// Sums over the images with the signs of every class (bit a of the class: odd under reflection
// a), in place; applied to the class sums it gives back the values at the images times 2^LOGB.
template <int LOGB, class T>
__device__ __forceinline__ void class_sums(T (&v)[1 << LOGB]) {
#pragma unroll
  for (int a = 0; a < LOGB; ++a)
#pragma unroll
    for (int g = 0; g < (1 << LOGB); ++g)
      if (!(g & (1 << a))) {
        const T p = v[g], q = v[g | (1 << a)];
        v[g] = p + q;
        v[g | (1 << a)] = p - q;
      }
}
typedef double v2d __attribute__((ext_vector_type(2)));

// Orbits k, k + 1 (k even, an even number of orbits along the third axis) of a row as 16-byte pairs.
template <int LOGB>
__device__ __forceinline__ v2d image_pair(const double* __restrict__ row, const int (&off)[1 << LOGB], int g) {
  if (LOGB == 3 && g >= 4) {
    const v2d t = *reinterpret_cast<const v2d*>(row + off[g] - 1);
    return v2d{t.y, t.x};
  }
  return *reinterpret_cast<const v2d*>(row + off[g]);
}
template <int LOGB>
__device__ __forceinline__ void image_pair_store(double* __restrict__ row, const int (&off)[1 << LOGB], int g, v2d v) {
  if (LOGB == 3 && g >= 4)
    *reinterpret_cast<v2d*>(row + off[g] - 1) = v2d{v.y, v.x};
  else
    *reinterpret_cast<v2d*>(row + off[g]) = v;
}

// Block row entries kk, kk + 1 (kk even) of class b, from one cell's rows X (minus Xref if given):
// the contraction tiles that read the cells themselves use it while staging.
template <int LOGB>
__device__ __forceinline__ double2 class_entry_pair(const SymMap& m, const double* __restrict__ X,
                                                    const double* __restrict__ Xref, int b, int kk) {
  double2 s = make_double2(0.0, 0.0);
  if (m.pairs) {
    if (kk >= m.kb) return s;
    const int sp = kk >= m.nvb;
    int off[1 << LOGB];
    orbit_images<LOGB>(m, kk - sp * m.nvb, off);
    const int64_t r0 = static_cast<int64_t>(sp) * m.nv;
    v2d v[1 << LOGB];
#pragma unroll
    for (int g = 0; g < (1 << LOGB); ++g) v[g] = image_pair<LOGB>(X + r0, off, g);
    if (Xref)
#pragma unroll
      for (int g = 0; g < (1 << LOGB); ++g) v[g] -= image_pair<LOGB>(Xref + r0, off, g);
#pragma unroll
    for (int g = 0; g < (1 << LOGB); ++g) {
      const bool neg = __builtin_popcount(b & g) & 1;
      s.x += neg ? -v[g].x : v[g].x;
      s.y += neg ? -v[g].y : v[g].y;
    }
    return s;
  }
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    if (kk + e >= m.kb) break;
    const int sp = kk + e >= m.nvb;
    int off[1 << LOGB];
    orbit_images<LOGB>(m, kk + e - sp * m.nvb, off);
    const int64_t r0 = static_cast<int64_t>(sp) * m.nv;
    double t = 0.0;
#pragma unroll
    for (int g = 0; g < (1 << LOGB); ++g) {
      const double v = Xref ? X[r0 + off[g]] - Xref[r0 + off[g]] : X[r0 + off[g]];
      t += (__builtin_popcount(b & g) & 1) ? -v : v;
    }
    (e ? s.y : s.x) = t;
  }
  return s;
}

// Blocks of the operator on the classes: with T_r = sum_g K[g i][(g ^ r) j] over the images g of
// the row and column orbits, class b has (1 / nb^2) sum_r (-1)^|b & r| T_r.
template <int LOGB>
__global__ __launch_bounds__(256) void class_operator_kernel(SymMap m, const double* __restrict__ op,
                                                             double* __restrict__ out) {
  constexpr int NB = 1 << LOGB;
  const int j = blockIdx.x * 256 + threadIdx.x, i = blockIdx.y;
  if (j >= m.ld) return;
  const int64_t n = static_cast<int64_t>(m.nsp) * m.nv;
  double t[NB];
#pragma unroll
  for (int r = 0; r < NB; ++r) t[r] = 0.0;
  if (j < m.kb) {
    const int si = i >= m.nvb, sj = j >= m.nvb;
    int oi[NB], oj[NB];
    orbit_images<LOGB>(m, i - si * m.nvb, oi);
    orbit_images<LOGB>(m, j - sj * m.nvb, oj);
#pragma unroll
    for (int g = 0; g < NB; ++g) {
      const double* row = op + (static_cast<int64_t>(si) * m.nv + oi[g]) * n + static_cast<int64_t>(sj) * m.nv;
#pragma unroll
      for (int r = 0; r < NB; ++r) t[r] += row[oj[g ^ r]];
    }
    class_sums<LOGB>(t);
  }
#pragma unroll
  for (int b = 0; b < NB; ++b)
    out[(static_cast<int64_t>(b) * m.kb + i) * m.ld + j] = t[b] * (1.0 / (NB * NB));
}

__device__ inline uint16_t bf16_rne(float f) {
  const uint32_t b = __float_as_uint(f);
  const uint32_t r = b + 0x7FFFu + ((b >> 16) & 1u);
  return static_cast<uint16_t>(r >> 16);
}
__device__ inline float bf16_to_f32(uint16_t h) { return __uint_as_float(static_cast<uint32_t>(h) << 16); }

__device__ __forceinline__ void bf16_pair(double x, uint32_t& hi, uint32_t& lo) {
  const uint16_t h = bf16_rne(static_cast<float>(x));
  hi = h;
  lo = bf16_rne(static_cast<float>(x - static_cast<double>(bf16_to_f32(h))));
}

// Cell operand of the contraction, once per launch: the class sums of x = X - Xref (Xref null: X)
// over each orbit's images, formed in FP64 and written as block rows
//   OUT 0: FP64 [cell][nb][ld];  1: rounded to FP32 [cell][nb][ld];
//   2, 3: the bf16 pair layout [cell][nb][2 Kp] (3: lo parts zero),
// entries past the classes' orbits zero.  Bound by HBM: it reads the distribution and writes as
// many values, 16 bytes per lane and access (the third axis is contiguous and keeps its order
// or is reversed whole): 24 576 cells of 6912 in FP64 0.52 ms = 5.2 TB/s.  What it buys there: the
// FP64 contraction of 4 blocks of 1728^2 takes 8.2 ms instead of 32.5 ms for the whole 6912^2.
template <int LOGB, int OUT, bool PAIR>
__global__ __launch_bounds__(256) void class_rows_kernel(SymMap m, const double* __restrict__ X,
                                                         const double* __restrict__ Xref,
                                                         const int32_t* __restrict__ active, int row_len, void* out) {
  constexpr int NB = 1 << LOGB;
  const int64_t cell = blockIdx.x;
  if (active && !active[cell]) return;
  const int kk = (blockIdx.y * 256 + threadIdx.x) * 2;
  if (kk >= row_len) return;
  const int64_t c0 = cell * m.nsp * static_cast<int64_t>(m.nv);
  v2d v[NB];
#pragma unroll
  for (int g = 0; g < NB; ++g) v[g] = v2d{0.0, 0.0};
  if constexpr (PAIR) {
    if (kk < m.kb) {
      const int sp = kk >= m.nvb;
      int off[NB];
      orbit_images<LOGB>(m, kk - sp * m.nvb, off);
      const int64_t r0 = c0 + static_cast<int64_t>(sp) * m.nv;
#pragma unroll
      for (int g = 0; g < NB; ++g) v[g] = image_pair<LOGB>(X + r0, off, g);
      if (Xref)
#pragma unroll
        for (int g = 0; g < NB; ++g) v[g] -= image_pair<LOGB>(Xref + r0, off, g);
    }
  } else {
#pragma unroll
    for (int e = 0; e < 2; ++e)
      if (kk + e < m.kb) {
        const int sp = kk + e >= m.nvb;
        int off[NB];
        orbit_images<LOGB>(m, kk + e - sp * m.nvb, off);
        const int64_t r0 = c0 + static_cast<int64_t>(sp) * m.nv;
#pragma unroll
        for (int g = 0; g < NB; ++g) v[g][e] = Xref ? X[r0 + off[g]] - Xref[r0 + off[g]] : X[r0 + off[g]];
      }
  }
  class_sums<LOGB>(v);
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int64_t row = cell * NB + b;
    if constexpr (OUT == 0) {
      *reinterpret_cast<v2d*>(static_cast<double*>(out) + row * row_len + kk) = v[b];
    } else if constexpr (OUT == 1) {
      *reinterpret_cast<float2*>(static_cast<float*>(out) + row * row_len + kk) =
          make_float2(static_cast<float>(v[b].x), static_cast<float>(v[b].y));
    } else {
      uint32_t h0, l0, h1, l1;
      bf16_pair(v[b].x, h0, l0);
      bf16_pair(v[b].y, h1, l1);
      uint16_t* p = static_cast<uint16_t*>(out) + row * 2 * row_len + (kk >> 5) * 64 + (kk & 31);
      *reinterpret_cast<uint32_t*>(p) = h0 | (h1 << 16);
      *reinterpret_cast<uint32_t*>(p + 32) = OUT == 2 ? l0 | (l1 << 16) : 0u;
    }
  }
}

// BF16 pair layout of the low-precision contraction operands (rows of K values,
// stored with Kp = K rounded up to 64): row r occupies 2 Kp bf16, and each block of
// 32 k-values holds its 32 hi parts followed by their 32 lo parts, so that one
// 128-byte line carries everything a 32-deep stage needs of the row.  Entries
// k >= K are zero in both halves; hi = RNE(x), lo = RNE(x - hi).  This kernel writes
// the operator's rows (row stride ld); class_rows_kernel writes the cells'.
__global__ void split_pairs_kernel(const double* __restrict__ X, int64_t rows, int K, int ld, int Kp,
                                   uint16_t* __restrict__ P) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= rows * Kp) return;
  const int64_t r = i / Kp;
  const int k = static_cast<int>(i - r * Kp);
  uint32_t h, l;
  bf16_pair(k < K ? X[r * ld + k] : 0.0, h, l);
  uint16_t* row = P + r * 2 * Kp + (k >> 5) * 64 + (k & 31);
  row[0] = static_cast<uint16_t>(h);
  row[32] = static_cast<uint16_t>(l);
}

// ------------------------------------------------------------------ FP64 MFMA GEMM
// acc[z][m][n] = sum_{k in [z*kps, min(K,(z+1)*kps))} X[m][k] * Op[n][k]
// Both operands are k-contiguous.  LDS tiles are stored k-major so that the
// 16 lanes of an MFMA operand column read 16 consecutive doubles.
constexpr int kBK = 16;
constexpr int kPad = 4;

// BK: k-depth of a stage; NBUF = 2: double-buffered LDS, software-pipelined: the next
// stage's global loads are issued at the start of a stage and written to the other LDS buffer
// two k-steps before its end, and the stage's one barrier sits before its last k-step's MFMAs,
// so that the next stage's first LDS reads overlap them.  NBUF = 1: one buffer (two barriers
// per stage, half the LDS, so deeper stages fit twice per CU).  PAD: row padding of the
// k-major LDS tiles (PAD = 1 with BK = 32 spreads the 64-lane stores of 16 k-rows x 4 rows
// over the banks).
// XCD-aware tile order of the contractions.  Workgroups go to the 8 XCDs
// round-robin in dispatch order, so each XCD's L2 would otherwise see cell and
// operator tiles from all over the grid.  Each XCD instead takes a contiguous
// run of the tile sequence, walked in groups of kGroup cell-tile rows (cell
// tile fastest), so the workgroups resident on one XCD share a few cell and
// operator tiles per k-stage.  A permutation of the (x, y) tiles: results are
// unchanged.  Returns the cell tile in .y and the operator tile in .x.
template <int kGroup = 8>
__device__ inline int2 xcd_tile() {
  const int gx = gridDim.x, gy = gridDim.y, total = gx * gy;
  int b = blockIdx.y * gx + blockIdx.x;
  if (total % 8 == 0) b = (b % 8) * (total / 8) + b / 8;
  const int first_y = (b / (kGroup * gx)) * kGroup;
  const int rows_in_group = min(kGroup, gy - first_y);
  const int in_group = b - first_y * gx;
  return make_int2(in_group / rows_in_group, first_y + in_group % rows_in_group);
}

// One output tile (operator tile bx, cell tile by, split bz) of the FP64 contraction; called by
// gemm_f64_kernel with the block indices and by the persistent 1-D iteration over virtual tiles.
// LOGB >= 0: X is the cells' own rows, their class sums formed while staging (few-cell tiles,
// which are bound by launch latency); otherwise block rows.
template <int BM, int BN, int WM, int WN, int BK = kBK, int NBUF = 2, int PAD = kPad, int LOGB = -1>
__device__ __forceinline__ void gemm_f64_tile(const GemmShape& sh, const double* __restrict__ X0,
                                              const double* __restrict__ Op0, double* __restrict__ C0, int bx,
                                              int by, int bz, const SymMap& sym) {
  constexpr int WAVES_N = BN / WN;
  constexpr int TM = WM / 16, TN = WN / 16;
  constexpr int A_LD = BM * BK / 2 / 256;
  constexpr int B_LD = BN * BK / 2 / 256;
  static_assert((BM / WM) * (BN / WN) == 4, "4 waves per workgroup");
  static_assert(A_LD >= 1 && B_LD >= 1, "tile too small");
  __shared__ double As[NBUF][BK][BM + PAD];
  __shared__ double Bs[NBUF][BK][BN + PAD];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave / WAVES_N) * WM, wn = (wave % WAVES_N) * WN;
  // plain grid order: the MFMA-bound FP64 tiles measured no faster (planar batch slower) with xcd_tile()
  const int64_t M = sh.M;
  const int N = sh.N, ldx = sh.ldx, ldo = sh.ldo;
  const int64_t m0 = static_cast<int64_t>(by) * BM;
  const int n0 = bx * BN;
  const int block = bz / sh.splits, split = bz - block * sh.splits;
  const int kbeg = split * sh.kps;
  const int kend = min(sh.K, kbeg + sh.kps);
  const double* X = LOGB >= 0 ? X0 : X0 + block * sh.xs;
  const double* Op = Op0 + block * sh.os;
  double* Cz = C0 + split * sh.cz + block * sh.cs;

  double2 ra[A_LD], rb[B_LD];
  auto gload = [&](int k0) {
#pragma unroll
    for (int i = 0; i < A_LD; ++i) {
      const int q = tid + 256 * i;
      const int r = q / (BK / 2), kc = (q % (BK / 2)) * 2;
      const int64_t gm = m0 + r;
      const int gk = k0 + kc;
      if constexpr (LOGB >= 0)
        ra[i] = (gm < M && gk < kend) ? class_entry_pair<LOGB>(sym, X + gm * ldx, nullptr, block, gk)
                                      : make_double2(0.0, 0.0);
      else
        ra[i] = (gm < M && gk < kend) ? *reinterpret_cast<const double2*>(X + gm * ldx + gk)
                                      : make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int i = 0; i < B_LD; ++i) {
      const int q = tid + 256 * i;
      const int r = q / (BK / 2), kc = (q % (BK / 2)) * 2;
      const int gn = n0 + r;
      const int gk = k0 + kc;
      rb[i] = (gn < N && gk < kend)
                  ? *reinterpret_cast<const double2*>(Op + static_cast<int64_t>(gn) * ldo + gk)
                  : make_double2(0.0, 0.0);
    }
  };
  auto sstore = [&](int buf) {
#pragma unroll
    for (int i = 0; i < A_LD; ++i) {
      const int q = tid + 256 * i;
      const int r = q / (BK / 2), kc = (q % (BK / 2)) * 2;
      As[buf][kc][r] = ra[i].x;
      As[buf][kc + 1][r] = ra[i].y;
    }
#pragma unroll
    for (int i = 0; i < B_LD; ++i) {
      const int q = tid + 256 * i;
      const int r = q / (BK / 2), kc = (q % (BK / 2)) * 2;
      Bs[buf][kc][r] = rb[i].x;
      Bs[buf][kc + 1][r] = rb[i].y;
    }
  };

  v4d acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = v4d{0.0, 0.0, 0.0, 0.0};

  const int nk = kend > kbeg ? (kend - kbeg + BK - 1) / BK : 0;
  if (nk > 0) {
    gload(kbeg);
    sstore(0);
  }
  __syncthreads();
  const int kr = lane >> 4, cc = lane & 15;
  if constexpr (NBUF == 2) {
    static_assert((BK / 4) % 2 == 0, "an even number of k-steps per stage");
    constexpr int KS = BK / 4, KW = KS - 2;
    double a[2][TM], b[2][TN];
    auto lread = [&](int buf, int kk, double* ar, double* br) {
#pragma unroll
      for (int i = 0; i < TM; ++i) ar[i] = As[buf][kk * 4 + kr][wm + i * 16 + cc];
#pragma unroll
      for (int j = 0; j < TN; ++j) br[j] = Bs[buf][kk * 4 + kr][wn + j * 16 + cc];
    };
    if (nk > 0) lread(0, 0, a[0], b[0]);
    for (int kt = 0; kt < nk; ++kt) {
      const int cur = kt & 1;
      const bool more = kt + 1 < nk;
      if (more) gload(kbeg + (kt + 1) * BK);
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) {
        const int c = kk & 1;
        if (kk + 1 < KS) lread(cur, kk + 1, a[c ^ 1], b[c ^ 1]);
        if (kk == KW && more) sstore(cur ^ 1);
        if (kk == KS - 1) {
          __syncthreads();       // next buffer written by every wave, this one read by every wave
          if (more) lread(cur ^ 1, 0, a[c ^ 1], b[c ^ 1]);
        }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[c][i], b[c][j], acc[i][j], 0, 0, 0);
      }
    }
  } else {
    static_assert(NBUF == 1, "one or two LDS buffers");
    for (int kt = 0; kt < nk; ++kt) {
      const int cur = 0;
      if (kt + 1 < nk) gload(kbeg + (kt + 1) * BK);
      // operands of k-step kk + 1 are read from LDS into the other register set
      // while the MFMAs of k-step kk run
      double a[2][TM], b[2][TN];
      auto lread = [&](int kk, double* ar, double* br) {
#pragma unroll
        for (int i = 0; i < TM; ++i) ar[i] = As[cur][kk * 4 + kr][wm + i * 16 + cc];
#pragma unroll
        for (int j = 0; j < TN; ++j) br[j] = Bs[cur][kk * 4 + kr][wn + j * 16 + cc];
      };
      lread(0, a[0], b[0]);
#pragma unroll
      for (int kk = 0; kk < BK / 4; ++kk) {
        const int c = kk & 1;
        if (kk + 1 < BK / 4) lread(kk + 1, a[c ^ 1], b[c ^ 1]);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[c][i], b[c][j], acc[i][j], 0, 0, 0);
      }
      // Schedule of the block above (a hint to the compiler's scheduler, which otherwise sinks
      // the reads behind the MFMAs that use the other register set): the first step's reads,
      // then per step one MFMA, the next step's LDS reads (ds_read2: two operands each), the
      // step's other MFMAs.
      constexpr int kReads = (TM + 1) / 2 + (TN + 1) / 2;
      __builtin_amdgcn_sched_group_barrier(0x100, kReads, 0);
#pragma unroll
      for (int kk = 0; kk + 1 < BK / 4; ++kk) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, kReads, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, TM * TN - 1, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, TM * TN, 0);
      __syncthreads();           // every wave is done with the buffer
      if (kt + 1 < nk) sstore(0);
      __syncthreads();
    }
  }
  // D layout of the 16x16x4 FP64 MFMA: lane l, element r -> row (l/16) + 4 r,
  // column l%16 (rows interleaved, unlike the FP32 forms)
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t gm = m0 + wm + i * 16 + kr + 4 * r;
        const int gn = n0 + wn + j * 16 + cc;
        if (gm < M && gn < N) Cz[gm * sh.ldc + gn] = acc[i][j][r];
      }
}

template <int BM, int BN, int WM, int WN, int BK = kBK, int NBUF = 2, int PAD = kPad, int LOGB = -1>
__global__ __launch_bounds__(256) void gemm_f64_kernel(const double* __restrict__ X, const double* __restrict__ Op,
                                                       double* __restrict__ C, GemmShape sh, SymMap sym) {
  gemm_f64_tile<BM, BN, WM, WN, BK, NBUF, PAD, LOGB>(sh, X, Op, C, blockIdx.x, blockIdx.y, blockIdx.z, sym);
}

// FP64 contraction on 128 x 128 tiles with LDS-DMA staging: the 128-row tile of the
// autotuner and the default heuristic.  Eight waves (4 along the cells x 2 along the
// operator rows) of 32 x 64 outputs: 2 x 4 blocks of the 16x16x4 FP64 MFMA, 64
// accumulator registers per lane, 127 registers in all, so two workgroups per CU give
// four waves per SIMD to cover each other's barrier and LDS waits.
// A stage is 16 deep and holds k pairs: slot (p, r) of an operand is the 16 bytes
// (k = 2p, 2p + 1) of its row r, 8 pairs x 128 rows per operand, 32 KB per stage with
// both operands.  Lane (kq, c) of an MFMA block reads one pair, (kq + 4 h, c), and feeds
// its first element to one MFMA and its second to the next, so a step of two MFMAs
// covers k = 2 kq + 8 h + {0, 1} over the four lane groups kq and a stage is two such
// ds_read_b128 steps (h = 0, 1) per block.  The stages are written by buffer-load LDS
// DMA (each lane's 16 bytes land at slot (8 j + wave) * 64 + lane of the operand's half
// of the stage for its instruction j, i.e. pair slot / 128, row slot % 128), so no registers or LDS stores
// carry the staging and the rows are copied without the transposing stores of the
// register-staged kernel.  The buffer descriptors start at the tile's first row and end
// after its last valid row; a pair past the split's k range gets an offset beyond the
// end: both read as zeros, which pads ragged cell, operator and k tails.
// Two stage buffers (distinct LDS objects, so that the compiler's LDS-DMA wait tracking
// lets reads of one proceed while the other is filled) and one barrier per stage: before
// it this wave's DMA of the next stage has landed (vmcnt(0)) and its reads of the current
// stage have completed; after it the next stage is visible to every wave and the current
// buffer is free, so the next stage's first reads are issued, then the DMA of the stage
// after it into the freed buffer, then the MFMAs of the current stage's second step.
// Preconditions (checked by the launcher): K even, row strides <= 2^20 (32-bit offsets within
// a tile's 128 rows).
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4))) void gemm_f64_dma_kernel(
    const double* __restrict__ X0, const double* __restrict__ Op0, double* __restrict__ C0, GemmShape sh) {
  __shared__ double2 buf0[2048];   // [operand][pair 0..7][row 0..127]
  __shared__ double2 buf1[2048];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // tiles to the XCDs in runs walked in groups of 8 cell-tile rows: the duct's fabric traffic
  // drops from 95 to 40 GB per launch at equal speed (groups of 2, 4, 16, 32: 68, 53, 45, 85 GB)
  const int2 tile = xcd_tile<8>();
  const int64_t M = sh.M;
  const int N = sh.N, ldx = sh.ldx, ldo = sh.ldo;
  const int64_t m0 = static_cast<int64_t>(tile.y) * 128;
  const int n0 = tile.x * 128;
  const int block = blockIdx.z / sh.splits, split = blockIdx.z - block * sh.splits;
  const int kbeg = split * sh.kps;
  const int kend = min(sh.K, kbeg + sh.kps);
  const int nk = kend > kbeg ? (kend - kbeg + 15) / 16 : 0;
  const double* X = X0 + block * sh.xs;
  const double* Op = Op0 + block * sh.os;
  double* Cz = C0 + split * sh.cz + block * sh.cs;

  // the last valid row ends after its K values (a block row may be the last of its array)
  const int rows_a = static_cast<int>(min<int64_t>(128, M - m0));
  const int rows_b = min(128, N - n0);
  const __amdgpu_buffer_rsrc_t rs_a = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<double*>(X + m0 * ldx), 0, ((rows_a - 1) * ldx + sh.K) * 8, 0x00020000);
  const __amdgpu_buffer_rsrc_t rs_b = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<double*>(Op + static_cast<int64_t>(n0) * ldo), 0, ((rows_b - 1) * ldo + sh.K) * 8, 0x00020000);
  // per DMA instruction j of this wave: the lane's pair and its byte offset within the tile
  uint32_t roff_a[2], roff_b[2];
  int pj[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int slot = (8 * j + wave) * 64 + lane;
    pj[j] = slot >> 7;
    roff_a[j] = static_cast<uint32_t>(((slot & 127) * ldx + 2 * pj[j]) * 8);
    roff_b[j] = static_cast<uint32_t>(((slot & 127) * ldo + 2 * pj[j]) * 8);
  }
  auto issue = [&](double2* buf, int k0) {
    const int krem = kend - k0;
    const uint32_t kb = static_cast<uint32_t>(k0) * 8u;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const uint32_t vo = 2 * pj[j] < krem ? roff_a[j] + kb : 0x80000000u;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_a, (lds_void_t*)&buf[(8 * j + wave) * 64], 16, vo, 0, 0, 0);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const uint32_t vo = 2 * pj[j] < krem ? roff_b[j] + kb : 0x80000000u;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_b, (lds_void_t*)&buf[1024 + (8 * j + wave) * 64], 16, vo, 0, 0,
                                               0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  const int kq = lane >> 4, cc = lane & 15;
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 64;
  v4d acc[2][4];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = v4d{0.0, 0.0, 0.0, 0.0};
  double2 a0[2], b0[4], a1[2], b1[4];
  auto lread = [&](const double2* buf, int h, double2* ar, double2* br) {
#pragma unroll
    for (int i = 0; i < 2; ++i) ar[i] = buf[(kq + 4 * h) * 128 + wm + 16 * i + cc];
#pragma unroll
    for (int j = 0; j < 4; ++j) br[j] = buf[1024 + (kq + 4 * h) * 128 + wn + 16 * j + cc];
  };
  auto mfma = [&](const double2* ar, const double2* br) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar[i].x, br[j].x, acc[i][j], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar[i].y, br[j].y, acc[i][j], 0, 0, 0);
  };
  // the stage in `cur` (its first step's operands already in a0, b0), the next one landing
  // in `nxt`; the DMA of stage k_dma goes to `cur` once every wave is past the barrier.  The
  // sched_barriers keep the MFMAs on their side of the barrier (they touch no memory, so the
  // scheduler would otherwise move them across it).
  // The wave's priority is raised from the barrier until the DMA is issued, so that the memory
  // instructions after the barrier are not held behind other waves' MFMAs (planar batch 1.74 ->
  // 1.70 ms, other shapes unchanged).
  auto stage = [&](double2* cur, double2* nxt, int k_dma) {
    lread(cur, 1, a1, b1);
    mfma(a0, b0);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
    __builtin_amdgcn_s_waitcnt(0x0f70);
    __syncthreads();
    lread(nxt, 0, a0, b0);
    __builtin_amdgcn_sched_barrier(0);
    issue(cur, k_dma);
    __builtin_amdgcn_s_setprio(0);
    mfma(a1, b1);
    __builtin_amdgcn_sched_barrier(0);
  };

  if (nk > 0) {
    issue(buf0, kbeg);
    __builtin_amdgcn_s_waitcnt(0x0f70);
    __syncthreads();
    issue(buf1, kbeg + (nk > 1 ? 16 : 0));
    lread(buf0, 0, a0, b0);
  }
  // stage pairs with the buffers named statically, then an odd last stage; past the last
  // stage the DMA target is clamped to the first stage (the freed buffer is not read again)
  int s = 0;
  for (; s + 1 < nk; s += 2) {
    stage(buf0, buf1, kbeg + (s + 2 < nk ? s + 2 : 0) * 16);
    stage(buf1, buf0, kbeg + (s + 3 < nk ? s + 3 : 0) * 16);
  }
  if (s < nk) {
    lread(buf0, 1, a1, b1);
    mfma(a0, b0);
    mfma(a1, b1);
  }
  // drain the clamped DMA before the workgroup can end
  __builtin_amdgcn_s_waitcnt(0x0f70);
  // D layout of the 16x16x4 FP64 MFMA: lane l, element r -> row l/16 + 4 r, column l%16
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t gm = m0 + wm + i * 16 + kq + 4 * r;
        const int gn = n0 + wn + j * 16 + cc;
        if (gm < M && gn < N) Cz[gm * sh.ldc + gn] = acc[i][j][r];
      }
}

// ------------------------------------------------------------------ FP32 MFMA GEMM
// Both operands are stored as float (class_rows_kernel rounds the cells' class sums), and so are the
// sums, which the MFMA holds in FP32 (finish_class_kernel adds splits and anchors in FP64).
template <int BM, int BN, int WM, int WN>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float* __restrict__ X0, const float* __restrict__ Op0,
                                                       float* __restrict__ C0, GemmShape sh) {
  constexpr int BK = 32;
  constexpr int WAVES_N = BN / WN;
  constexpr int TM = WM / 16, TN = WN / 16;
  constexpr int A_LD = BM * BK / 4 / 256;   // float4 loads of the (pre-rounded) cell operand
  constexpr int B_LD = BN * BK / 4 / 256;   // float4 loads of Op
  static_assert((BM / WM) * (BN / WN) == 4, "4 waves per workgroup");
  static_assert(A_LD >= 1 && B_LD >= 1, "tile too small");
  __shared__ float As[2][BK][BM + 4];
  __shared__ float Bs[2][BK][BN + 4];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave / WAVES_N) * WM, wn = (wave % WAVES_N) * WN;
  const int64_t M = sh.M;
  const int N = sh.N, ldx = sh.ldx, ldo = sh.ldo;
  const int64_t m0 = static_cast<int64_t>(blockIdx.y) * BM;
  const int n0 = blockIdx.x * BN;
  const int block = blockIdx.z / sh.splits, split = blockIdx.z - block * sh.splits;
  const int kbeg = split * sh.kps;
  const int kend = min(sh.K, kbeg + sh.kps);
  const float* X = X0 + block * sh.xs;
  const float* Op = Op0 + block * sh.os;
  float* Cz = C0 + split * sh.cz + block * sh.cs;

  float4 ra[A_LD];
  float4 rb[B_LD];
  auto gload = [&](int k0) {
#pragma unroll
    for (int i = 0; i < A_LD; ++i) {
      const int q = tid + 256 * i;
      const int r = q / (BK / 4), kc = (q % (BK / 4)) * 4;
      const int64_t gm = m0 + r;
      const int gk = k0 + kc;
      if (gm < M && gk + 3 < kend) {
        ra[i] = *reinterpret_cast<const float4*>(X + gm * ldx + gk);
      } else {
        float t[4];
        for (int e = 0; e < 4; ++e) t[e] = (gm < M && gk + e < kend) ? X[gm * ldx + gk + e] : 0.0f;
        ra[i] = make_float4(t[0], t[1], t[2], t[3]);
      }
    }
#pragma unroll
    for (int i = 0; i < B_LD; ++i) {
      const int q = tid + 256 * i;
      const int r = q / (BK / 4), kc = (q % (BK / 4)) * 4;
      const int gn = n0 + r;
      const int gk = k0 + kc;
      if (gn < N && gk + 3 < kend) {
        rb[i] = *reinterpret_cast<const float4*>(Op + static_cast<int64_t>(gn) * ldo + gk);
      } else {
        float t[4];
        for (int e = 0; e < 4; ++e)
          t[e] = (gn < N && gk + e < kend) ? Op[static_cast<int64_t>(gn) * ldo + gk + e] : 0.0f;
        rb[i] = make_float4(t[0], t[1], t[2], t[3]);
      }
    }
  };
  auto sstore = [&](int buf) {
#pragma unroll
    for (int i = 0; i < A_LD; ++i) {
      const int q = tid + 256 * i;
      const int r = q / (BK / 4), kc = (q % (BK / 4)) * 4;
      As[buf][kc][r] = ra[i].x;
      As[buf][kc + 1][r] = ra[i].y;
      As[buf][kc + 2][r] = ra[i].z;
      As[buf][kc + 3][r] = ra[i].w;
    }
#pragma unroll
    for (int i = 0; i < B_LD; ++i) {
      const int q = tid + 256 * i;
      const int r = q / (BK / 4), kc = (q % (BK / 4)) * 4;
      Bs[buf][kc][r] = rb[i].x;
      Bs[buf][kc + 1][r] = rb[i].y;
      Bs[buf][kc + 2][r] = rb[i].z;
      Bs[buf][kc + 3][r] = rb[i].w;
    }
  };

  v4f acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};

  const int nk = kend > kbeg ? (kend - kbeg + BK - 1) / BK : 0;
  if (nk > 0) {
    gload(kbeg);
    sstore(0);
  }
  __syncthreads();
  const int kr = lane >> 4, cc = lane & 15;
  for (int kt = 0; kt < nk; ++kt) {
    const int cur = kt & 1;
    if (kt + 1 < nk) gload(kbeg + (kt + 1) * BK);
#pragma unroll
    for (int kk = 0; kk < BK / 4; ++kk) {
      float a[TM], b[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) a[i] = As[cur][kk * 4 + kr][wm + i * 16 + cc];
#pragma unroll
      for (int j = 0; j < TN; ++j) b[j] = Bs[cur][kk * 4 + kr][wn + j * 16 + cc];
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    if (kt + 1 < nk) sstore(cur ^ 1);
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t gm = m0 + wm + i * 16 + kr * 4 + r;
        const int gn = n0 + wn + j * 16 + cc;
        if (gm < M && gn < N) Cz[gm * sh.ldc + gn] = acc[i][j][r];
      }
}

// FP32 contraction on 128 x 128 tiles with LDS-DMA staging: the form of gemm_f64_dma_kernel with 16-byte
// slots of four k values (quad p of a 32-deep stage, row r), so that a step of four MFMAs reads as
// many LDS bytes per MFMA cycle as its pairs: lane (kq, c) of a block reads quad kq + 4 h and feeds
// element e to the e-th MFMA (k = 4 kq + 16 h + e over the lane groups).  Waves, buffers, barriers, issue
// order, padding by the buffer descriptors and tile order as there.  Bound by the FP32 MFMA: 808 cells
// against two blocks of 4096^2 in 0.45-0.48 ms (113-120 of 157 TFLOP/s), where register-staged 64 x 128
// and 128 x 128 tiles took 0.60-0.75 ms.
// Preconditions (checked by the launcher): K, kps and the row strides multiples of 4, strides <= 2^21.
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4))) void gemm_f32_dma_kernel(
    const float* __restrict__ X0, const float* __restrict__ Op0, float* __restrict__ C0, GemmShape sh) {
  __shared__ float4 buf0[2048];   // [operand][quad 0..7][row 0..127]
  __shared__ float4 buf1[2048];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int2 tile = xcd_tile<8>();
  const int64_t M = sh.M;
  const int N = sh.N, ldx = sh.ldx, ldo = sh.ldo;
  const int64_t m0 = static_cast<int64_t>(tile.y) * 128;
  const int n0 = tile.x * 128;
  const int block = blockIdx.z / sh.splits, split = blockIdx.z - block * sh.splits;
  const int kbeg = split * sh.kps;
  const int kend = min(sh.K, kbeg + sh.kps);
  const int nk = kend > kbeg ? (kend - kbeg + 31) / 32 : 0;
  const float* X = X0 + block * sh.xs;
  const float* Op = Op0 + block * sh.os;
  float* Cz = C0 + split * sh.cz + block * sh.cs;

  const int rows_a = static_cast<int>(min<int64_t>(128, M - m0));
  const int rows_b = min(128, N - n0);
  const __amdgpu_buffer_rsrc_t rs_a = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(X + m0 * ldx), 0, ((rows_a - 1) * ldx + sh.K) * 4, 0x00020000);
  const __amdgpu_buffer_rsrc_t rs_b = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(Op + static_cast<int64_t>(n0) * ldo), 0, ((rows_b - 1) * ldo + sh.K) * 4, 0x00020000);
  uint32_t roff_a[2], roff_b[2];
  int pj[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int slot = (8 * j + wave) * 64 + lane;
    pj[j] = slot >> 7;
    roff_a[j] = static_cast<uint32_t>(((slot & 127) * ldx + 4 * pj[j]) * 4);
    roff_b[j] = static_cast<uint32_t>(((slot & 127) * ldo + 4 * pj[j]) * 4);
  }
  auto issue = [&](float4* buf, int k0) {
    const int krem = kend - k0;
    const uint32_t kb = static_cast<uint32_t>(k0) * 4u;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const uint32_t vo = 4 * pj[j] < krem ? roff_a[j] + kb : 0x80000000u;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_a, (lds_void_t*)&buf[(8 * j + wave) * 64], 16, vo, 0, 0, 0);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const uint32_t vo = 4 * pj[j] < krem ? roff_b[j] + kb : 0x80000000u;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_b, (lds_void_t*)&buf[1024 + (8 * j + wave) * 64], 16, vo, 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  const int kq = lane >> 4, cc = lane & 15;
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 64;
  v4f acc[2][4];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
  v4f a0[2], b0[4], a1[2], b1[4];
  auto lread = [&](const float4* buf, int h, v4f* ar, v4f* br) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
      ar[i] = *reinterpret_cast<const v4f*>(&buf[(kq + 4 * h) * 128 + wm + 16 * i + cc]);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      br[j] = *reinterpret_cast<const v4f*>(&buf[1024 + (kq + 4 * h) * 128 + wn + 16 * j + cc]);
  };
  auto mfma = [&](const v4f* ar, const v4f* br) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(ar[i][e], br[j][e], acc[i][j], 0, 0, 0);
  };
  auto stage = [&](float4* cur, float4* nxt, int k_dma) {
    lread(cur, 1, a1, b1);
    mfma(a0, b0);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
    __builtin_amdgcn_s_waitcnt(0x0f70);
    __syncthreads();
    lread(nxt, 0, a0, b0);
    __builtin_amdgcn_sched_barrier(0);
    issue(cur, k_dma);
    __builtin_amdgcn_s_setprio(0);
    mfma(a1, b1);
    __builtin_amdgcn_sched_barrier(0);
  };

  if (nk > 0) {
    issue(buf0, kbeg);
    __builtin_amdgcn_s_waitcnt(0x0f70);
    __syncthreads();
    issue(buf1, kbeg + (nk > 1 ? 32 : 0));
    lread(buf0, 0, a0, b0);
  }
  int s = 0;
  for (; s + 1 < nk; s += 2) {
    stage(buf0, buf1, kbeg + (s + 2 < nk ? s + 2 : 0) * 32);
    stage(buf1, buf0, kbeg + (s + 3 < nk ? s + 3 : 0) * 32);
  }
  if (s < nk) {
    lread(buf0, 1, a1, b1);
    mfma(a0, b0);
    mfma(a1, b1);
  }
  // drain the clamped DMA before the workgroup can end
  __builtin_amdgcn_s_waitcnt(0x0f70);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t gm = m0 + wm + i * 16 + kq * 4 + r;
        const int gn = n0 + wn + j * 16 + cc;
        if (gm < M && gn < N) Cz[gm * sh.ldc + gn] = acc[i][j][r];
      }
}

// ------------------------------------------------------------------ 3xBF16 MFMA GEMM
// x ~ xh + xl, op ~ oh + ol (bf16 pairs); acc += xl*oh + xh*ol + xh*oh on
// v_mfma_f32_16x16x32_bf16 with FP32 accumulation.  Both operands arrive in the
// pair layout of class_rows_kernel (the cell operand is split once per launch
// instead of once per output tile; Kp is a multiple of 64, so every stage is
// full).  k-stage of 64 staged through one LDS buffer per operand half; the next
// stage is prefetched into registers while the current one feeds the MFMAs.
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// NPROD = 1: the hi*hi product alone (lo halves neither loaded nor staged).
// LOGB >= 0 (32-row tile only): the cells' own rows are read in FP64 (X, minus Xref when given) and
// their class sums formed and split into hi and lo parts while they are staged, exactly as
// class_rows_kernel does, so that a launch on few cells needs no separate kernel; results are
// bit-identical.
// Row strides and block offsets of Xp and Op (sh.ldx, ldo, xs, os) are in bf16.
template <int BM, int BN, int WM, int WN, int NPROD = 3, int LOGB = -1>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void gemm_bf16x3_kernel(
    const uint16_t* __restrict__ Xp0, const uint16_t* __restrict__ Op0, float* __restrict__ C0, GemmShape sh,
    const double* __restrict__ X, const double* __restrict__ Xref, SymMap sym) {
  constexpr bool FUSED = LOGB >= 0;
  constexpr int BK = 64;                      // two MFMA k-steps per stage
  constexpr int WAVES_N = BN / WN;
  constexpr int TM = WM / 16, TN = WN / 16;
  constexpr int CH = BK / 8;                  // 16-byte chunks per row and stage
  constexpr int A_LD = BM * CH / 256;
  constexpr int B_LD = BN * CH / 256;
  static_assert(BM * CH % 256 == 0 && BN * CH % 256 == 0, "whole staging passes");
  static_assert((BM / WM) * (BN / WN) == 4, "4 waves per workgroup");
  // rows hold the 64 k-values of one m (or n) as eight 16-byte chunks, chunk c
  // of row r stored at slot c ^ ((r / 2) % 8): the 16 rows one MFMA operand read
  // touches and the two rows a 16-lane group of staging writes fills each
  // cover distinct banks.  A lane reads its 8 consecutive k values as one
  // 16-byte vector.
  constexpr int RS = BK;
  static_assert(CH == 8, "eight 16-byte chunks per row");
  __shared__ uint16_t sA[NPROD == 3 ? 2 : 1][BM][RS];
  __shared__ uint16_t sB[NPROD == 3 ? 2 : 1][BN][RS];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave / WAVES_N) * WM, wn = (wave % WAVES_N) * WN;
  // Swizzled slots are per-thread constants.  Staging: thread q = tid + 256 i
  // writes chunk tid % 8 of row tid / 8 + 32 i, so (row / 2) % 8 = (tid / 16) % 8.
  // Operand reads: rows wm + 16 i + lane % 16 (wm, 16 i multiples of 16), chunk
  // ks / 8 + lane / 16.
  const int wslot = ((tid & 7) ^ ((tid >> 4) & 7)) << 3;
  const int rsw = (lane & 15) >> 1;
  const int rslot0 = ((lane >> 4) ^ rsw) << 3, rslot1 = ((4 + (lane >> 4)) ^ rsw) << 3;
  const int2 tile = xcd_tile();
  const int64_t M = sh.M;
  const int N = sh.N;
  const int64_t m0 = static_cast<int64_t>(tile.y) * BM;
  const int n0 = tile.x * BN;
  const int block = blockIdx.z / sh.splits, split = blockIdx.z - block * sh.splits;
  const int kbeg = split * sh.kps;
  const int kend = min(sh.K, kbeg + sh.kps);
  const uint16_t* Xp = Xp0 + block * sh.xs;
  const uint16_t* Op = Op0 + block * sh.os;
  float* Cz = C0 + split * sh.cz + block * sh.cs;

  // (native vectors: HIP's uint4 struct copies from global memory kept the staging in scratch)
  u32x4 ra[2][A_LD], rb[2][B_LD];
  static_assert(!FUSED || A_LD == 1, "the fused split stages one chunk of eight values per thread");
  double2 xa[4];   // FUSED: the eight FP64 class sums of the thread's chunk
  // hi chunk of (row, k), k a multiple of 8 (its lo chunk sits 32 entries further);
  // rows past M or N read the last row: their products land in outputs that are
  // not stored
  auto pair_off = [&](int64_t row, int ld, int k) -> int64_t { return row * ld + (k >> 5) * 64 + (k & 31); };
  auto gload = [&](int k0) {
    if constexpr (FUSED) {
      const int64_t row = min<int64_t>(m0 + tid / CH, M - 1) * sym.nsp * static_cast<int64_t>(sym.nv);
      const int k = k0 + (tid % CH) * 8;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        xa[j] = class_entry_pair<FUSED ? LOGB : 1>(sym, X + row, Xref ? Xref + row : nullptr, block, k + 2 * j);
    } else {
#pragma unroll
      for (int i = 0; i < A_LD; ++i) {
        const int q = tid + 256 * i;
        const int64_t row = m0 + q / CH;
        const int64_t off = pair_off(row < M ? row : M - 1, sh.ldx, k0 + (q % CH) * 8);
        ra[0][i] = *reinterpret_cast<const u32x4*>(Xp + off);
        if constexpr (NPROD == 3) ra[1][i] = *reinterpret_cast<const u32x4*>(Xp + off + 32);
      }
    }
#pragma unroll
    for (int i = 0; i < B_LD; ++i) {
      const int q = tid + 256 * i;
      const int64_t row = n0 + q / CH;
      const int64_t off = pair_off(row < N ? row : N - 1, sh.ldo, k0 + (q % CH) * 8);
      rb[0][i] = *reinterpret_cast<const u32x4*>(Op + off);
      if constexpr (NPROD == 3) rb[1][i] = *reinterpret_cast<const u32x4*>(Op + off + 32);
    }
  };
  auto sstore = [&]() {
    if constexpr (FUSED) {
      // rounded to bf16 (hi), the remainder rounded again (lo), as in class_rows_kernel
      uint32_t hw[4], lw[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        uint32_t h0, l0, h1, l1;
        bf16_pair(xa[j].x, h0, l0);
        bf16_pair(xa[j].y, h1, l1);
        hw[j] = h0 | (h1 << 16);
        lw[j] = l0 | (l1 << 16);
      }
      ra[0][0] = u32x4{hw[0], hw[1], hw[2], hw[3]};
      if constexpr (NPROD == 3) ra[1][0] = u32x4{lw[0], lw[1], lw[2], lw[3]};
    }
#pragma unroll
    for (int i = 0; i < A_LD; ++i) {
      const int r = (tid + 256 * i) / CH, kc = wslot;
      *reinterpret_cast<u32x4*>(&sA[0][r][kc]) = ra[0][i];
      if constexpr (NPROD == 3) *reinterpret_cast<u32x4*>(&sA[NPROD == 3 ? 1 : 0][r][kc]) = ra[1][i];
    }
#pragma unroll
    for (int i = 0; i < B_LD; ++i) {
      const int r = (tid + 256 * i) / CH, kc = wslot;
      *reinterpret_cast<u32x4*>(&sB[0][r][kc]) = rb[0][i];
      if constexpr (NPROD == 3) *reinterpret_cast<u32x4*>(&sB[NPROD == 3 ? 1 : 0][r][kc]) = rb[1][i];
    }
  };

  v4f acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};

  const int nk = kend > kbeg ? (kend - kbeg + BK - 1) / BK : 0;
  if (nk > 0) {
    gload(kbeg);
    sstore();
  }
  __syncthreads();
  // operand layout of the 16x16x32 bf16 MFMA: lane l holds row (l % 16),
  // k = 8 * (l / 16) .. + 7
  const int rr = lane & 15, kq = (lane >> 4) * 8;
  for (int kt = 0; kt < nk; ++kt) {
    if (kt + 1 < nk) gload(kbeg + (kt + 1) * BK);
#pragma unroll
    for (int ks = 0; ks < BK; ks += 32) {
      v8bf ah[TM], al[TM], bh[TN], bl[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int r = wm + i * 16 + rr, c = ks == 0 ? rslot0 : rslot1;
        ah[i] = *reinterpret_cast<const v8bf*>(&sA[0][r][c]);
        if constexpr (NPROD == 3) al[i] = *reinterpret_cast<const v8bf*>(&sA[NPROD == 3 ? 1 : 0][r][c]);
      }
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int r = wn + j * 16 + rr, c = ks == 0 ? rslot0 : rslot1;
        bh[j] = *reinterpret_cast<const v8bf*>(&sB[0][r][c]);
        if constexpr (NPROD == 3) bl[j] = *reinterpret_cast<const v8bf*>(&sB[NPROD == 3 ? 1 : 0][r][c]);
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          if constexpr (NPROD == 3) {
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al[i], bh[j], acc[i][j], 0, 0, 0);
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[i], bl[j], acc[i][j], 0, 0, 0);
          }
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[i], bh[j], acc[i][j], 0, 0, 0);
        }
    }
    if (kt + 1 < nk) {
      __syncthreads();   // every wave is done reading the stage
      sstore();
      __syncthreads();
    }
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t gm = m0 + wm + i * 16 + (lane >> 4) * 4 + r;
        const int gn = n0 + wn + j * 16 + (lane & 15);
        if (gm < M && gn < N) Cz[gm * sh.ldc + gn] = acc[i][j][r];
      }
}

// 3xBF16 contraction on 256 x 256 output tiles, for large batches.  Eight waves
// (4 along the cells x 2 along the operator rows), each owning 64 x 128 outputs
// (128 FP32 accumulators per lane: two waves per SIMD fit the 256-register
// budget without spills).  Stages are 32 deep: the 256 cell rows and 256
// operator rows of a stage, hi and lo halves, are one 64 KB LDS buffer (rows of
// 128 bytes, chunk c of row r at slot c ^ ((r / 2) % 8), as in the 128-row
// kernel), and two buffers alternate.  The stages are written by LDS-DMA loads
// (global_load_lds_dwordx4: each lane's 16 bytes land at its own slot of a
// 1 KB run of eight rows; the swizzle is applied to the global address each
// lane fetches), issued one stage ahead, so no registers carry the staging.
// One barrier per stage: after it, the stage's data is visible to every wave and
// the other buffer (the previous stage) is free for the next DMA.  The two
// buffers are distinct LDS objects so that the compiler's LDS-DMA wait tracking
// lets reads of one proceed while the other is being filled.  Per stage and
// wave, right after the barrier: the four A fragments (hi and lo) and the first
// half of the operator fragments are read, then the DMA of the next stage is
// issued, then each operator half's 48 MFMAs run, product-major (lo*hi, hi*lo,
// hi*hi) so consecutive MFMAs update different accumulators.  Per output element
// the MFMA sequence is that of the 128-row kernel (same k blocks of 32, same
// product order), so the two agree to the last bit at equal split-K.
// Preconditions (checked by the launcher): rows times row stride under 2^32 bytes for
// both operands (32-bit DMA offsets).

__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2))) void gemm_bf16x3_wide_kernel(
    const uint16_t* __restrict__ Xp0, const uint16_t* __restrict__ Op0, float* __restrict__ C0, GemmShape sh) {
  __shared__ uint4 buf0[512][8];
  __shared__ uint4 buf1[512][8];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // groups of 4 cell-tile rows: an XCD's 32 resident workgroups then share 4 cell tiles and
  // 8 operator tiles per stage (2% faster on the duct than 8 x 4, which re-reads more of the
  // cell operand, the array that does not stay in the last-level cache)
  const int2 tile = xcd_tile<4>();
  const int64_t m0 = static_cast<int64_t>(tile.y) * 256;
  const int n0 = tile.x * 256;
  const int64_t M = sh.M;
  const int N = sh.N;
  const int block = blockIdx.z / sh.splits, split = blockIdx.z - block * sh.splits;
  const int kbeg = split * sh.kps;
  const int kend = min(sh.K, kbeg + sh.kps);
  const int nk = kend > kbeg ? (kend - kbeg) / 32 : 0;
  float* Cz = C0 + split * sh.cz + block * sh.cs;

  // DMA sources: waves 0-3 fill buffer rows 0-255 (cells), waves 4-7 rows 256-511
  // (operator rows), eight runs of eight rows each; rows past M or N read the last
  // row (their products land in outputs that are not stored)
  const bool isB = wave >= 4;
  const char* gbase = reinterpret_cast<const char*>(isB ? Op0 + block * sh.os : Xp0 + block * sh.xs);
  const int64_t rows = isB ? N : M;
  const int64_t row_bytes = 2 * static_cast<int64_t>(isB ? sh.ldo : sh.ldx);
  const int64_t row0 = isB ? n0 : m0;
  uint32_t off[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int r = (wave & 3) * 64 + i * 8 + (lane >> 3);
    const int c = (lane & 7) ^ ((r >> 1) & 7);
    const int64_t grow = min(row0 + r, rows - 1);
    off[i] = static_cast<uint32_t>(grow * row_bytes + (c >> 2) * 64 + (c & 3) * 16);
  }
  auto issue = [&](uint4(*buf)[8], int k0) {
    const uint32_t kb = static_cast<uint32_t>(k0) * 4u;
#pragma unroll
    for (int i = 0; i < 8; ++i)
      __builtin_amdgcn_global_load_lds((gbl_void_t*)(gbase + static_cast<uint64_t>(off[i] + kb)),
                                       (lds_void_t*)&buf[wave * 64 + i * 8][0], 16, 0, 0);
    // keep the loads ahead of the reads and MFMAs that follow
    __builtin_amdgcn_sched_barrier(0);
  };

  const int rr = lane & 15, q = lane >> 4, rsw = rr >> 1;
  const int s_hi = q ^ rsw, s_lo = (4 + q) ^ rsw;
  const int wm = (wave >> 1) * 64, wn = (wave & 1) * 128;
  v4f acc[4][8];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
  auto rd = [&](uint4(*buf)[8], int row, int slot) { return *reinterpret_cast<const v8bf*>(&buf[row][slot]); };
  // a stage: the A fragments and the operator's first half are read right after the barrier,
  // before the DMA of the next stage is issued (2.5% faster on the duct than issuing the DMA
  // first); then per operator half 48 MFMAs, product-major, with the second half's eight reads
  // spread over the first half's MFMAs
  v8bf ah[4], al[4], bh0[4], bl0[4];
  auto first_reads = [&](uint4(*buf)[8]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      ah[i] = rd(buf, wm + 16 * i + rr, s_hi);
      al[i] = rd(buf, wm + 16 * i + rr, s_lo);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      bh0[j] = rd(buf, 256 + wn + 16 * j + rr, s_hi);
      bl0[j] = rd(buf, 256 + wn + 16 * j + rr, s_lo);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto rest = [&](uint4(*buf)[8]) {
    v8bf bh1[4], bl1[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      bh1[j] = rd(buf, 256 + wn + 64 + 16 * j + rr, s_hi);
      bl1[j] = rd(buf, 256 + wn + 64 + 16 * j + rr, s_lo);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al[i], bh0[j], acc[i][j], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[i], bl0[j], acc[i][j], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[i], bh0[j], acc[i][j], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc[i][4 + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al[i], bh1[j], acc[i][4 + j], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc[i][4 + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[i], bl1[j], acc[i][4 + j], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc[i][4 + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[i], bh1[j], acc[i][4 + j], 0, 0, 0);
    for (int g = 0; g < 8; ++g) {
      __builtin_amdgcn_sched_group_barrier(0x008, 6, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 48, 0);
    __builtin_amdgcn_sched_barrier(0);
  };

  // Stage s sits in buffer s % 2.  The loop handles stage pairs with the buffers
  // named statically (no exit between the two halves: a mid-loop exit made the
  // register allocator shuffle the accumulators); an odd last stage follows it.
  // vmcnt(0) before each barrier: this wave's DMA of the stage has landed.  At the
  // end the DMA target is clamped to a valid stage: the buffer is free after the
  // barrier and nothing reads it again.
  if (nk > 0) issue(buf0, kbeg);
  int s = 0;
  for (; s + 1 < nk; s += 2) {
    __builtin_amdgcn_s_waitcnt(0x0f70);
    __syncthreads();
    first_reads(buf0);
    issue(buf1, kbeg + (s + 1) * 32);
    rest(buf0);
    __builtin_amdgcn_s_waitcnt(0x0f70);
    __syncthreads();
    first_reads(buf1);
    issue(buf0, kbeg + (s + 2 < nk ? s + 2 : 0) * 32);
    rest(buf1);
  }
  if (s < nk) {
    __builtin_amdgcn_s_waitcnt(0x0f70);
    __syncthreads();
    first_reads(buf0);
    rest(buf0);
  }
  // drain the clamped DMA of the last loop pass before the workgroup can end
  __builtin_amdgcn_s_waitcnt(0x0f70);
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t gm = m0 + wm + i * 16 + q * 4 + r;
        const int gn = n0 + wn + j * 16 + rr;
        if (gm < M && gn < N) Cz[gm * sh.ldc + gn] = acc[i][j][r];
      }
}

// ------------------------------------------------------------------ finish
// Projection and moments of a finished row (rhs and lh of the whole row written by this workgroup).
// LOGB >= 0: the correction by orbits, whose images share the tables' values (104 rows
// of 13 824: 28 us in all, 33 with the tables re-read whole).
template <int NT = 256, int LOGB = -1>   // NT: threads of the workgroup
__device__ __forceinline__ void finish_tail(const FinishArgs& a, int64_t c, double (&m)[9]) {
  __shared__ double sh[NT / 64 * 9];
  __shared__ double coef[5];
  if (a.project) {
    block_sum<9, NT>(m, sh);
  } else {   // the last four only: the sums across lanes are a tenth of a short row's time
    double am[4] = {m[5], m[6], m[7], m[8]};
    block_sum<4, NT>(am, sh);
    for (int k = 0; k < 4; ++k) m[5 + k] = am[k];
  }
  if (a.project) {
    if (threadIdx.x < 5) {
      double s = 0.0;
      for (int k = 0; k < 5; ++k) s += a.gram_inv[threadIdx.x * 5 + k] * m[k];
      coef[threadIdx.x] = s;
    }
    __syncthreads();
    const int n3 = a.n3;
    const int64_t base = c * n3;
    const double *vt1 = a.vtab, *vt2 = a.vtab + n3, *vt3 = a.vtab + 2 * static_cast<int64_t>(n3);
    const double* feq = a.feq + static_cast<int64_t>(c % a.nsp) * n3;
    double* rhs = a.rhs + base;
    double* lh = a.lh ? a.lh + base : nullptr;
    if constexpr (LOGB >= 0) {
      constexpr int NB = 1 << LOGB;
      for (int k = threadIdx.x; k < a.sym.nvb; k += NT) {
        int off[NB];
        orbit_images<LOGB>(a.sym, k, off);
        double r[NB], l[NB];
#pragma unroll
        for (int g = 0; g < NB; ++g) {
          r[g] = rhs[off[g]];
          l[g] = lh ? lh[off[g]] : 0.0;
        }
        const double v1 = vt1[off[0]], v2 = vt2[off[0]], v3 = vt3[off[0]], f = feq[off[0]];
        const double even = coef[0] + coef[4] * (v1 * v1 + v2 * v2 + v3 * v3);
        const double t1 = coef[1] * v1, t2 = coef[2] * v2, t3 = coef[3] * v3;
#pragma unroll
        for (int g = 0; g < NB; ++g) {
          const double corr = f * (even + ((g & 1) ? -t1 : t1) + ((g & 2) ? -t2 : t2) + ((g & 4) ? -t3 : t3));
          rhs[off[g]] = r[g] - corr;
          if (lh) lh[off[g]] = l[g] - corr;
        }
      }
    } else {
      for (int v = threadIdx.x; v < n3; v += blockDim.x) {
        const double v1 = vt1[v], v2 = vt2[v], v3 = vt3[v];
        const double vsq = v1 * v1 + v2 * v2 + v3 * v3;
        const double corr = feq[v] * (coef[0] + coef[1] * v1 + coef[2] * v2 + coef[3] * v3 + coef[4] * vsq);
        rhs[v] -= corr;
        if (lh) lh[v] -= corr;
      }
    }
  }
  if (a.amom && threadIdx.x == 0) {
    // with h stored for v2 > 0 only (h even in v2) the v2 v3 moments vanish identically
    a.amom[c * 4 + 0] = m[5];
    a.amom[c * 4 + 1] = m[6];
    a.amom[c * 4 + 2] = a.even_v2 ? 0.0 : m[7];
    a.amom[c * 4 + 3] = a.even_v2 ? 0.0 : m[8];
  }
}

// Row c = (cell, species) of the finish step; called by finish_kernel with the block index and by
// the persistent 1-D iteration.
__device__ __forceinline__ void finish_row(const FinishArgs& a, int64_t c_row, int nsplit, const double* acc_p) {
  const int64_t c = c_row;  // (cell, species) row of n3 values
  const int nsp = a.nsp, sp = static_cast<int>(c % nsp);
  const int64_t cell = c / nsp;
  if (a.active && !a.active[cell]) return;
  const int n3 = a.n3;
  const double del = a.delta[cell];
  const int fl = a.flow ? a.flow[cell] : 0;
  const double dUc = a.dU ? a.dU[c] : 0.0;
  const double dUq0 = a.dU ? a.dU[cell * nsp] : 0.0;
  const double dUq1 = (a.dU && nsp > 1) ? a.dU[cell * nsp + 1] : 0.0;
  const double ms = a.mass_ratio[sp];
  const double* feq = a.feq + static_cast<int64_t>(sp) * n3;
  const double* nu = a.nu + static_cast<int64_t>(sp) * n3;
  // L+ of the correction shapes of species 0 and 1 seen by species sp
  const double* kc0 = a.Kc + static_cast<int64_t>(sp) * n3;
  const double* kc1 = a.Kc + static_cast<int64_t>(nsp + sp) * n3;
  const double* vt1 = a.vtab;
  const double* vt2 = a.vtab + n3;
  const double* vt3 = a.vtab + 2 * static_cast<int64_t>(n3);
  const int64_t base = c * n3;
  const int64_t sstride = a.n_cells * static_cast<int64_t>(n3);
  double m[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) m[k] = 0.0;
  // one unknown: s = L+ h (partial sums and anchor), hv = h; returns the right side and L h
  auto unknown = [&](double s, double hv, double v1, double v2, double v3, double wv, double f, double nuv,
                     double k0, double k1, double& r, double& L) {
    const double vsq = v1 * v1 + v2 * v2 + v3 * v3;
    // L+ of the corrected iterate: the correction of every species of the cell enters
    double lp = s;
    if (a.dU) {
      lp += dUq0 * k0;
      if (nsp > 1) lp += dUq1 * k1;
    }
    const double hk = hv + dUc * 2.0 * ms * v3 * f;
    L = del * (lp - nuv * hk);
    double S = 0.0;
    if (fl == 1) S = v3 * f;
    else if (fl == 2 && nsp == 1) S = v3 * (vsq - 2.5) * f;
    r = del * lp + S;
    const double wL = wv * L;
    m[0] += wL;
    m[1] += wL * v1;
    m[2] += wL * v2;
    m[3] += wL * v3;
    m[4] += wL * vsq;
    m[5] += 2.0 * wv * v1 * v3 * L;
    m[6] += 2.0 * wv * v1 * v3 * hk;
    m[7] += 2.0 * wv * v2 * v3 * L;
    m[8] += 2.0 * wv * v2 * v3 * hk;
  };
  // U pairs (or unknowns) per lane and pass: the loads of all of them (partials, h, anchor) are
  // issued before any store (with one split the partial sum is the output row itself).  Rows
  // of even length are read and written in 16-byte pairs: the kernel is bound by its count of
  // vector-memory instructions.
  constexpr int U = 4;
  const int bs = blockDim.x;
  // pairs need 16-byte alignment of every row touched (caller arrays may be offset views)
  const uintptr_t align = reinterpret_cast<uintptr_t>(a.h + base) | reinterpret_cast<uintptr_t>(a.rhs + base) |
                          (a.lh ? reinterpret_cast<uintptr_t>(a.lh + base) : 0) |
                          (nsplit > 0 ? reinterpret_cast<uintptr_t>(acc_p + base) |
                                              reinterpret_cast<uintptr_t>(acc_p + sstride) : 0) |
                          (a.anchor_mode ? reinterpret_cast<uintptr_t>(a.accref + base) |
                                               reinterpret_cast<uintptr_t>(a.xref + base) : 0);
  if ((n3 & 1) == 0 && (align & 15) == 0) {
    constexpr int UP = U / 2;      // pairs per lane and pass
    const int np = n3 >> 1;
    auto d2p = [](const double* ptr) { return reinterpret_cast<const double2*>(ptr); };
    for (int p0 = threadIdx.x; p0 < np; p0 += UP * bs) {
      double2 sv[UP], hv[UP];
#pragma unroll
      for (int u = 0; u < UP; ++u) {
        sv[u] = make_double2(0.0, 0.0);
        hv[u] = p0 + u * bs < np ? d2p(a.h + base)[p0 + u * bs] : make_double2(0.0, 0.0);
      }
      // split-K partials four at a time, summed in split order
      for (int z0 = 0; z0 < nsplit; z0 += 4) {
        double2 t[4][UP];
#pragma unroll
        for (int dz = 0; dz < 4; ++dz)
#pragma unroll
          for (int u = 0; u < UP; ++u) {
            const int pp = p0 + u * bs;
            t[dz][u] = (z0 + dz < nsplit && pp < np) ? d2p(acc_p + (z0 + dz) * sstride + base)[pp]
                                                       : make_double2(0.0, 0.0);
          }
#pragma unroll
        for (int dz = 0; dz < 4; ++dz)
#pragma unroll
          for (int u = 0; u < UP; ++u)
            if (z0 + dz < nsplit) {
              sv[u].x += t[dz][u].x;
              sv[u].y += t[dz][u].y;
            }
      }
      if (a.anchor_mode == 2)
#pragma unroll
        for (int u = 0; u < UP; ++u)
          if (p0 + u * bs < np) {
            const double2 r = d2p(a.accref + base)[p0 + u * bs];
            sv[u].x += r.x;
            sv[u].y += r.y;
          }
#pragma unroll
      for (int u = 0; u < UP; ++u) {
        const int pp = p0 + u * bs;
        if (pp >= np) break;
        const double2 V1 = d2p(vt1)[pp], V2 = d2p(vt2)[pp], V3 = d2p(vt3)[pp], W = d2p(a.wtab)[pp];
        const double2 F = d2p(feq)[pp], NU = d2p(nu)[pp];
        double2 K0 = make_double2(0.0, 0.0), K1 = make_double2(0.0, 0.0);
        if (a.dU) {
          K0 = d2p(kc0)[pp];
          if (nsp > 1) K1 = d2p(kc1)[pp];
        }
        if (a.anchor_mode == 1) {
          reinterpret_cast<double2*>(a.accref + base)[pp] = sv[u];
          reinterpret_cast<double2*>(a.xref + base)[pp] = hv[u];
        }
        double2 R, L;
        unknown(sv[u].x, hv[u].x, V1.x, V2.x, V3.x, W.x, F.x, NU.x, K0.x, K1.x, R.x, L.x);
        unknown(sv[u].y, hv[u].y, V1.y, V2.y, V3.y, W.y, F.y, NU.y, K0.y, K1.y, R.y, L.y);
        reinterpret_cast<double2*>(a.rhs + base)[pp] = R;
        if (a.lh) reinterpret_cast<double2*>(a.lh + base)[pp] = L;
      }
    }
  } else {
    for (int v0 = threadIdx.x; v0 < n3; v0 += U * bs) {
      double sv[U], hv[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        sv[u] = 0.0;
        hv[u] = v0 + u * bs < n3 ? a.h[base + v0 + u * bs] : 0.0;
      }
      for (int z0 = 0; z0 < nsplit; z0 += 4) {
        double t[4][U];
#pragma unroll
        for (int dz = 0; dz < 4; ++dz)
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int v = v0 + u * bs;
            t[dz][u] = (z0 + dz < nsplit && v < n3) ? acc_p[(z0 + dz) * sstride + base + v] : 0.0;
          }
#pragma unroll
        for (int dz = 0; dz < 4; ++dz)
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (z0 + dz < nsplit) sv[u] += t[dz][u];
      }
      if (a.anchor_mode == 2)
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (v0 + u * bs < n3) sv[u] += a.accref[base + v0 + u * bs];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int v = v0 + u * bs;
        if (v >= n3) break;
        if (a.anchor_mode == 1) {
          a.accref[base + v] = sv[u];
          a.xref[base + v] = hv[u];
        }
        double r, L;
        unknown(sv[u], hv[u], vt1[v], vt2[v], vt3[v], a.wtab[v], feq[v], nu[v], a.dU ? kc0[v] : 0.0,
                (a.dU && nsp > 1) ? kc1[v] : 0.0, r, L);
        a.rhs[base + v] = r;
        if (a.lh) a.lh[base + v] = L;
      }
    }
  }
  finish_tail(a, c, m);
}

__global__ __launch_bounds__(256) void finish_kernel(FinishArgs a) { finish_row(a, blockIdx.x, a.splits, a.acc); }

// The finish step on the class sums of a reflected contraction: a lane takes an orbit (or two
// neighbouring ones, PAIR) of a row, adds the class sums of every split, turns them into L+ at the
// images and treats all images together.  Bound by HBM: 8 (splits + 2) bytes per unknown; the
// per-velocity tables, even (v3: odd) under the reflections, are read once per orbit instead of
// once per velocity (24 576 cells of 6912, one split: 0.74 ms = 5.5 TB/s, where finish_row on
// the whole matrix took 0.96 ms; 808 cells of 8192: 59 us with two splits, 76 us with four before).
// T: v2d (pairs) or double.
// A: double, or float for the sums of the low-precision contractions.
// UZ: splits whose loads are in flight together.
template <int LOGB, class T, class A, int UZ>
__device__ __forceinline__ void finish_class_row(const FinishArgs& a, int64_t row, double (&m)[9]) {
  constexpr int NB = 1 << LOGB;
  constexpr bool PAIR = sizeof(T) == 16;
  constexpr int STEP = PAIR ? 2 : 1;
  const SymMap& y = a.sym;
  const int nsp = a.nsp, sp = static_cast<int>(row % nsp);
  const int64_t cell = row / nsp;
  const int64_t nv = a.n3;
  const double del = a.delta[cell];
  const int fl = a.flow ? a.flow[cell] : 0;
  const double dUc = a.dU ? a.dU[row] : 0.0;
  const double dUq0 = a.dU ? a.dU[cell * nsp] : 0.0;
  const double dUq1 = (a.dU && nsp > 1) ? a.dU[cell * nsp + 1] : 0.0;
  const double ms = a.mass_ratio[sp];
  const double* feq = a.feq + sp * nv;
  const double* nu = a.nu + sp * nv;
  const double* kc0 = a.Kc + sp * nv;
  const double* kc1 = a.Kc + (nsp + sp) * nv;
  const double* vt1 = a.vtab;
  const double* vt2 = a.vtab + nv;
  const double* vt3 = a.vtab + 2 * nv;
  const double* h = a.h + row * nv;
  double* rhs = a.rhs + row * nv;
  double* lh = a.lh ? a.lh + row * nv : nullptr;
  const int64_t cr = cell * static_cast<int64_t>(NB) * y.ld + static_cast<int64_t>(sp) * y.nvb;  // class row of this species
  auto ld = [](const double* p) { return *reinterpret_cast<const T*>(p); };
  auto sum = [&](int64_t i) {
    const A* p = reinterpret_cast<const A*>(a.acc) + i;
    if constexpr (sizeof(A) == 8) {
      return *reinterpret_cast<const T*>(p);
    } else if constexpr (PAIR) {
      const float2 f = *reinterpret_cast<const float2*>(p);
      return T{f.x, f.y};
    } else {
      return static_cast<T>(*p);
    }
  };
  for (int k = threadIdx.x * STEP; k < y.nvb; k += blockDim.x * STEP) {
    int off[NB];
    orbit_images<LOGB>(y, k, off);
    T s[NB], hk[NB];
#pragma unroll
    for (int g = 0; g < NB; ++g) {
      s[g] = T{};
      if constexpr (PAIR) hk[g] = image_pair<LOGB>(h, off, g);
      else hk[g] = h[off[g]];
    }
    if (a.anchor_mode == 1) {
#pragma unroll
      for (int g = 0; g < NB; ++g) {
        if constexpr (PAIR) image_pair_store<LOGB>(a.xref + row * nv, off, g, hk[g]);
        else a.xref[row * nv + off[g]] = hk[g];
      }
    }
    const T V1 = ld(vt1 + off[0]), V2 = ld(vt2 + off[0]), V3 = ld(vt3 + off[0]), W = ld(a.wtab + off[0]);
    const T F = ld(feq + off[0]), NU = ld(nu + off[0]);
    T K = T{};
    if (a.dU) {
      K = dUq0 * ld(kc0 + off[0]);
      if (nsp > 1) K += dUq1 * ld(kc1 + off[0]);
    }
    int z = 0;
    for (; z + UZ <= a.splits; z += UZ) {
      T t[UZ][NB];
#pragma unroll
      for (int u = 0; u < UZ; ++u)
#pragma unroll
        for (int b = 0; b < NB; ++b) t[u][b] = sum((z + u) * a.acc_stride + cr + static_cast<int64_t>(b) * y.ld + k);
#pragma unroll
      for (int u = 0; u < UZ; ++u)
#pragma unroll
        for (int b = 0; b < NB; ++b) s[b] += t[u][b];
    }
    for (; z < a.splits; ++z)
#pragma unroll
      for (int b = 0; b < NB; ++b) s[b] += sum(z * a.acc_stride + cr + static_cast<int64_t>(b) * y.ld + k);
    if (a.anchor_mode) {
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        T* r = reinterpret_cast<T*>(a.accref + cr + static_cast<int64_t>(b) * y.ld + k);
        if (a.anchor_mode == 1) *r = s[b];
        else s[b] += *r;
      }
    }
    class_sums<LOGB>(s);   // L+ h at the images
    const T vsq = V1 * V1 + V2 * V2 + V3 * V3;
    T S = T{};
    if (fl == 1) S = V3 * F;
    else if (fl == 2 && nsp == 1) S = V3 * (vsq - 2.5) * F;
    const T dh = dUc * 2.0 * ms * V3 * F;
#pragma unroll
    for (int g = 0; g < NB; ++g) {
      const double o3 = LOGB == 3 && g >= 4 ? -1.0 : 1.0;   // correction and source are odd in v3
      const T lp = s[g] + o3 * K;
      hk[g] += o3 * dh;
      const T L = del * (lp - NU * hk[g]);
      const T r = del * lp + o3 * S;
      if constexpr (PAIR) {
        image_pair_store<LOGB>(rhs, off, g, r);
        if (lh) image_pair_store<LOGB>(lh, off, g, L);
      } else {
        rhs[off[g]] = r;
        if (lh) lh[off[g]] = L;
      }
      s[g] = L;
    }
    // sums of L and h over the images with the signs of the moments' velocity products
    class_sums<LOGB>(s);
    class_sums<LOGB>(hk);
    auto add = [&](double& acc, T v) {
      if constexpr (PAIR) acc += v.x + v.y;
      else acc += v;
    };
    constexpr int C1 = 1, C2 = LOGB >= 2 ? 2 : 0, C3 = LOGB == 3 ? 4 : 0;   // classes odd in v1, v2, v3
    if (a.project) {
      add(m[0], W * s[0]);
      add(m[1], W * V1 * s[C1]);
      add(m[2], W * V2 * s[C2]);
      add(m[3], W * V3 * s[C3]);
      add(m[4], W * vsq * s[0]);
    }
    const T w13 = 2.0 * W * V1 * V3, w23 = 2.0 * W * V2 * V3;
    add(m[5], w13 * s[C1 | C3]);
    add(m[6], w13 * hk[C1 | C3]);
    add(m[7], w23 * s[C2 | C3]);
    add(m[8], w23 * hk[C2 | C3]);
  }
}

// splits whose loads are in flight together
constexpr int finish_splits(int logb, bool deep) { return (logb == 1 ? 4 : logb == 2 ? 2 : 1) * (deep ? 2 : 1); }

// pairs: every row, and the class rows, in 16-byte pairs (lh may be offset by 8 bytes)
// NT threads a row: 256, or more where there are no more rows than compute units; DEEP: more splits in
// flight, at the price of waves a SIMD that few rows do not have.
template <int LOGB, class A, int NT, bool DEEP>
__global__ __launch_bounds__(NT) void finish_class_kernel(FinishArgs a) {
  constexpr int UZ = finish_splits(LOGB, DEEP);
  const int64_t row = blockIdx.x;
  if (a.active && !a.active[row / a.nsp]) return;
  double m[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) m[k] = 0.0;
  const uintptr_t align = reinterpret_cast<uintptr_t>(a.h) | reinterpret_cast<uintptr_t>(a.rhs) |
                          reinterpret_cast<uintptr_t>(a.lh);
  // (eight images of a pair would not fit the registers)
  bool pairs = false;
  if constexpr (LOGB < 3) {
    pairs = a.sym.pairs && (align & 15) == 0;
    if (pairs) finish_class_row<LOGB, v2d, A, UZ>(a, row, m);
  }
  if (!pairs) finish_class_row<LOGB, double, A, UZ>(a, row, m);
  finish_tail<NT, LOGB>(a, row, m);
}

// ------------------------------------------------------------------ sweep

// One thread per (case, species, |v1| > 0 velocity pair).  The two marches of a velocity are
// serial in x1 and there are few threads (a wave or less for each SIMD), so what bounds it is
// latency, of memory and of the instructions of a node.  Each thread keeps the right sides of
// the next AHEAD nodes in flight, for the second march from the start.  Waits for one of
// them count the loads and stores issued after it, so the code between them has no branches
// (else the counts are those of the shortest path through them): whole chunks of AHEAD nodes,
// then the remainder, for which nothing is left to load.  The stencil coefficients, which the
// workgroup shares, come through LDS, the next chunk's loaded while this one is marched, and
// the diagonals of kSweepGroup nodes are inverted before the march through them.
// With the division on the chain, 8 nodes in flight and branches among them: 51 us for 8
// cases of 101 nodes at 32^3, 106 us for the mixture's 16 cases of up to 201 at 24^3, 8.1 us for
// 17 nodes at 16^3; now 27, 52 and 5.0.
// Moments are taken afterwards by moments_kernel.
constexpr int kSweepNT = 64;      // a wave a workgroup, over all compute units
constexpr int kSweepAhead = 24;
constexpr int kSweepGroup = 8;

// One march: node i of it, counted from its first one, is cell first + dir * i (dir = +-1).
// The pointers walk from row to row (a row's address as a product of 64 bits takes more
// scalar instructions than the node itself).
template <int NT, int AHEAD>   // NT: threads of the workgroup
struct SweepMarch {
  static constexpr int kPer = (3 * AHEAD + NT - 1) / NT;
  const char* rhs;      // row of this species at the first node, advanced by the loads
  char* h;              // the same of h, advanced by the stores
  const double* coef;   // the direction's three coefficients at the first node
  int64_t step;         // bytes from node to node of rhs and h
  int dir, count;
  uint32_t off;         // bytes of the velocity
  double v1, dn;        // its speed, and its collision frequency times delta

  // the right side of node i, then on to the next (which stays at the last one)
  __device__ __forceinline__ double load(int i) {
    const double x = *reinterpret_cast<const double*>(rhs + off);
    rhs += i < count - 1 ? step : 0;
    return x;
  }
  __device__ __forceinline__ void load(double (&r)[AHEAD]) {
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) r[u] = load(u);
  }
  // the coefficients of a chunk (what is left over of the threads repeats the last ones)
  __device__ __forceinline__ void stage(int base, double (&c)[kPer]) const {
#pragma unroll
    for (int p = 0; p < kPer; ++p) {
      const int e = min(static_cast<int>(threadIdx.x) + p * NT, 3 * AHEAD - 1);
      c[p] = coef[dir * min(base + e / 3, count - 1) * 6 + e % 3];
    }
  }
  __device__ __forceinline__ void put(double x) {
    *reinterpret_cast<double*>(h + off) = x;
    h += step;
  }

  // nodes base .. of a chunk: NODES of them (TAIL: `left`, with nothing more to load)
  template <bool TAIL>
  __device__ __forceinline__ void chunk(int base, int left, const double* sh, double& h1, double& h2,
                                        double (&r)[AHEAD]) {
#pragma unroll
    for (int g0 = 0; g0 < AHEAD; g0 += kSweepGroup) {
      if (TAIL && g0 >= left) break;
      double den[kSweepGroup], inv[kSweepGroup], b[kSweepGroup], c[kSweepGroup];
#pragma unroll
      for (int u = 0; u < kSweepGroup; ++u) {
        den[u] = __builtin_fma(v1, sh[3 * (g0 + u)], dn);
        b[u] = sh[3 * (g0 + u) + 1];
        c[u] = sh[3 * (g0 + u) + 2];
      }
#pragma unroll
      for (int u = 0; u < kSweepGroup; ++u) inv[u] = 1.0 / den[u];
#pragma unroll
      for (int u = 0; u < kSweepGroup; ++u) asm volatile("" : "+v"(inv[u]));   // all of them before the march
#pragma unroll
      for (int u = 0; u < kSweepGroup; ++u) {
        if (TAIL && g0 + u >= left) break;
        const double val = div_known(r[g0 + u] - v1 * (b[u] * h1 + c[u] * h2), den[u], inv[u]);
        put(val);
        h2 = h1;
        h1 = val;
        if (!TAIL) r[g0 + u] = load(base + g0 + u + AHEAD);
      }
    }
  }

  // Marches from the values h1, h2 of the two nodes before the first; r holds the first right
  // sides, next the first coefficients.
  __device__ __forceinline__ void run(double& h1, double& h2, double (&r)[AHEAD], double (&next)[kPer], double* sh) {
    auto staged = [&] {
      __syncthreads();
#pragma unroll
      for (int p = 0; p < kPer; ++p) sh[min(static_cast<int>(threadIdx.x) + p * NT, 3 * AHEAD - 1)] = next[p];
      __syncthreads();
    };
    int base = 0;
    for (; base + AHEAD <= count; base += AHEAD) {
      staged();
      stage(base + AHEAD, next);
      chunk<false>(base, AHEAD, sh, h1, h2, r);
    }
    if (base < count) {
      staged();
      chunk<true>(base, count - base, sh, h1, h2, r);
    }
  }
};

template <int NT, int AHEAD>
__device__ __forceinline__ void sweep1d_block(const SweepArgs& a, int bx, int cs, int sp) {
  __shared__ double sh[3 * AHEAD];
  const int nsp = a.nsp;
  if (a.case_active && !a.case_active[cs]) return;   // uniform over the workgroup
  const int half = a.n3 / 2, n3 = a.n3;
  const int64_t c0 = a.node_off[cs];
  const int nodes = static_cast<int>(a.node_off[cs + 1] - c0);
  // threads beyond the last velocity march it once more (and store the same values)
  const int t = min(bx * NT + static_cast<int>(threadIdx.x), half - 1);
  const int d23 = a.d2 * a.d3;
  const int j1h = t / d23, r = t % d23;
  const int jp = a.n / 2 + j1h, jm = a.n / 2 - 1 - j1h;
  const int vp = jp * d23 + r, vm = jm * d23 + r;
  const double* nu = a.nu + static_cast<int64_t>(sp) * n3;
  const double v1 = a.v1d[jp], del = a.delta_case[cs], dnp = del * nu[vp], dnm = del * nu[vm];
  const uint32_t op = vp * 8u, om = vm * 8u;
  // v1 > 0: wall value 0, march towards the symmetry plane (nodes 1 .. nodes-1); v1 < 0:
  // specular reflection at the last node, march to the wall (nodes nodes-2 .. 0)
  const int64_t step = static_cast<int64_t>(nsp) * n3 * 8, row0 = (c0 * nsp + sp) * n3 * 8;
  const int64_t row1 = row0 + step, row2 = row0 + (nodes - 2) * step;
  const char* rhs = reinterpret_cast<const char*>(a.rhs);
  char* h = reinterpret_cast<char*>(a.h);
  using March = SweepMarch<NT, AHEAD>;
  March out = {rhs + row1, h + row0, a.coef + (c0 + 1) * 6, step, 1, nodes - 1, op, v1, dnp};
  March in = {rhs + row2, h + row2 + step, a.coef + (c0 + nodes - 2) * 6 + 3, -step, -1, nodes - 1, om, v1, dnm};
  double r_out[AHEAD], r_in[AHEAD], c_out[March::kPer], c_in[March::kPer];
  out.stage(0, c_out);
  out.load(r_out);
  in.stage(0, c_in);
  in.load(r_in);
  double h1 = 0.0, h2 = 0.0;
  out.put(0.0);
  out.run(h1, h2, r_out, c_out, sh);
  h2 = 0.0;
  in.put(h1);
  in.run(h1, h2, r_in, c_in, sh);
}

template <int NT>
__global__ __launch_bounds__(NT) void sweep1d_kernel(SweepArgs a) {
  sweep1d_block<NT, kSweepAhead>(a, blockIdx.x, blockIdx.y, blockIdx.z);
}

// Calls f(v1, v2, v3, h) for every unknown of row `row` (n3 values): in 16-byte pairs for
// rows of even length (the moment kernels are bound by their count of memory instructions).
template <typename F>
__device__ inline void for_row(int n3, const double* __restrict__ vtab, const double* __restrict__ h, int64_t row,
                               F&& f) {
  const double* hr = h + row * n3;
  if ((n3 & 1) == 0 && (reinterpret_cast<uintptr_t>(hr) & 15) == 0) {
    const int np = n3 >> 1;
    const double2* h2 = reinterpret_cast<const double2*>(hr);
    const double2* a1 = reinterpret_cast<const double2*>(vtab);
    const double2* a2 = reinterpret_cast<const double2*>(vtab + n3);
    const double2* a3 = reinterpret_cast<const double2*>(vtab + 2 * static_cast<int64_t>(n3));
#pragma unroll 2
    for (int p = threadIdx.x; p < np; p += blockDim.x) {
      const double2 x = h2[p], v1 = a1[p], v2 = a2[p], v3 = a3[p];
      f(v1.x, v2.x, v3.x, x.x);
      f(v1.y, v2.y, v3.y, x.y);
    }
  } else {
    for (int v = threadIdx.x; v < n3; v += blockDim.x)
      f(vtab[v], vtab[n3 + v], vtab[2 * static_cast<int64_t>(n3) + v], hr[v]);
  }
}

__device__ __forceinline__ void moments_row(int n3, int nsp, double ms0, double ms1, const double* __restrict__ vtab,
                                            const double* __restrict__ h, double w, double* __restrict__ mom,
                                            int64_t c) {   // c: (cell, species) row
  __shared__ double sh[4 * 4];
  const double ms = (c % nsp) == 0 ? ms0 : ms1;
  double m[4] = {0.0, 0.0, 0.0, 0.0};
  for_row(n3, vtab, h, c, [&](double v1, double v2, double v3, double hv) {
    const double vsq = v1 * v1 + v2 * v2 + v3 * v3;
    const double x = w * hv;
    m[0] += v3 * x;
    m[1] += (ms * vsq - 2.5) * v3 * x;
    m[2] += v3 * (2.0 * v1 * v1 - 1.0) * x;
    m[3] += 2.0 * ms * v1 * v3 * x;
  });
  block_sum<4>(m, sh);
  if (threadIdx.x == 0)
    for (int k = 0; k < 4; ++k) mom[c * 4 + k] = m[k];
}

__global__ __launch_bounds__(256) void moments_kernel(int n3, int nsp, double ms0, double ms1,
                                                      const double* __restrict__ vtab,
                                                      const double* __restrict__ h, double w,
                                                      double* __restrict__ mom) {
  moments_row(n3, nsp, ms0, ms1, vtab, h, w, mom, blockIdx.x);
}

// ------------------------------------------------------------------ diffusion (1-D)
// One workgroup per case.  The march from the wall is a serial recurrence, so one lane
// carries it, and nothing but it: the whole workgroup stages the nodes' equations into LDS
// with the inverses of their diagonals, and takes the outputs and the flow-rate integrals
// from the lane's values afterwards.  101 nodes: 8 us (7 without flow rates), and 26 with all of it on the lane.
constexpr int kDiffChunk = 256;

__device__ __forceinline__ void diffusion1d_case(const DiffusionArgs& a, int cs) {
  __shared__ double in[9][kDiffChunk];    // Uh, qh, G1, x, and a y_i = s - b y_{i-1} - c y_{i-2}: s, b, c, a, 1/a
  __shared__ double ys[kDiffChunk];       // y
  __shared__ double prev[3];              // x, U3 and q3 of the node before the chunk
  __shared__ double red[4 * 2];
  if (a.case_active && !a.case_active[cs]) return;   // uniform over the workgroup
  const int64_t c0 = a.node_off[cs];
  const int nodes = static_cast<int>(a.node_off[cs + 1] - c0);
  const double del = a.delta_case[cs];
  const bool pois = a.flow_case[cs] == 1;
  double y1 = 0.0, y2 = 0.0;
  double flow[2] = {0.0, 0.0};            // M, Q integrals
  for (int base = 0; base < nodes; base += kDiffChunk) {
    const int cnt = min(kDiffChunk, nodes - base);
    for (int t = threadIdx.x; t < cnt; t += blockDim.x) {
      const int64_t cell = c0 + base + t;
      const double Uh = a.mom[cell * 4 + 0], G1 = a.mom[cell * 4 + 2], x = a.x[cell];
      in[0][t] = Uh;
      in[1][t] = a.mom[cell * 4 + 1];
      in[2][t] = G1;
      in[3][t] = x;
      if (a.sis) {
        double s = Uh + G1, b = 0.0, c = 0.0, ca = 1.0;
        if (base + t > 0) {
          double A1 = 0.0;
          if (a.amom) A1 = a.amom[cell * 4 + 0] + a.N * del * a.amom[cell * 4 + 1];
          s = A1 - (pois ? a.N * del * x : 0.0);
          ca = a.coef[cell * 6 + 0];
          b = a.coef[cell * 6 + 1];
          c = a.coef[cell * 6 + 2];
        }
        in[4][t] = s;
        in[5][t] = b;
        in[6][t] = c;
        in[7][t] = ca;
        in[8][t] = 1.0 / ca;
      }
    }
    __syncthreads();
    if (threadIdx.x == 0 && a.sis) {
#pragma unroll 8
      for (int t = 0; t < cnt; ++t) {
        const double y = div_known((in[4][t] - in[6][t] * y2) - in[5][t] * y1, in[7][t], in[8][t]);
        y2 = y1;
        y1 = y;
        ys[t] = y;
      }
    }
    __syncthreads();
    // moments of h^{k+1} = h^{k+1/2} + dU 2 v3 f_eq (eq. guided)
    auto moved = [&](int t, double& U, double& dU, double& Un, double& qn) {
      const double Uh = in[0][t];
      U = a.sis ? ys[t] - in[2][t] : Uh;
      dU = U - Uh;
      Un = Uh + dU * a.cU;
      qn = in[1][t] + dU * a.cq;
    };
    for (int t = threadIdx.x; t < cnt; t += blockDim.x) {
      const int64_t cell = c0 + base + t;
      double U, dU, Un, qn;
      moved(t, U, dU, Un, qn);
      if (a.U) a.U[cell] = U;
      if (a.dU) a.dU[cell] = dU;
      if (a.qfield) a.qfield[cell] = qn;
      if (a.ufield) a.ufield[cell] = Un;
      if (base + t > 0) {
        double xp, Up, qp;
        if (t > 0) {
          double u_, d_;
          moved(t - 1, u_, d_, Up, qp);
          xp = in[3][t - 1];
        } else {
          xp = prev[0];
          Up = prev[1];
          qp = prev[2];
        }
        flow[0] += 0.5 * (Un + Up) * (in[3][t] - xp);
        flow[1] += 0.5 * (qn + qp) * (in[3][t] - xp);
      }
    }
    if (base + cnt < nodes) {
      __syncthreads();
      if (threadIdx.x == 0) {
        double u_, d_;
        moved(cnt - 1, u_, d_, prev[1], prev[2]);
        prev[0] = in[3][cnt - 1];
      }
      __syncthreads();
    }
  }
  if (!a.state) return;   // (no flow rates: the sums are a third of a short march)
  block_sum<2>(flow, red);
  if (threadIdx.x == 0) {
    const double M = 2.0 * flow[0], Q = 2.0 * flow[1];
    double* st = a.state + cs * 4;
    const double dM = fabs(M - st[0]) / fmax(fabs(M), 1e-300);
    const double dQ = fabs(Q - st[1]) / fmax(fabs(Q), 1e-300);
    const double res = fmax(dM, dQ);
    st[0] = M;
    st[1] = Q;
    st[2] = (M != M || Q != Q) ? __builtin_nan("") : res;
    const int it = a.iters[cs] + 1;
    a.iters[cs] = it;
    if (!(res >= a.eps) || M != M || Q != Q) a.case_active[cs] = 0;
    st[3] = static_cast<double>(it);
  }
}


// The case's flag, as its march left it, copied to the flags of its cells (what the next
// iteration's finish and sweep read), so that no separate expansion launch is needed.
__device__ __forceinline__ void case_flag_to_cells(const DiffusionArgs& a, int cs) {
  __shared__ int32_t flag;
  if (!a.cell_active || !a.case_active) return;
  __syncthreads();
  if (threadIdx.x == 0) flag = __hip_atomic_load(&a.case_active[cs], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  const int64_t c0 = a.node_off[cs], c1 = a.node_off[cs + 1];
  for (int64_t c = c0 + threadIdx.x; c < c1; c += blockDim.x) a.cell_active[c] = flag;
}

__global__ __launch_bounds__(kDiffChunk) void diffusion1d_kernel(DiffusionArgs a) {
  diffusion1d_case(a, blockIdx.x);
  case_flag_to_cells(a, blockIdx.x);
}

// Binary mixture (planar): the velocity equations of species B (own shear
// stress) and A (total stress minus B's), integrated once from the symmetry
// plane and marched from the wall; rows are (cell, species) with species A
// first.  mom[row][4] = {int v3 h, q, G1, P13}; U is per unit molar fraction.
// The two species march independently (lane s carries species s); staging, outputs and
// integrals as in diffusion1d_case.
__device__ __forceinline__ void diffusion1d_mix_case(const DiffusionArgs& a, int cs) {
  __shared__ double in_s[2][4][kDiffChunk];   // per species: Uh, qh, G, s
  __shared__ double in_c[5][kDiffChunk];      // per node: x, and b, c, a, 1/a (as in diffusion1d_case)
  __shared__ double ys[2][kDiffChunk];        // per species: y
  __shared__ double prev[5];                  // x, then U3 and q3 per species, of the node before the chunk
  __shared__ double red[4 * 4];
  if (a.case_active && !a.case_active[cs]) return;   // uniform over the workgroup
  const int64_t c0 = a.node_off[cs];
  const int nodes = static_cast<int>(a.node_off[cs + 1] - c0);
  const double del = a.delta_case[cs];
  const double pois = a.flow_case[cs] == 1 ? 1.0 : 0.0;
  const int sp = threadIdx.x;                 // marching lane: species sp (lanes 0, 1)
  double y1 = 0.0, y2 = 0.0;
  double flow[4] = {0.0, 0.0, 0.0, 0.0};      // (M, Q) integrals per species
  for (int base = 0; base < nodes; base += kDiffChunk) {
    const int cnt = min(kDiffChunk, nodes - base);
    for (int t = threadIdx.x; t < cnt; t += blockDim.x) {
      const int64_t cell = c0 + base + t;
      const double x = a.x[cell];
      const double PB = a.mom[(cell * 2 + 1) * 4 + 3];
      const bool inner = base + t > 0;
      in_c[0][t] = x;
      if (a.sis) {
        const double ca = inner ? a.coef[cell * 6 + 0] : 1.0;
        in_c[1][t] = inner ? a.coef[cell * 6 + 1] : 0.0;
        in_c[2][t] = inner ? a.coef[cell * 6 + 2] : 0.0;
        in_c[3][t] = ca;
        in_c[4][t] = 1.0 / ca;
      }
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int64_t r = cell * 2 + s;
        const double Uh = a.mom[r * 4 + 0] / a.chi[s], G = a.mom[r * 4 + 2];
        in_s[s][0][t] = Uh;
        in_s[s][1][t] = a.mom[r * 4 + 1];
        in_s[s][2][t] = G;
        if (a.sis) {
          double q = a.chi[s] * Uh + G;
          if (inner) {
            const double Nd = a.Ns[s] * del;
            double A = 0.0;
            if (a.amom) A = a.amom[r * 4 + 0] + Nd * a.amom[r * 4 + 1];
            q = s == 1 ? A - Nd * PB / a.mass_ratio[1] : A - Nd * (pois * x - PB);
          }
          in_s[s][3][t] = q;
        }
      }
    }
    __syncthreads();
    if (sp < 2 && a.sis) {
#pragma unroll 8
      for (int t = 0; t < cnt; ++t) {
        const double y = div_known((in_s[sp][3][t] - in_c[2][t] * y2) - in_c[1][t] * y1, in_c[3][t], in_c[4][t]);
        y2 = y1;
        y1 = y;
        ys[sp][t] = y;
      }
    }
    __syncthreads();
    auto moved = [&](int s, int t, double& U, double& dU, double& Un, double& qn) {
      const double Uh = in_s[s][0][t];
      U = a.sis ? (ys[s][t] - in_s[s][2][t]) / a.chi[s] : Uh;
      dU = U - Uh;
      Un = Uh + dU * a.cUs[s];
      qn = in_s[s][1][t] + dU * a.cqs[s];
    };
    for (int t = threadIdx.x; t < cnt; t += blockDim.x) {
      const double dx = base + t == 0 ? 0.0 : in_c[0][t] - (t > 0 ? in_c[0][t - 1] : prev[0]);
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int64_t r = (c0 + base + t) * 2 + s;
        double U, dU, Un, qn;
        moved(s, t, U, dU, Un, qn);
        if (a.U) a.U[r] = U;
        if (a.dU) a.dU[r] = dU;
        if (a.qfield) a.qfield[r] = qn;
        if (a.ufield) a.ufield[r] = Un;
        if (base + t > 0) {
          double Up, qp, u_, d_;
          if (t > 0) {
            moved(s, t - 1, u_, d_, Up, qp);
          } else {
            Up = prev[1 + 2 * s];
            qp = prev[2 + 2 * s];
          }
          flow[2 * s] += 0.5 * (Un + Up) * dx;
          flow[2 * s + 1] += 0.5 * (qn + qp) * dx;
        }
      }
    }
    if (base + cnt < nodes) {
      __syncthreads();
      if (sp < 2) {
        double u_, d_;
        moved(sp, cnt - 1, u_, d_, prev[1 + 2 * sp], prev[2 + 2 * sp]);
        if (sp == 0) prev[0] = in_c[0][cnt - 1];
      }
      __syncthreads();
    }
  }
  if (!a.state) return;
  block_sum<4>(flow, red);
  if (threadIdx.x == 0) {
    double* st = a.state + cs * 6;  // M_A, M_B, Q_A, Q_B, residual, iterations
    double res = 0.0;
    bool bad = false;
    for (int s = 0; s < 2; ++s) {
      const double M = 2.0 * a.flow_factor * flow[2 * s], Q = 2.0 * a.flow_factor * flow[2 * s + 1];
      res = fmax(res, fmax(fabs(M - st[s]) / fmax(fabs(M), 1e-300), fabs(Q - st[2 + s]) / fmax(fabs(Q), 1e-300)));
      bad = bad || M != M || Q != Q;
      st[s] = M;
      st[2 + s] = Q;
    }
    st[4] = bad ? __builtin_nan("") : res;
    const int it = a.iters[cs] + 1;
    a.iters[cs] = it;
    if (!(res >= a.eps) || bad) a.case_active[cs] = 0;
    st[5] = static_cast<double>(it);
  }
}

__global__ __launch_bounds__(kDiffChunk) void diffusion1d_mix_kernel(DiffusionArgs a) {
  diffusion1d_mix_case(a, blockIdx.x);
  case_flag_to_cells(a, blockIdx.x);
}

// ------------------------------------------------------------------ 2-D sweep
// One workgroup per (case, group of kSweepV velocity quadruples (+-|v1|, +-|v2|, v3)).
// The quadrants are swept in the order (+,+), (-,+), (+,-), (-,-).  Within a
// quadrant every upwind reference of a cell lies on an earlier anti-diagonal of
// the sweep order (ii + jj smaller), mirror ghosts read an earlier quadrant and
// the wrapped periodic references read later anti-diagonals (the previous
// iterate), so the anti-diagonals are processed in order with a workgroup
// barrier between them and the cells of one anti-diagonal in parallel: the
// values read are exactly those of the row-by-row sweep.
constexpr int kSweepV = 4;       // velocity quadruples per workgroup
constexpr int kSweepThreads = 256;

__global__ __launch_bounds__(kSweepThreads) void sweep2d_kernel(Sweep2DArgs a) {
  const int cs = blockIdx.y;
  if (a.case_active && !a.case_active[cs]) return;   // uniform over the workgroup
  const int n = a.n, hn = n / 2, n3 = a.n3, d3 = a.d3;
  const int nsp = a.nsp, sp = blockIdx.z;
  const double* __restrict__ nu = a.nu + static_cast<int64_t>(sp) * n3;
  const int quads = hn * hn * d3;
  // neighbouring velocity groups share cache lines of h and the right sides: with the group
  // count a multiple of 8, consecutive groups go to the same XCD (dispatch is round-robin)
  const int gx = gridDim.x;
  const int grp = (gx % 8 == 0) ? (blockIdx.x % 8) * (gx / 8) + blockIdx.x / 8 : blockIdx.x;
  const int tq = grp * kSweepV + threadIdx.x % kSweepV;
  const bool vvalid = tq < quads;
  const int t = vvalid ? tq : 0;
  const int jq1 = t / (hn * d3), jq2 = (t / d3) % hn, j3 = t % d3;
  const int slot = threadIdx.x / kSweepV, slots = kSweepThreads / kSweepV;
  const int n1 = a.n1[cs], n2 = a.n2[cs];
  const int64_t g0 = a.grid_off[cs];
  const double del = a.delta_case[cs];
  for (int q = 0; q < 4; ++q) {
    const int s1 = (q & 1) ? -1 : 1, s2 = (q & 2) ? -1 : 1;
    const int j1 = s1 > 0 ? hn + jq1 : hn - 1 - jq1;
    const int j2 = s2 > 0 ? hn + jq2 : hn - 1 - jq2;
    const int v = (j1 * n + j2) * d3 + j3;
    const int vm1 = ((n - 1 - j1) * n + j2) * d3 + j3;
    const int vm2 = (j1 * n + (n - 1 - j2)) * d3 + j3;
    const double av1 = fabs(a.v1d[j1]), av2 = fabs(a.v1d[j2]);
    const double dnu = del * nu[v];
    const int sg1 = s1 > 0 ? 0 : 1, sg2 = s2 > 0 ? 0 : 1;
    for (int d = 0; d < n1 + n2 - 1; ++d) {
      const int lo = max(0, d - (n2 - 1)), hi = min(d, n1 - 1);   // ii range of the anti-diagonal
      for (int c0 = lo; c0 <= hi; c0 += slots) {
        const int ii = c0 + slot;
        if (vvalid && ii <= hi) {
          const int jj = d - ii;
          const int i = s1 > 0 ? ii : n1 - 1 - ii;
          const int j = s2 > 0 ? jj : n2 - 1 - jj;
          const int cell = a.gcell[g0 + static_cast<int64_t>(i) * n2 + j];
          if (cell >= 0) {
            const int64_t o1 = (static_cast<int64_t>(cell) * 2 + 0) * 2 + sg1;
            const int64_t o2 = (static_cast<int64_t>(cell) * 2 + 1) * 2 + sg2;
            const int64_t row = static_cast<int64_t>(cell) * nsp + sp;
            double acc = a.rhs[row * n3 + v];
            const double c1[3] = {a.coef[o1 * 3], a.coef[o1 * 3 + 1], a.coef[o1 * 3 + 2]};
            const double c2[3] = {a.coef[o2 * 3], a.coef[o2 * 3 + 1], a.coef[o2 * 3 + 2]};
#pragma unroll
            for (int k = 0; k < 2; ++k) {
              const int8_t k1 = a.kind[o1 * 2 + k];
              if (k1) {
                const int64_t r = static_cast<int64_t>(a.ref[o1 * 2 + k]) * nsp + sp;
                acc -= av1 * c1[k + 1] * a.h[r * n3 + (k1 == 2 ? vm1 : v)];
              }
              const int8_t k2 = a.kind[o2 * 2 + k];
              if (k2) {
                const int64_t r = static_cast<int64_t>(a.ref[o2 * 2 + k]) * nsp + sp;
                acc -= av2 * c2[k + 1] * a.h[r * n3 + (k2 == 2 ? vm2 : v)];
              }
            }
            a.h[row * n3 + v] = acc / (dnu + av1 * c1[0] + av2 * c2[0]);
          }
        }
      }
      __syncthreads();
    }
  }
}

// Pipelined form of the same sweep for cross sections whose anti-diagonals hold at most
// P * 64 cells (min(n1, n2) <= 64 P): each slot owns up to P cells of a diagonal, and the
// read-only data of its cells on the next diagonal (cell index, stencil coefficients,
// upwind references, right side) are loaded while the current diagonal is computed, so
// that after each barrier only the upwind values of h are waited for.  The values and the
// order of the updates are those of sweep2d_kernel.  P is the smallest that covers the
// longest anti-diagonal: the per-cell state of two diagonals sits in registers, so a
// smaller P leaves room for more resident workgroups.
constexpr int kSweepMaxP = 3;

// The four words lane K of each group of four lanes holds, in every lane of the group
// (DPP quad_perm broadcast; every lane of the group must be active).
template <int K>
__device__ inline void quad_broadcast(const uint4& w, uint32_t* out) {
  constexpr int ctrl = K * 0x55;   // quad_perm(K, K, K, K)
  out[0] = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(w.x), ctrl, 0xF, 0xF, false));
  out[1] = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(w.y), ctrl, 0xF, 0xF, false));
  out[2] = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(w.z), ctrl, 0xF, 0xF, false));
  out[3] = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(w.w), ctrl, 0xF, 0xF, false));
}

struct Sweep2DPoint {
  int64_t row;          // (cell * nsp + species), -1: no fluid cell
  double rhs, c1[3], c2[3];
  int32_t r1[2], r2[2];
  int8_t k1[2], k2[2];
};

template <int kSweepP>
__global__ __launch_bounds__(kSweepThreads) void sweep2d_pipelined_kernel(Sweep2DArgs a) {
  const int cs = blockIdx.y;
  if (a.case_active && !a.case_active[cs]) return;   // uniform over the workgroup
  const int n = a.n, hn = n / 2, n3 = a.n3, d3 = a.d3;
  const int nsp = a.nsp, sp = blockIdx.z;
  const double* __restrict__ nu = a.nu + static_cast<int64_t>(sp) * n3;
  const int quads = hn * hn * d3;
  // neighbouring velocity groups share cache lines of h and the right sides: with the group
  // count a multiple of 8, consecutive groups go to the same XCD (dispatch is round-robin)
  const int gx = gridDim.x;
  const int grp = (gx % 8 == 0) ? (blockIdx.x % 8) * (gx / 8) + blockIdx.x / 8 : blockIdx.x;
  const int tq = grp * kSweepV + threadIdx.x % kSweepV;
  const bool vvalid = tq < quads;
  const int t = vvalid ? tq : 0;
  const int jq1 = t / (hn * d3), jq2 = (t / d3) % hn, j3 = t % d3;
  const int slot = threadIdx.x / kSweepV, slots = kSweepThreads / kSweepV;
  const int n1 = a.n1[cs], n2 = a.n2[cs];
  const int64_t g0 = a.grid_off[cs];
  const double del = a.delta_case[cs];
  for (int q = 0; q < 4; ++q) {
    const int s1 = (q & 1) ? -1 : 1, s2 = (q & 2) ? -1 : 1;
    const int j1 = s1 > 0 ? hn + jq1 : hn - 1 - jq1;
    const int j2 = s2 > 0 ? hn + jq2 : hn - 1 - jq2;
    const int v = (j1 * n + j2) * d3 + j3;
    const int vm1 = ((n - 1 - j1) * n + j2) * d3 + j3;
    const int vm2 = (j1 * n + (n - 1 - j2)) * d3 + j3;
    const double av1 = fabs(a.v1d[j1]), av2 = fabs(a.v1d[j2]);
    const double dnu = del * nu[v];
    const int sg1 = s1 > 0 ? 0 : 1, sg2 = s2 > 0 ? 0 : 1;
    static_assert(kSweepV == 4, "the four lanes of a slot (one velocity each) form a DPP quad");
    const int quad = threadIdx.x & 3;
    auto load = [&](int d, int p, Sweep2DPoint& pt) {
      pt.row = -1;
      const int lo = max(0, d - (n2 - 1)), hi = min(d, n1 - 1);
      const int ii = lo + slot + p * slots;
      int cell = -1;                     // the same for the four lanes of the quad
      if (d <= n1 + n2 - 2 && ii <= hi) {
        const int jj = d - ii;
        const int i = s1 > 0 ? ii : n1 - 1 - ii;
        const int j = s2 > 0 ? jj : n2 - 1 - jj;
        cell = a.gcell[g0 + static_cast<int64_t>(i) * n2 + j];
      }
      // the cell's two 32-byte stencil records (axis 1 with the sign of v1, axis 2 with the sign
      // of v2) are loaded 16 bytes per lane and broadcast within the quad: one load instruction
      // instead of fifteen (lanes of cells that do not exist read record 0 and discard it)
      const int64_t o = (static_cast<int64_t>(cell >= 0 ? cell : 0) * 2 + (quad >> 1)) * 2 + ((quad >> 1) ? sg2 : sg1);
      const uint4 w = *reinterpret_cast<const uint4*>(a.rec + o * 8 + (quad & 1) * 4);
      uint32_t r[16];
      quad_broadcast<0>(w, r);
      quad_broadcast<1>(w, r + 4);
      quad_broadcast<2>(w, r + 8);
      quad_broadcast<3>(w, r + 12);
      if (!vvalid || cell < 0) return;
      auto f64 = [&](int k) { return __builtin_bit_cast(double, (static_cast<uint64_t>(r[k + 1]) << 32) | r[k]); };
      pt.c1[0] = f64(0);
      pt.c1[1] = f64(2);
      pt.c1[2] = f64(4);
      pt.c2[0] = f64(8);
      pt.c2[1] = f64(10);
      pt.c2[2] = f64(12);
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        pt.k1[k] = static_cast<int8_t>(r[6 + k] & 3u);
        pt.r1[k] = static_cast<int32_t>(r[6 + k] >> 2);
        pt.k2[k] = static_cast<int8_t>(r[14 + k] & 3u);
        pt.r2[k] = static_cast<int32_t>(r[14 + k] >> 2);
      }
      pt.row = static_cast<int64_t>(cell) * nsp + sp;
      pt.rhs = a.rhs[pt.row * n3 + v];
    };
    Sweep2DPoint cur[kSweepP], nxt[kSweepP];
#pragma unroll
    for (int p = 0; p < kSweepP; ++p) load(0, p, cur[p]);
    for (int d = 0; d < n1 + n2 - 1; ++d) {
      double up[kSweepP][4];
#pragma unroll
      for (int p = 0; p < kSweepP; ++p) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          up[p][k] = (cur[p].row >= 0 && cur[p].k1[k])
                         ? a.h[(static_cast<int64_t>(cur[p].r1[k]) * nsp + sp) * n3 + (cur[p].k1[k] == 2 ? vm1 : v)]
                         : 0.0;
          up[p][2 + k] = (cur[p].row >= 0 && cur[p].k2[k])
                             ? a.h[(static_cast<int64_t>(cur[p].r2[k]) * nsp + sp) * n3 + (cur[p].k2[k] == 2 ? vm2 : v)]
                             : 0.0;
        }
      }
#pragma unroll
      for (int p = 0; p < kSweepP; ++p) load(d + 1, p, nxt[p]);
#pragma unroll
      for (int p = 0; p < kSweepP; ++p) {
        const Sweep2DPoint& c = cur[p];
        if (c.row >= 0) {
          double acc = c.rhs;
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            if (c.k1[k]) acc -= av1 * c.c1[k + 1] * up[p][k];
            if (c.k2[k]) acc -= av2 * c.c2[k + 1] * up[p][2 + k];
          }
          a.h[c.row * n3 + v] = acc / (dnu + av1 * c.c1[0] + av2 * c.c2[0]);
        }
      }
      __syncthreads();
#pragma unroll
      for (int p = 0; p < kSweepP; ++p) cur[p] = nxt[p];
    }
  }
}

// Row-blocked form of the same sweep, for cross sections of up to 128 cells along axis 2
// whose distributions fit 2 GiB (32-bit row offsets).  A lane owns one velocity quadruple,
// and every value it reads during the sweep belongs to that quadruple: in-quadrant upwind
// cells (this sweep), mirror ghosts (the quadrant with the mirrored axis's sign flipped: this
// sweep if it came earlier, else the previous iterate) and periodic wraps (cells later in the
// sweep order: the previous iterate).  Any order in which each cell follows its upwind cells
// along both axes therefore reads the values the anti-diagonal order reads; the update of
// each cell is the same expression in the same order (a reference of kind 0 enters with
// coefficient 0 in place of being skipped), so the results agree to the sign of zeros.
//
// A workgroup holds W <= 16 waves of 64 quadruples each, of one case and species, and sweeps
// the four quadrants in the same order (one workgroup per quadrant where no reference is a
// mirror ghost: then the quadrants do not read each other).  Within a quadrant the cells are
// taken in the sweep's orientation (row r, column c counted from the upwind corner); the
// columns are split into W blocks of cw <= CW (4 or 8) columns, and each wave runs over all
// rows of its block, column by column.  The two values left of the block come from wave
// w - 1 through LDS, double-buffered by row parity and handed on by two counters per wave
// (rows published, rows of the left neighbour's values read) instead of a workgroup barrier,
// so the waves run skewed by about a row each.  The two rows above are the lane's registers;
// only references that leave the grid are read from h: those of rows 0 and 1 (axis 1) when
// the quadrant starts, those of columns 0 and 1 (axis 2) with the right sides.  A block
// row's uniform data (grid-ordered stencil records and 32-bit row offsets) is loaded one word
// per lane four rows ahead into a ring of four LDS slots per wave and read back by broadcast
// (coefficients) or into scalar registers (offsets, reference words); the right sides are
// loaded two rows (CW = 4) or one row (CW = 8) ahead into registers that alternate between
// two sets (the row loop is unrolled by two), so that no register copy waits for a load.
// Rows of h and of the right sides are addressed through buffer descriptors, the row offset
// as the scalar offset: a solid or missing cell uses an empty descriptor, whose loads return
// 0 and whose stores are dropped, and gets a finite placeholder update (a = 1).  Lanes past
// the last quadruple repeat it (same values, same stores).  The full barrier at the end of a
// quadrant makes its stores visible to the mirror reads of the next.
constexpr int kRowWaves = 16;
constexpr int kRowSpinMax = 1 << 22; // bound on a wave's wait for its neighbour (never reached)

// Waits until *flag >= target (a counter another wave of the workgroup advances), then
// orders the LDS reads that follow after the writes published before the counter.
__device__ inline void lds_wait_at_least(const int* flag, int target) {
  for (int it = 0; it < kRowSpinMax; ++it) {
    if (__builtin_amdgcn_readfirstlane(__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) >=
        target)
      break;
    __builtin_amdgcn_s_sleep(1);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Publishes value in *flag after the wave's earlier LDS accesses.
__device__ inline void lds_publish(int* flag, int value) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __hip_atomic_store(flag, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

template <int CW>
__global__ __launch_bounds__(64 * kRowWaves) void sweep2d_rows_kernel(
    Sweep2DArgs a, const uint32_t* __restrict__ grec, const uint32_t* __restrict__ growb,
    const double* __restrict__ rhs, double* __restrict__ h) {
  // right sides are loaded two rows ahead for 4 columns per wave, one row ahead for 8 (registers)
  constexpr int kAhead = CW == 4 ? 2 : 1;
  constexpr int kRowWords = 17 * CW;                // 16 record words and a row offset per cell
  constexpr int kRegs = (kRowWords + 63) / 64;
  __shared__ double carry[2][kRowWaves][2][64];     // [row parity][wave][column c - 1, c - 2][lane]
  __shared__ __align__(16) uint32_t stage[kRowWaves][4][kRegs * 64];
  __shared__ double row1[kRowWaves][CW][64];        // second out-of-grid axis-1 reference of row 1
  __shared__ int published[kRowWaves];              // rows whose carry the wave has written
  __shared__ int consumed[kRowWaves];               // rows of its left neighbour's carry it has read
  const int n = a.n, hn = n / 2, n3 = a.n3, d3 = a.d3;
  const int nsp = a.nsp;
  const int quads = hn * hn * d3, groups = (quads + 63) / 64;
  // Workgroups are dispatched round-robin over the 8 XCDs (each with its own L2); numbering
  // them so that consecutive velocity groups of a case share an XCD lets the cache lines they
  // share (their 512-byte segments of a row are not line-aligned) be fetched once.
  const int nwg = gridDim.x, lin = blockIdx.x, per = nwg / 8, rem = nwg % 8, xcd = lin % 8, slot = lin / 8;
  const int logical = xcd < rem ? xcd * (per + 1) + slot : rem * (per + 1) + (xcd - rem) * per + slot;
  const int grp = logical % groups, cs = (logical / groups) % a.n_cases;
  const int sp = (logical / (groups * a.n_cases)) % nsp;
  // without mirror ghosts the quadrants do not read each other: one workgroup per quadrant
  const int qsplit = logical / (groups * a.n_cases * nsp);
  const int q0 = a.quad_split ? qsplit : 0, q1 = a.quad_split ? qsplit + 1 : 4;
  if (a.case_active && !a.case_active[cs]) return;   // uniform over the workgroup
  const int W = blockDim.x >> 6, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const double* __restrict__ nu = a.nu + static_cast<int64_t>(sp) * n3;
  const uint32_t row_bytes = static_cast<uint32_t>(nsp * n3 * 8);
  // Rows of species sp through buffer descriptors: cell c's row at byte offset growb (a 32-bit
  // scalar offset; the launcher checks that h fits), the lane's velocity in the vector offset.
  // A cell that is not there (solid, outside the grid) uses the empty descriptor: its loads
  // return 0 and its stores are dropped.
  const __amdgpu_buffer_rsrc_t rs_rhs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(rhs + static_cast<int64_t>(sp) * n3), 0, 0x7fffffff, 0x00020000);
  const __amdgpu_buffer_rsrc_t rs_h =
      __builtin_amdgcn_make_buffer_rsrc(h + static_cast<int64_t>(sp) * n3, 0, 0x7fffffff, 0x00020000);
  const __amdgpu_buffer_rsrc_t rs_none = __builtin_amdgcn_make_buffer_rsrc(h, 0, 0, 0x00020000);
  // lanes past the last quadruple repeat the last one (same wave, same values, same stores)
  const int tq = grp * 64 + lane;
  const int t = tq < quads ? tq : quads - 1;
  const int jq1 = t / (hn * d3), jq2 = (t / d3) % hn, j3 = t % d3;
  const int n1 = a.n1[cs], n2 = a.n2[cs];
  const int64_t g0 = a.grid_off[cs];
  const double del = a.delta_case[cs];
  const int cw = (n2 + W - 1) / W;                   // <= CW (checked by the launcher)
  const int jb0 = min(w * cw, n2), nb = min(cw, n2 - jb0);
  const int rows = (n1 + 1) & ~1;                    // an even count: row n1 of odd n1 is a placeholder
  auto ld = [&](const __amdgpu_buffer_rsrc_t& rs, uint32_t vo, uint32_t so) {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rs, vo, so, 0));
  };
  for (int q = q0; q < q1; ++q) {
    const int s1 = (q & 1) ? -1 : 1, s2 = (q & 2) ? -1 : 1;
    const int j1 = s1 > 0 ? hn + jq1 : hn - 1 - jq1;
    const int j2 = s2 > 0 ? hn + jq2 : hn - 1 - jq2;
    const int v = (j1 * n + j2) * d3 + j3;
    const int vm1 = ((n - 1 - j1) * n + j2) * d3 + j3;
    const int vm2 = (j1 * n + (n - 1 - j2)) * d3 + j3;
    const uint32_t vb = v * 8u, vm1b = vm1 * 8u, vm2b = vm2 * 8u;
    const double av1 = fabs(a.v1d[j1]), av2 = fabs(a.v1d[j2]);
    const double dnu = del * nu[v];
    const int sg1 = s1 > 0 ? 0 : 1, sg2 = s2 > 0 ? 0 : 1;
    if (lane == 0) {
      published[w] = 0;
      consumed[w] = 0;
    }
    __syncthreads();
    // grid index of the block's column k in oriented row r: rbase(r) + dj k
    const int dj = s2, jstart = s2 > 0 ? jb0 : n2 - 1 - jb0;
    auto rbase = [&](int r) { return g0 + static_cast<int64_t>(s1 > 0 ? r : n1 - 1 - r) * n2 + jstart; };
    // Staging slot of row r: 16 record words per cell (axis 1 with the sign of v1, then axis 2
    // with the sign of v2), then the cells' row offsets (0xffffffff: none), one word per lane.
    // Where there is no cell (outside the block or the grid) the words are read from the
    // tables' extra solid entry (a = 1, no references, no row): every lane loads, and uses
    // the word as loaded, so that all rows issue the same memory instructions and the waits
    // for them stay counted.
    auto load_row = [&](int r, uint32_t (&sv)[kRegs]) {
      const bool rv = r < n1;
      const int64_t gb = rbase(rv ? r : 0);
#pragma unroll
      for (int u = 0; u < kRegs; ++u) {
        const int x = 64 * u + lane;
        const bool isrec = x < 16 * CW;
        const int k = isrec ? x >> 4 : x - 16 * CW, d = x & 15, axis = d >> 3;
        const int64_t gk = rv && k < nb ? gb + dj * k : a.grid_none;
        sv[u] = isrec ? grec[(gk * 4 + axis * 2 + (axis ? sg2 : sg1)) * 8 + (d & 7)] : growb[gk];
      }
    };
    auto put_row = [&](int r, const uint32_t (&sv)[kRegs]) {
#pragma unroll
      for (int u = 0; u < kRegs; ++u) stage[w][r & 3][64 * u + lane] = sv[u];
    };
    auto coef = [&](int r, int k, int wd) {
      return *reinterpret_cast<const double*>(&stage[w][r & 3][16 * k + wd]);
    };
    auto word = [&](int r, int i) { return __builtin_amdgcn_readfirstlane(stage[w][r & 3][i]); };
    auto row_of = [&](int r, int k) { return word(r, 16 * CW + k); };
    auto load_rhs = [&](int r, double (&rr)[CW]) {
#pragma unroll
      for (int k = 0; k < CW; ++k) {
        const uint32_t o = row_of(r, k);
        rr[k] = ld(o != 0xffffffffu ? rs_rhs : rs_none, vb, o);
      }
    };
    // value of a reference word (ref << 2 | kind) at the lane's velocity (mirrored for kind 2)
    auto ref_at = [&](uint32_t x, uint32_t vmir) {
      return ld(x & 3u ? rs_h : rs_none, (x & 3u) == 2 ? vmir : vb, (x >> 2) * row_bytes);
    };
    // out-of-grid axis-2 references: column c, reference st (one and two cells upwind), of the
    // block's first two columns if it holds them
    auto load_edge = [&](int r, double (&ge)[3]) {
#pragma unroll
      for (int e = 0; e < 3; ++e) {
        const int c = e == 2 ? 1 : 0, st = e == 0 ? 0 : 1;
        const bool mine = c >= jb0 && c < jb0 + nb;
        ge[e] = ref_at(mine ? word(r, 16 * (c - jb0) + 14 + st) : 0u, vm2b);
      }
    };
    // out-of-grid axis-1 references take the places of rows r - 1, r - 2: both of row 0 in
    // pr1, pr2, the second one of row 1 in LDS until row 1
    double pr1[CW], pr2[CW];              // rows r - 1, r - 2 of the block
#pragma unroll
    for (int k = 0; k < CW; ++k) {
      const bool have = k < nb;
      const uint32_t* p0 = grec + ((have ? rbase(0) + dj * k : a.grid_none) * 4 + sg1) * 8;
      const uint32_t* p1 = grec + ((have ? rbase(1) + dj * k : a.grid_none) * 4 + sg1) * 8;
      pr1[k] = ref_at(p0[6], vm1b);
      pr2[k] = ref_at(p0[7], vm1b);
      row1[w][k][lane] = ref_at(p1[7], vm1b);
    }
    uint32_t sA[kRegs], sB[kRegs];        // staging words of row r + 3 (A / B alternate)
    double rA[CW], rB[CW], eA[3], eB[3];  // right sides and edge references of even / odd rows
    load_row(0, sA);
    load_row(1, sB);
    put_row(0, sA);
    put_row(1, sB);
    load_row(2, sA);
    put_row(2, sA);
    load_row(3, sB);
    load_rhs(0, rA);
    load_edge(0, eA);
    if (kAhead == 2) {
      load_rhs(1, rB);
      load_edge(1, eB);
    }
    // row r with (rc, ec) of row r, loaded kAhead rows earlier, and the staging words ss of row
    // r + 3 loaded by the previous row; stages them, loads row r + 4's words into sn and, once
    // this row's are consumed, row r + kAhead's right sides and edge references into (rn, en)
    // (the same registers two rows ahead; the other set one row ahead).  Calls alternate the
    // A / B sets.
    auto row = [&](int r, double (&rc)[CW], double (&ec)[3], double (&rn)[CW], double (&en)[3],
                   uint32_t (&ss)[kRegs], uint32_t (&sn)[kRegs]) {
      put_row(r + 3, ss);
      load_row(r + 4, sn);
      if (__builtin_expect(r == 1, 0)) {
#pragma unroll
        for (int k = 0; k < CW; ++k) pr2[k] = row1[w][k][lane];
      }
      double acc0[CW];
#pragma unroll
      for (int k = 0; k < CW; ++k) acc0[k] = rc[k] - av1 * coef(r, k, 2) * pr1[k];
      const double e0 = ec[0], e1 = ec[1], e2 = ec[2];
      load_rhs(r + kAhead, rn);
      load_edge(r + kAhead, en);
      double p1 = 0.0, p2 = 0.0;              // columns c - 1, c - 2 of this row
      if (w > 0) {
        lds_wait_at_least(&published[w - 1], r + 1);
        p1 = carry[r & 1][w - 1][0][lane];
        p2 = carry[r & 1][w - 1][1][lane];
        lds_publish(&consumed[w], r + 1);
      }
      if (__builtin_expect(jb0 == 0, 0)) {
        p1 = e0;
        p2 = e1;
      }
      const double in1 = p1, in2 = p2;
      // column 1's second reference leaves the grid: it replaces the shifted value at k = 1
      // (block from column 0) or k = 0 (block from column 1)
      const double p2k1 = jb0 == 0 ? e2 : in1;
      if (__builtin_expect(jb0 == 1, 0)) p2 = e2;
      double hv[CW];
#pragma unroll
      for (int k = 0; k < CW; ++k) {
        if (k == 1) p2 = p2k1;
        double acc = acc0[k];
        acc -= av2 * coef(r, k, 10) * p1;
        acc -= av1 * coef(r, k, 4) * pr2[k];
        acc -= av2 * coef(r, k, 12) * p2;
        hv[k] = acc / (dnu + av1 * coef(r, k, 0) + av2 * coef(r, k, 8));
        const uint32_t o = row_of(r, k);
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, hv[k]), o != 0xffffffffu ? rs_h : rs_none,
                                              vb, o, 0);
        p2 = p1;
        p1 = hv[k];
        pr2[k] = pr1[k];
        pr1[k] = hv[k];
      }
      if (__builtin_expect(nb < CW, 0)) {     // the carry is the block's last two columns
        p1 = in1;
        p2 = in2;
#pragma unroll
        for (int k = 0; k < CW; ++k)
          if (k < nb) {
            p2 = p1;
            p1 = hv[k];
          }
      }
      if (w < W - 1) {
        lds_wait_at_least(&consumed[w + 1], r - 1);  // its read of row r - 2 (same parity) is done
        carry[r & 1][w][0][lane] = p1;
        carry[r & 1][w][1][lane] = p2;
        lds_publish(&published[w], r + 1);
      }
    };
    if (kAhead == 2) {
      for (int r = 0; r < rows; r += 2) {
        row(r, rA, eA, rA, eA, sB, sA);
        row(r + 1, rB, eB, rB, eB, sA, sB);
      }
    } else {
      for (int r = 0; r < rows; r += 2) {
        row(r, rA, eA, rB, eB, sB, sA);
        row(r + 1, rB, eB, rA, eA, sA, sB);
      }
    }
    __syncthreads();
  }
}

// The same for few cases.  What bounds the form above there is the instructions of a cell (about
// 80, most of the FP64 ones of four cycles) on the few compute units that it reaches: a case has
// few quadruples (1728 at 24^3), and one workgroup of 16 waves carries 64 of them through all the
// cells.  Here a wave takes 16 quadruples by 16 columns: lane 16 g + i carries quadruple i
// through the four columns of group g, one row behind group g - 1, and a workgroup has a quarter
// of the quadruples and of the waves.  One 64 x 64 duct at 24^3 (27 workgroups before, 108
// now): 552 -> 289 us, two of 48 x 47: 370 -> 212.  What is left is latency: one wave a SIMD,
// 280 instructions a step of four cells and six rounds of LDS, 2400 cycles.  The coefficients
// that a wave reads from LDS serve 16 quadruples here and 64 above, so where the workgroups
// above fill the chip that form is the faster one: six ducts 800 against 915 us, two periodic
// 128 x 128 cells (a workgroup a quadrant) 600 against 820.
//
// A workgroup holds W <= 8 waves, side by side along axis 2, of one case and species, and sweeps
// the four quadrants in the same order (one workgroup per quadrant where no reference is a
// mirror ghost: then the quadrants do not read each other).  Within a quadrant the cells are
// taken in the sweep's orientation (row r, column c counted from the upwind corner).  At step s
// group g is at row s - g of its columns.  The two values left of a group come from the group
// before through LDS (`carry`, by step parity): from its own wave's step before, or, for the
// first group, from the last group of wave w - 1, handed on by two counters per wave (rows
// published, steps whose value has been read) instead of a workgroup barrier.  The two rows
// above are the lane's registers; only references that leave the grid are read from h: those
// of rows 0 and 1 (axis 1) when the quadrant starts, those of columns 0 and 1 (axis 2, first
// group of the first wave) with the right sides.  A row's stencil records and row offsets,
// uniform over the quadruples, are loaded by the wave, 16 bytes a lane, six rows ahead, put
// into a ring of eight LDS slots four rows ahead and read from there; the right sides are
// loaded two rows ahead into registers that alternate between two sets (the loop is unrolled
// by two), so that no register copy waits for a load.  Rows of h and of the right sides are
// addressed through buffer descriptors of 2 GiB: a solid or missing cell has an offset beyond
// the end, where loads return 0 and stores are dropped, and gets a finite placeholder update
// (a = 1).  Lanes past the last quadruple repeat it (same values, same stores).  The full
// barrier at the end of a quadrant makes its stores visible to the mirror reads of the next.
constexpr int kLaneWaves = 8;
constexpr int kLaneCols = 4;          // columns of a lane
constexpr int kLaneQuads = 16;        // quadruples of a wave
constexpr int kLaneWaveCols = 16;     // columns of a wave: kLaneCols by 64 / kLaneQuads groups
constexpr int kLaneSlots = 8;
constexpr uint32_t kNoRow = 0x80000000u;   // beyond the descriptors' 2 GiB
// One wave's share of LDS.
struct LaneWave {
  u32x4 rec[kLaneSlots][64];                  // per slot and cell: axis 1 (a, b), (c, references), axis 2 the same
  uint32_t off[kLaneSlots][kLaneWaveCols];     // byte offsets of the cells' rows
  double2 carry[2][64];                      // by step parity: the last two columns of the lane's group
  double row1[kLaneCols][64];                 // second out-of-grid axis-1 reference of row 1
};

// 1 / x for x > 0 well inside the range of normal numbers (the diagonals of the sweeps).
__device__ __forceinline__ double reciprocal(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = __builtin_fma(__builtin_fma(-x, y, 1.0), y, y);
  return __builtin_fma(__builtin_fma(-x, y, 1.0), y, y);
}

__global__ __launch_bounds__(64 * kLaneWaves) void sweep2d_lanes_kernel(
    Sweep2DArgs a, const uint32_t* __restrict__ grec, const uint32_t* __restrict__ growb,
    const double* __restrict__ rhs, double* __restrict__ h) {
  extern __shared__ __align__(16) unsigned char lane_lds[];
  const int W = blockDim.x >> 6, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  LaneWave* waves = reinterpret_cast<LaneWave*>(lane_lds);
  LaneWave& me = waves[w];
  int* published = reinterpret_cast<int*>(waves + W);   // rows whose carry the wave's last group has written
  int* consumed = published + W;                        // steps whose carry of its left neighbour it has read
  const int n = a.n, hn = n / 2, n3 = a.n3, d3 = a.d3;
  const int nsp = a.nsp;
  const int quads = hn * hn * d3, groups = (quads + kLaneQuads - 1) / kLaneQuads;
  // Workgroups are dispatched round-robin over the 8 XCDs (each with its own L2); numbering
  // them so that consecutive velocity groups of a case share an XCD lets the cache lines they
  // share (their 128-byte segments of a row are not line-aligned) be fetched once.
  const int nwg = gridDim.x, lin = blockIdx.x, per = nwg / 8, rem = nwg % 8, xcd = lin % 8, slot = lin / 8;
  const int logical = xcd < rem ? xcd * (per + 1) + slot : rem * (per + 1) + (xcd - rem) * per + slot;
  const int grp = logical % groups, cs = (logical / groups) % a.n_cases;
  const int sp = (logical / (groups * a.n_cases)) % nsp;
  // without mirror ghosts the quadrants do not read each other: one workgroup per quadrant
  const int qsplit = logical / (groups * a.n_cases * nsp);
  const int q0 = a.quad_split ? qsplit : 0, q1 = a.quad_split ? qsplit + 1 : 4;
  if (a.case_active && !a.case_active[cs]) return;   // uniform over the workgroup
  const double* __restrict__ nu = a.nu + static_cast<int64_t>(sp) * n3;
  const uint32_t row_bytes = static_cast<uint32_t>(nsp * n3 * 8);
  // rows of species sp (the launcher checks that h fits), the lane's velocity in the offset
  const __amdgpu_buffer_rsrc_t rs_rhs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(rhs + static_cast<int64_t>(sp) * n3), 0, 0x7fffffff, 0x00020000);
  const __amdgpu_buffer_rsrc_t rs_h =
      __builtin_amdgcn_make_buffer_rsrc(h + static_cast<int64_t>(sp) * n3, 0, 0x7fffffff, 0x00020000);
  const int g = lane / kLaneQuads;
  const int t = min(grp * kLaneQuads + lane % kLaneQuads, quads - 1);
  const int jq1 = t / (hn * d3), jq2 = (t / d3) % hn, j3 = t % d3;
  const int n1 = a.n1[cs], n2 = a.n2[cs];
  const int64_t g0 = a.grid_off[cs];
  const double del = a.delta_case[cs];
  const int jb = kLaneWaveCols * w + kLaneCols * g;     // the lane's first column
  const int steps = (n1 + 64 / kLaneQuads) & ~1;       // an even count, the last group's last row included
  auto ld = [&](const __amdgpu_buffer_rsrc_t& rs, uint32_t o) {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rs, o, 0, 0));
  };
  for (int q = q0; q < q1; ++q) {
    const int s1 = (q & 1) ? -1 : 1, s2 = (q & 2) ? -1 : 1;
    const int j1 = s1 > 0 ? hn + jq1 : hn - 1 - jq1;
    const int j2 = s2 > 0 ? hn + jq2 : hn - 1 - jq2;
    const int v = (j1 * n + j2) * d3 + j3;
    const int vm1 = ((n - 1 - j1) * n + j2) * d3 + j3;
    const int vm2 = (j1 * n + (n - 1 - j2)) * d3 + j3;
    const uint32_t vb = v * 8u, vm1b = vm1 * 8u, vm2b = vm2 * 8u;
    const double av1 = fabs(a.v1d[j1]), av2 = fabs(a.v1d[j2]);
    const double dnu = del * nu[v];
    const int sg1 = s1 > 0 ? 0 : 1, sg2 = s2 > 0 ? 0 : 1;
    if (lane == 0) {
      published[w] = 0;
      consumed[w] = 0;
    }
    __syncthreads();
    // grid index of column c of oriented row r: rbase(r) + s2 c
    auto rbase = [&](int r) { return g0 + static_cast<int64_t>(s1 > 0 ? r : n1 - 1 - r) * n2 + (s2 > 0 ? 0 : n2 - 1); };
    // Staging of row r: lane 4 c + part loads 16 bytes of the records of the wave's column c
    // (axis part / 2 with the sign of its velocity), and lane c (mod 16) the offset of its row.
    // Beyond the grid the last row or column is read again, but for its offset: nothing inside
    // depends on what comes of it there.
    auto grid_col = [&](int c) { return s2 > 0 ? min(c, n2 - 1) : n2 - 1 - min(c, n2 - 1); };
    const uint32_t rec_byte = grid_col(kLaneWaveCols * w + (lane >> 2)) * 128 + ((lane & 2) ? 2 + sg2 : sg1) * 32 + (lane & 1) * 16;
    const int off_col = kLaneWaveCols * w + (lane & 15);
    const uint32_t off_byte = grid_col(off_col) * 4;
    auto load_row = [&](int r, u32x4& rec, uint32_t& off) {
      const int rr = min(r, n1 - 1);
      const int64_t row = g0 + static_cast<int64_t>(s1 > 0 ? rr : n1 - 1 - rr) * n2;
      rec = *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(grec + row * 32) + rec_byte);
      off = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(growb + row) + off_byte);
    };
    auto put_row = [&](int r, const u32x4& rec, uint32_t off) {
      me.rec[r % kLaneSlots][lane] = rec;
      me.off[r % kLaneSlots][lane & 15] = r < n1 && off_col < n2 ? min(off, kNoRow) : kNoRow;
    };
    // byte offsets of the lane's row r, and its right sides
    auto offsets = [&](int r, uint32_t (&o)[kLaneCols]) {
      const u32x4 ov = *reinterpret_cast<const u32x4*>(&me.off[r & (kLaneSlots - 1)][kLaneCols * g]);
#pragma unroll
      for (int k = 0; k < kLaneCols; ++k) o[k] = ov[k] + vb;
    };
    auto load_rhs = [&](int r, double (&rr)[kLaneCols]) {
      uint32_t o[kLaneCols];
      offsets(r, o);
#pragma unroll
      for (int k = 0; k < kLaneCols; ++k) rr[k] = ld(rs_rhs, o[k]);
    };
    // value of a reference word (ref << 2 | kind) at the lane's velocity (mirrored for kind 2)
    auto ref_at = [&](uint32_t x, uint32_t vmir) {
      const uint32_t o = (x >> 2) * row_bytes + ((x & 3u) == 2 ? vmir : vb);
      return ld(rs_h, x & 3u ? o : kNoRow);
    };
    // out-of-grid axis-2 references of the first group's row r: both of column 0, the second of column 1
    auto load_edge = [&](int r, double (&ge)[3]) {
      const u32x4* c = me.rec[r & (kLaneSlots - 1)];
      ge[0] = ref_at(g == 0 ? c[3][2] : 0u, vm2b);
      ge[1] = ref_at(g == 0 ? c[3][3] : 0u, vm2b);
      ge[2] = ref_at(g == 0 ? c[7][3] : 0u, vm2b);
    };
    // out-of-grid axis-1 references take the places of rows r - 1, r - 2: both of row 0 in
    // pr1, pr2, the second one of row 1 in LDS until row 1
    double pr1[kLaneCols], pr2[kLaneCols];      // rows r - 1, r - 2 of the lane's columns
#pragma unroll
    for (int k = 0; k < kLaneCols; ++k) {
      const bool have = jb + k < n2;
      const uint32_t* p0 = grec + ((have ? rbase(0) + s2 * (jb + k) : a.grid_none) * 4 + sg1) * 8;
      const uint32_t* p1 = grec + ((have && n1 > 1 ? rbase(1) + s2 * (jb + k) : a.grid_none) * 4 + sg1) * 8;
      pr1[k] = ref_at(p0[6], vm1b);
      pr2[k] = ref_at(p0[7], vm1b);
      me.row1[k][lane] = ref_at(p1[7], vm1b);
    }
    u32x4 sA, sB;                             // staging words of row s + 4 (A / B alternate)
    uint32_t fA, fB;
    double rA[kLaneCols], rB[kLaneCols], eA[3] = {}, eB[3] = {};
    for (int r = 0; r < 4; r += 2) {
      load_row(r, sA, fA);
      load_row(r + 1, sB, fB);
      put_row(r, sA, fA);
      put_row(r + 1, sB, fB);
    }
    // rows -3 .. -1 of the groups that have not begun: no cells (their slots are filled later)
    for (int r = 5; r < kLaneSlots; ++r) me.off[r][lane & 15] = kNoRow;
    load_rhs(-g, rA);
    // of the row to come: right side less the term of the row above, the other three
    // coefficients, the diagonal and its inverse
    double acc0[kLaneCols], b2[kLaneCols], c1[kLaneCols], c2[kLaneCols], den[kLaneCols], inv[kLaneCols];
    auto prepare = [&](int r, const double (&rc)[kLaneCols], const double (&up)[kLaneCols]) {
      const double2* cf = reinterpret_cast<const double2*>(&me.rec[r & (kLaneSlots - 1)][4 * kLaneCols * g]);
#pragma unroll
      for (int k = 0; k < kLaneCols; ++k) {
        const double2 ab1 = cf[4 * k], ab2 = cf[4 * k + 2];
        den[k] = dnu + av1 * ab1.x + av2 * ab2.x;
        inv[k] = reciprocal(den[k]);
        b2[k] = av2 * ab2.y;
        c1[k] = av1 * cf[4 * k + 1].x;
        c2[k] = av2 * cf[4 * k + 3].x;
        acc0[k] = rc[k] - av1 * ab1.y * up[k];
      }
    };
    prepare(-g, rA, pr1);
    auto sweep = [&](auto first) {
      constexpr bool FIRST = decltype(first)::value;   // the wave of column 0
      const double2* left = g > 0 ? &me.carry[0][lane - kLaneQuads]
                                  : FIRST ? &me.carry[0][lane] : &waves[w - 1].carry[0][lane + 64 - kLaneQuads];
      const int* left_rows = FIRST ? published : published + w - 1;
      const int* right_steps = consumed + min(w + 1, W - 1);
      // in the order of the loop below: its waits count the loads and stores since the one waited
      // for, and allow no more of them than there are on the way into the loop
      load_row(4, sA, fA);
      if (FIRST) load_edge(0, eA);
      __builtin_amdgcn_sched_barrier(0);
      load_rhs(1 - g, rB);
      __builtin_amdgcn_sched_barrier(0);
      load_row(5, sB, fB);
      if (FIRST) load_edge(1, eB);
      __builtin_amdgcn_sched_barrier(0);
      load_rhs(2 - g, rA);
      __builtin_amdgcn_sched_barrier(0);
      // Step s, prepared by the step before; up1 and up2 hold rows r - 1 and r - 2 and are left
      // holding r - 1 and r.  While the chain through the row's cells runs, what does not depend
      // on it: the staging, the next step's coefficients and inverses (its right sides rn) and the
      // loads of the right sides of the step after the one after it.
      auto step = [&](int s, double (&rn)[kLaneCols], double (&ec)[3], u32x4& sr, uint32_t& fr, double (&up1)[kLaneCols],
                      double (&up2)[kLaneCols]) {
        const int r = s - g;
        if (s <= 4) {
#pragma unroll
          for (int k = 0; k < kLaneCols; ++k) {
            double x = me.row1[k][lane];
            asm volatile("" : "+v"(x));   // a value, not one of two addresses
            up2[k] = r == 1 ? x : up2[k];
          }
        }
        // LDS serves a wave's accesses in order: the carry read after a counter that is high enough
        // is the one published before it
        double2 in;
        for (int it = 0; it < kRowSpinMax; ++it) {
          const int rows = __hip_atomic_load(left_rows, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
          __builtin_amdgcn_sched_barrier(0);
          in = left[((s + 1) & 1) * 64];
          if (FIRST || __builtin_amdgcn_readfirstlane(rows) >= min(s + 1, n1)) break;
          __builtin_amdgcn_s_sleep(1);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        if (!FIRST) lds_publish(&consumed[w], s + 1);
        const int taken = __hip_atomic_load(right_steps, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        put_row(s + 4, sr, fr);
        load_row(s + 6, sr, fr);
        uint32_t o[kLaneCols];
        offsets(r, o);
        double p1 = in.x, p2 = in.y;            // columns c - 1, c - 2 of this row
        if (FIRST) {
          p1 = g == 0 ? ec[0] : p1;
          p2 = g == 0 ? ec[1] : p2;
        }
        const double e2 = ec[2];
        double hv[kLaneCols];
#pragma unroll
        for (int k = 0; k < kLaneCols; ++k) {
          if (FIRST && k == 1) p2 = g == 0 ? e2 : p2;
          double acc = acc0[k];
          acc -= b2[k] * p1;
          acc -= c1[k] * up2[k];
          acc -= c2[k] * p2;
          hv[k] = div_known(acc, den[k], inv[k]);
          __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, hv[k]), rs_h, o[k], 0, 0);
          p2 = p1;
          p1 = hv[k];
        }
        if (s < 3) {                            // groups that have not begun keep the references
#pragma unroll
          for (int k = 0; k < kLaneCols; ++k) {
            const double u1 = up1[k], u2 = up2[k];
            up1[k] = r < 0 ? u2 : u1;
            up2[k] = r < 0 ? u1 : hv[k];
          }
        } else {
#pragma unroll
          for (int k = 0; k < kLaneCols; ++k) up2[k] = hv[k];
        }
        if (FIRST) load_edge(s + 2, ec);
        prepare(r + 1, rn, up2);
#pragma unroll
        for (int k = 0; k < kLaneCols; ++k) asm volatile("" : "+v"(acc0[k]), "+v"(inv[k]));   // in this step, rn free
        load_rhs(r + 3, rn);
        if (w < W - 1 && __builtin_amdgcn_readfirstlane(taken) < s - 4)
          lds_wait_at_least(right_steps, s - 4);   // its read of what is overwritten
        me.carry[s & 1][lane] = make_double2(p1, p2);
        if (w < W - 1) lds_publish(&published[w], s - 2);
      };
      for (int s = 0; s < steps; s += 2) {
        step(s, rB, eA, sA, fA, pr1, pr2);
        step(s + 1, rA, eB, sB, fB, pr2, pr1);
      }
    };
    if (w == 0)
      sweep(std::true_type{});
    else
      sweep(std::false_type{});
    __syncthreads();
  }
}

// Few cases: up to six of the lanes kernel's waves a compute unit, fewer for the widths whose
// workgroups then share units unevenly.  Time against the rows kernel over 12, 40 and 100 rows at
// 16^3 and 24^3 (least and greatest): three and more waves a workgroup 0.45-1.00 up to six waves a
// unit (1.2-1.7 beyond for three), but five-wave ones (65 to 80 columns) 0.50-0.69 at five and
// 0.87-1.26 at six; two-wave ones of 17 to 20 columns 0.72-0.95 at two and 0.85-1.10 at three, of 24
// to 32 columns 0.68-0.94 up to three and a half and 1.05-1.11 at four to six; one wave 0.45-1.03.
bool sweep2d_by_lanes(const Sweep2DArgs& a) {
  const int hn = a.n / 2;
  const int64_t quads = static_cast<int64_t>(hn) * hn * a.d3;
  const int W = (a.max_n2 + kLaneWaveCols - 1) / kLaneWaveCols;
  const int half_waves = W == 2 ? (a.max_n2 > 24 ? 7 : 4) : W == 5 ? 10 : 12;   // allowed a unit, twice
  return (quads + kLaneQuads - 1) / kLaneQuads * a.n_cases * a.nsp * (a.quad_split ? 4 : 1) * W * 2 <= half_waves * 256;
}

// Per (cell, species) row: U3, q3 = int (a v^2 - 5/2) v3 h, G1, G12, G2, P13 = 2a int v1 v3 h,
// P23 = 2a int v2 v3 h (a = m_s / m_A; 1 for one gas).
// A workgroup takes R cells of one species, whose values share the per-velocity tables: the
// texture-address units are what a row by itself is bound by (three table loads to one of h).
// 24 576 cells of 6912: 395 -> 296 us (4.6 TB/s), 4096 cells 65 -> 56 (R = 4; the launcher says where).
template <int R>
__global__ __launch_bounds__(256) void moments2d_kernel(int64_t n_cells, int n3, int nsp, double ms0, double ms1,
                                                        const double* __restrict__ vtab,
                                                        const double* __restrict__ h, double w,
                                                        const int32_t* __restrict__ active,
                                                        double* __restrict__ mom) {
  __shared__ double sh[4 * 7 * R];
  const int64_t cell0 = static_cast<int64_t>(blockIdx.x) * R;
  const int sp = blockIdx.y;
  auto live = [&](int u) { return cell0 + u < n_cells && (!active || active[cell0 + u]); };
  bool any = false;
#pragma unroll
  for (int u = 0; u < R; ++u) any = any || live(u);
  if (!any) return;   // uniform over the workgroup
  const double ms = sp == 0 ? ms0 : ms1;
  const double* hr[R];
#pragma unroll
  for (int u = 0; u < R; ++u) hr[u] = h + (min(cell0 + u, n_cells - 1) * nsp + sp) * n3;
  double m[7 * R];
#pragma unroll
  for (int k = 0; k < 7 * R; ++k) m[k] = 0.0;
  auto add = [&](double v1, double v2, double v3, const double (&x)[R]) {
    const double vsq = v1 * v1 + v2 * v2 + v3 * v3, t = w * v3;
    const double f[7] = {t, (ms * vsq - 2.5) * t, (2.0 * v1 * v1 - 1.0) * t, 2.0 * v1 * v2 * t, (2.0 * v2 * v2 - 1.0) * t,
                         2.0 * ms * v1 * t, 2.0 * ms * v2 * t};
#pragma unroll
    for (int u = 0; u < R; ++u)
#pragma unroll
      for (int k = 0; k < 7; ++k) m[7 * u + k] += f[k] * x[u];
  };
  const double *t1 = vtab, *t2 = vtab + n3, *t3 = vtab + 2 * static_cast<int64_t>(n3);
  if ((n3 & 1) == 0 && (reinterpret_cast<uintptr_t>(h) & 15) == 0) {
    for (int p = 2 * threadIdx.x; p < n3; p += 2 * blockDim.x) {
      double x0[R], x1[R];
#pragma unroll
      for (int u = 0; u < R; ++u) {
        const double2 x = *reinterpret_cast<const double2*>(hr[u] + p);
        x0[u] = x.x;
        x1[u] = x.y;
      }
      const double2 v1 = *reinterpret_cast<const double2*>(t1 + p), v2 = *reinterpret_cast<const double2*>(t2 + p),
                    v3 = *reinterpret_cast<const double2*>(t3 + p);
      add(v1.x, v2.x, v3.x, x0);
      add(v1.y, v2.y, v3.y, x1);
    }
  } else {
    for (int v = threadIdx.x; v < n3; v += blockDim.x) {
      double x[R];
#pragma unroll
      for (int u = 0; u < R; ++u) x[u] = hr[u][v];
      add(t1[v], t2[v], t3[v], x);
    }
  }
  block_sum<7 * R>(m, sh);
  if (threadIdx.x < 8 * R) {
    const int u = threadIdx.x >> 3, k = threadIdx.x & 7;
    double x = 0.0;
#pragma unroll
    for (int e = 0; e < 7 * R; ++e) x = e == 7 * u + k && k < 7 ? m[e] : x;
    if (live(u)) mom[((cell0 + u) * nsp + sp) * 8 + k] = x;
  }
}

// ------------------------------------------------------------------ 2-D diffusion
// Finite-volume form of the SIS velocity equation on one case per workgroup,
// Jacobi-preconditioned conjugate gradients in FP64, then flow rates.
constexpr int kD2Threads = 1024;

__device__ inline double par_sign(int bits, int p1, int p2) {
  return ((bits & 1) ? p1 : 1) * ((bits & 2) ? p2 : 1);
}

template <int K>
__device__ inline void block_sum_big(double (&v)[K], double* sh /* >= 16*K */) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int nw = blockDim.x >> 6;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const double s = wave_sum(v[k]);
    if (lane == 0) sh[wave * K + k] = s;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < K; ++k) {
    double s = 0.0;
    for (int w = 0; w < nw; ++w) s += sh[w * K + k];
    v[k] = s;
  }
  __syncthreads();
}

// Workspace of case cs for CG (one gas): per grid cell Uh G1 G12 G2 A1 A2, x r p Ap.
__device__ inline double* d2_work(const Diff2DArgs& a, int cs) { return a.work + a.grid_off[cs] * kDiffWork; }

__device__ void d2_fill_work(const Diff2DArgs& a, int cs, double* W, int ng, bool warm) {
  const int64_t g0 = a.grid_off[cs];
  const double Nd = a.Ns[0] * a.delta_case[cs];
  for (int g = threadIdx.x; g < ng; g += blockDim.x) {
    const int cell = a.gcell[g0 + g];
    double* w = W + static_cast<int64_t>(g) * kDiffWork;
    if (cell >= 0) {
      const double* m = a.mom + static_cast<int64_t>(cell) * 8;
      w[0] = m[0] / a.chi[0]; w[1] = m[2]; w[2] = m[3]; w[3] = m[4];
      if (a.amom) {
        const double* am = a.amom + static_cast<int64_t>(cell) * 4;
        w[4] = am[0] + Nd * am[1];
        w[5] = am[2] + Nd * am[3];
      } else {
        w[4] = 0.0; w[5] = 0.0;
      }
      if (!warm) w[6] = w[0];
    } else {
      for (int k = 0; k < 6; ++k) w[k] = 0.0;
      w[6] = 0.0;
    }
    w[7] = 0.0; w[8] = 0.0; w[9] = 0.0;
  }
}

// The fields 0 .. 5 of that workspace at grid cell g of a case: as filled, or straight from the
// moments (the inverse form needs them once, and its cells are then independent; there 10 and 11 are the
// shear stresses P_B13, P_B23 of a mixture's species B).
struct D2Work {
  const double* W;
  __device__ double operator()(int g, int f) const { return W[static_cast<int64_t>(g) * kDiffWork + f]; }
};
struct D2Moments {
  const Diff2DArgs& a;
  int s;
  int64_t g0;
  double chi, Nd;
  __device__ double operator()(int g, int f) const {
    const int cell = a.gcell[g0 + g];
    if (cell < 0) return 0.0;
    const int64_t row = static_cast<int64_t>(cell) * a.nsp + s;
    if (f == 0) return a.mom[row * 8] / chi;
    if (f < 4) return a.mom[row * 8 + f + 1];
    if (f < 6) return a.amom ? a.amom[row * 4 + 2 * (f - 4)] + Nd * a.amom[row * 4 + 2 * (f - 4) + 1] : 0.0;
    return a.nsp == 2 ? a.mom[(static_cast<int64_t>(cell) * 2 + 1) * 8 + f - 5] : 0.0;
  }
};

// Right side of the finite-volume velocity equation of species s at an unknown grid
// cell G (Dirichlet neighbours moved to the right) and the diagonal of its row:
// chi_s lap U_s = source_s - (d11 G1 + 2 d12 G12 + d22 G2) + d1 A1 + d2 A2, with
// source = -N delta [Poiseuille] for one gas; for mixtures N_A delta (div P_B - [P])
// (species A) and -N_B delta (m_A/m_B) div P_B (species B).
template <class Field>
__device__ double d2_rhs(const Diff2DArgs& a, int s, int64_t g0, int64_t G, const Field& W, bool pois, double del,
                         double& diag) {
  const int g = static_cast<int>(G - g0);
  const int32_t* nbr = a.nb + G * 8;
  const int8_t* bits = a.nbm + G * 8;
  const double* np = a.npos + G * 4;
  const double xc = a.cpos[G * 2], yc = a.cpos[G * 2 + 1];
  auto val = [&](int q, int f, int p1, int p2) {
    const int r = nbr[q];
    return r < 0 ? 0.0 : par_sign(bits[q], p1, p2) * W(r, f);
  };
  const double xE = np[0], xW = np[1], yN = np[2], yS = np[3];
  const double w1 = a.width[G * 2], w2 = a.width[G * 2 + 1];
  auto d11 = [&](int f, int p1, int p2) {
    const double w = W(g, f);
    return ((val(0, f, p1, p2) - w) / (xE - xc) - (w - val(1, f, p1, p2)) / (xc - xW)) / w1;
  };
  auto d22 = [&](int f, int p1, int p2) {
    const double w = W(g, f);
    return ((val(2, f, p1, p2) - w) / (yN - yc) - (w - val(3, f, p1, p2)) / (yc - yS)) / w2;
  };
  const double Nd = a.Ns[s] * del;
  double rhs = 0.0;
  if (a.nsp == 1) {
    rhs = pois ? -Nd : 0.0;
  } else {
    const double coef = s == 1 ? -Nd / a.mass_ratio[1] : Nd;
    if (s == 0 && pois) rhs -= Nd;
    rhs += coef * ((val(0, 10, -1, 1) - val(1, 10, -1, 1)) / (xE - xW) +
                   (val(2, 11, 1, -1) - val(3, 11, 1, -1)) / (yN - yS));
  }
  const double cross = ((val(4, 2, -1, -1) - val(6, 2, -1, -1)) / (yN - yS) -
                        (val(5, 2, -1, -1) - val(7, 2, -1, -1)) / (yN - yS)) / (xE - xW);
  rhs -= d11(1, 1, 1) + 2.0 * cross + d22(3, 1, 1);
  rhs += (val(0, 4, -1, 1) - val(1, 4, -1, 1)) / (xE - xW);
  rhs += (val(2, 5, 1, -1) - val(3, 5, 1, -1)) / (yN - yS);
  double b = -(rhs / a.chi[s]) * a.dA[G];
  diag = 0.0;
  for (int q = 0; q < 4; ++q) {
    const double fw = a.fw[G * 4 + q];
    if (fw == 0.0) continue;
    const int r = nbr[q];
    diag += fw;
    if (a.dflag[g0 + r] != 2) b += fw * W(r, 0);
  }
  return b;
}

// New velocities, corrections, moments of h^{k+1}, flow rates and the convergence
// test of one case (all species).  usol: the solutions at the unknown cells (null:
// the CG iterate in the workspace; CIS: no solve).
template <bool INVERSE>
__device__ void d2_outputs(const Diff2DArgs& a, int cs, int ng, const double* usol, int it, double* sh) {
  const int64_t g0 = a.grid_off[cs];
  const int nsp = a.nsp;
  double fr[4] = {0.0, 0.0, 0.0, 0.0};   // (M, Q) per species
  for (int s = 0; s < nsp; ++s) {
    const double* W = INVERSE ? nullptr : d2_work(a, cs);
    const int64_t voff = nsp * a.uoff[cs] + static_cast<int64_t>(s) * a.n_unknown[cs];
    for (int g = threadIdx.x; g < ng; g += blockDim.x) {
      const int64_t G = g0 + g;
      const int cell = a.gcell[G];
      if (cell < 0) continue;
      const int64_t row = static_cast<int64_t>(cell) * nsp + s;
      const double Uh = INVERSE ? a.mom[row * 8] / a.chi[s] : W[static_cast<int64_t>(g) * kDiffWork];
      double U = Uh;
      if (a.sis && a.dflag[G] == 2) U = INVERSE ? usol[voff + a.uidx[G]] : W[static_cast<int64_t>(g) * kDiffWork + 6];
      const double dU = U - Uh;
      const double Un = Uh + dU * a.cUs[s];
      const double qn = a.mom[row * 8 + 1] + dU * a.cqs[s];
      if (a.U) a.U[row] = U;
      if (a.dU) a.dU[row] = dU;
      if (a.ufield) a.ufield[row] = Un;
      if (a.qfield) a.qfield[row] = qn;
      fr[2 * s] += Un * a.dA[G];
      fr[2 * s + 1] += qn * a.dA[G];
    }
  }
  block_sum_big<4>(fr, sh);
  if (threadIdx.x == 0) {
    // the CG iterate in the workspace is a valid warm start only after a CG solve (the
    // inverse path leaves the workspace's iterate untouched)
    if (a.have_x) a.have_x[cs] = (a.sis && !INVERSE) ? 1 : 0;
    if (a.cg_iters) a.cg_iters[cs] = it;
    if (a.state) {
      double* st = a.state + cs * (2 * nsp + 2);   // M[nsp], Q[nsp], residual, iterations
      double res = 0.0;
      bool bad = false;
      for (int s = 0; s < nsp; ++s) {
        double M = fr[2 * s] / a.area[cs], Q = fr[2 * s + 1] / a.area[cs];
        if (nsp == 2) {
          M *= a.flow_factor;
          Q *= a.flow_factor;
        }
        const double dM = fabs(M - st[s]) / fmax(fabs(M), 1e-300);
        const double dQ = fabs(Q - st[nsp + s]) / fmax(fabs(Q), 1e-300);
        res = fmax(res, fmax(dM, dQ));
        bad = bad || M != M || Q != Q;
        st[s] = M;
        st[nsp + s] = Q;
      }
      st[2 * nsp] = bad ? __builtin_nan("") : res;
      const int k = a.iters[cs] + 1;
      a.iters[cs] = k;
      if (!(res >= a.eps) || bad) a.case_active[cs] = 0;
      st[2 * nsp + 1] = static_cast<double>(k);
    }
  }
}

// Conjugate-gradient form (one gas; cases without a precomputed inverse).
__global__ __launch_bounds__(kD2Threads) void diffusion2d_kernel(Diff2DArgs a) {
  __shared__ double sh[16 * 4];
  const int cs = blockIdx.x;
  if (a.case_active && !a.case_active[cs]) return;
  if (a.direct && a.direct[cs]) return;   // solved by the inverse path
  const int64_t g0 = a.grid_off[cs];
  const int ng = static_cast<int>(a.grid_off[cs + 1] - g0);
  const double del = a.delta_case[cs];
  const bool pois = a.flow_case[cs] == 1;
  double* W = d2_work(a, cs);
  const bool warm = a.have_x && a.have_x[cs];
  d2_fill_work(a, cs, W, ng, warm);
  __syncthreads();
  int it = 0;
  if (a.sis) {
    // right side, initial residual, preconditioned direction
    double red[3] = {0.0, 0.0, 0.0};   // r.z, b.b, r.r
    for (int g = threadIdx.x; g < ng; g += blockDim.x) {
      const int64_t G = g0 + g;
      if (a.dflag[G] != 2) continue;
      double* w = W + static_cast<int64_t>(g) * kDiffWork;
      double diag;
      const double b = d2_rhs(a, 0, g0, G, D2Work{W}, pois, del, diag);
      double Ax = 0.0;
      for (int q = 0; q < 4; ++q) {
        const double fw = a.fw[G * 4 + q];
        if (fw == 0.0) continue;
        const int r = a.nb[G * 8 + q];
        if (a.dflag[g0 + r] == 2) Ax -= fw * W[static_cast<int64_t>(r) * kDiffWork + 6];
      }
      Ax += diag * w[6];
      const double r0 = b - Ax;
      w[7] = r0;
      w[8] = r0 / diag;
      w[9] = b;     // keep b for the norm only during setup
      red[0] += r0 * r0 / diag;
      red[1] += b * b;
      red[2] += r0 * r0;
    }
    block_sum_big<3>(red, sh);
    double rz = red[0];
    const double bnorm = sqrt(red[1]);
    double rnorm = sqrt(red[2]);
    while (rnorm > a.tol * bnorm && it < a.max_iter) {
      // Ap and p.Ap
      double pap[1] = {0.0};
      for (int g = threadIdx.x; g < ng; g += blockDim.x) {
        const int64_t G = g0 + g;
        if (a.dflag[G] != 2) continue;
        double* w = W + static_cast<int64_t>(g) * kDiffWork;
        double diag = 0.0, Ap = 0.0;
        for (int q = 0; q < 4; ++q) {
          const double fw = a.fw[G * 4 + q];
          if (fw == 0.0) continue;
          const int r = a.nb[G * 8 + q];
          diag += fw;
          if (a.dflag[g0 + r] == 2) Ap -= fw * W[static_cast<int64_t>(r) * kDiffWork + 8];
        }
        Ap += diag * w[8];
        w[9] = Ap;
        pap[0] += w[8] * Ap;
      }
      block_sum_big<1>(pap, sh);
      const double alpha = rz / pap[0];
      double nr[2] = {0.0, 0.0};
      for (int g = threadIdx.x; g < ng; g += blockDim.x) {
        const int64_t G = g0 + g;
        if (a.dflag[G] != 2) continue;
        double* w = W + static_cast<int64_t>(g) * kDiffWork;
        double diag = 0.0;
        for (int q = 0; q < 4; ++q) diag += a.fw[G * 4 + q];
        w[6] += alpha * w[8];
        w[7] -= alpha * w[9];
        nr[0] += w[7] * w[7] / diag;
        nr[1] += w[7] * w[7];
      }
      block_sum_big<2>(nr, sh);
      const double beta = nr[0] / rz;
      rz = nr[0];
      rnorm = sqrt(nr[1]);
      for (int g = threadIdx.x; g < ng; g += blockDim.x) {
        const int64_t G = g0 + g;
        if (a.dflag[G] != 2) continue;
        double* w = W + static_cast<int64_t>(g) * kDiffWork;
        double diag = 0.0;
        for (int q = 0; q < 4; ++q) diag += a.fw[G * 4 + q];
        w[8] = w[7] / diag + beta * w[8];
      }
      __syncthreads();
      ++it;
    }
  }
  d2_outputs<false>(a, cs, ng, nullptr, it, sh);
}

// Inverse form, step 1: right sides of the unknown cells of every species (compact per case), by
// cells over the chip (one workgroup a case, its fields staged in the workspace first: 110 us
// for a 64 x 64 duct, 390 for two periodic 128 x 128 cells; now 12 and 36).
__global__ __launch_bounds__(256) void diffusion2d_rhs_kernel(Diff2DArgs a) {
  const int cs = blockIdx.y, s = blockIdx.z;
  if (a.case_active && !a.case_active[cs]) return;
  if (!a.direct[cs] || !a.sis) return;
  const int64_t g0 = a.grid_off[cs];
  const int ng = static_cast<int>(a.grid_off[cs + 1] - g0);
  const double del = a.delta_case[cs];
  const bool pois = a.flow_case[cs] == 1;
  const D2Moments W = {a, s, g0, a.chi[s], a.Ns[s] * del};
  const int64_t voff = a.nsp * a.uoff[cs] + static_cast<int64_t>(s) * a.n_unknown[cs];
  for (int g = blockIdx.x * blockDim.x + threadIdx.x; g < ng; g += gridDim.x * blockDim.x) {
    const int64_t G = g0 + g;
    if (a.dflag[G] != 2) continue;
    double diag;
    a.bvec[voff + a.uidx[G]] = d2_rhs(a, s, g0, G, W, pois, del, diag);
  }
}

// Inverse form, step 2: y = A^-1 b for the right sides of one group (same cross
// section), one wave per row of the shared inverse, which is read once for all of them.
template <int G>
__device__ void d2_gemv_rows(const Diff2DArgs& a, int grp, int row, int lane) {
  const int nu = a.grp_n[grp];
  const double* Ar = a.ainv + a.grp_aoff[grp] + static_cast<int64_t>(row) * nu;
  const double* b[G];
  double s[G];
#pragma unroll
  for (int m = 0; m < G; ++m) {
    b[m] = a.bvec + a.grp_vec[grp * kInverseGroup + m];
    s[m] = 0.0;
  }
  for (int j = lane; j < nu; j += 64) {
    const double v = Ar[j];
#pragma unroll
    for (int m = 0; m < G; ++m) s[m] += v * b[m][j];
  }
#pragma unroll
  for (int m = 0; m < G; ++m) {
    const double t = wave_sum(s[m]);
    if (lane == 0) a.yvec[a.grp_vec[grp * kInverseGroup + m] + row] = t;
  }
}

__global__ __launch_bounds__(256) void diffusion2d_gemv_kernel(Diff2DArgs a) {
  const int grp = blockIdx.y;
  if (!a.sis) return;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= a.grp_n[grp]) return;
  switch (a.grp_size[grp]) {
    case 1: d2_gemv_rows<1>(a, grp, row, lane); break;
    case 2: d2_gemv_rows<2>(a, grp, row, lane); break;
    case 3: d2_gemv_rows<3>(a, grp, row, lane); break;
    case 4: d2_gemv_rows<4>(a, grp, row, lane); break;
    case 5: d2_gemv_rows<5>(a, grp, row, lane); break;
    case 6: d2_gemv_rows<6>(a, grp, row, lane); break;
    case 7: d2_gemv_rows<7>(a, grp, row, lane); break;
    default: d2_gemv_rows<8>(a, grp, row, lane); break;
  }
}

// Inverse form, step 3: outputs, flow rates, convergence.
__global__ __launch_bounds__(kD2Threads) void diffusion2d_out_kernel(Diff2DArgs a) {
  __shared__ double sh[16 * 4];
  const int cs = blockIdx.x;
  if (a.case_active && !a.case_active[cs]) return;
  if (!a.direct[cs]) return;
  const int64_t g0 = a.grid_off[cs];
  const int ng = static_cast<int>(a.grid_off[cs + 1] - g0);
  d2_outputs<true>(a, cs, ng, a.yvec, 0, sh);
}

// Newton-Schulz steps for the inverse of a Jacobi-scaled SPD matrix (plan time).
// Per-block sum of squares of I - P (Frobenius residual, an upper bound of the 2-norm).
__global__ void ns_residual_kernel(const double* __restrict__ P, int n, double* __restrict__ part) {
  __shared__ double sh[4];
  const int64_t count = static_cast<int64_t>(n) * n;
  double m = 0.0;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < count;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int64_t r = i / n, c = i % n;
    const double e = (r == c ? 1.0 : 0.0) - P[i];
    m += e * e;
  }
  m = wave_sum(m);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    double v = 0.0;
    for (int w = 0; w < (blockDim.x >> 6); ++w) v += sh[w];
    part[blockIdx.x] = v;
  }
}

__global__ void ns_two_minus_kernel(double* __restrict__ P, int n) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= static_cast<int64_t>(n) * n) return;
  const int64_t r = i / n, c = i % n;
  P[i] = (r == c ? 2.0 : 0.0) - P[i];
}

// out[r][c] = X[r][c] s[r] s[c] for r, c < n (X has leading dimension ldx, out has n)
__global__ void ns_scale_kernel(const double* __restrict__ X, int ldx, int n, const double* __restrict__ s,
                                double* __restrict__ out) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= static_cast<int64_t>(n) * n) return;
  const int64_t r = i / n, c = i % n;
  out[i] = X[r * ldx + c] * s[r] * s[c];
}

// X = alpha I (n x n); S = I, then S[row][col] = val for the listed entries
__global__ void ns_init_kernel(double* __restrict__ X, int n, double alpha) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= static_cast<int64_t>(n) * n) return;
  X[i] = (i / n == i % n) ? alpha : 0.0;
}

__global__ void ns_scatter_kernel(double* __restrict__ S, int n, const int32_t* __restrict__ rc,
                                  const double* __restrict__ val, int64_t count) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= count) return;
  S[static_cast<int64_t>(rc[2 * i]) * n + rc[2 * i + 1]] = val[i];
}

// ------------------------------------------------------------------ polar velocity grid (tube)
__global__ void polar_fhat_kernel(int nm, const double* __restrict__ xi, int nv, const double* __restrict__ vnode,
                                  const double* __restrict__ wf, double* __restrict__ fhat) {
  const int m = blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= nm) return;
  const double x0 = xi[m], x1 = xi[nm + m], x2 = xi[2 * nm + m];
  double s = 0.0;
  for (int j = 0; j < nv; ++j)
    s += wf[j] * cos(x0 * vnode[j]) * cos(x1 * vnode[nv + j]) * cos(x2 * vnode[2 * nv + j]);
  fhat[m] = 4.0 * s;
}

__global__ void polar_cos_kernel(int nv, int nm, const double* __restrict__ vnode, const double* __restrict__ xi,
                                 double* __restrict__ X) {
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (idx >= static_cast<int64_t>(nv) * nm) return;
  const int i = static_cast<int>(idx / nm), m = static_cast<int>(idx % nm);
  X[idx] = cos(xi[m] * vnode[i] + xi[nm + m] * vnode[nv + i] + xi[2 * nm + m] * vnode[2 * nv + i]);
}

__global__ void polar_scale_terms_kernel(int Tp, int nm, const double* __restrict__ mt,
                                         const double* __restrict__ fhat, const double* __restrict__ sc,
                                         double* __restrict__ out) {
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (idx >= static_cast<int64_t>(Tp) * nm) return;
  const int m = static_cast<int>(idx % nm);
  out[idx] = mt[idx] * fhat[m] * sc[m];
}

__global__ void polar_coef_kernel(int nv, int Tp, const double* __restrict__ AB, const int32_t* __restrict__ srcT,
                                  const double* __restrict__ c, const double* __restrict__ feq, int inu,
                                  double* __restrict__ aT, double* __restrict__ nu) {
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (idx >= static_cast<int64_t>(nv) * Tp) return;
  const int i = static_cast<int>(idx / Tp), t = static_cast<int>(idx % Tp);
  const int sidx = srcT[t];
  aT[idx] = sidx >= 0 ? c[t] * AB[static_cast<int64_t>(i) * Tp + sidx] : (sidx == -1 ? -feq[i] : 0.0);
  if (t == 0) nu[i] = AB[static_cast<int64_t>(i) * Tp + inu];
}

__global__ void polar_xc_kernel(int nv, int nm, const double* __restrict__ vnode, const double* __restrict__ xi,
                                const double* __restrict__ sc, const double* __restrict__ C, double* __restrict__ Xc) {
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (idx >= static_cast<int64_t>(nv) * nm) return;
  const int i = static_cast<int>(idx / nm), m = static_cast<int>(idx % nm);
  const double ph = xi[m] * vnode[i] + xi[nm + m] * vnode[nv + i] + xi[2 * nm + m] * vnode[2 * nv + i];
  const double cm = C[idx] * sc[m];
  double sn, cs;
  sincos(ph, &sn, &cs);
  Xc[2 * idx] = cm * cs;
  Xc[2 * idx + 1] = cm * sn;
}

__global__ void polar_op2_kernel(int nv, int nm, const double* __restrict__ vnode, const double* __restrict__ xi,
                                 const double* __restrict__ wp, double* __restrict__ Op2) {
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (idx >= static_cast<int64_t>(nv) * nm) return;
  const int j = static_cast<int>(idx / nm), m = static_cast<int>(idx % nm);
  double sa, ca, sc_, cc;
  sincos(xi[m] * vnode[j], &sa, &ca);
  const double cb = cos(xi[nm + m] * vnode[nv + j]);
  sincos(xi[2 * nm + m] * vnode[2 * nv + j], &sc_, &cc);
  const double w4 = 4.0 * wp[j] * cb * sc_;
  Op2[2 * idx] = -w4 * sa;
  Op2[2 * idx + 1] = w4 * ca;
}

// ------------------------------------------------------------------ tube
// One workgroup per (case, group of kTubeV (v_r, v_z) pairs).  Inward molecules
// (th > pi/2) are swept from the wall to the centre, then outward ones from the
// centre to the wall; in both passes a node depends on its two r-upwind nodes and
// its two th-upwind (larger th) nodes, so the anti-diagonals of (r, th) are processed
// in order.  What bounds it is the latency of one diagonal, there being little work in
// one: a thread keeps to one th column, so that its r-upwind values stay in registers,
// hands its value to the next columns through LDS (the one barrier of a diagonal), loads
// what it needs kTubeAhead diagonals before, and has all of the next node's equation but that
// value, and its inverted diagonal, by the time the value arrives.  150 nodes, 20 columns:
// 86 us, of which the instructions of a diagonal (70 of four cycles, one wave a SIMD) are
// about half and the waits for LDS and the barrier a third; 394 us with the values passed on
// through global memory and the division after them.
// Two more columns in front hand on the values that the first two depend on: none where the
// columns begin at th = pi, else those of the columns before, read from h (the outward pass
// goes on from the inward one, and more columns than kTubeCols are swept in strips).  The
// coefficients of a node are loaded once for all columns and stay in LDS while they pass it.
constexpr int kTubeV = 8;
constexpr int kTubeCols = 62;
constexpr int kTubeAhead = 24;   // even: LDS holds this diagonal and the one before
constexpr int kTubeNodes = 128;  // >= kTubeCols + 2 + 2 kTubeAhead

struct TubeLds {
  double ring[2][(kTubeCols + 4) * kTubeV];
  alignas(16) double node[kTubeNodes][4];   // of node j at j mod kTubeNodes: three coefficients, r
};

template <bool OUT>
__device__ __forceinline__ void tube_march(const TubeSweepArgs& a, TubeLds& lds, int64_t n0, int n, double del, int q,
                                           bool valid, int kk0) {
  const int nth = a.n_th, half = nth / 2, nvz = a.n_vz, nv = a.nv;
  const int ivr = q / nvz, iz = q % nvz;
  const int t = threadIdx.x, kl = t / kTubeV, cols = min(kTubeCols, half - kk0);
  const bool hand = kl < 2;
  // column kk of the pass is th node k; columns -1 and -2 of the outward pass are inward ones
  const int top = (OUT ? half : nth) - 1;
  const int kk = min(kk0 + kl - 2, half - 1), k = min(top - kk, nth - 1);
  const bool none = top - kk > nth - 1;   // beyond th = pi
  const int count = OUT ? n : n - 1;
  const int diagonals = count + cols + 1;
  const unsigned stored = valid && !hand && kl < cols + 2 ? count : 0;   // nodes of this thread
  const double vr = a.vr[ivr], S = vr * a.sth[k] / (2.0 * a.dth), c1 = vr * a.cth[k];
  auto vix = [&](int kx) { return (ivr * nth + kx) * nvz + iz; };
  const int v = vix(k);
  const double dn = del * a.nu[v];
  // the last column has no th-upwind term, the one before it uses the last twice (4 h - h)
  const bool last = k == nth - 1, second = k == nth - 2;
  const double s4 = last ? 0.0 : (second ? 3.0 : 4.0) * S, s2 = last || second ? 0.0 : S, s3 = last ? 0.0 : 3.0 * S;
  // what the thread loads at its first node, and the bytes to the next: its right side; the
  // values handed on, 0 (h at the wall, inward) beyond th = pi
  double* h = a.h + n0 * nv;
  const int64_t first = OUT ? 0 : n - 2, step = (OUT ? 8 : -8) * static_cast<int64_t>(nv);
  const char* in = reinterpret_cast<const char*>((hand ? h : a.rhs + n0 * nv) + (none ? n - 1 : first) * nv + v);
  const int64_t in_step = none ? 0 : step;
  char* out = reinterpret_cast<char*>(h + first * nv + v);
  auto load = [&](int d) {   // at diagonal d: the first node until it has come, the last one from then on
    const double x = *reinterpret_cast<const double*>(in);
    in += static_cast<unsigned>(d - kl) < static_cast<unsigned>(count - 1) ? in_step : 0;
    return x;
  };
  // coefficients of kTubeAhead nodes from node j on
  constexpr int kPer = 4 * kTubeAhead / (4 * kTubeV);   // of a thread of the smallest workgroup
  const double* coef = (OUT ? a.cout : a.cin) + n0 * 3;
  const double* radius = a.r + n0;
  auto load_coef = [&](int j, double (&c)[kPer]) {
#pragma unroll
    for (int p = 0; p < kPer; ++p) {
      const int e = t + p * static_cast<int>(blockDim.x), jn = min(j + e / 4, count - 1), i = OUT ? jn : n - 2 - jn;
      c[p] = 0.0;
      if (e < 4 * kTubeAhead) c[p] = (e & 3) == 3 ? radius[i] : coef[i * 3 + (e & 3)];
    }
  };
  auto keep_coef = [&](int j, const double (&c)[kPer]) {
#pragma unroll
    for (int p = 0; p < kPer; ++p) {
      const int e = t + p * static_cast<int>(blockDim.x);
      if (e < 4 * kTubeAhead) lds.node[(j + e / 4) % kTubeNodes][e & 3] = c[p];
    }
  };
  double buf[kTubeAhead], next[kPer];
  load_coef(0, next);
#pragma unroll
  for (int u = 0; u < kTubeAhead; ++u) buf[u] = load(u);
  double y1 = 0.0, y2 = 0.0;
  if (OUT) {   // ghosts across the centre hold h(r, pi - th)
    y1 = h[vix(nth - 1 - k)];
    y2 = h[nv + vix(nth - 1 - k)];
  }
  keep_coef(0, next);
  load_coef(kTubeAhead, next);
  keep_coef(kTubeAhead, next);
  __syncthreads();
  // the node's equation times r: D h = base + s4 h1, base = r (rhs - c1 (cb y1 + cc y2)) - s2 h2; the first nodes
  // of the computed columns come at diagonal 2 and later, so what is set up here (and from
  // slots not yet written) for diagonal 0 is not used
  double D = 1.0, inv = 1.0, base = 0.0, handed = buf[0];
  auto slot = [&](int d) { return lds.node[static_cast<unsigned>(d - kl) % kTubeNodes]; };
  double ca, cb, cc, cr;
  auto read_coef = [&](int d) {
    const double* c = slot(d);
    ca = c[0];
    cb = c[1];
    cc = c[2];
    cr = c[3];
  };
  read_coef(1);
  for (int d0 = 0; d0 < diagonals; d0 += kTubeAhead) {
    load_coef(d0 + 2 * kTubeAhead, next);
#pragma unroll
    for (int u = 0; u < kTubeAhead; ++u) {
      const int d = d0 + u, j = d - kl;
      const double* before = lds.ring[(u + 1) % 2] + t;   // diagonal d - 1, two columns of padding in front
      const double near = before[kTubeV], far = before[0];
      __builtin_amdgcn_sched_barrier(0);   // the reads first
      // the next node of this column but for its neighbour's value: the division in the shadow of
      // the reads
      const double next_D = __builtin_fma(cr, __builtin_fma(c1, ca, dn), s3);
      double next_inv = 1.0 / next_D;
      asm volatile("" : "+v"(next_inv));
      double val = div_known(__builtin_fma(s4, near, base), D, inv);
      val = hand ? handed : val;
      lds.ring[u % 2][t + 2 * kTubeV] = val;
      y2 = j >= 0 ? y1 : y2;
      y1 = j >= 0 ? val : y1;
      const double x = buf[(u + 1) % kTubeAhead];
      D = next_D;
      inv = next_inv;
      handed = x;
      base = __builtin_fma(-(cr * c1), cb * y1 + cc * y2, __builtin_fma(-s2, far, cr * x));
      read_coef(d + 2);
      buf[u] = load(d + kTubeAhead);
      if (u == kTubeAhead - 1) keep_coef(d0 + 2 * kTubeAhead, next);
      if (static_cast<unsigned>(j) < stored) {
        *reinterpret_cast<double*>(out) = val;
        out += step;
      }
      __syncthreads();
    }
  }
}

__global__ __launch_bounds__(kTubeV * (kTubeCols + 2)) void sweep_tube_kernel(TubeSweepArgs a) {
  __shared__ TubeLds lds;
  const int cs = blockIdx.y;
  if (a.case_active && !a.case_active[cs]) return;
  const int nth = a.n_th, half = nth / 2, nvz = a.n_vz;
  const int tq = blockIdx.x * kTubeV + threadIdx.x % kTubeV;
  const bool valid = tq < a.n_vr * nvz;
  const int q = valid ? tq : 0;
  const int64_t n0 = a.node_off[cs];
  const int n = static_cast<int>(a.node_off[cs + 1] - n0);
  const double del = a.delta_case[cs];
  // wall node, inward velocities: molecules leaving a diffuse wall carry h = 0
  for (int k = half + threadIdx.x / kTubeV; k < nth; k += blockDim.x / kTubeV)
    if (valid) a.h[(n0 + n - 1) * a.nv + ((q / nvz) * nth + k) * nvz + q % nvz] = 0.0;
  __syncthreads();
  for (int kk0 = 0; kk0 < half; kk0 += kTubeCols) tube_march<false>(a, lds, n0, n, del, q, valid, kk0);
  __syncthreads();
  for (int kk0 = 0; kk0 < half; kk0 += kTubeCols) tube_march<true>(a, lds, n0, n, del, q, valid, kk0);
}

__global__ __launch_bounds__(256) void moments_tube_kernel(int nv, const double* __restrict__ vnode,
                                                           const double* __restrict__ wnode,
                                                           const double* __restrict__ h,
                                                           const int32_t* __restrict__ active,
                                                           double* __restrict__ mom) {
  __shared__ double sh[4 * 5];
  const int64_t c = blockIdx.x;
  if (active && !active[c]) return;
  double m[5] = {0, 0, 0, 0, 0};
  for (int v = threadIdx.x; v < nv; v += blockDim.x) {
    const double v1 = vnode[v], v2 = vnode[nv + v], v3 = vnode[2 * nv + v];
    const double x = wnode[v] * h[c * nv + v];
    m[0] += v3 * x;
    m[1] += (v1 * v1 + v2 * v2 + v3 * v3 - 2.5) * v3 * x;
    m[2] += v3 * (2.0 * v1 * v1 - 1.0) * x;
    m[3] += 2.0 * v3 * (v1 * v1 - v2 * v2) * x;
    m[4] += 2.0 * v1 * v3 * x;
  }
  block_sum<5>(m, sh);
  if (threadIdx.x == 0) {
    for (int k = 0; k < 5; ++k) mom[c * 8 + k] = m[k];
    mom[c * 8 + 5] = 0.0;
    mom[c * 8 + 6] = 0.0;
    mom[c * 8 + 7] = 0.0;
  }
}

// Velocity equation of the tube, one workgroup per case: a march over the radial nodes
// from the wall inwards (staged, carried and finished as in diffusion1d_case), outputs,
// flow rates 2 int_0^1 f r dr and the convergence test.
__global__ __launch_bounds__(kDiffChunk) void diffusion_tube_kernel(TubeDiffArgs a) {
  __shared__ double in[5][kDiffChunk];    // a y_i = s - b y_{i+1} - c y_{i+2}: s, b, c, a, 1/a
  __shared__ double ys[kDiffChunk];       // y
  __shared__ double red[4 * 2];
  const int cs = blockIdx.x;
  if (a.case_active && !a.case_active[cs]) return;   // uniform over the workgroup
  const int64_t n0 = a.node_off[cs];
  const int n = static_cast<int>(a.node_off[cs + 1] - n0);
  const double del = a.delta_case[cs];
  const bool pois = a.flow_case[cs] == 1;
  const double Nd = a.N * del;
  double y1 = 0.0, y2 = 0.0;
  double flow[2] = {0.0, 0.0};            // M, Q
  for (int end = n; end > 0; end -= kDiffChunk) {
    const int lo = max(0, end - kDiffChunk), cnt = end - lo;
    const int i = lo + threadIdx.x;       // one node a thread
    const int64_t node = n0 + i;
    const bool mine = static_cast<int>(threadIdx.x) < cnt;
    double U3 = 0.0, q3 = 0.0, G = 0.0;
    if (mine) {
      const double* m = a.mom + node * 8;
      U3 = m[0];
      q3 = m[1];
      G = m[2];
      if (a.sis) {
        double s = U3 + G, b = 0.0, c = 0.0, ca = 1.0;
        if (i < n - 1) {
          double A = 0.0;
          if (a.amom) A = a.amom[node * 4 + 0] + Nd * a.amom[node * 4 + 1];
          const double r = a.r[node];
          s = A - m[3] / r - (pois ? Nd * r / 2.0 : 0.0);
          ca = a.cin[node * 3 + 0];
          b = a.cin[node * 3 + 1];
          if (i < n - 2) c = a.cin[node * 3 + 2];
        }
        in[0][threadIdx.x] = s;
        in[1][threadIdx.x] = b;
        in[2][threadIdx.x] = c;
        in[3][threadIdx.x] = ca;
        in[4][threadIdx.x] = 1.0 / ca;
      }
    }
    __syncthreads();
    if (threadIdx.x == 0 && a.sis) {
#pragma unroll 8
      for (int t = cnt - 1; t >= 0; --t) {
        const double y = div_known((in[0][t] - in[2][t] * y2) - in[1][t] * y1, in[3][t], in[4][t]);
        y2 = y1;
        y1 = y;
        ys[t] = y;
      }
    }
    __syncthreads();
    if (mine) {
      const double U = a.sis ? ys[threadIdx.x] - G : U3;
      const double dU = U - U3, Un = U3 + dU * a.cU, qn = q3 + dU * a.cq;
      if (a.U) a.U[node] = U;
      if (a.dU) a.dU[node] = dU;
      if (a.ufield) a.ufield[node] = Un;
      if (a.qfield) a.qfield[node] = qn;
      flow[0] += a.tw[node] * Un;
      flow[1] += a.tw[node] * qn;
    }
  }
  if (!a.state) return;
  block_sum<2>(flow, red);
  const double M = flow[0], Q = flow[1];
  if (threadIdx.x == 0) {
    double* st = a.state + cs * 4;
    const double dM = fabs(M - st[0]) / fmax(fabs(M), 1e-300);
    const double dQ = fabs(Q - st[1]) / fmax(fabs(Q), 1e-300);
    const double res = fmax(dM, dQ);
    st[0] = M;
    st[1] = Q;
    st[2] = (M != M || Q != Q) ? __builtin_nan("") : res;
    const int k = a.iters[cs] + 1;
    a.iters[cs] = k;
    if (!(res >= a.eps) || M != M || Q != Q) a.case_active[cs] = 0;
    st[3] = static_cast<double>(k);
  }
}

// ------------------------------------------------------------------ persistent 1-D iteration
// Small planar batches (a few dozen cells, the coarse-grid setting) are bound by launch
// latency: one iteration is six dependent launches of a few microseconds of work each.
// This kernel runs n_iters whole iterations in one cooperative launch: the same phases
// as the launched path (contraction over virtual 32 x 128 tiles and split-K slices,
// finish rows, sweep blocks, moment rows, one velocity-equation march per case, which
// also writes its cells' active flags), each a grid-stride loop over the phase's units,
// separated by grid barriers.  Results equal the launched path's to rounding (the
// split-K slicing of the contraction differs).
//
// Grid barrier: one arrival counter that only grows within a launch (barrier number t
// completes when it reaches t * gridDim.x) and a release word; agent-scope fences on
// both sides make each phase's writes visible to every XCD's caches.  The wait is
// bounded: a wait that runs out sets the abort word, every later barrier returns at
// once, and the host reports the launch as failed (no hang).
constexpr int kBarrierSpin = 1 << 22;

__device__ inline void grid_barrier(unsigned* bar, unsigned& gen) {
  __syncthreads();
  if (threadIdx.x == 0) {
    __threadfence();
    const unsigned target = ++gen;
    if (__hip_atomic_load(&bar[2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0) {
      const unsigned arrived = __hip_atomic_fetch_add(&bar[0], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1;
      if (arrived == target * gridDim.x) {
        __hip_atomic_store(&bar[1], target, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } else {
        int n = 0;
        while (__hip_atomic_load(&bar[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
          if (++n > kBarrierSpin) {
            __hip_atomic_store(&bar[2], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            break;
          }
          if (__hip_atomic_load(&bar[2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) break;
          __builtin_amdgcn_s_sleep(1);
        }
      }
    }
    __threadfence();
  } else {
    ++gen;
  }
  __syncthreads();
}

__global__ __launch_bounds__(256, 2) void sis1d_persistent_kernel(Persist1DArgs a) {
  __shared__ int32_t case_flag;
  unsigned gen = 0;
  const int G = gridDim.x;
  const int n_n = (a.n3 + 127) / 128;
  const int n_m = static_cast<int>((a.n_cells + 31) / 32);
  const int n_tiles = n_n * n_m * a.splits;
  const GemmShape sh{a.n_cells, a.n3, a.n3, a.kps, a.splits, a.n3, a.n3, a.n3, 0, 0, 0, a.n_cells * a.n3};
  const int nbx = (a.sw.n3 / 2 + 255) / 256;
  const int n_sweep = nbx * a.sw.n_cases;
  for (int it = 0; it < a.n_iters; ++it) {
    const bool zero = a.first_from_zero && it == 0;   // h = 0: L+ h = 0, no contraction
    if (!zero) {
      for (int t = blockIdx.x; t < n_tiles; t += G) {
        const int bz = t / (n_n * n_m), r = t - bz * (n_n * n_m);
        gemm_f64_tile<32, 128, 32, 32>(sh, a.h, a.op, a.acc, r % n_n, r / n_n, bz, SymMap{});
        __syncthreads();
      }
      grid_barrier(a.bar, gen);
    }
    for (int64_t c = blockIdx.x; c < a.fin.n_cells; c += G) {
      finish_row(a.fin, c, zero ? 0 : a.splits, zero ? nullptr : a.acc);
      __syncthreads();
    }
    grid_barrier(a.bar, gen);
    for (int t = blockIdx.x; t < n_sweep; t += G) sweep1d_block<256, 8>(a.sw, t % nbx, t / nbx, 0);
    grid_barrier(a.bar, gen);
    for (int64_t c = blockIdx.x; c < a.n_cells; c += G) {
      moments_row(a.sw.n3, 1, 1.0, 1.0, a.vtab, a.sw.h, a.w, a.mom, c);
      __syncthreads();
    }
    grid_barrier(a.bar, gen);
    for (int cs = blockIdx.x; cs < a.dif.n_cases; cs += G) {
      diffusion1d_case(a.dif, cs);
      __syncthreads();
      // the case's flag, as its march left it, for the cell-level flags of the next finish
      if (threadIdx.x == 0) case_flag = __hip_atomic_load(&a.dif.case_active[cs], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __syncthreads();
      const int64_t c0 = a.dif.node_off[cs], c1 = a.dif.node_off[cs + 1];
      for (int64_t c = c0 + threadIdx.x; c < c1; c += blockDim.x) a.cell_active[c] = case_flag;
      __syncthreads();
    }
    grid_barrier(a.bar, gen);
  }
}

__global__ void zero_u32_kernel(unsigned* p, int n) {
  if (static_cast<int>(threadIdx.x) < n) p[threadIdx.x] = 0u;
}

__global__ void expand_active_kernel(const int32_t* __restrict__ case_active,
                                     const int32_t* __restrict__ case_of_cell, int64_t n_cells,
                                     int32_t* __restrict__ cell_active) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n_cells) cell_active[i] = case_active[case_of_cell[i]];
}

}  // namespace

// ------------------------------------------------------------------ launchers
hipError_t launch_assemble(int n, int T, const double* X, const double* Y, const double* feq,
                           double loss_coef, const double* beta_r, double* op, int64_t ldo, int accumulate,
                           hipStream_t s) {
  const int nd = 2 * n - 1;
  const size_t shm = static_cast<size_t>(kAsmPB) * (nd + n) * sizeof(double);
  dim3 grid(n * n, n * n);
  hipLaunchKernelGGL(assemble_kernel, grid, dim3(256), shm, s, n, T, X, Y, feq, loss_coef, beta_r, op, ldo,
                     accumulate);
  return hipGetLastError();
}

hipError_t launch_reduce_operator(const double* op, int64_t ld, double* red, int nsp, int n, int parity,
                                  hipStream_t s) {
  const int d2 = parity == 2 ? n / 2 : n, d3 = n / 2;
  const int64_t ldr = static_cast<int64_t>(nsp) * n * d2 * d3;
  const int64_t count = ldr * ldr;
  hipLaunchKernelGGL(reduce_operator_kernel, dim3(static_cast<unsigned>((count + 255) / 256)), dim3(256), 0, s, op,
                     ld, red, nsp, n, parity);
  return hipGetLastError();
}

int pair_stride(int K) { return (K + 63) / 64 * 64; }

hipError_t launch_split_pairs(const double* X, int64_t rows, int K, int ld, uint16_t* P, hipStream_t s) {
  const int Kp = pair_stride(K);
  const int64_t n = rows * Kp;
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(split_pairs_kernel, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, s, X, rows, K, ld,
                     Kp, P);
  return hipGetLastError();
}

bool make_sym_map(SymMap& m, int nsp, const int (&dim)[3], const bool (&mirror)[3]) {
  m = SymMap{};
  m.nsp = nsp;
  m.nv = dim[0] * dim[1] * dim[2];
  int rep[3], axes = 0;
  bool ok = true;
  for (int a = 0; a < 3; ++a) {
    if (mirror[a] && dim[a] % 2) ok = false;
    rep[a] = mirror[a] ? dim[a] / 2 : dim[a];
    axes += mirror[a];
  }
  // the reflected axes the kernels take: 1; 2 (polar); 1 and 2; all
  if (axes == 0 || (mirror[2] && axes != 3) || (axes == 2 && !mirror[0])) ok = false;
  const int64_t nvb = static_cast<int64_t>(rep[0]) * rep[1] * rep[2], d23 = static_cast<int64_t>(rep[1]) * rep[2];
  if (nvb * d23 >= (int64_t(1) << 32) || nvb > (1 << 28)) ok = false;   // orbit_images divides by multiplication
  if (!ok) return false;
  m.logb = axes;
  m.nvb = static_cast<int>(nvb);
  m.kb = nsp * m.nvb;
  m.ld = (m.kb + 7) / 8 * 8;
  m.d23r = static_cast<int>(d23);
  m.d3r = rep[2];
  m.mul23 = static_cast<uint32_t>(((uint64_t(1) << 32) + m.d23r - 1) / m.d23r);
  m.mul3 = static_cast<uint32_t>(((uint64_t(1) << 32) + m.d3r - 1) / m.d3r);
  m.s1 = dim[1] * dim[2];
  m.s2 = dim[2];
  m.lo1 = mirror[0] ? rep[0] : 0;
  m.lo2 = mirror[1] ? rep[1] : 0;
  m.lo3 = mirror[2] ? rep[2] : 0;
  m.pairs = rep[2] % 2 == 0;
  return true;
}

hipError_t launch_class_operator(const SymMap& m, const double* op, double* out, hipStream_t s) {
  const dim3 grid((m.ld + 255) / 256, m.kb);
  if (m.logb == 1) hipLaunchKernelGGL(class_operator_kernel<1>, grid, dim3(256), 0, s, m, op, out);
  else if (m.logb == 2) hipLaunchKernelGGL(class_operator_kernel<2>, grid, dim3(256), 0, s, m, op, out);
  else if (m.logb == 3) hipLaunchKernelGGL(class_operator_kernel<3>, grid, dim3(256), 0, s, m, op, out);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

namespace {
template <int LOGB, int OUT>
hipError_t class_rows(const SymMap& m, const double* X, const double* Xref, const int32_t* active, int64_t cells,
                      int row_len, void* out, hipStream_t s) {
  const dim3 grid(static_cast<unsigned>(cells), (row_len / 2 + 255) / 256);
  const bool aligned = ((reinterpret_cast<uintptr_t>(X) | reinterpret_cast<uintptr_t>(Xref)) & 15) == 0;
  if (m.pairs && aligned)
    hipLaunchKernelGGL((class_rows_kernel<LOGB, OUT, true>), grid, dim3(256), 0, s, m, X, Xref, active, row_len, out);
  else
    hipLaunchKernelGGL((class_rows_kernel<LOGB, OUT, false>), grid, dim3(256), 0, s, m, X, Xref, active, row_len, out);
  return hipGetLastError();
}
template <int LOGB>
hipError_t class_rows_out(const SymMap& m, int precision, const double* X, const double* Xref, const int32_t* active,
                          int64_t cells, void* out, hipStream_t s) {
  switch (precision) {
    case 0: return class_rows<LOGB, 0>(m, X, Xref, active, cells, m.ld, out, s);
    case 1: return class_rows<LOGB, 1>(m, X, Xref, active, cells, m.ld, out, s);
    case 2: return class_rows<LOGB, 2>(m, X, Xref, active, cells, pair_stride(m.kb), out, s);
    default: return class_rows<LOGB, 3>(m, X, Xref, active, cells, pair_stride(m.kb), out, s);
  }
}
}  // namespace

hipError_t launch_class_rows(const SymMap& m, int precision, const double* X, const double* Xref, const int32_t* active,
                             int64_t cells, void* out, hipStream_t s) {
  if (cells == 0) return hipSuccess;
  switch (m.logb) {
    case 1: return class_rows_out<1>(m, precision, X, Xref, active, cells, out, s);
    case 2: return class_rows_out<2>(m, precision, X, Xref, active, cells, out, s);
    default: return class_rows_out<3>(m, precision, X, Xref, active, cells, out, s);
  }
}

hipError_t launch_convert_f32(const double* op, float* out, int64_t count, hipStream_t s) {
  hipLaunchKernelGGL(convert_f32_kernel, dim3((count + 255) / 256), dim3(256), 0, s, op, out, count);
  return hipGetLastError();
}

int gemm_k_per_split(int K, int splits) {
  const int unit = 64;  // multiple of every BK
  int kps = (K + splits - 1) / splits;
  kps = (kps + unit - 1) / unit * unit;
  return kps;
}

int gemm_tile_rows(int tile) {
  return tile == 5 ? 256 : (tile == 0 || tile == 3) ? 128 : (tile == 2 || tile == 4) ? 64 : 32;
}

int gemm_tile_depth(int tile, int precision) {
  if (tile == 5) return 32;        // 3xBF16, 256 x 256: 32-deep stages in two LDS buffers
  if (precision >= 2) return 64;   // bf16 forms: both operands staged in 64-deep stages
  return tile >= 3 ? 32 : 16;
}

bool gemm_wide_fits(int64_t M, int N, int K, int nb) {
  const int64_t row_bytes = 4 * static_cast<int64_t>(pair_stride(K));
  return M * nb * row_bytes < (int64_t(1) << 32) && N * row_bytes < (int64_t(1) << 32);
}

hipError_t launch_gemm(const GemmArgs& g, hipStream_t s) {
  const int BN = 128;
  const int BM = gemm_tile_rows(g.tile);
  const int nb = g.sym ? 1 << g.sym->logb : 1;
  const SymMap sym = g.sym ? *g.sym : SymMap{};
  // the few-cell tile of FP64 and the bf16 forms reads the cells' own rows
  const bool own_rows = g.sym && g.cells_own_rows;
  if (own_rows && (g.tile != 1 || g.precision == 1)) return hipErrorInvalidValue;
  if (g.tile >= 3 && g.precision == 1) return hipErrorInvalidValue;
  if (g.tile == 5 && g.precision != 2) return hipErrorInvalidValue;
  if ((g.tile == 3 || g.tile == 4) && g.precision != 0) return hipErrorInvalidValue;
  GemmShape sh{};
  sh.M = g.M;
  sh.splits = g.splits > 0 ? g.splits : 1;
  if (g.sym) {
    sh.N = sym.kb;
    sh.ldc = nb * sym.ld;
    sh.cs = sym.ld;
  } else {
    sh.N = g.N;
    sh.ldc = g.N;
  }
  sh.cz = sh.M * sh.ldc;
  const dim3 grid((sh.N + BN - 1) / BN, static_cast<unsigned>((g.M + BM - 1) / BM), sh.splits * nb);
  if (g.precision <= 1) {
    // block rows are padded with zeros to ld (a multiple of 8)
    sh.K = !g.sym ? g.K : g.precision == 1 ? sym.ld : (sym.kb + 1) / 2 * 2;
    sh.kps = gemm_k_per_split(g.sym ? sym.kb : g.K, sh.splits);
    sh.ldo = g.sym ? sym.ld : g.K;
    sh.ldx = own_rows ? sym.nsp * sym.nv : g.sym ? nb * sym.ld : g.K;
    sh.xs = g.sym ? sym.ld : 0;
    sh.os = g.sym ? static_cast<int64_t>(sym.kb) * sym.ld : 0;
  } else {
    const int Kp = pair_stride(g.sym ? sym.kb : g.K);
    sh.K = Kp;
    sh.kps = gemm_k_per_split(Kp, sh.splits);
    sh.ldo = 2 * Kp;
    sh.ldx = 2 * Kp * nb;
    sh.xs = 2 * Kp;
    sh.os = static_cast<int64_t>(sh.N) * 2 * Kp;
  }
#define SIS_GEMM(kernel, threads, ...) hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, s, __VA_ARGS__, sh)
  double* acc64 = static_cast<double*>(g.acc);
  float* acc32 = static_cast<float*>(g.acc);
  if (g.precision == 0) {
    if (sh.K % 2 || sh.ldx % 2 || sh.ldo % 2) return hipErrorInvalidValue;   // rows are loaded in 16-byte k pairs
#define SIS_F64(...) hipLaunchKernelGGL((gemm_f64_kernel<__VA_ARGS__>), grid, dim3(256), 0, s, g.X, g.op64, acc64, sh, sym)
    if (g.tile == 0 && sh.ldx <= (1 << 20) && sh.ldo <= (1 << 20)) SIS_GEMM(gemm_f64_dma_kernel, 512, g.X, g.op64, acc64);
    else if (g.tile == 0) SIS_F64(128, 128, 64, 64);
    else if (g.tile == 2) SIS_F64(64, 128, 32, 64);
    else if (g.tile == 3) SIS_F64(128, 128, 64, 64, 32, 1, 1);
    else if (g.tile == 4) SIS_F64(64, 128, 32, 64, 32, 1, 1);
    else if (!own_rows) SIS_F64(32, 128, 32, 32);
    else if (sym.logb == 1) SIS_F64(32, 128, 32, 32, kBK, 2, kPad, 1);
    else if (sym.logb == 2) SIS_F64(32, 128, 32, 32, kBK, 2, kPad, 2);
    else SIS_F64(32, 128, 32, 32, kBK, 2, kPad, 3);
#undef SIS_F64
  } else if (g.precision == 1) {
    if (!g.X32 || !g.op32) return hipErrorInvalidValue;
    if (sh.ldx % 4 || sh.ldo % 4 || sh.K % 4 || sh.ldx > (1 << 21) || sh.ldo > (1 << 21)) return hipErrorInvalidValue;
    if (g.tile == 0) SIS_GEMM(gemm_f32_dma_kernel, 512, g.X32, g.op32, acc32);
    else if (g.tile == 2) SIS_GEMM((gemm_f32_kernel<64, 128, 32, 64>), 256, g.X32, g.op32, acc32);
    else SIS_GEMM((gemm_f32_kernel<32, 128, 32, 32>), 256, g.X32, g.op32, acc32);
  } else {
    // bf16 forms: operands in the pair layout, k running over the padded Kp (zeros past K)
    if (!g.opp || (own_rows ? !g.X : !g.Xp)) return hipErrorInvalidValue;
#define SIS_BF(...) \
  hipLaunchKernelGGL((gemm_bf16x3_kernel<__VA_ARGS__>), grid, dim3(256), 0, s, g.Xp, g.opp, acc32, sh, g.X, g.Xref, sym)
    if (g.tile == 5) {
      if (!gemm_wide_fits(g.M, sh.N, g.sym ? sym.kb : g.K, nb)) return hipErrorInvalidValue;
      const dim3 wgrid((sh.N + 255) / 256, static_cast<unsigned>((g.M + 255) / 256), sh.splits * nb);
      hipLaunchKernelGGL(gemm_bf16x3_wide_kernel, wgrid, dim3(512), 0, s, g.Xp, g.opp, acc32, sh);
    } else if (g.precision == 3) {
      if (own_rows) {
        if (sym.logb == 1) SIS_BF(32, 128, 32, 32, 1, 1);
        else if (sym.logb == 2) SIS_BF(32, 128, 32, 32, 1, 2);
        else SIS_BF(32, 128, 32, 32, 1, 3);
      } else if (g.tile == 0) SIS_BF(128, 128, 64, 64, 1);
      else if (g.tile == 2) SIS_BF(64, 128, 32, 64, 1);
      else SIS_BF(32, 128, 32, 32, 1);
    } else if (own_rows) {
      if (sym.logb == 1) SIS_BF(32, 128, 32, 32, 3, 1);
      else if (sym.logb == 2) SIS_BF(32, 128, 32, 32, 3, 2);
      else SIS_BF(32, 128, 32, 32, 3, 3);
    } else if (g.tile == 0) SIS_BF(128, 128, 64, 64);
    else if (g.tile == 2) SIS_BF(64, 128, 32, 64);
    else SIS_BF(32, 128, 32, 32);
#undef SIS_BF
  }
#undef SIS_GEMM
  return hipGetLastError();
}

hipError_t launch_finish(const FinishArgs& a, hipStream_t s) {
  const dim3 grid(static_cast<unsigned>(a.n_cells));
  const int logb = a.sym.logb;
  const bool few = a.n_cells <= 256;
  // Few rows leave most compute units without one, and a row's orbits are then a chain of loads: 1024
  // threads a row (512 of the 161-register form; 104 rows of 13 824: 43 -> 33 us).  With more rows than
  // units 256 stream as well.  Four classes gain 1 to 11% at every length.  Two classes, by orbits or pairs
  // of them a row: 864 pairs 0 to 4%, 1331 orbits 3 to 7%, 729 orbits 1% without the projection and -8% with
  // it, 500 pairs -2 to -7%.  Eight, against the form with more splits in flight: 1331 orbits 1 to 2%,
  // 1000 -2%.
  const int items = a.sym.pairs ? a.sym.nvb / 2 : a.sym.nvb;
  const bool wide = few && (logb == 1 ? items > (a.project ? 768 : 512) : logb == 2 || a.sym.nvb > 1024);
  // Short rows, few of them, have as many splits as it takes to fill the chip, and the rounds of loads
  // are what they wait for (17 rows of 1024, eight splits: 7.5 -> 6.1 us) -- where more at once are
  // fewer rounds: four splits of two classes are one round of four and would be four of one (0.7 us).
  auto rounds = [&](bool deep) { return a.splits / finish_splits(logb, deep) + a.splits % finish_splits(logb, deep); };
  const bool deep = few && logb && rounds(true) < rounds(false);
#define SIS_FINISH_(LOGB, A)                                                                             \
  if (wide) hipLaunchKernelGGL((finish_class_kernel<LOGB, A, LOGB == 2 ? 512 : 1024, false>), grid,      \
                               dim3(LOGB == 2 ? 512 : 1024), 0, s, a);                                   \
  else if (LOGB != 2 && deep)                                                                            \
    hipLaunchKernelGGL((finish_class_kernel<LOGB, A, 256, LOGB != 2>), grid, dim3(256), 0, s, a);        \
  else hipLaunchKernelGGL((finish_class_kernel<LOGB, A, 256, false>), grid, dim3(256), 0, s, a)
#define SIS_FINISH(LOGB) if (a.acc_f32) { SIS_FINISH_(LOGB, float); } else { SIS_FINISH_(LOGB, double); }
  switch (a.sym.logb) {
    case 0: hipLaunchKernelGGL(finish_kernel, grid, dim3(256), 0, s, a); break;
    case 1: SIS_FINISH(1); break;
    case 2: SIS_FINISH(2); break;
    default: SIS_FINISH(3); break;
  }
#undef SIS_FINISH
#undef SIS_FINISH_
  return hipGetLastError();
}

hipError_t launch_sweep1d(const SweepArgs& a, hipStream_t s) {
  const int half = a.n3 / 2;
  // A wave a workgroup, but where there are more than two waves a SIMD: then bandwidth counts, and rows
  // whose halves are not whole 128-byte lines leave lines shared by workgroups (of other XCDs) between
  // every 64 velocities.  256 cases of 401 nodes, two species of 432 velocities: 453 -> 329 us with four
  // waves, 404 with the form before this one; whole lines 2-10% slower with four, and halves that fill
  // less than four fifths of them up to 47%.
  const int waves = (half + kSweepNT - 1) / kSweepNT, fours = (half + 255) / 256;
  const bool full = static_cast<int64_t>(waves) * a.n_cases * a.nsp >= 2 * 1024;
  if (full && half % 16 != 0 && half * 5 >= fours * 256 * 4)
    hipLaunchKernelGGL(sweep1d_kernel<256>, dim3(fours, a.n_cases, a.nsp), dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL(sweep1d_kernel<kSweepNT>, dim3(waves, a.n_cases, a.nsp), dim3(kSweepNT), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_moments(int n3, int nsp, const double* mass_ratio, int64_t n_rows, const double* vtab,
                          const double* h, double w, double* mom, hipStream_t s) {
  const double m0 = mass_ratio ? mass_ratio[0] : 1.0, m1 = mass_ratio && nsp > 1 ? mass_ratio[1] : 1.0;
  hipLaunchKernelGGL(moments_kernel, dim3(static_cast<unsigned>(n_rows)), dim3(256), 0, s, n3, nsp, m0, m1, vtab, h,
                     w, mom);
  return hipGetLastError();
}

hipError_t launch_diffusion1d(const DiffusionArgs& a, hipStream_t s) {
  if (a.nsp == 2)
    hipLaunchKernelGGL(diffusion1d_mix_kernel, dim3(a.n_cases), dim3(kDiffChunk), 0, s, a);
  else
    hipLaunchKernelGGL(diffusion1d_kernel, dim3(a.n_cases), dim3(kDiffChunk), 0, s, a);
  return hipGetLastError();
}


int sweep2d_form(int max_diag, int max_n2, int64_t row_bytes_total) {
  if (max_n2 <= kRowWaves * 8 && row_bytes_total < (int64_t(1) << 31)) return 1;
  const int slots = kSweepThreads / kSweepV;
  return (max_diag + slots - 1) / slots <= kSweepMaxP ? 2 : 3;
}

hipError_t launch_sweep2d(const Sweep2DArgs& a, hipStream_t s) {
  const int hn = a.n / 2;
  const int count = hn * hn * a.d3;
  const int form = sweep2d_form(a.max_diag, a.max_n2, a.row_bytes_total);
  if (form == 1) {
    if (sweep2d_by_lanes(a)) {
      const int W = (a.max_n2 + kLaneWaveCols - 1) / kLaneWaveCols;
      const size_t lds = W * (sizeof(LaneWave) + 2 * sizeof(int));
      if (lds > 65536) {   // has to be asked for
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(sweep2d_lanes_kernel),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
        if (e != hipSuccess) return e;
      }
      dim3 grid(((count + kLaneQuads - 1) / kLaneQuads) * a.n_cases * a.nsp * (a.quad_split ? 4 : 1));
      hipLaunchKernelGGL(sweep2d_lanes_kernel, grid, dim3(64 * W), lds, s, a, a.grec, a.growb, a.rhs, a.h);
      return hipGetLastError();
    }
    const int cwmax = a.max_n2 <= kRowWaves * 4 ? 4 : 8;
    const int W = (a.max_n2 + cwmax - 1) / cwmax;
    dim3 grid(((count + 63) / 64) * a.n_cases * a.nsp * (a.quad_split ? 4 : 1));
    if (cwmax == 4)
      hipLaunchKernelGGL(sweep2d_rows_kernel<4>, grid, dim3(64 * W), 0, s, a, a.grec, a.growb, a.rhs, a.h);
    else
      hipLaunchKernelGGL(sweep2d_rows_kernel<8>, grid, dim3(64 * W), 0, s, a, a.grec, a.growb, a.rhs, a.h);
    return hipGetLastError();
  }
  dim3 grid((count + kSweepV - 1) / kSweepV, a.n_cases, a.nsp);
  const int slots = kSweepThreads / kSweepV;
  const int P = (a.max_diag + slots - 1) / slots;
  if (form == 3)
    hipLaunchKernelGGL(sweep2d_kernel, grid, dim3(kSweepThreads), 0, s, a);
  else if (P <= 1)
    hipLaunchKernelGGL(sweep2d_pipelined_kernel<1>, grid, dim3(kSweepThreads), 0, s, a);
  else if (P == 2)
    hipLaunchKernelGGL(sweep2d_pipelined_kernel<2>, grid, dim3(kSweepThreads), 0, s, a);
  else
    hipLaunchKernelGGL(sweep2d_pipelined_kernel<3>, grid, dim3(kSweepThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_moments2d(int n3, int nsp, const double* mass_ratio, int64_t n_cells, const double* vtab,
                            const double* h, double w, const int32_t* cell_active, double* mom, hipStream_t s) {
  const double m0 = mass_ratio[0], m1 = nsp > 1 ? mass_ratio[1] : 1.0;
  // Four cells a workgroup where the rows come from HBM and are long: rows that the sweep left in the
  // 256 MB cache come so fast that the 28 sums across lanes at the end of a workgroup decide, at few
  // workgroups a unit.  Four against one: 3000 cells of 2048 29 against 21 us, 24 576 129 against 110; of 4096
  // 5929 cells 51 against 43, 8190 66 against 68, 24 576 154 against 199; of 6912 2970 cells 41 against 35, 4096
  // 48 against 57; 2025 cells of 13 824 49 against 59.
  const double values = static_cast<double>(n_cells) * nsp * n3;
  if (n3 >= 5120 ? values >= 25e6 : n3 >= 4000 && values >= 33e6)
    hipLaunchKernelGGL(moments2d_kernel<4>, dim3(static_cast<unsigned>((n_cells + 3) / 4), nsp), dim3(256), 0, s, n_cells,
                       n3, nsp, m0, m1, vtab, h, w, cell_active, mom);
  else
    hipLaunchKernelGGL(moments2d_kernel<1>, dim3(static_cast<unsigned>(n_cells), nsp), dim3(256), 0, s, n_cells, n3, nsp,
                       m0, m1, vtab, h, w, cell_active, mom);
  return hipGetLastError();
}

hipError_t launch_diffusion2d(const Diff2DArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(diffusion2d_kernel, dim3(a.n_cases), dim3(kD2Threads), 0, s, a);
  if (a.direct) {
    const unsigned blocks = std::max(1, (a.max_unknown + 255) / 256);
    hipLaunchKernelGGL(diffusion2d_rhs_kernel, dim3(blocks, a.n_cases, a.nsp), dim3(256), 0, s, a);
    if (a.max_unknown > 0 && a.n_groups > 0)
      hipLaunchKernelGGL(diffusion2d_gemv_kernel, dim3((a.max_unknown + 3) / 4, a.n_groups), dim3(256), 0, s, a);
    hipLaunchKernelGGL(diffusion2d_out_kernel, dim3(a.n_cases), dim3(kD2Threads), 0, s, a);
  }
  return hipGetLastError();
}

hipError_t launch_ns_residual(const double* P, int n, double* part, int blocks, hipStream_t s) {
  hipLaunchKernelGGL(ns_residual_kernel, dim3(blocks), dim3(256), 0, s, P, n, part);
  return hipGetLastError();
}

hipError_t launch_ns_two_minus(double* P, int n, hipStream_t s) {
  const int64_t count = static_cast<int64_t>(n) * n;
  hipLaunchKernelGGL(ns_two_minus_kernel, dim3(static_cast<unsigned>((count + 255) / 256)), dim3(256), 0, s, P, n);
  return hipGetLastError();
}

hipError_t launch_ns_scale(const double* X, int ldx, int n, const double* sc, double* out, hipStream_t s) {
  const int64_t count = static_cast<int64_t>(n) * n;
  if (count == 0) return hipSuccess;
  hipLaunchKernelGGL(ns_scale_kernel, dim3(static_cast<unsigned>((count + 255) / 256)), dim3(256), 0, s, X, ldx, n,
                     sc, out);
  return hipGetLastError();
}

hipError_t launch_ns_scatter(double* S, int n, const int32_t* rc, const double* val, int64_t count, hipStream_t s) {
  if (count == 0) return hipSuccess;
  hipLaunchKernelGGL(ns_scatter_kernel, dim3(static_cast<unsigned>((count + 255) / 256)), dim3(256), 0, s, S, n, rc,
                     val, count);
  return hipGetLastError();
}

hipError_t launch_ns_init(double* X, int n, double alpha, hipStream_t s) {
  const int64_t count = static_cast<int64_t>(n) * n;
  hipLaunchKernelGGL(ns_init_kernel, dim3(static_cast<unsigned>((count + 255) / 256)), dim3(256), 0, s, X, n, alpha);
  return hipGetLastError();
}

int persist1d_max_blocks() {
  int dev = 0, cus = 0, per = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, sis1d_persistent_kernel, 256, 0) != hipSuccess) return 0;
  return cus * per;
}

hipError_t launch_persist1d(const Persist1DArgs& a, int blocks, hipStream_t s) {
  if (blocks < 1 || blocks > persist1d_max_blocks()) return hipErrorInvalidConfiguration;
  if (a.sw.nsp != 1 || a.fin.nsp != 1 || a.n3 != a.sw.n3) return hipErrorInvalidValue;
  // the barrier words start at zero in every launch (a fill kernel, not a memset node, in
  // case the caller captures the stream)
  hipLaunchKernelGGL(zero_u32_kernel, dim3(1), dim3(64), 0, s, a.bar, 4);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  Persist1DArgs arg = a;
  void* params[] = {&arg};
  return hipLaunchCooperativeKernel(reinterpret_cast<const void*>(sis1d_persistent_kernel), dim3(blocks), dim3(256),
                                    params, 0, s);
}

hipError_t launch_expand_active(const int32_t* case_active, const int32_t* case_of_cell,
                                int64_t n_cells, int32_t* cell_active, hipStream_t s) {
  hipLaunchKernelGGL(expand_active_kernel, dim3(static_cast<unsigned>((n_cells + 255) / 256)), dim3(256), 0, s,
                     case_active, case_of_cell, n_cells, cell_active);
  return hipGetLastError();
}

hipError_t launch_polar_fhat(int nm, const double* xi, int nv, const double* vnode, const double* wf, double* fhat,
                             hipStream_t s) {
  hipLaunchKernelGGL(polar_fhat_kernel, dim3((nm + 255) / 256), dim3(256), 0, s, nm, xi, nv, vnode, wf, fhat);
  return hipGetLastError();
}

static dim3 grid_for(int64_t count) { return dim3(static_cast<unsigned>((count + 255) / 256)); }

hipError_t launch_polar_cos(int nv, int nm, const double* vnode, const double* xi, double* X, hipStream_t s) {
  hipLaunchKernelGGL(polar_cos_kernel, grid_for(static_cast<int64_t>(nv) * nm), dim3(256), 0, s, nv, nm, vnode, xi, X);
  return hipGetLastError();
}

hipError_t launch_polar_scale_terms(int Tp, int nm, const double* mt, const double* fhat, const double* sc,
                                    double* out, hipStream_t s) {
  hipLaunchKernelGGL(polar_scale_terms_kernel, grid_for(static_cast<int64_t>(Tp) * nm), dim3(256), 0, s, Tp, nm, mt,
                     fhat, sc, out);
  return hipGetLastError();
}

hipError_t launch_polar_coef(int nv, int Tp, const double* AB, const int32_t* src, const double* c,
                             const double* feq, int inu, double* aT, double* nu, hipStream_t s) {
  hipLaunchKernelGGL(polar_coef_kernel, grid_for(static_cast<int64_t>(nv) * Tp), dim3(256), 0, s, nv, Tp, AB, src, c,
                     feq, inu, aT, nu);
  return hipGetLastError();
}

hipError_t launch_polar_xc(int nv, int nm, const double* vnode, const double* xi, const double* sc,
                           const double* C, double* Xc, hipStream_t s) {
  hipLaunchKernelGGL(polar_xc_kernel, grid_for(static_cast<int64_t>(nv) * nm), dim3(256), 0, s, nv, nm, vnode, xi,
                     sc, C, Xc);
  return hipGetLastError();
}

hipError_t launch_polar_op2(int nv, int nm, const double* vnode, const double* xi, const double* wp, double* Op2,
                            hipStream_t s) {
  hipLaunchKernelGGL(polar_op2_kernel, grid_for(static_cast<int64_t>(nv) * nm), dim3(256), 0, s, nv, nm, vnode, xi,
                     wp, Op2);
  return hipGetLastError();
}

hipError_t launch_sweep_tube(const TubeSweepArgs& a, hipStream_t s) {
  if (a.max_nodes < 3) return hipErrorInvalidValue;
  const int pairs = a.n_vr * a.n_vz;
  dim3 grid((pairs + kTubeV - 1) / kTubeV, a.n_cases);
  const int cols = std::min(a.n_th / 2, kTubeCols);
  hipLaunchKernelGGL(sweep_tube_kernel, grid, dim3(kTubeV * (cols + 2)), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_moments_tube(int64_t n_nodes, int nv, const double* vnode, const double* wnode, const double* h,
                               const int32_t* active, double* mom, hipStream_t s) {
  if (n_nodes == 0) return hipSuccess;
  hipLaunchKernelGGL(moments_tube_kernel, dim3(static_cast<unsigned>(n_nodes)), dim3(256), 0, s, nv, vnode, wnode,
                     h, active, mom);
  return hipGetLastError();
}

hipError_t launch_diffusion_tube(const TubeDiffArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(diffusion_tube_kernel, dim3(a.n_cases), dim3(kDiffChunk), 0, s, a);
  return hipGetLastError();
}

}  // namespace sis
