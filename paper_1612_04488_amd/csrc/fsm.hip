// The fast spectral method (the collision evaluation the paper cites for eq.
// LBE_collision) on the device: per cell, the forward transform of every parity class
// of the distribution, then for every one of the 2D + 1 terms its multiplier,
// the inverse transform back to the velocities and the product with the
// term's f_eq field, summed over the terms; and the plan's tables.  Every transform is
// separable: each axis is a small dense GEMM against a factor matrix, run on the FP64 MFMA
// (v_mfma_f64_16x16x4) with the operands staged in LDS.  Declarations in fsm.h.
#include "fsm.h"

#include <algorithm>

namespace sis {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));
constexpr int kThreads = 256;   // four wave64s

__device__ inline v4d mfma(double a, double b, v4d c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// C(m, n) = sum_{k < K} A(m, k) B(k, n) for the 16 x 16 NT block at (m0, n0),
// complex planar: la(m, k, re, im), lb(k, n, re, im) fetch the operands (zero
// outside the matrices).  Lane l holds, for tile j and element r, the entry
// (m0 + l/16 + 4r, n0 + 16 j + l%16) (the 16x16x4 FP64 layout: A from lane
// (row l%16, k l/16), B from lane (k l/16, column l%16)).
template <int NT, class LA, class LB>
__device__ inline void cgemm_block(int K, int m0, int n0, LA la, LB lb, v4d (&cr)[NT], v4d (&ci)[NT]) {
  const int lane = threadIdx.x & 63, kr = lane >> 4, cc = lane & 15;
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    cr[j] = v4d{0.0, 0.0, 0.0, 0.0};
    ci[j] = v4d{0.0, 0.0, 0.0, 0.0};
  }
  for (int k0 = 0; k0 < K; k0 += 4) {
    double ar, ai;
    la(m0 + cc, k0 + kr, ar, ai);
    const double nai = -ai;
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      double br, bi;
      lb(k0 + kr, n0 + 16 * j + cc, br, bi);
      cr[j] = mfma(ar, br, cr[j]);
      ci[j] = mfma(ar, bi, ci[j]);
      cr[j] = mfma(nai, bi, cr[j]);
      ci[j] = mfma(ai, br, ci[j]);
    }
  }
}

// Every (16 x 16 NT) block of an M x N complex product, blocks dealt round-robin
// to the four waves; st(m, n, re, im) stores the entries inside the matrix.
template <int NT, class LA, class LB, class ST>
__device__ inline void cgemm(int M, int N, int K, LA la, LB lb, ST st) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, kr = lane >> 4, cc = lane & 15;
  const int mb = (M + 15) / 16, nbk = (N + 16 * NT - 1) / (16 * NT);
  for (int blk = wave; blk < mb * nbk; blk += 4) {
    const int m0 = (blk / nbk) * 16, n0 = (blk % nbk) * 16 * NT;
    v4d cr[NT], ci[NT];
    cgemm_block<NT>(K, m0, n0, la, lb, cr, ci);
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + kr + 4 * r, n = n0 + 16 * j + cc;
        if (m < M && n < N) st(m, n, cr[j][r], ci[j][r]);
      }
  }
}

// ---------------------------------------------------------------- multipliers
__device__ double phi_closed(double s, double R, double Lp) {
  // 2 int_0^R rho cos(b rho) d rho, b = |pi s / Lp|; power series for small b R
  const double b = fabs(M_PI * s / Lp);
  const double x = b * R;
  if (x < 0.5) {
    double term = 1.0, acc = 0.5;
    for (int k = 1; k < 12; ++k) {
      term *= -(x * x) / ((2.0 * k - 1.0) * (2.0 * k));
      acc += term / (2.0 * k + 2.0);
    }
    return 2.0 * R * R * acc;
  }
  return 2.0 * (R * sin(x) / b + (cos(x) - 1.0) / (b * b));
}

__global__ __launch_bounds__(256) void fsm_mult_kernel(FsmMultArgs a) {
  const FsmDims d = a.d;
  const int64_t qll = static_cast<int64_t>(d.Q) * d.L * d.L;
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (idx >= qll) return;
  const int l2i = static_cast<int>(idx % d.L);
  const int l1i = static_cast<int>((idx / d.L) % d.L);
  const int l3 = static_cast<int>(idx / (static_cast<int64_t>(d.L) * d.L));
  const double l1 = l1i - (d.P / 2 - 1), l2 = l2i - (d.P / 2 - 1), l3d = l3;
  double beta = 0.0;
  for (int p = 0; p < a.D; ++p) {
    const double ex = a.dirs[3 * p], ey = a.dirs[3 * p + 1], ez = a.dirs[3 * p + 2];
    const double s = l1 * ex + l2 * ey + l3d * ez;
    const double q0 = l1 - s * ex, q1 = l2 - s * ey, q2 = l3d - s * ez;
    const double perp = sqrt(fmax(q0 * q0 + q1 * q1 + q2 * q2, 0.0));
    double ph, ps;
    if (a.phi_closed) {
      ph = phi_closed(s, a.R, a.Lp);
    } else {
      const double b = fabs(M_PI * s / a.Lp);
      double acc = 0.0;
      for (int k = 0; k < a.n_phi; ++k) acc += a.phi_w[k] * cos(b * a.phi_x[k]);
      ph = 2.0 * acc;
    }
    if (a.psi_closed) {
      const double c = M_PI * a.R * perp / a.Lp;
      ps = c == 0.0 ? M_PI * a.R * a.R : 2.0 * M_PI * a.R * a.R * j1(c) / c;
    } else {
      const double b = M_PI * perp / a.Lp;
      double acc = 0.0;
      for (int k = 0; k < a.n_psi; ++k) acc += a.psi_w[k] * j0(b * a.psi_x[k]);
      ps = 2.0 * M_PI * acc;
    }
    a.mult[static_cast<int64_t>(2 * p) * qll + idx] = ps;
    a.mult[static_cast<int64_t>(2 * p + 1) * qll + idx] = ph;
    beta += a.W[p] * ph * ps;
  }
  a.mult[static_cast<int64_t>(2 * a.D) * qll + idx] = 4.0 * a.b0 * beta;
}

// ---------------------------------------------------------------- per-cell transforms
// One workgroup per (range of terms, slab of B modes l1, cell, parity class of the cell's distribution).  A
// function of one class (even or odd in every velocity axis) lives on the octant v > 0 and has a
// real spectrum on the octant l >= 0, and the multipliers and fields are split into their own
// parity parts (launch_fsm_fold), so every transform is real, Q^3 modes to H^3 velocities (H = n/2,
// cosine or sine factors by the parities), and one term per direction and multiplier kind
// serves all mirror images of the direction.  With the class sums x of the cell:
//   forward  R(l) = sum_i x(i) c1(l1, i1) c2(l2, i2) c3(l3, i3)            (the slab's l1 only)
//   stage 1  T1(l2; b, i3) = sum_l3 m_t(l) R(l) E3(l3, i3)                 (l1 = l10 + b)
//   stage 2  T2(b; i2, i3) = sum_l2 T1(l2; b, i3) E2(l2, i2)
//   stage 3  G(i1; i2, i3) += X_t(i) sum_b E1(l1, i1) T2(b; i2, i3)
// (E = w(l) c(l, .), w = 1 for l = 0 and 2 otherwise; the same table for the three axes).  Bound by
// the FP64 MFMA: a term of a (24-mode, 12-velocity, B = 8) slab is 126 MFMAs against 37 KB of
// multipliers from L2.  R stays in LDS for all terms; the waves take stage 1 of a term and stage 3
// of the one before between the same two barriers, two workgroups share a CU, and the
// multipliers of the next term are in flight across the barrier.  512 cells of the duct's gas (24^3
// velocities on the v3 > 0 half, 129 terms): 5.2 ms with the MFMA pipes 57% busy, where complex
// transforms of the whole spectrum (2.06e9 executed flops per cell, 4.0e8 now) took 33 ms at 39%; one
// cell 51 us instead of 1.44 ms (its terms split over workgroups).  Six waves per workgroup left one
// workgroup per CU (7.3 ms): the waves of two do not spread evenly over the SIMDs.
struct SlabShape {
  int BQ, BH, HH;        // columns of stage 1 (b, l2), 2 (b, i3) and 3 (i2, i3)
  int rs, ts, hs;        // LDS row strides of R, T1, T2
  int t1, t2, t3;        // 16 x 16 tiles of the stages
  int kb4;               // 4-deep k-steps of stage 3
};
__host__ __device__ inline SlabShape slab_shape(const FsmClassDims& d, int B) {
  SlabShape z;
  z.BQ = B * d.Q;
  z.BH = B * d.H;
  z.HH = d.H * d.H;
  const int mt = (d.H + 15) / 16;
  z.t1 = (z.BQ + 15) / 16 * mt;
  z.t2 = (z.BH + 15) / 16 * mt;
  z.t3 = (z.HH + 15) / 16 * mt;
  z.rs = (z.BQ + 15) / 16 * 16 + 16;   // rows k and k + 1 half the banks apart
  z.ts = (z.BH + 15) / 16 * 16 + 1;    // odd: 16 lanes down a column hit distinct banks
  z.hs = (z.HH + 15) / 16 * 16;
  z.kb4 = (B + 3) / 4;   // (LDS rows of T2: 4 per k-step of the kernel, one or two)
  return z;
}
// 4-deep k-steps that the kernel is built for: at least ceil(Q / 4)
inline int class_ksteps(const FsmClassDims& d) { return d.H > 16 ? 8 : d.Q <= 16 ? 4 : (d.Q + 3) / 4; }

// KS, KB: 4-deep k-steps of stages 1 and 2, and of stage 3 (zeros past Q and B); NT1, NT2, NT3: tiles per
// wave of the stages; MT: 16-wide tiles along a velocity axis.  Without GUARD the term loop has no
// branch: a wave without a tile computes one that goes to `trash` (or is never stored).
template <int KS, int KB, int NT1, int NT2, int NT3, int MT, bool GUARD>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(NT3 == 2 ? 4 : 2))) void fsm_class_kernel(FsmClassDims d, int B, const double* __restrict__ X,
                                                        const double* __restrict__ Etab,
                                                        const double* __restrict__ mult,
                                                        const double* __restrict__ field,
                                                        const int* __restrict__ parts, double* __restrict__ accp,
                                                        int64_t acc_stride) {
  extern __shared__ double sm[];
  constexpr int HP = 16 * MT, KP = 4 * KS;
  const SlabShape z = slab_shape(d, B);
  const int Q = d.Q, H = d.H;
  double* E = sm;                       // [2][KP][HP]: cosines, sines; zero past Q and H
  double* R = E + 2 * KP * HP;          // [KP][rs]
  double* T1 = R + KP * z.rs;           // [KP][ts]
  double* T2 = T1 + KP * z.ts;          // [4 KB][hs]
  // then 64 doubles that idle tiles write
  const int tid = threadIdx.x, nthr = blockDim.x, W = nthr >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, kr = lane >> 4, cc = lane & 15;
  const int l10 = blockIdx.y * B;
  const int64_t cell = blockIdx.x / d.nb;
  const int cls = static_cast<int>(blockIdx.x - cell * d.nb);
  // parity of the class along each axis; the axes stored by parity carry theirs
  const int x1 = cls & 1, x2 = d.nb >= 4 ? (cls >> 1) & 1 : 0, x3 = d.nb == 8 ? (cls >> 2) & 1 : 1;
  const double* xr = X + (cell * d.nb + cls) * static_cast<int64_t>(d.ld);

  for (int i = tid; i < 2 * KP * HP; i += nthr) {
    const int l = (i / HP) % KP;
    E[i] = l < Q ? Etab[((i >= KP * HP ? Q : 0) + l) * HP + i % HP] : 0.0;
  }
  for (int i = tid; i < KP * (z.rs + z.ts) + 4 * KB * z.hs + 64; i += nthr) R[i] = 0.0;
  __syncthreads();
  // forward: E carries w(l), taken out again by halving (exact)
  auto fac = [&](int odd, int l, int i) { return (l == 0 ? 1.0 : 0.5) * E[(odd * KP + l) * HP + i]; };
  for (int o = tid; o < B * z.HH; o += nthr) {
    const int b = o / z.HH, r = o - b * z.HH;
    if (l10 + b < Q) {
      double a = 0.0;
      for (int i = 0; i < H; ++i) a += fac(x1, l10 + b, i) * xr[i * z.HH + r];
      T2[b * z.hs + r] = a;
    }
  }
  __syncthreads();
  for (int o = tid; o < B * Q * H; o += nthr) {
    const int i3 = o % H, l2 = (o / H) % Q, b = o / (H * Q);
    double a = 0.0;
    for (int i = 0; i < H; ++i) a += fac(x2, l2, i) * T2[b * z.hs + i * H + i3];
    T1[l2 * z.ts + b * H + i3] = a;
  }
  __syncthreads();
  for (int o = tid; o < Q * z.BQ; o += nthr) {
    const int c = o % z.BQ, l3 = o / z.BQ, b = c / Q, l2 = c - b * Q;
    double a = 0.0;
    for (int i = 0; i < H; ++i) a += fac(x3, l3, i) * T1[l2 * z.ts + b * H + i];
    R[l3 * z.rs + c] = a;
  }
  __syncthreads();

  // This wave's tiles of the stages and the lane's addresses in them, once for all terms (the index
  // divisions would cost more than a term's MFMAs): tile (c0, i0) = (column, velocity) origin.
  // Stage 1: multiplier offset (clamped in bounds: the slab's columns are contiguous in a row of the
  // table, and the last slab may end inside them), R column, T1 slots of the lane's four results.
  // Stage 2: T1 column and T2 slots.  Stage 3: T2 column, field offsets (clamped), E column.
  const int Q2 = Q * Q;
  const int ct1 = z.t1 / MT, ct2 = z.t2 / MT, ct3 = z.t3 / MT;
  // (all as offsets: LDS ones from sm)
  const int oR = 2 * KP * HP, oT1 = oR + KP * z.rs, oT2 = oT1 + KP * z.ts, trash = oT2 + 4 * KB * z.hs + lane;
  int mcol[NT1], rcol[NT1], tcol[NT2], ycol[NT3], e3col[NT1], e2col[NT2], e1col[NT3];
  int slot1[NT1][4], slot2[NT2][4];
#pragma unroll
  for (int j = 0; j < NT1; ++j) {
    const int tile = min(wave + W * j, z.t1 - 1);
    const int m = MT == 1 ? 0 : tile / ct1, c0 = (tile - m * ct1) * 16, i3 = m * 16 + cc;
    rcol[j] = oR + kr * z.rs + c0 + cc;
    e3col[j] = kr * HP + i3;
    mcol[j] = (kr * Q2 + min(l10 * Q + min(c0 + cc, z.BQ - 1), Q2 - 1)) * 8;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int c = c0 + kr + 4 * r, b = c / Q, l2 = c - b * Q;
      slot1[j][r] = wave + W * j < z.t1 && c < z.BQ && i3 < H ? oT1 + l2 * z.ts + b * H + i3 : trash;
    }
  }
#pragma unroll
  for (int j = 0; j < NT2; ++j) {
    const int tile = min(wave + W * j, z.t2 - 1);
    const int m = MT == 1 ? 0 : tile / ct2, c0 = (tile - m * ct2) * 16, i2 = m * 16 + cc;
    tcol[j] = oT1 + kr * z.ts + c0 + cc;
    e2col[j] = kr * HP + i2;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int c = c0 + kr + 4 * r, b = c / H, i3 = c - b * H;
      slot2[j][r] = wave + W * j < z.t2 && c < z.BH && i2 < H ? oT2 + b * z.hs + i2 * H + i3 : trash;
    }
  }
  int foff[NT3];
#pragma unroll
  for (int q = 0; q < NT3; ++q) {
    const int tile = min(wave + W * q, z.t3 - 1);
    const int m = MT == 1 ? 0 : tile / ct3, c0 = (tile - m * ct3) * 16;
    ycol[q] = oT2 + kr * z.hs + c0 + cc;
    e1col[q] = min(l10 + kr, KP - 1) * HP + m * 16 + cc;   // rows of T2 past the slab are zero
    foff[q] = ((m * 16 + kr) * z.HH + min(c0 + cc, z.HH - 1)) * 8;
  }
  const int e1step = KB == 2 ? (min(l10 + 4 + kr, KP - 1) - min(l10 + kr, KP - 1)) * HP : 0;
  double mv[NT1][KS], fv[NT3][4];
  // a scalar base (the tables' rows are padded to whole k-steps and tiles) and a 32-bit byte offset
  auto at = [](const double* base, int off) {
    return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(base) + static_cast<unsigned>(off));
  };
  const int64_t mterm = static_cast<int64_t>(KP) * Q2, fterm = static_cast<int64_t>(HP) * z.HH;
  auto load_mult = [&](int t) {
    const double* mt = mult + t * mterm;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int j = 0; j < NT1; ++j) mv[j][ks] = at(mt + 4 * ks * Q2, mcol[j]);
  };
  auto load_field = [&](int t) {
    const double* ft = field + t * fterm;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int q = 0; q < NT3; ++q) fv[q][r] = at(ft + 4 * r * z.HH, foff[q]);
  };
  v4d G[NT3];
#pragma unroll
  for (int q = 0; q < NT3; ++q) G[q] = v4d{0.0, 0.0, 0.0, 0.0};
  auto stage1 = [&](int part) {
    const int e = (x3 ^ ((part >> 2) & 1)) * KP * HP;
    v4d o[NT1];
#pragma unroll
    for (int j = 0; j < NT1; ++j) o[j] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int j = 0; j < NT1; ++j)
        if (!GUARD || wave + W * j < z.t1) o[j] = mfma(mv[j][ks] * sm[rcol[j] + 4 * ks * z.rs], sm[e3col[j] + e + 4 * ks * HP], o[j]);
#pragma unroll
    for (int j = 0; j < NT1; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) sm[slot1[j][r]] = o[j][r];
  };
  auto stage2 = [&](int part) {
    const int e = (x2 ^ ((part >> 1) & 1)) * KP * HP;
    v4d o[NT2];
#pragma unroll
    for (int j = 0; j < NT2; ++j) o[j] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int j = 0; j < NT2; ++j)
        if (!GUARD || wave + W * j < z.t2) o[j] = mfma(sm[tcol[j] + 4 * ks * z.ts], sm[e2col[j] + e + 4 * ks * HP], o[j]);
#pragma unroll
    for (int j = 0; j < NT2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) sm[slot2[j][r]] = o[j][r];
  };
  auto stage3 = [&](int part) {
    const int e = (x1 ^ (part & 1)) * KP * HP;
    // i^(odd axes after - odd axes before): the phases of the sine axes
    const int after = (x1 ^ (part & 1)) + (x2 ^ ((part >> 1) & 1)) + (x3 ^ ((part >> 2) & 1));
    const double sgn = after == x1 + x2 + x3 ? 1.0 : -1.0;
    v4d o[NT3];
#pragma unroll
    for (int q = 0; q < NT3; ++q) o[q] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int q = 0; q < NT3; ++q)
        if (!GUARD || wave + W * q < z.t3) o[q] = mfma(sm[e1col[q] + e + kb * e1step], sm[ycol[q] + 4 * kb * z.hs], o[q]);
#pragma unroll
    for (int q = 0; q < NT3; ++q)
#pragma unroll
      for (int r = 0; r < 4; ++r) G[q][r] += fv[q][r] * (sgn * o[q][r]);
  };
  // Between two barriers: stage 1 of a term with stage 3 of the one before, then stage 2.  The next
  // term's multipliers are loaded once stage 1 has used this term's, its fields before stage 2; the
  // scheduler must not pull their first use across the barrier (it would wait for them there).
  const int t0 = static_cast<int>(static_cast<int64_t>(d.T) * blockIdx.z / gridDim.z);
  const int last = static_cast<int>(static_cast<int64_t>(d.T) * (blockIdx.z + 1) / gridDim.z) - 1;
  load_mult(t0);
  int part = parts[t0];
  stage1(part);
  load_mult(min(t0 + 1, last));
  __syncthreads();
  for (int t = t0; t < last; ++t) {
    const int next = parts[t + 1];
    load_field(t);
    stage2(part);
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
    stage1(next);
    load_mult(min(t + 2, last));
    stage3(part);
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
    part = next;
  }
  load_field(last);
  stage2(part);
  __syncthreads();
  stage3(part);
  double* out = accp + (blockIdx.z * gridDim.y + blockIdx.y) * acc_stride + (cell * d.nb + cls) * static_cast<int64_t>(d.ld);
#pragma unroll
  for (int q = 0; q < NT3; ++q) {
    const int tile = wave + W * q;
    if (tile < z.t3) {
      const int c = (tile % ct3) * 16 + cc, i0 = (tile / ct3) * 16 + kr;
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (c < z.HH && i0 + 4 * r < H) out[(i0 + 4 * r) * z.HH + c] = G[q][r];
    }
  }
}

// Parity parts of the multipliers and fields (see launch_fsm_fold): part k of term t, odd along
// the axes of the bits of part[t] (none or two; every table is even under inversion), is the mean over
// the images (l1, l2, l3), (-l1, l2, l3), (l1, l2, -l3), (-l1, l2, -l3) with the signs of axes 1 and 3.
__global__ __launch_bounds__(256) void fsm_fold_mult_kernel(FsmDims d, int T, int rows, const double* __restrict__ mult,
                                                            const int* __restrict__ row, const int* __restrict__ part,
                                                            double* __restrict__ out) {
  const int Q = d.Q, L = d.L, half = d.P / 2 - 1;
  const int64_t len = static_cast<int64_t>(rows) * Q * Q;
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i >= T * len) return;
  const int t = static_cast<int>(i / len);
  const int r = static_cast<int>(i - t * len);
  const int l2 = r % Q, l1 = (r / Q) % Q, l3 = r / (Q * Q);
  if (l3 >= Q) {
    out[i] = 0.0;
    return;
  }
  const double* m = mult + static_cast<int64_t>(row[t]) * Q * L * L;
  auto at = [&](int a, int b) { return m[(static_cast<int64_t>(l3) * L + half + a) * L + half + b]; };
  const double s1 = part[t] & 1 ? -1.0 : 1.0, s3 = part[t] & 4 ? -1.0 : 1.0;
  // (-l1, l2, l3); (l1, l2, -l3) ~ (-l1, -l2, l3); (-l1, l2, -l3) ~ (l1, -l2, l3)
  out[i] = 0.25 * ((at(l1, l2) + s1 * at(-l1, l2)) + s3 * (at(-l1, -l2) + s1 * at(l1, -l2)));
}

__global__ __launch_bounds__(256) void fsm_fold_field_kernel(int n, int T, int rows, const double* __restrict__ in,
                                                             const double* __restrict__ feq,
                                                             const int* __restrict__ src, const int* __restrict__ part,
                                                             const double* __restrict__ coef,
                                                             double* __restrict__ out) {
  const int H = n / 2;
  const int64_t len = static_cast<int64_t>(rows) * H * H;
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i >= T * len) return;
  const int t = static_cast<int>(i / len);
  const int r = static_cast<int>(i - t * len);
  const int i3 = r % H, i2 = (r / H) % H, i1 = r / (H * H);
  if (i1 >= H) {
    out[i] = 0.0;
    return;
  }
  const double* f = src[t] >= 0 ? in + static_cast<int64_t>(src[t]) * n * n * n : feq;
  auto at = [&](int m1, int m3) {   // reflected along axes 1, 3
    const int a = m1 ? H - 1 - i1 : H + i1, c = m3 ? H - 1 - i3 : H + i3;
    return f[(static_cast<int64_t>(a) * n + H + i2) * n + c];
  };
  const double s1 = part[t] & 1 ? -1.0 : 1.0, s3 = part[t] & 4 ? -1.0 : 1.0;
  out[i] = coef[t] * 0.25 * ((at(0, 0) + s1 * at(1, 0)) + s3 * (at(0, 1) + s1 * at(1, 1)));
}

// ---------------------------------------------------------------- plan tables
// One workgroup per (term, slab of K1 output rows a1):
//   Z(a1, l3, l2)  = sum_l1 E1(a1, l1) m_t(l3, l1, l2) X(l1, l3, l2)
//   W(a1, l3, a2)  = sum_l2 Z(a1, l3, l2) E2(a2, l2)
//   O(a1, a2, a3)  = Re sum_l3 W(a1, l3, a2) E3(a3, l3)
__global__ __launch_bounds__(kThreads) void fsm_table_kernel(FsmTableArgs a, int K1) {
  extern __shared__ double sm[];
  const FsmDims d = a.d;
  const int t = a.t0 + blockIdx.y;
  const int slot = a.slot[t];
  if (slot < 0) return;
  const int L = d.L, Q = d.Q, m2 = a.m2, m3 = a.m3;
  const double* e1r = a.e1r + t * a.e1_ts;
  const double* e1i = a.e1i + t * a.e1_ts;
  const double* e2r = a.e2r + t * a.e2_ts;
  const double* e2i = a.e2i + t * a.e2_ts;
  const double* e3r = a.e3r + t * a.e3_ts;
  const double* e3i = a.e3i + t * a.e3_ts;
  const int r0 = blockIdx.x * K1, kr1 = min(K1, a.m1 - r0);
  double* Zr = sm;                    // [K1][Q][L]
  double* Zi = Zr + K1 * Q * L;
  double* Wr = Zi + K1 * Q * L;       // [K1][Q][m2]
  double* Wi = Wr + K1 * Q * m2;
  const int64_t LL = static_cast<int64_t>(L) * L;
  const double* mt = a.mult + static_cast<int64_t>(a.mrow ? a.mrow[t] : t) * Q * LL;
  const int64_t sQL = static_cast<int64_t>(Q) * L;
  {
    const int M = kr1, K = L, N = Q * L;   // column c = (l3, l2)
    auto la = [&](int m, int k, double& re, double& im) {
      const bool ok = m < M && k < K;
      re = ok ? e1r[(r0 + m) * L + k] : 0.0;
      im = ok ? e1i[(r0 + m) * L + k] : 0.0;
    };
    auto lb = [&](int k, int c, double& re, double& im) {
      if (k < K && c < N) {
        const int l3 = c / L, l2 = c - l3 * L;
        const double mv = mt[l3 * LL + static_cast<int64_t>(k) * L + l2];
        if (a.X) {
          const int64_t o = (static_cast<int64_t>(k) * 2 * Q + l3) * L + l2;
          re = mv * a.X[o];
          im = mv * a.X[o + sQL];
        } else {
          re = mv;
          im = 0.0;
        }
      } else {
        re = im = 0.0;
      }
    };
    auto st = [&](int m, int c, double re, double im) {
      Zr[m * N + c] = re;
      Zi[m * N + c] = im;
    };
    cgemm<2>(M, N, K, la, lb, st);
  }
  __syncthreads();
  {
    const int M = kr1 * Q, K = L, N = m2;  // row r = (a1, l3)
    auto la = [&](int m, int k, double& re, double& im) {
      const bool ok = m < M && k < K;
      re = ok ? Zr[m * L + k] : 0.0;
      im = ok ? Zi[m * L + k] : 0.0;
    };
    auto lb = [&](int k, int c, double& re, double& im) {
      const bool ok = k < K && c < N;
      re = ok ? e2r[c * L + k] : 0.0;
      im = ok ? e2i[c * L + k] : 0.0;
    };
    auto st = [&](int m, int c, double re, double im) {
      Wr[m * m2 + c] = re;
      Wi[m * m2 + c] = im;
    };
    cgemm<2>(M, N, K, la, lb, st);
  }
  __syncthreads();
  {
    const int M = kr1 * m2, K = Q, N = m3;  // row r = (a1, a2)
    auto la = [&](int m, int k, double& re, double& im) {
      const bool ok = m < M && k < K;
      const int a1 = ok ? m / m2 : 0, a2 = m - a1 * m2;
      re = ok ? Wr[(a1 * Q + k) * m2 + a2] : 0.0;
      im = ok ? Wi[(a1 * Q + k) * m2 + a2] : 0.0;
    };
    auto lb = [&](int k, int c, double& re, double& im) {
      const bool ok = k < K && c < N;
      re = ok ? e3r[c * Q + k] : 0.0;
      im = ok ? e3i[c * Q + k] : 0.0;
    };
    const double sc = a.scale[t];
    double* out = a.out + static_cast<int64_t>(slot) * a.m1 * m2 * m3;
    auto st = [&](int m, int c, double re, double) {
      out[(static_cast<int64_t>(r0) * m2 + m) * m3 + c] = sc * re;
    };
    cgemm<2>(M, N, K, la, lb, st);
  }
}

__global__ void fsm_shift_factor_kernel(int nt, int m, int nl, int lmin, int doubled, const int* __restrict__ base,
                                        const double* __restrict__ shift, int shift_stride, int P,
                                        double* __restrict__ er, double* __restrict__ ei) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= static_cast<int64_t>(nt) * m * nl) return;
  const int k = static_cast<int>(i % nl), a = static_cast<int>((i / nl) % m), t = static_cast<int>(i / (static_cast<int64_t>(nl) * m));
  const int l = lmin + k;
  // the angle pi q / P with q = l (base + 2 z) reduced mod 2P before the sine and cosine
  double q = l * (base[a] + 2.0 * shift[static_cast<int64_t>(t) * shift_stride]);
  q -= 2.0 * P * floor(q / (2.0 * P));
  const double ang = M_PI * q / P;
  const double w = (doubled && l > 0) ? 2.0 : 1.0;
  er[i] = w * cos(ang);
  ei[i] = w * sin(ang);
}

__global__ void band_profile_kernel(int nt, int m, int off, const double* __restrict__ g, int ng,
                                    const double* __restrict__ z, int P, double* __restrict__ S) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= static_cast<int64_t>(nt) * 3 * m) return;
  const int a = static_cast<int>(i % m), k = static_cast<int>((i / m) % 3), t = static_cast<int>(i / (3 * m));
  const double zz = z[3 * t + k];
  auto dirichlet = [&](double w) {
    double s = 1.0;
    for (int l = 1; l < P / 2; ++l) s += 2.0 * cos(2.0 * M_PI * l * w / P);
    return s / P;
  };
  double acc = 0.0;
  if (ng == 0) {
    acc = dirichlet(off + a + zz);
  } else {
    for (int j = 0; j < ng; ++j) acc += g[j] * dirichlet(off + a - j + zz);
  }
  S[i] = acc;
}

__global__ void separable_kernel(int nt, int m, const double* __restrict__ S, const double* __restrict__ w,
                                 double* __restrict__ out) {
  const int64_t m3 = static_cast<int64_t>(m) * m * m;
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= nt * m3) return;
  const int t = static_cast<int>(i / m3);
  const int64_t r = i - t * m3;
  const int a0 = static_cast<int>(r / (m * m)), a1 = static_cast<int>((r / m) % m), a2 = static_cast<int>(r % m);
  const double* St = S + static_cast<int64_t>(t) * 3 * m;
  out[i] = w[t] * St[a0] * St[m + a1] * St[2 * m + a2];
}

__global__ void scale_rows_kernel(int nt, int64_t len, const double* __restrict__ in, const int* __restrict__ src,
                                  const double* __restrict__ sc, double* __restrict__ out) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= nt * len) return;
  const int t = static_cast<int>(i / len);
  out[i] = sc[t] * in[static_cast<int64_t>(src[t]) * len + (i - t * len)];
}

size_t table_lds_bytes(const FsmDims& d, int m2, int K1) {
  return static_cast<size_t>(2 * K1 * d.Q * d.L + 2 * K1 * d.Q * m2) * sizeof(double);
}

size_t class_lds_bytes(const FsmClassDims& d, int B) {
  const SlabShape z = slab_shape(d, B);
  const int KP = 4 * class_ksteps(d);
  return (static_cast<size_t>(KP) * (z.rs + z.ts) + 8 * z.hs +
          2 * static_cast<size_t>(KP) * ((d.H + 15) / 16 * 16) + 64) * sizeof(double);
}

// Kernel of a slab and its waves (4 or 8: a whole number per SIMD, so that two workgroups share a CU), by
// the tiles per wave of the stages: four waves with up to (3, 2, 3) tiles for slabs of more than 4 and
// (2, 1, 4) for narrower ones (the default slabs of 16 to 24 and of 25 to 32 modes), else eight with up to
// (2, 1, 2); velocity axes of more than 16 nodes have a kernel of their own.  W = 0: none.
struct ClassKernel {
  int W, kind;
  bool exact;   // every wave has its full share: no guards
};
ClassKernel class_kernel(const FsmClassDims& d, int B) {
  const SlabShape z = slab_shape(d, B);
  auto fits = [&](int w, int n1, int n2, int n3) { return z.t1 <= n1 * w && z.t2 <= n2 * w && z.t3 <= n3 * w; };
  const int ks = class_ksteps(d);
  if (d.H > 16) return {fits(8, 4, 3, 6) ? 8 : 0, 3, false};
  if (fits(4, 2, 1, 2)) return {4, 0, false};
  if (z.kb4 == 2 && ks <= 6 && fits(4, 3, 2, 3)) return {4, 1, z.t1 > 8 && z.t2 > 4 && z.t3 > 8 && z.t1 % 4 == 0};
  if (z.kb4 == 1 && ks >= 7 && fits(4, 2, 1, 4)) return {4, 2, z.t1 == 8 && z.t2 == 4 && z.t3 > 12};
  return {fits(8, 2, 1, 2) ? 8 : 0, 0, false};
}

constexpr size_t kLdsMax = 160 * 1024;

}  // namespace

hipError_t launch_fsm_multipliers(const FsmMultArgs& a, hipStream_t s) {
  const int64_t qll = static_cast<int64_t>(a.d.Q) * a.d.L * a.d.L;
  hipLaunchKernelGGL(fsm_mult_kernel, dim3(static_cast<unsigned>((qll + 255) / 256)), dim3(256), 0, s, a);
  return hipGetLastError();
}

int fsm_mult_rows(const FsmClassDims& d) { return 4 * class_ksteps(d); }
int fsm_field_rows(const FsmClassDims& d) { return (d.H + 15) / 16 * 16; }

hipError_t launch_fsm_fold(const FsmDims& d, const FsmClassDims& c, const double* mult, const int* row, const int* part,
                           double* out, hipStream_t s) {
  const int rows = fsm_mult_rows(c);
  const int64_t total = static_cast<int64_t>(c.T) * rows * c.Q * c.Q;
  hipLaunchKernelGGL(fsm_fold_mult_kernel, dim3(static_cast<unsigned>((total + 255) / 256)), dim3(256), 0, s, d, c.T, rows,
                     mult, row, part, out);
  return hipGetLastError();
}

hipError_t launch_fsm_fold_fields(const FsmClassDims& c, const double* in, const double* feq, const int* src,
                                  const int* part, const double* coef, double* out, hipStream_t s) {
  const int rows = fsm_field_rows(c);
  const int64_t total = static_cast<int64_t>(c.T) * rows * c.H * c.H;
  hipLaunchKernelGGL(fsm_fold_field_kernel, dim3(static_cast<unsigned>((total + 255) / 256)), dim3(256), 0, s, 2 * c.H,
                     c.T, rows, in, feq, src, part, coef, out);
  return hipGetLastError();
}

hipError_t launch_fsm_shift_factors(int nt, int m, int nl, int lmin, int doubled, const int* base, const double* shift,
                                    int shift_stride, int P, double* er, double* ei, hipStream_t s) {
  const int64_t total = static_cast<int64_t>(nt) * m * nl;
  if (total <= 0) return hipSuccess;
  hipLaunchKernelGGL(fsm_shift_factor_kernel, dim3(static_cast<unsigned>((total + 255) / 256)), dim3(256), 0, s, nt, m,
                     nl, lmin, doubled, base, shift, shift_stride, P, er, ei);
  return hipGetLastError();
}

hipError_t launch_band_profiles(int nt, int m, int off, const double* g, int ng, const double* z, int P, double* S,
                                hipStream_t s) {
  const int64_t total = static_cast<int64_t>(nt) * 3 * m;
  if (total <= 0) return hipSuccess;
  hipLaunchKernelGGL(band_profile_kernel, dim3(static_cast<unsigned>((total + 255) / 256)), dim3(256), 0, s, nt, m, off,
                     g, ng, z, P, S);
  return hipGetLastError();
}

hipError_t launch_separable(int nt, int m, const double* S, const double* w, double* out, hipStream_t s) {
  const int64_t total = static_cast<int64_t>(nt) * m * m * m;
  if (total <= 0) return hipSuccess;
  hipLaunchKernelGGL(separable_kernel, dim3(static_cast<unsigned>((total + 255) / 256)), dim3(256), 0, s, nt, m, S, w,
                     out);
  return hipGetLastError();
}

hipError_t launch_scale_rows(int nt, int64_t len, const double* in, const int* src, const double* sc, double* out,
                             hipStream_t s) {
  const int64_t total = static_cast<int64_t>(nt) * len;
  if (total <= 0) return hipSuccess;
  hipLaunchKernelGGL(scale_rows_kernel, dim3(static_cast<unsigned>((total + 255) / 256)), dim3(256), 0, s, nt, len, in,
                     src, sc, out);
  return hipGetLastError();
}

bool fsm_tables_fit(const FsmDims& d, int m2) { return table_lds_bytes(d, m2, 1) <= kLdsMax; }

hipError_t launch_fsm_tables(const FsmTableArgs& a, hipStream_t s) {
  if (a.nt <= 0) return hipSuccess;
  int K1 = 4;
  while (K1 > 1 && table_lds_bytes(a.d, a.m2, K1) > kLdsMax) --K1;
  const size_t lds = table_lds_bytes(a.d, a.m2, K1);
  if (lds > kLdsMax) return hipErrorInvalidValue;
  dim3 grid((a.m1 + K1 - 1) / K1, a.nt);
  hipLaunchKernelGGL(fsm_table_kernel, grid, dim3(kThreads), lds, s, a, K1);
  return hipGetLastError();
}

int fsm_slab_count(const FsmClassDims& d, int slab_l1) { return (d.Q + slab_l1 - 1) / slab_l1; }

int fsm_default_slab(const FsmClassDims& d) {
  // the widest (up to 8) of which two workgroups fit a CU's LDS and four waves hold the tiles
  int B = 8;
  auto good = [&](int b) {
    const int W = class_kernel(d, b).W;
    return b <= d.Q && class_lds_bytes(d, b) <= kLdsMax / 2 && (W == 4 || (W && d.H > 16));
  };
  while (B > 1 && !good(B)) --B;
  return B;
}

bool fsm_slab_fits(const FsmClassDims& d, int slab_l1) {
  return slab_l1 >= 1 && slab_l1 <= 8 && class_lds_bytes(d, slab_l1) <= kLdsMax && class_kernel(d, slab_l1).W;
}

const char* fsm_unsupported(const FsmDims& d) {
  const int tiles = ((d.n + 15) / 16) * ((d.n2 * d.n3 + 15) / 16);
  if (tiles > 64) return "the per-cell transform path holds at most 64 x 16 x 16 outputs per cell (use parity storage)";
  if (d.Q > 32) return "the per-cell transform path takes n_pad <= 64";
  return nullptr;
}

int fsm_sums(const FsmClassDims& d, int slab_l1, int64_t n_cells) {
  // few cells: the terms are split over workgroups (at least four each) until two fit every CU twice
  const int slabs = fsm_slab_count(d, slab_l1);
  const int64_t groups = n_cells * d.nb * slabs;
  return slabs * static_cast<int>(std::max<int64_t>(1, std::min<int64_t>({1024 / std::max<int64_t>(groups, 1), 16, d.T / 4})));
}

hipError_t launch_fsm_class(const FsmClassDims& d, int slab_l1, int64_t n_cells, const double* X, const double* E,
                            const double* mult, const double* field, const int* part, double* acc, int64_t acc_stride,
                            hipStream_t s) {
  if (n_cells <= 0) return hipSuccess;
  const SlabShape z = slab_shape(d, slab_l1);
  const size_t lds = class_lds_bytes(d, slab_l1);
  const ClassKernel k = class_kernel(d, slab_l1);
  const int ks = class_ksteps(d);
  if (lds > kLdsMax || d.Q > 4 * ks || ks > 8 || d.H > 32 || !k.W) return hipErrorInvalidValue;
  // consecutive workgroups take the same slab: the CUs of an XCD read the same multipliers
  const int slabs = fsm_slab_count(d, slab_l1);
  const dim3 grid(static_cast<unsigned>(n_cells * d.nb), slabs, fsm_sums(d, slab_l1, n_cells) / slabs);
#define SIS_FSM(...)                                                                                                  \
  hipLaunchKernelGGL((fsm_class_kernel<__VA_ARGS__>), grid, dim3(64 * k.W), lds, s, d, slab_l1, X, E, mult, field, part, \
                     acc, acc_stride)
  if (k.kind == 3) {
    SIS_FSM(8, 2, 4, 3, 6, 2, true);
  } else if (k.kind == 1) {
    if (ks == 4) SIS_FSM(4, 2, 3, 2, 3, 1, true);
    else if (ks == 5) SIS_FSM(5, 2, 3, 2, 3, 1, true);
    else if (!k.exact) SIS_FSM(6, 2, 3, 2, 3, 1, true);
    else SIS_FSM(6, 2, 3, 2, 3, 1, false);
  } else if (k.kind == 2) {
    if (ks == 7) SIS_FSM(7, 1, 2, 1, 4, 1, true);
    else if (!k.exact) SIS_FSM(8, 1, 2, 1, 4, 1, true);
    else SIS_FSM(8, 1, 2, 1, 4, 1, false);
  } else if (ks == 4) {
    SIS_FSM(4, 2, 2, 1, 2, 1, true);
  } else if (ks == 5) {
    SIS_FSM(5, 2, 2, 1, 2, 1, true);
  } else if (ks == 6) {
    SIS_FSM(6, 2, 2, 1, 2, 1, true);
  } else if (ks == 7) {
    SIS_FSM(7, 2, 2, 1, 2, 1, true);
  } else {
    SIS_FSM(8, 2, 2, 1, 2, 1, true);
  }
#undef SIS_FSM
  return hipGetLastError();
}

double fsm_flops_per_cell(const FsmClassDims& d, int slab_l1) {
  // MFMAs issued (2048 flops each) by every class and slab, and the forward sums
  const SlabShape z = slab_shape(d, slab_l1);
  const int ks = class_ksteps(d), slabs = fsm_slab_count(d, slab_l1);
  const double mfma = static_cast<double>(d.T) * ((z.t1 + z.t2) * ks + z.t3 * z.kb4);
  const double fwd = 2.0 * d.H * (slab_l1 * z.HH + static_cast<double>(z.BQ) * d.H + static_cast<double>(d.Q) * z.BQ);
  return d.nb * slabs * (2048.0 * mfma + fwd);
}

}  // namespace sis
