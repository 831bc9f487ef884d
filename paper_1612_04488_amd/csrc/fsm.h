// The fast spectral method on the device: separable pruned DFTs of the velocity grid as
// small GEMMs on the FP64 MFMA, staged in LDS (fsm.hip), per cell and for the plan's
// tables.  All pointers are device pointers.
//
// Modes of the tables: l1, l2 take the P - 1 signed values -(P/2 - 1) .. P/2 - 1 (index
// l + P/2 - 1; the Nyquist mode -P/2 carries no multiplier), l3 the Q = P/2
// values 0 .. P/2 - 1 (half spectrum: h is real, so its transform is
// Hermitian).  Frequencies xi_l = pi l / L_p, velocities v_j = (j + 1/2 - n/2) dv.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sis {

struct FsmDims {
  int n;        // velocity nodes per axis
  int P;        // padded DFT size per axis
  int L;        // P - 1 modes on axes 1, 2
  int Q;        // P / 2 modes on axis 3
  int n2, n3;   // stored nodes on axes 2, 3
  int nv;       // n * n2 * n3 stored velocities per cell
  int T;        // terms: 2 D gain terms and the loss
};

// Multipliers m[T][Q][L][L] (term 2p: psi_p, 2p + 1: phi_p, 2D: beta) of the
// half spectrum, evaluated on the device.  dirs[D][3], W[D]; the radial rule as
// RadialRule (planner.h): phi_closed / psi_closed select the closed forms, else
// the node tables (nodes, weights) are used.
struct FsmMultArgs {
  FsmDims d;
  int D;
  double b0, R, Lp;
  const double* dirs;
  const double* W;
  int phi_closed, psi_closed;
  int n_phi, n_psi;
  const double *phi_x, *phi_w, *psi_x, *psi_w;
  double* mult;
};
hipError_t launch_fsm_multipliers(const FsmMultArgs& a, hipStream_t s);

// ---- per-cell transforms on parity classes (see SymMap in kernels.h for the classes and their rows)
// A function that is even or odd in every velocity axis is given by its values at the H^3 velocities
// of the octant v > 0 (H = n/2, v = (i + 1/2) dv) and has a real spectrum on the Q^3 modes
// l >= 0 (Q = n_pad/2, the Nyquist modes dropped) up to a phase per odd axis.  The terms:
// for a direction e and its mirror images, with psi^k, X^k the parts of the multiplier and field
// that are odd along the axes of k (none or two axes), sum over the images X (psi * h) =
// (number of images) sum_k X^k (psi^k * h); every product keeps the class of h.
struct FsmClassDims {
  int Q, H;     // modes and velocities per axis
  int T;        // terms: (direction up to reflection, part k, kind of multiplier), and the loss
  int nb, ld;   // classes and their row length (SymMap)
};
// mult [T][l3][l1][l2], l3 padded with zeros to fsm_mult_rows: part[t] (bits: odd axes 1, 2, 3) of row
// row[t] of the multipliers m[.][Q][L][L]
int fsm_mult_rows(const FsmClassDims& d);
hipError_t launch_fsm_fold(const FsmDims& d, const FsmClassDims& c, const double* mult, const int* row, const int* part,
                           double* out, hipStream_t s);
// field [T][i1][i2][i3], i1 padded with zeros to fsm_field_rows: coef[t] times part[t] of the full-grid
// field in[src[t]] (feq for src[t] < 0)
int fsm_field_rows(const FsmClassDims& d);
hipError_t launch_fsm_fold_fields(const FsmClassDims& c, const double* in, const double* feq, const int* src,
                                  const int* part, const double* coef, double* out, hipStream_t s);
// Transforms of every term with their field products, summed, from the class rows X [cells][nb][ld]:
//   acc[s][cell][class][i] = sum_{t in range} field[t][i] sum_{l1 in slab} sum_{l2, l3} mult[t][l] R(l) E E E
// for the slabs of slab_l1 modes l1 each (n_slabs = ceil(Q / slab_l1)) and, for few cells, ranges of
// terms; the fsm_sums partial sums (acc_stride elements apart) add up to the class sums of L+ of each
// cell at delta = 1.  E [2][Q][H rounded up to 16]: w(l) cos, w(l) sin of pi l (2 i + 1) / n_pad, w = 1 for
// l = 0 and 2 otherwise, zero past H.
int fsm_sums(const FsmClassDims& d, int slab_l1, int64_t n_cells);
int fsm_slab_count(const FsmClassDims& d, int slab_l1);
int fsm_default_slab(const FsmClassDims& d);
// whether the transform kernel's LDS holds a slab of slab_l1 modes
bool fsm_slab_fits(const FsmClassDims& d, int slab_l1);
// null if the grid is within what the path takes, else the reason.
const char* fsm_unsupported(const FsmDims& d);
hipError_t launch_fsm_class(const FsmClassDims& d, int slab_l1, int64_t n_cells, const double* X, const double* E,
                            const double* mult, const double* field, const int* part, double* acc, int64_t acc_stride,
                            hipStream_t s);
// Per-term pruned inverse DFTs of the multipliers (plan-time tables), times a
// spectrum X (layout of S, one cell) or X = 1 when X is null:
//   out[slot[t]][a1][a2][a3] = scale[t] Re sum_l E1(a1, l1) E2(a2, l2) E3(a3, l3) m_t(l) X(l)
// for the terms t in [t0, t0 + nt), on output nodes given by the factor matrices
// E1 [m1][L], E2 [m2][L], E3 [m3][Q] (E3 doubled for l3 > 0: the conjugate half).
// Terms with slot[t] < 0 are skipped.
struct FsmTableArgs {
  FsmDims d;
  int m1, m2, m3;
  const double *e1r, *e1i, *e2r, *e2i, *e3r, *e3i;
  int64_t e1_ts, e2_ts, e3_ts;  // per-term strides of the factor arrays (0: one set for all terms)
  const double* mult;
  const int* mrow;      // [T] multiplier row of each term, or null (row t)
  const double* X;
  const int* slot;      // [T]
  const double* scale;  // [T]
  double* out;
  int t0, nt;
};
hipError_t launch_fsm_tables(const FsmTableArgs& a, hipStream_t s);
// whether launch_fsm_tables holds the modes of d and m2 output nodes on axis 2 in LDS
bool fsm_tables_fit(const FsmDims& d, int m2);

// Shifted factor matrices of nt terms on m nodes and nl modes l = lmin .. lmin + nl - 1:
//   e[t][a][k] = w(l) e^{i pi l (base[a] + 2 shift[t]) / P},  w = 1, or (doubled != 0) 2 for l > 0,
// re and im parts in er, ei ([nt][m][nl] each); base[a] are integers (2a + 1 - n for the velocity
// nodes, 2(a - (n - 1)) for the difference grid), shift[t] in grid spacings.
hipError_t launch_fsm_shift_factors(int nt, int m, int nl, int lmin, int doubled, const int* base, const double* shift,
                                    int shift_stride, int P, double* er, double* ei, hipStream_t s);

// One-dimensional band-limited profiles of nt terms on three axes:
//   S[t][k][a] = sum_{j < ng} g[j] D_P(off + a - j + z[t][k])   (ng = 0: D_P(off + a + z[t][k])),
// D_P(w) = (1/P) sum over the non-Nyquist modes l of e^{2 pi i l w / P}; and their products
//   out[t][a0][a1][a2] = w[t] S[t][0][a0] S[t][1][a1] S[t][2][a2].
hipError_t launch_band_profiles(int nt, int m, int off, const double* g, int ng, const double* z, int P, double* S,
                                hipStream_t s);
hipError_t launch_separable(int nt, int m, const double* S, const double* w, double* out, hipStream_t s);
// out[t][i] = s[t] in[src[t]][i], i < len
hipError_t launch_scale_rows(int nt, int64_t len, const double* in, const int* src, const double* sc, double* out,
                             hipStream_t s);

// Executed flops of one cell update (every MFMA issued, padding included)
double fsm_flops_per_cell(const FsmClassDims& d, int slab_l1);

}  // namespace sis
