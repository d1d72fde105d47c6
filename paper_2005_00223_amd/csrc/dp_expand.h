// Piecewise Chebyshev expansions of the embedding nets.
//
// An embedding net maps ONE number, s, to M1 features, so G(s) and dG/ds can
// be laid out once per set of weights as polynomials on a few intervals of
// s, to below the rounding of the precision they are used in.  An interval
// ("piece") [lo, hi] carries K coefficients per feature of
//   G_m(s) = sum_k C[k][m] T_k(x),  dG_m/ds = sum_k C'[k][m] T_k(x),
//   x = (s - mid) ih,  T_k the Chebyshev polynomials.
// The descriptor sum is then linear in what a neighbour contributes:
//   T = (1/Nc) sum_j G(s_j) R_j^T = (1/Nc) sum_pieces C^T H,
//   H[k][c] = sum_{j in piece} T_k(x_j) R_j[c]      (K x 4 per atom),
// and so is the backward,
//   dE/dR_j[c] = sum_k T_k(x_j) M[k][c],    M  = C  dE/dT   (K x 4),
//   dE/ds_j    = sum_k T_k(x_j) (M'[k] . R_j),  M' = C' dE/dT,
// so a pair costs 3 K x 4 products instead of the net's layers, and the
// layers' width enters only once per atom.
//
// Both polynomials are interpolated at the K Chebyshev nodes of the piece
// from the net itself, evaluated with its tangent on the host (in extended
// precision for double, in double for float), with the weights as the
// kernels of the precision hold them.  A piece is halved until its last two
// coefficients are below `tol` of the largest value of the net on it (of
// its slope for C'), so the truncation stays under the arithmetic's own
// rounding.  Pieces cover s in [0, smax]; a net that would need too many
// covers less, and one that covers too little has no expansion (the layer
// kernels evaluate it, as they do a frame with a pair beyond the range).
#pragma once
#include <vector>

#include "dp_internal.h"

namespace dpk {

constexpr int EXP_KP = 16;        // coefficient rows per piece (K <= EXP_KP, zero padded)
constexpr int EXP_K64 = 16;       // coefficients per piece in double
constexpr int EXP_K32 = 12;       // and in float
constexpr int EXP_PMAX = 32;      // pieces per net, at most
constexpr int EXP_BITS = 64;      // (neighbour type, piece) pairs of one centre type: one mask bit each
constexpr double EXP_SMAX = 32.0; // range of s: pairs down to 0.03 A
constexpr double EXP_SMIN = 2.0;  // a net covering less has no expansion
constexpr int EXP_SEG = 12;       // pieces one atom's neighbours may lie in (all types together)

// One net as the host evaluates it: layer l maps in[l] to in[l + 1] features,
// W[l] row-major [in][out]; weights already rounded as the kernels hold them.
struct ExpNetIn {
  int n_layers = 0;
  int w[MAXL + 1] = {0};
  bool lin = false;  // affine last layer
  std::vector<double> W[MAXL], b[MAXL];
};

struct ExpTables {
  bool ok = false;
  int P = 0;           // pieces per net (shorter nets padded with unreachable ones)
  int K = 0, M1p = 0;  // coefficients in use, padded features
  double smax = 0.0;   // pairs beyond it take the layer kernels
  std::vector<double> lo, mid, ih;  // [nets][P]
  std::vector<double> C;            // [nets][P][2][EXP_KP][M1p]: C, then C'
};

// nets: ntypes^2 of them, net (t, u) at t * ntypes + u.  f64: for double kernels
// (K = EXP_K64, interpolated in extended precision to 2^-52), else for float
// (EXP_K32, in double to 2^-25).
ExpTables exp_build(const std::vector<ExpNetIn> &nets, int ntypes, int M1p, bool f64);

// Device tables of one set of nets (Real = double or float).
template <typename Real>
struct ExpTab {
  int P, M1p;
  Real smax;
  const Real *piece;  // [nets][P][4]: lo, mid, ih, -
  const Real *Cf;     // [nets][P][KP][M1p]     forward: features contiguous
  const Real *Cb;     // [nets][P][2][M1p][KP]  backward: C and C', coefficients contiguous
};

template <typename Real>
struct ExpArgs {
  Dims d;
  ExpTab<Real> tab;
  int seg;                    // segments an atom's H / M rows hold
  const int32_t *atom_of_pos; // [rows]
  int64_t rows;
  const double4 *xw;
  double L[3];
  const int32_t *nlist, *nreal;
  uint32_t *flags;            // FLAG_FAR: a pair beyond smax, or more segments than an atom's rows hold
  unsigned long long *mask;   // [natoms] bit u * P + (P - 1 - piece): the atom's segments, in that order
  Real *H;                    // [natoms][seg][EXP_KP][4]
  Real *M;                    // [natoms][seg][2][EXP_KP][4] (the same memory as H)
  Real *T;                    // [natoms][M1][4]
  Real *D;                    // [rows][M1*M2], or NULL (the fitting kernels form it)
  const Real *dD;             // [rows][M1*M2], or NULL: dT holds dE/dT of the unscaled sum
  const Real *dT;             // [natoms][M1][4]
  double *force;              // [natoms][3]
  double *vir_part;           // [grid][9]
  double *net_deriv;          // optional [natoms][nnei][4]
};

template <typename Real>
void launch_exp_fwd(hipStream_t s, const ExpArgs<Real> &a);             // H, T (and D)
template <typename Real>
void launch_exp_bwd(hipStream_t s, const ExpArgs<Real> &a, int grid);   // M, forces, virial parts
int exp_bwd_grid(int64_t rows);

}  // namespace dpk
