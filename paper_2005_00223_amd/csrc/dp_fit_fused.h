// Declarations of the fused FP64 / FP32 fitting-net kernels
// (k_fit_fused.hip).  Not part of the public ABI.
#pragma once
#include "dp_internal.h"

namespace dpk {

template <typename Real>
struct V4;
template <>
struct V4<double> {
  typedef double t __attribute__((ext_vector_type(4)));
};
template <>
struct V4<float> {
  typedef float t __attribute__((ext_vector_type(4)));
};

// four sums over the four lane groups: group g ends with component g
template <typename Real>
__device__ inline Real group_columns(const typename V4<Real>::t &p, int g) {
  const bool b1 = g & 2, b0 = g & 1;
  const Real s0 = (b0 ? p[1] : p[0]) + __shfl_xor(b0 ? p[0] : p[1], 16);
  const Real s1 = (b0 ? p[3] : p[2]) + __shfl_xor(b0 ? p[2] : p[3], 16);
  return (b1 ? s1 : s0) + __shfl_xor(b1 ? s0 : s1, 32);
}

constexpr int FITX_TILES = 16;  // 16-column tiles of a hidden layer, at most

// Element offsets of the weights packed as MFMA A operands, per type and
// layer: forward [chunk of 16 inputs][output tile][lane][4], backward
// [chunk of 16 outputs][input tile][lane][4] (layer 0: [row a of D][chunk]).
// In layer 0 a chunk is one row a of D, its M2 columns padded to 16.
struct FitPack {
  int64_t f[MAXT][MAXF], b[MAXT][MAXF];
  int64_t total;
};

template <typename Real>
struct FitFusedArgs {
  Dims d;
  FitOffsets fo;
  const Real *fwt;            // fitting weights (biases, output layer)
  FitPack pk;
  const Real *pack;           // packed hidden-layer weights
  const int32_t *type_start;  // [ntypes + 1] padded row starts (device)
  const int32_t *atom_of_pos; // [rows]
  int64_t rows;
  int maxw;                   // widest hidden layer
  const Real *T;              // [natoms][M1][4], T / Nc
  Real *Tt[MAXF + 1];         // tanh outputs, per 16 rows [tile][lane][4]
  Real *dT;                   // [natoms][M1][4] dE/dT of the unscaled sum (pass 2)
  double *eatom;              // [natoms] (pass 1)
  // small systems, or NULL: gz of layer 0 [rows][fw[1]] and the sums over rows
  // of D [4][rows][16][4] on their way between the kernels of pass 2
  Real *gz, *low;
};

// Whether the kernels take the model: M1 <= 128, hidden widths multiples of
// 16 up to 256, no doubling skip.
bool fit_fused_supported(const Dims &d);
FitPack fit_pack_layout(const Dims &d);
template <typename Real>
void launch_fit_pack(hipStream_t s, const Dims &d, const FitOffsets &fo, const Real *W, const FitPack &pk, Real *out);
// pass 1: forward and E_i; pass 2: backward to dE/dT; n: atoms with rows
template <typename Real>
void launch_fit_fused(hipStream_t s, const FitFusedArgs<Real> &a, int64_t n, int pass);
// D = T T_<^T of n atoms, in atom order
void launch_form_d(hipStream_t s, int64_t n, int M1, int M2, const double *T, double *D);

}  // namespace dpk
