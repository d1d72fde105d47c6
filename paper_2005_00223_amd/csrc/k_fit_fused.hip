// Fitting net in FP64 / FP32, forward and backward each in one kernel: a
// workgroup takes 16 RT rows (atoms of one type) through every layer.
//
//   forward   D = T T_<^T is formed from T as the first layer's A operand (it
//             never reaches memory), the hidden layers chain through an LDS
//             tile, the tanh outputs are kept for the backward, E_i at the end.
//   backward  dE/dY through the hidden layers, then dE/dD = gz W_0^T one row a
//             of D (16 columns) at a time, contracted at once into
//             dT[a][c] = (sum_b dD[a][b] T[b][c] + [a < M2] sum_a' dD[a'][a] T[a'][c]) / Nc,
//             so dE/dD never reaches memory either.
//
// Before: one GEMM launch per layer, D (1,600 values an atom) written and read
// twice, dE/dD likewise; 32,000 atoms, FP64, 1600-240-240-240: 755 + 900 us,
// and 65 + 315 us more in the descriptor kernels.  These two: 664 + 677 us
// (48 TFLOP/s of the 72 a large FP64 product reaches here); FP32 1,053 ->
// 368 + 333 us.
//
// k_fitx_*: the eight waves of a workgroup split the columns of a layer, so
// each weight is read by one wave only: the weights are packed as MFMA A
// operands (the rows are the N dimension; four k-steps of a lane contiguous,
// k_fit_pack) and go from L2 straight to registers, four chunks of 16 input
// features ahead; the activations come from an LDS tile shared by all.  What
// bounds it is the matrix pipe once RT >= 2; at RT = 1 the loads of the
// weights (4.0 MB of L2 reads per 16 rows in FP64).
//
// k_fitr_bwd: one wave per 16 rows, activations in registers throughout, the
// weights shared by four waves through LDS.  One wave per SIMD (FP64) leaves
// no other to hide its LDS reads (63 % of cycles on the matrix pipe).
#include "dp_fit_fused.h"
#include "dp_f64.h"

namespace dpk {

template <typename Real>
__global__ void k_fit_pack(Dims d, FitOffsets fo, const Real *__restrict__ W, FitPack pk, Real *__restrict__ out) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= pk.total) return;
  int t = 0, l = 0, back = 0;
  for (int tt = 0; tt < d.ntypes; ++tt)
    for (int ll = 0; ll < d.n_fit; ++ll) {
      if (q >= pk.f[tt][ll]) {
        t = tt;
        l = ll;
        back = 0;
      }
    }
  for (int tt = 0; tt < d.ntypes; ++tt)
    for (int ll = 0; ll < d.n_fit; ++ll)
      if (q >= pk.b[tt][ll]) {
        t = tt;
        l = ll;
        back = 1;
      }
  const int in = d.fw[l], o_ = d.fw[l + 1];
  int64_t e = q - (back ? pk.b[t][l] : pk.f[t][l]);
  // a block of 64 lanes x 4 k-steps holds 16 bytes of every lane at a time
  constexpr int V = 16 / sizeof(Real);
  const int lane = (int)(e / V & 63), g = lane >> 4, col = lane & 15;
  const int k4 = MF<Real>::row((int)(e & 255) / (64 * V) * V + (int)(e % V), g);  // the k-step's input of the chunk's 16
  e >>= 8;
  const Real *w = W + fo.w[t][l];
  int i, o;  // weight W[i][o]
  bool in_range = true;
  if (!back) {
    const int nt = o_ / 16, kc = (int)(e / nt), ct = (int)(e % nt), k = k4;
    o = 16 * ct + col;
    if (l == 0) {
      i = kc * d.M2 + k;
      in_range = k < d.M2;
    } else {
      i = 16 * kc + k;
    }
  } else if (l == 0) {
    const int kn = o_ / 16, a = (int)(e / kn), kc = (int)(e % kn);
    i = a * d.M2 + col;
    in_range = col < d.M2;
    o = 16 * kc + k4;
  } else {
    const int nt = in / 16, kc = (int)(e / nt), ct = (int)(e % nt);
    i = 16 * ct + col;
    o = 16 * kc + k4;
  }
  out[q] = in_range ? w[(int64_t)i * o_ + o] : Real(0);
}

bool fit_fused_supported(const Dims &d) {
  if (d.M1 > 128 || d.n_fit < 1) return false;
  for (int l = 1; l <= d.n_fit; ++l) {
    if (d.fw[l] % 16 || d.fw[l] > 16 * FITX_TILES) return false;
    if (l > 1 && d.fw[l] == 2 * d.fw[l - 1]) return false;  // the doubling skip crosses the waves' columns
  }
  return d.fw[1] != d.fw[0] && d.fw[1] != 2 * d.fw[0];
}

FitPack fit_pack_layout(const Dims &d) {
  FitPack p{};
  int64_t at = 0;
  for (int back = 0; back < 2; ++back)
    for (int t = 0; t < d.ntypes; ++t)
      for (int l = 0; l < d.n_fit; ++l) {
        (back ? p.b : p.f)[t][l] = at;
        at += (int64_t)(l == 0 ? d.M1 * 16 : d.fw[l]) * d.fw[l + 1];
      }
  p.total = at;
  return p;
}

template <typename Real>
void launch_fit_pack(hipStream_t s, const Dims &d, const FitOffsets &fo, const Real *W, const FitPack &pk, Real *out) {
  hipLaunchKernelGGL(k_fit_pack<Real>, dim3((unsigned)((pk.total + 255) / 256)), dim3(256), 0, s, d, fo, W, pk, out);
}
template void launch_fit_pack<double>(hipStream_t, const Dims &, const FitOffsets &, const double *, const FitPack &,
                                      double *);
template void launch_fit_pack<float>(hipStream_t, const Dims &, const FitOffsets &, const float *, const FitPack &,
                                     float *);

// a lane's four k-steps of a packed block (64 lanes, 16 bytes of each at a time)
__device__ inline V4<double>::t wblock(const double *b, int lane) {
  typedef double v2 __attribute__((ext_vector_type(2)));
  const v2 lo = *(const v2 *)(b + 2 * lane), hi = *(const v2 *)(b + 128 + 2 * lane);
  return V4<double>::t{lo[0], lo[1], hi[0], hi[1]};
}
__device__ inline V4<float>::t wblock(const float *b, int lane) { return *(const V4<float>::t *)(b + 4 * lane); }

// the block's type and first row (type blocks start at multiples of ROW_TILE)
template <typename Real>
__device__ inline bool fit_block(const FitFusedArgs<Real> &a, int R, int &t, int64_t &r0, int64_t &r1) {
  int64_t b = blockIdx.x;
  for (t = 0; t < a.d.ntypes; ++t) {
    const int64_t s = a.type_start[t], e = a.type_start[t + 1], nb = (e - s + R - 1) / R;
    if (b < nb) {
      r0 = s + b * R;
      r1 = e;
      return true;
    }
    b -= nb;
  }
  return false;
}

constexpr int FX_PD = 4;       // chunks of weights in flight per wave
constexpr int NW = 8, CT = 2;  // waves, and column tiles of each (sixteen waves of one: 2 % slower)
static_assert(NW * CT >= FITX_TILES, "every column tile has a wave");

// acc = (LDS tile) x (packed weights): nk chunks of 16 input features; xr = the tile's row lane % 16, XS its row
// stride
template <typename Real, int RT>
__device__ inline void fitx_layer(const Real *__restrict__ W, int nk, int nt, const int (&ct)[CT], const Real *xr,
                                  int XS, int lane, typename MF<Real>::acc (&acc)[RT][CT]) {
  const int g = lane >> 4;
  typedef typename V4<Real>::t v4;
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int c = 0; c < CT; ++c) acc[r][c] = typename MF<Real>::acc{0, 0, 0, 0};
  v4 w[FX_PD][CT];
  auto wload = [&](int kc, v4(&q)[CT]) {
#pragma unroll
    for (int c = 0; c < CT; ++c) q[c] = wblock(W + ((int64_t)(kc < nk ? kc : nk - 1) * nt + ct[c]) * 256, lane);
  };
#pragma unroll
  for (int k = 0; k < FX_PD; ++k) wload(k, w[k]);
  for (int kc = 0; kc < nk; kc += FX_PD) {
#pragma unroll
    for (int k = 0; k < FX_PD; ++k) {
      if (kc + k >= nk) continue;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        Real x[RT];
#pragma unroll
        for (int r = 0; r < RT; ++r) x[r] = xr[16 * r * XS + 16 * (kc + k) + MF<Real>::row(j, g)];
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
          for (int c = 0; c < CT; ++c) acc[r][c] = MF<Real>::mma(w[k][c][j], x[r], acc[r][c]);
      }
      wload(kc + k + FX_PD, w[k]);
    }
  }
}

// ---------------------------------------------------------------------------
// forward
// ---------------------------------------------------------------------------
template <typename Real, int RT, int W>
struct FwdShape {
  static constexpr int R = 16 * RT;
  static constexpr int AG = 64 * W / (4 * R);             // rows of D formed at a time
  static constexpr int AS = AG < FX_PD ? FX_PD : AG;      // rows of D per stage
  static constexpr int DS = 16 * AS + 1;                  // row stride of the staged D
  static size_t lds(int maxw) {
    const size_t x = (size_t)R * (maxw + 1), s = (size_t)2 * R * DS;
    return sizeof(Real) * (x > s ? x : s);
  }
};

// layer 0 of the workgroup's rows for the wave's C column tiles: K = (a, b), D
// formed by the W waves in LDS stages of AS rows a (at X)
template <typename Real, int RT, int W, int C>
__device__ inline void fitx_first(const FitFusedArgs<Real> &a, int t, int64_t r0, int64_t r1, const int (&ct)[C], Real *X,
                                  int tid, typename MF<Real>::acc (&acc)[RT][C]) {
  typedef FwdShape<Real, RT, W> S;
  typedef typename MF<Real>::acc acc_t;
  typedef typename V4<Real>::t v4;
  constexpr int R = S::R, AS = S::AS, DS = S::DS;
  static_assert(AS % S::AG == 0 && AS % FX_PD == 0, "stages of whole row groups and weight rings");
  const Dims &d = a.d;
  const int lane = tid & 63, g = lane >> 4, col = lane & 15, M1 = d.M1, M2 = d.M2;
  const int row = (tid >> 2) % R, bq = tid & 3, ag = (tid >> 2) / R;
  const bool maker = ag < S::AG;
  const int at = r0 + row < r1 ? a.atom_of_pos[r0 + row] : -1;
  const Real *Ti = a.T + (int64_t)(at < 0 ? 0 : at) * M1 * 4;
  v4 tb[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int b = 4 * bq + k;
    const v4 v = *(const v4 *)(Ti + (b < M2 ? b : 0) * 4);
    tb[k] = at >= 0 && b < M2 ? v : v4{0, 0, 0, 0};
  }
  const int nt = d.fw[1] / 16;
  const Real *Wp = a.pack + a.pk.f[t][0];
  auto wload = [&](int k, v4(&w)[C]) {
    const int kc = k < M1 ? k : M1 - 1;
#pragma unroll
    for (int c = 0; c < C; ++c) w[c] = wblock(Wp + ((int64_t)kc * nt + ct[c]) * 256, lane);
  };
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int c = 0; c < C; ++c) acc[r][c] = acc_t{0, 0, 0, 0};
  constexpr int NG = AS / S::AG;  // rows of D a maker forms per stage
  v4 ta[NG];
  auto tload = [&](int st) {
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      const int k = st * AS + q * S::AG + ag;
      const v4 v = *(const v4 *)(Ti + (k < M1 ? k : 0) * 4);
      ta[q] = k < M1 ? v : v4{0, 0, 0, 0};
    }
  };
  auto form = [&](Real *Ds) {
    if (maker)
#pragma unroll
      for (int q = 0; q < NG; ++q)
#pragma unroll
        for (int k = 0; k < 4; ++k)
          Ds[row * DS + 16 * (q * S::AG + ag) + 4 * bq + k] =
              ta[q][0] * tb[k][0] + ta[q][1] * tb[k][1] + ta[q][2] * tb[k][2] + ta[q][3] * tb[k][3];
  };
  const int nst = (M1 + AS - 1) / AS;
  v4 w[FX_PD][C];
  tload(0);
#pragma unroll
  for (int k = 0; k < FX_PD; ++k) wload(k, w[k]);
  form(X);
  __syncthreads();
  for (int st = 0; st < nst; ++st) {
    const Real *Ds = X + (st & 1) * R * DS;
    if (st + 1 < nst) tload(st + 1);
#pragma unroll
    for (int al = 0; al < AS; ++al) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        Real x[RT];
#pragma unroll
        for (int r = 0; r < RT; ++r) x[r] = Ds[(16 * r + col) * DS + 16 * al + MF<Real>::row(j, g)];
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
          for (int c = 0; c < C; ++c) acc[r][c] = MF<Real>::mma(w[al % FX_PD][c][j], x[r], acc[r][c]);
      }
      wload(st * AS + al + FX_PD, w[al % FX_PD]);
    }
    if (st + 1 < nst) form(X + ((st + 1) & 1) * R * DS);
    __syncthreads();
  }
}

// FIRST = false: layer 0 has been evaluated by k_fitx_l0
template <typename Real, int RT, bool FIRST>
__global__ void __launch_bounds__(64 * NW, 1) k_fitx_fwd(FitFusedArgs<Real> a) {
  typedef typename MF<Real>::acc acc_t;
  typedef typename V4<Real>::t v4;
  constexpr int R = 16 * RT;
  extern __shared__ __align__(16) unsigned char fitx_smem[];
  __shared__ Real es[NW][R];
  Real *X = (Real *)fitx_smem;
  const Dims &d = a.d;
  int t;
  int64_t r0, r1;
  if (!fit_block(a, R, t, r0, r1) || a.atom_of_pos[r0] < 0) return;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, g = lane >> 4, col = lane & 15;
  acc_t acc[RT][CT];
  if constexpr (FIRST) {
    const int nt = d.fw[1] / 16;
    int ct[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) ct[c] = wv * CT + c < nt ? wv * CT + c : nt - 1;
    fitx_first<Real, RT, NW, CT>(a, t, r0, r1, ct, X, tid, acc);
  }
  // ---- epilogues and hidden layers ----
  const int XS = a.maxw + 1;
  for (int l = 0; l < d.n_fit; ++l) {
    const int out = d.fw[l + 1], nt = out / 16;
    const Real *bias = a.fwt + a.fo.b[t][l];
    const bool last = l + 1 == d.n_fit;
    const Real *wo = a.fwt + a.fo.w[t][d.n_fit];
    Real *Tt = a.Tt[l + 1];
    Real ep[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) ep[r] = 0;
    const bool skip = l > 0 && out == d.fw[l];
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      const int ct = wv * CT + c;
      if (ct >= nt) continue;
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        v4 th, *const tp = (v4 *)(Tt + (((r0 >> 4) + r) * nt + ct) * 256 + lane * 4);
        const bool done = !FIRST && l == 0;
        if (done) th = *tp;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int o = 16 * ct + MF<Real>::row(q, g);
          if (!done) th[q] = MF<Real>::tanh_(acc[r][c][q] + bias[o]);
          Real y = th[q];
          if (skip) y += X[(16 * r + col) * XS + o];
          acc[r][c][q] = y;
          if (last) ep[r] += y * wo[o];
        }
        if (!done && r0 + 16 * r < r1) *tp = th;
      }
    }
    if (last) {
      // E_i: the lane groups of a row, then the waves, in order
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        Real e = ep[r];
        e += __shfl_xor(e, 16);
        e += __shfl_xor(e, 32);
        if (g == 0) es[wv][16 * r + col] = e;
      }
      __syncthreads();
      if (tid < R && r0 + tid < r1) {
        const int at = a.atom_of_pos[r0 + tid];
        Real e = 0;
        for (int w = 0; w < NW; ++w) e += es[w][tid];
        if (at >= 0) a.eatom[at] = (double)(e + a.fwt[a.fo.b[t][d.n_fit]]);
      }
      return;
    }
    __syncthreads();  // the tile's readers are done
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      const int ct = wv * CT + c;
      if (ct >= nt) continue;
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int q = 0; q < 4; ++q) X[(16 * r + col) * XS + 16 * ct + MF<Real>::row(q, g)] = acc[r][c][q];
    }
    __syncthreads();
    const int nk = out / 16, nn = d.fw[l + 2] / 16;
    const Real *W = a.pack + a.pk.f[t][l + 1];
    int ctn[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) ctn[c] = wv * CT + c < nn ? wv * CT + c : nn - 1;
    fitx_layer<Real, RT>(W, nk, nn, ctn, X + col * XS, XS, lane, acc);
  }
}

// Layer 0 alone, four column tiles a workgroup (blockIdx.y: which), for
// systems of so few rows that one workgroup per 16 rows leaves most CUs idle.
constexpr int FS_W = 4;
template <typename Real>
__global__ void __launch_bounds__(64 * FS_W, 1) k_fitx_l0(FitFusedArgs<Real> a) {
  typedef FwdShape<Real, 1, FS_W> S;
  typedef typename V4<Real>::t v4;
  __shared__ __align__(16) Real X[2 * S::R * S::DS];
  int t;
  int64_t r0, r1;
  if (!fit_block(a, S::R, t, r0, r1) || a.atom_of_pos[r0] < 0) return;
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, nt = a.d.fw[1] / 16, tile = blockIdx.y * FS_W + (tid >> 6);
  const int ct[1] = {tile < nt ? tile : nt - 1};
  typename MF<Real>::acc acc[1][1];
  fitx_first<Real, 1, FS_W, 1>(a, t, r0, r1, ct, X, tid, acc);
  if (tile >= nt) return;
  const Real *bias = a.fwt + a.fo.b[t][0];
  v4 th;
#pragma unroll
  for (int q = 0; q < 4; ++q) th[q] = MF<Real>::tanh_(acc[0][0][q] + bias[16 * tile + MF<Real>::row(q, g)]);
  *(v4 *)(a.Tt[1] + ((r0 >> 4) * nt + tile) * 256 + lane * 4) = th;
}

// ---------------------------------------------------------------------------
// backward
// ---------------------------------------------------------------------------
// dE/dD, one row a of D at a time (this wave: a = a0, a0 + step, ..): lane (g, n)
// gets b = row(q, g) of row n.  X: gz of layer 0, row stride XS; Tl: T_<, at the
// end the sums over the workgroup's rows a of dD[a][b] T[a].
template <typename Real, int RT, int W>
__device__ inline void fitx_last(const FitFusedArgs<Real> &a, int t, int64_t r0, int64_t r1, const Real *X, int XS, Real *Tl,
                                 int a0, int step, int tid) {
  typedef typename MF<Real>::acc acc_t;
  typedef typename V4<Real>::t v4;
  const Dims &d = a.d;
  const int lane = tid & 63, wv = tid >> 6, g = lane >> 4, col = lane & 15, M1 = d.M1;
  int at[RT];
#pragma unroll
  for (int r = 0; r < RT; ++r) at[r] = r0 + 16 * r + col < r1 ? a.atom_of_pos[r0 + 16 * r + col] : -1;
  const int nk = d.fw[1] / 16;
  const Real *W0 = a.pack + a.pk.b[t][0];
  const Real *xr = X + col * XS;
  const Real sc = (Real)d.inv_nc;
  v4 low[RT][4];  // sum over this wave's a of dD[a][b = row(q, g)] T[a]
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int q = 0; q < 4; ++q) low[r][q] = v4{0, 0, 0, 0};
  // the wave's weights are one stream over (a, chunk): FX_PD of them in flight
  v4 w[FX_PD];
  int wa = a0, wk = 0;
  auto wload = [&](v4 &q) {
    q = wblock(W0 + ((int64_t)(wa < M1 ? wa : M1 - 1) * nk + wk) * 256, lane);
    if (++wk == nk) {
      wk = 0;
      wa += step;
    }
  };
#pragma unroll
  for (int k = 0; k < FX_PD; ++k) wload(w[k]);
  for (int ar = a0; ar < M1; ar += step) {
    acc_t z[RT], z2[RT];
    v4 ta[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      z[r] = z2[r] = acc_t{0, 0, 0, 0};
      ta[r] = *(const v4 *)(a.T + ((int64_t)(at[r] < 0 ? 0 : at[r]) * M1 + ar) * 4);
    }
    for (int kc = 0; kc < nk; ++kc) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int r = 0; r < RT; ++r) {
          acc_t &zj = j & 1 ? z2[r] : z[r];
          zj = MF<Real>::mma(w[0][j], xr[16 * r * XS + 16 * kc + MF<Real>::row(j, g)], zj);
        }
#pragma unroll
      for (int k = 0; k + 1 < FX_PD; ++k) w[k] = w[k + 1];
      wload(w[FX_PD - 1]);
    }
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      z[r] += z2[r];
      v4 p = {0, 0, 0, 0};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        p += z[r][q] * *(const v4 *)(Tl + ((16 * r + col) * 16 + MF<Real>::row(q, g)) * 4);
        low[r][q] += z[r][q] * ta[r];
      }
      const Real v = group_columns<Real>(p, g);
      if (at[r] >= 0) a.dT[((int64_t)at[r] * M1 + ar) * 4 + g] = v * sc;
    }
  }
  // the sums over a of the waves, in order, into the LDS area of T_<
  __syncthreads();
  for (int wi = 0; wi < W; ++wi) {
    if (wi == wv)
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          v4 *o = (v4 *)(Tl + ((16 * r + col) * 16 + MF<Real>::row(q, g)) * 4);
          *o = wi == 0 ? low[r][q] : *o + low[r][q];
        }
    __syncthreads();
  }
}

// LAST = false: leaves gz of layer 0 in a.gz for k_fitx_d0
template <typename Real, int RT, bool LAST>
__global__ void __launch_bounds__(64 * NW, 1) k_fitx_bwd(FitFusedArgs<Real> a) {
  typedef typename MF<Real>::acc acc_t;
  typedef typename V4<Real>::t v4;
  constexpr int R = 16 * RT;
  extern __shared__ __align__(16) unsigned char fitx_smem[];
  const Dims &d = a.d;
  int t;
  int64_t r0, r1;
  if (!fit_block(a, R, t, r0, r1) || a.atom_of_pos[r0] < 0) return;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, g = lane >> 4, col = lane & 15;
  const int M1 = d.M1, M2 = d.M2, XS = a.maxw + 1;
  Real *X = (Real *)fitx_smem;   // [R][XS] gz
  Real *Tl = X + R * XS;         // [R][16][4] T_<, later the sums over the rows of D
  for (int o = tid; o < R * 16; o += 64 * NW) {
    const int row = o >> 4, b = o & 15;
    const int at = r0 + row < r1 ? a.atom_of_pos[r0 + row] : -1;
    v4 v = *(const v4 *)(a.T + ((int64_t)(at < 0 ? 0 : at) * M1 + (b < M2 ? b : 0)) * 4);
    if (at < 0 || b >= M2) v = v4{0, 0, 0, 0};
    *(v4 *)(Tl + o * 4) = v;
  }
  acc_t gy[RT][CT];  // dE/dY of the layer above, then of this one
  {
    const Real *wo = a.fwt + a.fo.w[t][d.n_fit];
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      const int ct = wv * CT + c;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int o = 16 * ct + MF<Real>::row(q, g);
        const Real w = o < d.fw[d.n_fit] ? wo[o] : Real(0);
#pragma unroll
        for (int r = 0; r < RT; ++r) gy[r][c][q] = w;
      }
    }
  }
  for (int l = d.n_fit - 1; l >= 0; --l) {
    // gz = gy (1 - t^2) into the tile
    const int out = d.fw[l + 1], nt = out / 16;
    const Real *Tt = a.Tt[l + 1];
    if (l < d.n_fit - 1) __syncthreads();
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      const int ct = wv * CT + c;
      if (ct >= nt) continue;
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        const int64_t rt = (r0 >> 4) + (r0 + 16 * r < r1 ? r : 0);
        const v4 th = *(const v4 *)(Tt + (rt * nt + ct) * 256 + lane * 4);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int o = 16 * ct + MF<Real>::row(q, g);
          const Real gz = gy[r][c][q] * (Real(1) - th[q] * th[q]);
          if (!LAST && l == 0) a.gz[(r0 + 16 * r + col) * out + o] = gz;
          else X[(16 * r + col) * XS + o] = gz;
        }
      }
    }
    __syncthreads();
    if (l == 0) break;
    const int nn = d.fw[l] / 16;
    const Real *W = a.pack + a.pk.b[t][l];
    int ctn[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) ctn[c] = wv * CT + c < nn ? wv * CT + c : nn - 1;
    acc_t acc[RT][CT];
    fitx_layer<Real, RT>(W, nt, nn, ctn, X + col * XS, XS, lane, acc);
    const bool skip = out == d.fw[l];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int q = 0; q < 4; ++q) gy[r][c][q] = skip ? acc[r][c][q] + gy[r][c][q] : acc[r][c][q];
  }
  if constexpr (!LAST) return;
  fitx_last<Real, RT, NW>(a, t, r0, r1, X, XS, Tl, wv, NW, tid);
  const Real sc = (Real)d.inv_nc;
  for (int o = tid; o < R * M2; o += 64 * NW) {
    const int row = o / M2, b = o % M2;
    const int i = r0 + row < r1 ? a.atom_of_pos[r0 + row] : -1;
    if (i < 0) continue;
    v4 *dt = (v4 *)(a.dT + ((int64_t)i * M1 + b) * 4);
    *dt = *dt + *(const v4 *)(Tl + (row * 16 + b) * 4) * sc;
  }
}

// dE/dT from gz of layer 0, the rows a of D dealt to gridDim.y workgroups of
// 16 rows; their sums over a go to a.low and are added by k_fitx_low.
template <typename Real>
__global__ void __launch_bounds__(64 * FS_W, 1) k_fitx_d0(FitFusedArgs<Real> a) {
  typedef typename V4<Real>::t v4;
  __shared__ __align__(16) Real X[16 * (16 * FITX_TILES + 1)];
  __shared__ __align__(32) Real Tl[16 * 16 * 4];
  const Dims &d = a.d;
  int t;
  int64_t r0, r1;
  if (!fit_block(a, 16, t, r0, r1) || a.atom_of_pos[r0] < 0) return;
  const int tid = threadIdx.x, w1 = d.fw[1], M1 = d.M1, M2 = d.M2, XS = w1 + 1;
  for (int o = tid; o < 16 * w1; o += 64 * FS_W) X[o / w1 * XS + o % w1] = a.gz[(r0 + o / w1) * w1 + o % w1];
  for (int o = tid; o < 16 * 16; o += 64 * FS_W) {
    const int b = o & 15, at = a.atom_of_pos[r0 + (o >> 4)];
    v4 v = *(const v4 *)(a.T + ((int64_t)(at < 0 ? 0 : at) * M1 + (b < M2 ? b : 0)) * 4);
    if (at < 0 || b >= M2) v = v4{0, 0, 0, 0};
    *(v4 *)(Tl + o * 4) = v;
  }
  __syncthreads();
  fitx_last<Real, 1, FS_W>(a, t, r0, r1, X, XS, Tl, blockIdx.y * FS_W + (tid >> 6), FS_W * gridDim.y, tid);
  for (int o = tid; o < 16 * 16; o += 64 * FS_W)
    *(v4 *)(a.low + ((int64_t)blockIdx.y * a.rows + r0) * 64 + o * 4) = *(const v4 *)(Tl + o * 4);
}

// dE/dT of the first M2 rows += the workgroups' sums, in order
template <typename Real>
__global__ void k_fitx_low(FitFusedArgs<Real> a, int ny) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, row = q >> 6;
  const int b = (int)(q >> 2) & 15;
  if (row >= a.rows || row >= a.type_start[a.d.ntypes] || b >= a.d.M2) return;
  const int i = a.atom_of_pos[row];
  if (i < 0) return;
  Real v = 0;
  for (int y = 0; y < ny; ++y) v += a.low[(int64_t)y * a.rows * 64 + q];
  a.dT[((int64_t)i * a.d.M1 + b) * 4 + (q & 3)] += v * (Real)a.d.inv_nc;
}

template <typename Real, int RT, bool ALL = true>
static void launch_fitx(hipStream_t s, const FitFusedArgs<Real> &a, int pass) {
  constexpr int R = 16 * RT;
  const unsigned grid = (unsigned)(a.rows / R + 2 * a.d.ntypes);
  if (pass == 1) {
    const size_t lds = FwdShape<Real, RT, NW>::lds(a.maxw);
    (void)hipFuncSetAttribute((const void *)k_fitx_fwd<Real, RT, ALL>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)lds);
    hipLaunchKernelGGL((k_fitx_fwd<Real, RT, ALL>), dim3(grid), dim3(64 * NW), lds, s, a);
  } else if constexpr (RT <= 2) {
    const size_t lds = sizeof(Real) * ((size_t)R * (a.maxw + 1) + (size_t)R * 64);
    (void)hipFuncSetAttribute((const void *)k_fitx_bwd<Real, RT, ALL>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)lds);
    hipLaunchKernelGGL((k_fitx_bwd<Real, RT, ALL>), dim3(grid), dim3(64 * NW), lds, s, a);
  }
}

// 16 rows at a time with the wide layer 0 spread over FS_Y workgroups each
constexpr int FS_Y = 4;
template <typename Real>
static void launch_fitx_spread(hipStream_t s, const FitFusedArgs<Real> &a, int pass) {
  const unsigned gx = (unsigned)(a.rows / 16 + 2 * a.d.ntypes);
  if (pass == 1) {
    hipLaunchKernelGGL(k_fitx_l0<Real>, dim3(gx, (unsigned)(a.d.fw[1] / 16 + FS_W - 1) / FS_W), dim3(64 * FS_W), 0, s, a);
    launch_fitx<Real, 1, false>(s, a, pass);
  } else {
    launch_fitx<Real, 1, false>(s, a, pass);
    hipLaunchKernelGGL(k_fitx_d0<Real>, dim3(gx, FS_Y), dim3(64 * FS_W), 0, s, a);
    hipLaunchKernelGGL(k_fitx_low<Real>, dim3((unsigned)((a.rows * 64 + 255) / 256)), dim3(256), 0, s, a, FS_Y);
  }
}

// ---------------------------------------------------------------------------
// backward of large systems: one wave per 16 rows.  With the rows as the MFMA
// N dimension an output tile's registers are the next layer's B operands
// (k-step r of chunk mt takes register r of tile mt), so activations never
// leave registers.  The four waves of a workgroup share the weights through
// LDS, one chunk of 16 inputs per stage, loaded two stages ahead.
// ---------------------------------------------------------------------------
constexpr int FR_NT = 15;                   // output tiles: hidden width 240
constexpr int FR_WAVES = 4, FR_ROWS = 16 * FR_WAVES;
template <typename Real>
constexpr int fr_chunk() { return FR_NT * 64 * 4 * (int)sizeof(Real); }  // bytes of a stage: a chunk of 16 inputs

// One stage on its way from L2 to LDS through registers: load() while the
// stage before it is in use, store() after that (a direct global-to-LDS copy
// was waited for at the next LDS read, whichever buffer it went to).
template <typename Real>
struct FrStage {
  typedef uint32_t u4 __attribute__((ext_vector_type(4)));
  static constexpr int BLK = fr_chunk<Real>() / 1024;        // 1 KB blocks
  static constexpr int N = (BLK + FR_WAVES - 1) / FR_WAVES;  // per wave
  u4 r[N];
  // chunk k of nk (blocks past the last reread it)
  __device__ void load(const Real *__restrict__ W, int k, int nk, int wv, int lane) {
    const int last = nk * BLK - 1;
    const unsigned char *src = (const unsigned char *)W;
#pragma unroll
    for (int q = 0; q < N; ++q) {
      const int b = k * BLK + q * FR_WAVES + wv;
      r[q] = *(const u4 *)(src + (size_t)(b < last ? b : last) * 1024 + 16u * (unsigned)lane);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  __device__ void store(unsigned char *buf, int wv, int lane) const {
#pragma unroll
    for (int q = 0; q < N; ++q) {
      const int b = q * FR_WAVES + wv;
      if (b < BLK) *(u4 *)(buf + b * 1024 + 16 * lane) = r[q];
    }
  }
};

// The operands of a stage's products are read GR blocks at a time, while the
// GR before them are multiplied; the first of the next stage at the end of
// this one (its LDS buffer is one barrier old), so the matrix cores do not
// wait for LDS behind a barrier.
template <typename Real>
struct FrOps {
  typedef typename V4<Real>::t v4;
  static constexpr int GR = sizeof(Real) == 8 ? 3 : 5, NG = FR_NT / GR;
  static_assert(NG & 1, "a stage's last group leaves the next one's first in slot 1");
  v4 w[2][GR];
  // blocks of group q of the stage at buf, into slot
  __device__ void read(const unsigned char *buf, int q, int slot, int lane) {
#pragma unroll
    for (int c = 0; c < GR; ++c) w[slot][c] = wblock((const Real *)buf + (q * GR + c) * 256, lane);
  }
  // group q of the stage at buf is in slot q % 2: read the one after it
  __device__ void ahead(const unsigned char *buf, const unsigned char *next, int q, int lane) {
    if (q + 1 < NG) read(buf, q + 1, (q + 1) & 1, lane);
    else if (next) read(next, 0, (q + 1) & 1, lane);
    __builtin_amdgcn_sched_barrier(0);
  }
  __device__ void wrap() {
#pragma unroll
    for (int c = 0; c < GR; ++c) w[0][c] = w[1][c];
  }
};

// A layer's first two stages into the buffers, and the first group of
// operands.  The buffers' last readers are behind a barrier.
template <typename Real>
__device__ inline void fr_begin(FrStage<Real> &st, FrOps<Real> &o, const Real *__restrict__ W, int nk,
                                unsigned char *smem, int wv, int lane) {
  st.store(smem, wv, lane);
  st.load(W, 1, nk, wv, lane);
  st.store(smem + fr_chunk<Real>(), wv, lane);
  __syncthreads();
  o.read(smem, 0, 0, lane);
}

// acc += W y, y in the layer's register layout; st holds its first stage
template <typename Real>
__device__ inline void fr_layer(FrStage<Real> &st, const Real *__restrict__ W, unsigned char *smem, int wv, int lane,
                                const typename MF<Real>::acc (&y)[FR_NT], typename MF<Real>::acc (&acc)[FR_NT]) {
  constexpr int SB = fr_chunk<Real>(), GR = FrOps<Real>::GR, NG = FrOps<Real>::NG;
  FrOps<Real> o;
  fr_begin(st, o, W, FR_NT, smem, wv, lane);
#pragma unroll
  for (int k = 0; k < FR_NT; ++k) {
    if (k + 2 < FR_NT) st.load(W, k + 2, FR_NT, wv, lane);
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      o.ahead(smem + k % 3 * SB, k + 1 < FR_NT ? smem + (k + 1) % 3 * SB : nullptr, q, lane);
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int c = 0; c < GR; ++c)
          acc[q * GR + c] = MF<Real>::mma(o.w[q & 1][c][j], y[k][j], acc[q * GR + c]);
      __builtin_amdgcn_sched_barrier(0);
    }
    o.wrap();
    if (k + 2 < FR_NT) st.store(smem + (k + 2) % 3 * SB, wv, lane);
    __syncthreads();
  }
}

template <typename Real>
__global__ void __launch_bounds__(64 * FR_WAVES, sizeof(Real) == 8 ? 1 : 2) k_fitr_bwd(FitFusedArgs<Real> a) {
  typedef typename MF<Real>::acc acc_t;
  typedef typename V4<Real>::t v4;
  extern __shared__ __align__(16) unsigned char fitx_smem[];
  constexpr int SB = fr_chunk<Real>(), GR = FrOps<Real>::GR, NG = FrOps<Real>::NG;  // three stages of SB bytes
  FrStage<Real> st;
  const Dims &d = a.d;
  int t;
  int64_t r0, r1;
  if (!fit_block(a, FR_ROWS, t, r0, r1) || a.atom_of_pos[r0] < 0) return;
  const int lane = threadIdx.x & 63, g = lane >> 4, col = lane & 15;
  // uniform over the wave: weight addresses stay in scalar registers
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int M1 = d.M1, M2 = d.M2;
  r0 += 16 * wv;
  const int at = a.atom_of_pos[r0 + col];
  const Real *Ti = a.T + (int64_t)(at < 0 ? 0 : at) * M1 * 4;
  acc_t gy[FR_NT], gz[FR_NT];
  {
    const Real *wo = a.fwt + a.fo.w[t][d.n_fit];
#pragma unroll
    for (int c = 0; c < FR_NT; ++c)
#pragma unroll
      for (int q = 0; q < 4; ++q) gy[c][q] = wo[16 * c + MF<Real>::row(q, g)];
  }
  for (int l = d.n_fit - 1; l >= 0; --l) {
    st.load(a.pack + a.pk.b[t][l], 0, l > 0 ? FR_NT : M1, wv, lane);
    const Real *Tt = a.Tt[l + 1] + (r0 >> 4) * FR_NT * 256 + lane * 4;
#pragma unroll
    for (int c = 0; c < FR_NT; ++c) {
      const v4 th = *(const v4 *)(Tt + c * 256);
#pragma unroll
      for (int q = 0; q < 4; ++q) gz[c][q] = gy[c][q] * (Real(1) - th[q] * th[q]);
    }
    if (l == 0) break;
    // the skip's share stays in the accumulators
    fr_layer<Real>(st, a.pack + a.pk.b[t][l], fitx_smem, wv, lane, gz, gy);
  }
  // dE/dD, one row a of D at a time: lane (g, n) gets b = row(r, g) of row n
  v4 tb[4], low[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int b = MF<Real>::row(j, g);
    const v4 v = *(const v4 *)(Ti + (b < M2 ? b : 0) * 4);
    tb[j] = b < M2 ? v : v4{0, 0, 0, 0};
    low[j] = v4{0, 0, 0, 0};
  }
  const Real *W = a.pack + a.pk.b[t][0];
  const Real sc = (Real)d.inv_nc;
  v4 tn = *(const v4 *)Ti;
  FrOps<Real> o;
  fr_begin(st, o, W, M1, fitx_smem, wv, lane);
  unsigned char *cur = fitx_smem, *nxt = fitx_smem + SB, *third = fitx_smem + 2 * SB;
  for (int k = 0; k < M1; ++k) {
    const v4 ta = tn;
    tn = *(const v4 *)(Ti + (k + 1 < M1 ? k + 1 : 0) * 4);
    st.load(W, k + 2, M1, wv, lane);
    acc_t z[4];  // partial sums of the row of dE/dD
#pragma unroll
    for (int j = 0; j < 4; ++j) z[j] = acc_t{0, 0, 0, 0};
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      o.ahead(cur, nxt, q, lane);
#pragma unroll
      for (int c = 0; c < GR; ++c)
#pragma unroll
        for (int j = 0; j < 4; ++j) z[j] = MF<Real>::mma(o.w[q & 1][c][j], gz[q * GR + c][j], z[j]);
      __builtin_amdgcn_sched_barrier(0);
    }
    o.wrap();
    st.store(third, wv, lane);
    v4 p = {0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const Real v = (z[0][j] + z[1][j]) + (z[2][j] + z[3][j]);
      p += v * tb[j];
      low[j] += v * ta;
    }
    const Real v = group_columns<Real>(p, g);
    if (at >= 0) a.dT[((int64_t)at * M1 + k) * 4 + g] = v * sc;
    __syncthreads();
    unsigned char *const c0 = cur;
    cur = nxt;
    nxt = third;
    third = c0;
  }
  // + the sums over a, onto rows this wave has written
  __threadfence_block();
  if (at >= 0)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int b = MF<Real>::row(j, g);
      if (b < M2) {
        v4 *o = (v4 *)(a.dT + ((int64_t)at * M1 + b) * 4);
        *o = *o + low[j] * sc;
      }
    }
}

template <typename Real>
static void launch_fitr_bwd(hipStream_t s, const FitFusedArgs<Real> &a) {
  const int lds = 3 * fr_chunk<Real>();
  (void)hipFuncSetAttribute((const void *)k_fitr_bwd<Real>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  hipLaunchKernelGGL(k_fitr_bwd<Real>, dim3((unsigned)(a.rows / FR_ROWS)), dim3(64 * FR_WAVES), lds, s, a);
}

// Atoms up to which layer 0 is spread: one workgroup per 16 rows leaves CUs
// idle (us, forward + backward, as one kernel each | spread: FP64 192 atoms
// 94 + 106 | 61 + 74, 1,367 97 + 110 | 79 + 85, 2,048 101 + 113 | 92 + 102,
// 3,000 103 + 116 | 112 + 107; FP32 192 56 + 64 | 40 + 47, 2,048 60 + 70 |
// 60 + 70).
constexpr int64_t FIT_SPREAD = 2048;

// Time of a launch whose workgroups take R atoms each: the rounds that 256
// CUs need for them, times a round's time (us, 1600-240-240-240).
static int64_t fit_rounds(int64_t n, int R) { return (n + 256 * R - 1) / (256 * R); }

// The variant is the one with the least (rounds x time of a round); more rows
// a workgroup read fewer weights a row, but a round is longer, and a launch
// lasts whole rounds.  Measured (us, RT = 1 | 2 | 4 or the row-wave backward):
//   atoms           500         6,144        12,288       24,576        32,768
//   FP64 forward  95 161 298  199 176 308  304 340 323  604 533 646  809 718 671
//   FP64 backward 108 165 318 222 183 325  342 351 338  674 549 664  896 738 690
//   FP32 forward  57 94 168   110 106 181  169 182 188  325 287 374  429 373 386
//   FP32 backward 65 101 167  120 114 175  189 221 184  368 340 321  478 456 341
// (RT = 4 backward needs more LDS than a CU has at the widest layers; FP32
// forward takes 1 or 2.)  Hidden widths other than 240 have no row-wave kernel.
template <typename Real>
void launch_fit_fused(hipStream_t s, const FitFusedArgs<Real> &a, int64_t n, int pass) {
  constexpr bool F64 = sizeof(Real) == 8;
  if (a.rows <= 0) return;
  if (n <= FIT_SPREAD && a.gz) {
    launch_fitx_spread(s, a, pass);
    return;
  }
  const int64_t r1 = fit_rounds(n, 16), r2 = fit_rounds(n, 32), r4 = fit_rounds(n, 64);
  if (pass == 1) {
    const int64_t t1 = r1 * (F64 ? 100 : 56), t2 = r2 * (F64 ? 176 : 95);
    if constexpr (F64) {
      if (r4 * 326 < (t1 < t2 ? t1 : t2)) {
        launch_fitx<Real, 4>(s, a, pass);
        return;
      }
    }
    if (t1 <= t2) launch_fitx<Real, 1>(s, a, pass);
    else launch_fitx<Real, 2>(s, a, pass);
    return;
  }
  bool rows = true;
  for (int l = 1; l <= a.d.n_fit; ++l) rows = rows && a.d.fw[l] == 16 * FR_NT;
  const int64_t t1 = r1 * (F64 ? 111 : 62), t2 = r2 * (F64 ? 182 : 114), tr = r4 * (F64 ? 341 : 180);
  if (rows && tr < t1 && tr < t2) launch_fitr_bwd(s, a);
  else if (t1 <= t2) launch_fitx<Real, 1>(s, a, pass);
  else launch_fitx<Real, 2>(s, a, pass);
}
template void launch_fit_fused<double>(hipStream_t, const FitFusedArgs<double> &, int64_t, int);
template void launch_fit_fused<float>(hipStream_t, const FitFusedArgs<float> &, int64_t, int);

// D[i] = T[i] T_<[i]^T of every atom (when a caller asks for it)
template <typename Real>
__global__ void k_form_d(int64_t n, int M1, int M2, const Real *__restrict__ T, Real *__restrict__ D) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t MM = (int64_t)M1 * M2;
  if (q >= n * MM) return;
  const int64_t i = q / MM;
  const int f = (int)(q % MM) / M2, b = (int)(q % M2);
  const Real *x = T + (i * M1 + f) * 4, *y = T + (i * M1 + b) * 4;
  D[q] = x[0] * y[0] + x[1] * y[1] + x[2] * y[2] + x[3] * y[3];
}

void launch_form_d(hipStream_t s, int64_t n, int M1, int M2, const double *T, double *D) {
  const int64_t q = n * M1 * M2;
  if (q > 0)
    hipLaunchKernelGGL(k_form_d<double>, dim3((unsigned)((q + 255) / 256)), dim3(256), 0, s, n, M1, M2, T, D);
}

}  // namespace dpk
