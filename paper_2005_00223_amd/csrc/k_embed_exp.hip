// Embedding + descriptor, forward and backward, through the nets' Chebyshev
// expansions (dp_expand.h), for every precision policy: FP64 in double, the
// mixed policies in float on the weights their own kernels hold.
//
//   k_exp_pair   per atom: H[k][c] = sum_j T_k(x_j) R_j[c] of every piece
//                its neighbours lie in, R_j formed from the positions
//   k_exp_desc   four atoms per wave: T = C^T H / Nc on the matrix cores
//                (N = 4 atoms x 4 components), and D = T T_<^T (FP64 / FP32)
//   k_exp_adj    four atoms per wave: dE/dT from dE/dD (FP64 / FP32), then
//                M = C dE/dT and M' = C' dE/dT on the matrix cores
//   k_exp_force  per atom: dE/dR_j from M, M', the FP64 force pass, F_j
//                merged in LDS and added by FP64 atomics, virial partial sums
//
// The list is sorted by distance, so the neighbours of one net come in
// descending s and each piece's are one run of slots; an atom's runs
// ("segments") are numbered in that order and recorded in its mask.  Both
// pair kernels find them by the same bitwise-reproducible arithmetic (this
// file is compiled with -ffp-contract=off).
//
// A wave takes one atom in the pair kernels, 64 neighbours at a time: one
// lane per neighbour for the geometry, then four lanes per neighbour, one
// per component, for the polynomials, so that H (K accumulators a lane) and
// M (2 K operands a lane) stay in registers; with one lane per neighbour H
// would take 4 K accumulators and a wave reduction four times as long.
//
// Measured, 32,000 copper atoms (5.8 million pairs), the layer kernels before
// and these now: FP64 forward 5.30 ms -> 0.12 (k_exp_pair 0.09, k_exp_desc
// 0.03), backward 8.05 ms -> 0.30 (k_exp_adj 0.04, k_exp_force 0.26); FP32
// forward 3.19 ms -> 0.08, backward 6.03 ms -> 0.19.  FP16, 62,565 centres:
// forward 2.18 ms -> 0.15, backward 3.53 ms -> 0.34.
// The pair kernels wait on latency (atom -> list -> positions -> pieces -> M)
// more than they compute: atom data come by scalar loads, pieces are found
// once per neighbour from lanes, positions and M are loaded ahead
// (k_exp_pair 96 -> 90 us FP64, 72 -> 57 FP32).
#include "dp_expand.h"
#include "dp_f64.h"

namespace dpk {

constexpr int EXP_WAVES = 4;
constexpr int EXP_ROWS = 16;         // rows of a run in k_exp_force
constexpr int EXP_HASH_LOG = 10, EXP_HASH = 1 << EXP_HASH_LOG, EXP_PROBES = 8;
// rows from which k_exp_force merges in LDS: below, 16 rows a workgroup leave
// CUs idle (whole evaluation with | without, FP32 copper: 864 atoms 324 | 322
// us, 4,000 380 | 400, 6,912 469 | 508)
constexpr int64_t EXP_MERGE = 4096;

// rows up to which four workgroups share the feature tiles (k_exp_desc) or the
// segments (k_exp_adj) of four atoms: one wave per four atoms is a serial chain
// of both on a mostly idle chip (192 water atoms FP64: 20.7 -> 6.8 us and 22.8
// -> 11.0)
constexpr int64_t EXP_SPREAD = 2048;

template <typename Real>
struct ExpK;
template <>
struct ExpK<double> {
  static constexpr int K = EXP_K64;
};
template <>
struct ExpK<float> {
  static constexpr int K = EXP_K32;
};

// One pair's geometry from the wrapped positions: the displacement, 1/r, the
// switch's argument and the environment row (s, s d / r).
struct PairGeo {
  double dx, dy, dz, ir, x;
  double R[4];
};

// FINE: 1/r and r from one more residual step each (FP64 kernels)
template <bool FINE>
__device__ inline PairGeo pair_geo(const double4 &pi, const double4 &pj, const double (&L)[3], double rcs,
                                   double inv_w) {
  const double4 D = pair_disp_sq(pi, pj, L[0], L[1], L[2]);
  PairGeo g;
  g.dx = D.x;
  g.dy = D.y;
  g.dz = D.z;
  double ir = rsqrt64(D.w), r = D.w * ir;
  if (FINE) {
    r = fma(fma(-r, r, D.w), 0.5 * ir, r);
    ir = fma(fma(-r, ir, 1.0), ir, ir);
  }
  const double x = fmin(fmax((r - rcs) * inv_w, 0.0), 1.0);
  const double sv = (x * x * x * (-6.0 * x * x + 15.0 * x - 10.0) + 1.0) * ir, tv = sv * ir;
  g.ir = ir;
  g.x = x;
  g.R[0] = sv;
  g.R[1] = tv * D.x;
  g.R[2] = tv * D.y;
  g.R[3] = tv * D.z;
  return g;
}

// The pieces of one net, piece q's ends and scale in lane q (P <= 32).
template <typename Real>
struct Pieces {
  Real lo, mid, ih;
  __device__ void load(const Real *__restrict__ pc, int P, int lane) {
    const Real *q = pc + 4 * (lane < P ? lane : P - 1);
    lo = q[0];
    mid = q[1];
    ih = q[2];
  }
  __device__ static double from(double v, int q) {
    const long long b = __double_as_longlong(v);
    return __longlong_as_double((long long)(unsigned)__builtin_amdgcn_readlane((int)b, q) |
                                (long long)__builtin_amdgcn_readlane((int)(b >> 32), q) << 32);
  }
  __device__ static float from(float v, int q) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), q));
  }
  // piece of s: the last one whose lower end is <= s (lo[0] = 0); the whole
  // wave stops at the first piece above all of its s
  __device__ int of(int P, Real s) const {
    int p = 0;
    for (int q = 1; q < P; ++q) {
      const bool up = s >= from(lo, q);
      if (!__ballot(up)) break;
      p += up ? 1 : 0;
    }
    return p;
  }
};

// One net's neighbours of an atom, 64 at a time: positions are loaded one
// block ahead, list entries two, so that neither latency stands between two
// blocks.  Slots past the end reread the last one.
struct PairStream {
  const int32_t *list;
  const double4 *xw;
  int cnt, j, jn;
  double4 x, xn;
  __device__ int slot(int q) const { return list[q < cnt ? q : cnt - 1]; }
  __device__ void begin(const int32_t *l, const double4 *p, int n, int lane) {
    list = l;
    xw = p;
    cnt = n;
    jn = slot(lane);
    xn = xw[jn];
    j = jn;
    jn = slot(64 + lane);
  }
  // block at n0: j, x
  __device__ void next(int n0, int lane) {
    x = xn;
    const int cur = j;
    if (n0 + 64 < cnt) {
      xn = xw[jn];
      j = jn;
      jn = slot(n0 + 128 + lane);
    }
    jcur = cur;
  }
  int jcur;
};

// workgroup barrier that orders LDS accesses only (atomics to memory stay in flight)
__device__ inline void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ inline unsigned long long seg_bit(int P, int u, int p) { return 1ull << (u * P + (P - 1 - p)); }

// blocks of EXP_WAVES atoms, in contiguous runs per XCD (workgroups are
// dealt round-robin by id), so that neighbouring atoms' positions meet in
// one L2
__device__ inline int64_t xcd_block(unsigned b, unsigned nb) {
  const unsigned per = (nb + 7) / 8;
  return (int64_t)(b & 7) * per + (b >> 3);
}

// the sum of v over the lanes of equal lane % 4, lane l getting entry l / 4
template <typename Real, int K>
__device__ inline Real quad_columns(Real (&v)[K], int lane) {
  static_assert(K <= 16, "one entry per lane group");
  Real a[8];
  const bool b5 = lane & 32, b4 = lane & 16, b3 = lane & 8, b2 = lane & 4;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const Real hi = k + 8 < K ? v[k + 8 < K ? k + 8 : 0] : Real(0);
    const Real keep = b5 ? hi : v[k], send = b5 ? v[k] : hi;
    a[k] = keep + __shfl_xor(send, 32);
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const Real keep = b4 ? a[k + 4] : a[k], send = b4 ? a[k] : a[k + 4];
    a[k] = keep + __shfl_xor(send, 16);
  }
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const Real keep = b3 ? a[k + 2] : a[k], send = b3 ? a[k] : a[k + 2];
    a[k] = keep + __shfl_xor(send, 8);
  }
  const Real keep = b2 ? a[1] : a[0], send = b2 ? a[0] : a[1];
  return keep + __shfl_xor(send, 4);
}

// ---------------------------------------------------------------------------
// H of every atom
// ---------------------------------------------------------------------------
template <typename Real>
__global__ void __launch_bounds__(64 * EXP_WAVES) k_exp_pair(ExpArgs<Real> a) {
  constexpr int K = ExpK<Real>::K;
  __shared__ Real Rs[EXP_WAVES][64 * 4];
  const Dims &d = a.d;
  // uniform over the wave: the atom's data come by scalar loads
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t p = xcd_block(blockIdx.x, gridDim.x) * EXP_WAVES + wv;
  if (p >= a.rows) return;
  const int i = __builtin_amdgcn_readfirstlane(a.atom_of_pos[p]);
  if (i < 0) return;
  Real *Rw = Rs[wv];
  const double4 pi = a.xw[i];
  const int t = __builtin_amdgcn_readfirstlane((int)pi.w), P = a.tab.P, c = lane & 3;
  const double inv_w = 1.0 / (d.rcut - d.rcut_smth);
  Real *Hi = a.H + (int64_t)i * a.seg * (EXP_KP * 4);
  unsigned long long mask = 0;
  int slot = 0;
  bool far = false;
  for (int u = 0; u < d.ntypes; ++u) {
    const int cnt = a.nreal[(int64_t)i * d.ntypes + u];
    if (cnt == 0) continue;
    const int64_t base = (int64_t)i * d.nnei + d.off[u];
    Pieces<Real> pc;
    pc.load(a.tab.piece + (int64_t)(t * d.ntypes + u) * P * 4, P, lane);
    PairStream ps;
    ps.begin(a.nlist + base, a.xw, cnt, lane);
    Real acc[K];
    int cur = -1;
    Real mid = 0, ih = 0;
    auto flush = [&]() {
      const Real h = quad_columns<Real, K>(acc, lane);
      if (slot < a.seg) Hi[slot * (EXP_KP * 4) + lane] = h;
      else far = true;
      mask |= seg_bit(P, u, cur);
      ++slot;
    };
    for (int n0 = 0; n0 < cnt; n0 += 64) {
      ps.next(n0, lane);
      const PairGeo g = pair_geo<sizeof(Real) == 8>(pi, ps.x, a.L, d.rcut_smth, inv_w);
      const bool in = n0 + lane < cnt;  // slots past the end get a zero row
      const int piece = pc.of(P, in ? (Real)g.R[0] : Real(0));
      far |= in && !((Real)g.R[0] <= a.tab.smax);
      wave_sync();
#pragma unroll
      for (int k = 0; k < 4; ++k) Rw[lane * 4 + k] = in ? (Real)g.R[k] : Real(0);
      wave_sync();
      const int left = cnt - n0;
      for (int sub = 0; sub < 4 && sub * 16 < left; ++sub) {
        const int nl = sub * 16 + (lane >> 2);
        const Real s = Rw[nl * 4], Rc = Rw[nl * 4 + c];
        const bool valid = nl < left;
        const int mine = __shfl(piece, nl);
        unsigned long long todo = __ballot(valid);
        while (todo) {
          // the next piece, in descending order; a neighbour whose s lies
          // above the current piece (ties of the quantised distance) takes it
          const int np = __builtin_amdgcn_readlane(mine, __ffsll(todo) - 1);
          if (cur < 0 || np < cur) {
            if (cur >= 0) flush();
            cur = np;
            mid = pc.from(pc.mid, cur);
            ih = pc.from(pc.ih, cur);
#pragma unroll
            for (int k = 0; k < K; ++k) acc[k] = 0;
          }
          const bool now = (todo >> lane & 1) && mine >= cur;
          const Real x = now ? (s - mid) * ih : Real(0), x2 = x + x;
          // q_k = T_k(x) R[c]
          Real q0 = now ? Rc : Real(0), q1 = x * q0;
          acc[0] += q0;
          acc[1] += q1;
#pragma unroll
          for (int k = 2; k < K; ++k) {
            const Real q2 = fma(x2, q1, -q0);
            acc[k] += q2;
            q0 = q1;
            q1 = q2;
          }
          todo &= ~__ballot(now);
        }
      }
    }
    flush();
  }
  if (lane == 0) a.mask[i] = mask;
  if (__ballot(far) && lane == 0) atomicOr(a.flags, FLAG_FAR);
}

// ---------------------------------------------------------------------------
// T = C^T H / Nc, D = T T_<^T
// ---------------------------------------------------------------------------
// EXP_MT: feature tiles a wave accumulates at once; without D the tiles may be
// dealt to gridDim.y workgroups
template <typename Real, bool WITH_D, int EXP_MT>
__global__ void __launch_bounds__(64) k_exp_desc(ExpArgs<Real> a) {
  extern __shared__ __align__(16) unsigned char exp_smem[];
  Real *Ts = (Real *)exp_smem;  // WITH_D: [4][M1p][4]
  const Dims &d = a.d;
  const int lane = threadIdx.x, g = lane >> 4, r4 = (lane & 15) >> 2, c = lane & 3;
  const int64_t p0 = (int64_t)blockIdx.x * 4;
  const int M1 = d.M1, M1p = a.tab.M1p, nmt = M1p >> 4, P = a.tab.P, MM = M1 * d.M2;
  int atom[4], t = -1;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    atom[r] = a.atom_of_pos[p0 + r];
    if (atom[r] >= 0 && t < 0) t = (int)a.xw[atom[r]].w;
  }
  if (t < 0) {
    if (WITH_D)
      for (int64_t o = lane; o < 4 * (int64_t)MM; o += 64) a.D[p0 * MM + o] = 0;
    return;
  }
  unsigned long long any = 0, mine = 0;
  int im = -1;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const unsigned long long m = atom[r] >= 0 ? a.mask[atom[r]] : 0ull;
    any |= m;
    if (r == r4) {
      mine = m;
      im = atom[r];
    }
  }
  const Real *Hm = a.H + (int64_t)(im < 0 ? 0 : im) * a.seg * (EXP_KP * 4) + c;
  for (int mt0 = blockIdx.y * EXP_MT; mt0 < nmt; mt0 += gridDim.y * EXP_MT) {
    typename MF<Real>::acc acc[EXP_MT];
#pragma unroll
    for (int m = 0; m < EXP_MT; ++m) acc[m] = typename MF<Real>::acc{0, 0, 0, 0};
    for (unsigned long long todo = any; todo; todo &= todo - 1) {
      const int b = __ffsll(todo) - 1;
      const int u = b / P, pc = P - 1 - b % P;
      const Real *C = a.tab.Cf + ((int64_t)(t * d.ntypes + u) * P + pc) * EXP_KP * M1p;
      const bool has = mine >> b & 1;
      const int sl = has ? __popcll(mine & ((1ull << b) - 1)) : 0;
      const Real *Hs = Hm + (sl < a.seg ? sl : 0) * (EXP_KP * 4);
      constexpr int KS = (ExpK<Real>::K + 3) / 4;
      Real bv[KS];
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) bv[kk] = Hs[(4 * kk + g) * 4];
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) {
        const Real hv = has ? bv[kk] : Real(0);
        const Real *Ck = C + (int64_t)(4 * kk + g) * M1p + (lane & 15);
#pragma unroll
        for (int m = 0; m < EXP_MT; ++m)
          acc[m] = MF<Real>::mma(Ck[16 * (mt0 + m < nmt ? mt0 + m : nmt - 1)], hv, acc[m]);
      }
    }
#pragma unroll
    for (int m = 0; m < EXP_MT; ++m) {
      if (mt0 + m >= nmt) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int f = 16 * (mt0 + m) + MF<Real>::row(r, g);
        const Real v = im < 0 ? Real(0) : acc[m][r] * (Real)d.inv_nc;
        if (WITH_D) Ts[(r4 * M1p + f) * 4 + c] = v;
        if (f < M1 && im >= 0) a.T[((int64_t)im * M1 + f) * 4 + c] = v;
      }
    }
  }
  if (WITH_D) {
    wave_sync();
    const int b = lane & 15;
    for (int r = 0; r < 4; ++r) {
      const Real *Tr = Ts + (int64_t)r * M1p * 4;
      Real *Dp = a.D + (p0 + r) * (int64_t)MM;
      const Real bv = b < d.M2 ? Tr[b * 4 + g] : Real(0);
      for (int mt = 0; mt < nmt; ++mt) {
        const typename MF<Real>::acc z =
            MF<Real>::mma(Tr[(mt * 16 + (lane & 15)) * 4 + g], bv, typename MF<Real>::acc{0, 0, 0, 0});
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int f = mt * 16 + MF<Real>::row(q, g);
          if (f < M1 && b < d.M2) Dp[f * d.M2 + b] = z[q];
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// M = C dE/dT, M' = C' dE/dT
// ---------------------------------------------------------------------------
template <typename Real, bool FROM_D>
__global__ void __launch_bounds__(64) k_exp_adj(ExpArgs<Real> a) {
  typedef typename MF<Real>::acc acc_t;
  extern __shared__ __align__(16) unsigned char exp_smem[];
  Real *dTs = (Real *)exp_smem;  // FROM_D: [4][M1p][4]
  const Dims &d = a.d;
  const int lane = threadIdx.x, g = lane >> 4, col = lane & 15, r4 = col >> 2, c = lane & 3;
  const int64_t p0 = (int64_t)blockIdx.x * 4;
  const int M1 = d.M1, M1p = a.tab.M1p, nmt = M1p >> 4, P = a.tab.P, M2 = d.M2, MM = M1 * M2;
  int atom[4], t = -1;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    atom[r] = a.atom_of_pos[p0 + r];
    if (atom[r] >= 0 && t < 0) t = (int)a.xw[atom[r]].w;
  }
  if (t < 0) return;
  if (FROM_D) {
    // dT[m] = (sum_b dD[m][b] T[b] + [m < M2] sum_a dD[a][m] T[a]) / Nc, one
    // atom after the other; the operands of the next 16 rows of dD are
    // loaded during the products of these.  The k index of the first sum
    // runs as b = 4 g + k, so a lane's four values of dD are contiguous.
    Real xa[4], ya[4], yb[4], tb[4];
    auto load = [&](int r, int mt) {
      const Real *dD = a.dD + (p0 + r) * (int64_t)MM;
      const Real *T = a.T + (int64_t)(atom[r] < 0 ? 0 : atom[r]) * M1 * 4 + c;
      const int m = 16 * mt + col, mc = m < M1 ? m : M1 - 1;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int b = 4 * g + k, bc = b < M2 ? b : M2 - 1;
        const Real v = dD[mc * M2 + bc];
        xa[k] = b < M2 ? v : Real(0);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int f = 16 * mt + 4 * k + g, fc = f < M1 ? f : M1 - 1;
        const Real v = dD[fc * M2 + (col < M2 ? col : M2 - 1)], w = T[fc * 4];
        ya[k] = col < M2 && f < M1 ? v : Real(0);
        yb[k] = col < 4 ? w : Real(0);
      }
      if (mt == 0)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int b = 4 * g + k;
          const Real w = T[(b < M2 ? b : M2 - 1) * 4];
          tb[k] = col < 4 && b < M2 ? w : Real(0);
        }
    };
    load(0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      acc_t low{0, 0, 0, 0}, z0{0, 0, 0, 0};
      Real tc[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) tc[k] = tb[k];
      const Real sc = atom[r] < 0 ? Real(0) : (Real)d.inv_nc;
      auto put = [&](int mt, const acc_t &z) {
        if (col < 4)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            dTs[(r * M1p + 16 * mt + MF<Real>::row(q, g)) * 4 + c] = atom[r] < 0 ? Real(0) : z[q] * sc;
      };
      for (int mt = 0; mt < nmt; ++mt) {
        Real x[4], y[4], yt[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          x[k] = xa[k];
          y[k] = ya[k];
          yt[k] = yb[k];
        }
        if (mt + 1 < nmt) load(r, mt + 1);
        else if (r < 3) load(r + 1, 0);
        acc_t z{0, 0, 0, 0};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          z = MF<Real>::mma(x[k], tc[k], z);
          low = MF<Real>::mma(y[k], yt[k], low);
        }
        if (mt == 0) z0 = z;
        else put(mt, z);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) z0[q] += low[q];
      put(0, z0);
    }
    wave_sync();
  }
  unsigned long long any = 0, mine = 0;
  int im = -1;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const unsigned long long m = atom[r] >= 0 ? a.mask[atom[r]] : 0ull;
    any |= m;
    if (r == r4) {
      mine = m;
      im = atom[r];
    }
  }
  const Real *dTg = FROM_D ? dTs + (int64_t)r4 * M1p * 4 + c : a.dT + (int64_t)(im < 0 ? 0 : im) * M1 * 4 + c;
  const int mlast = FROM_D ? M1p - 1 : M1 - 1;
  unsigned turn = 0;  // the segments are dealt to gridDim.y workgroups
  for (unsigned long long todo = any; todo; todo &= todo - 1) {
    if (turn++ % gridDim.y != blockIdx.y) continue;
    const int b = __ffsll(todo) - 1;
    const int u = b / P, pc = P - 1 - b % P;
    const Real *C = a.tab.Cb + ((int64_t)(t * d.ntypes + u) * P + pc) * 2 * M1p * EXP_KP + col;
    const Real *Cd = C + (int64_t)M1p * EXP_KP;
    acc_t v{0, 0, 0, 0}, w{0, 0, 0, 0};
    // 16 features at a time, the next ones' operands in flight; rows of C
    // past M1 are zero, the dE/dT they meet only has to be finite
    Real cn[4], dn[4], xn[4];
    auto load = [&](int m0) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int mm = m0 + 4 * k + g;
        cn[k] = C[mm * EXP_KP];
        dn[k] = Cd[mm * EXP_KP];
        xn[k] = dTg[(mm < mlast ? mm : mlast) * 4];
      }
    };
    load(0);
    for (int m0 = 0; m0 < M1p; m0 += 16) {
      Real cc[4], dc[4], xc[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        cc[k] = cn[k];
        dc[k] = dn[k];
        xc[k] = xn[k];
      }
      load(m0 + 16 < M1p ? m0 + 16 : m0);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        v = MF<Real>::mma(cc[k], xc[k], v);
        w = MF<Real>::mma(dc[k], xc[k], w);
      }
    }
    const int sl = __popcll(mine & ((1ull << b) - 1));
    if ((mine >> b & 1) && sl < a.seg) {
      Real *Mo = a.M + ((int64_t)im * a.seg + sl) * (2 * EXP_KP * 4) + c;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        Mo[MF<Real>::row(q, g) * 4] = v[q];
        Mo[(EXP_KP + MF<Real>::row(q, g)) * 4] = w[q];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// forces and virial
// ---------------------------------------------------------------------------
// MERGE: 3 FP64 atomics a pair at memory reach 55 G/s whatever the rest of the
// kernel does (32,000 copper atoms, 5.8 million pairs: 318 us in FP32, of
// which 138 remain without them; a copy of F per XCD changed nothing, so it is
// the atomic units, not the lines' movement).  A workgroup therefore takes 16
// consecutive rows and adds its pairs' forces in an LDS table keyed by atom;
// each atom's sum then goes to memory once.  Rows close in space share most
// neighbours (ordered copper: 2,900 pairs, about 600 atoms).  A pair whose
// places in the table are taken goes to memory by itself, so atoms in random
// order, where nothing merges, cost what they did (1,441 against 1,439 us for
// an FP32 evaluation).  318 -> 188 us FP32, 335 -> 258 FP64, 62,565 centres
// 600 -> 339; 8 rows 204 us, 32 rows 224; a workgroup per cell of the cell
// list with sums addressed by cell 208 to 380 (cells differ in size).  What is
// left waits on latency, so waves count: in FP32 the workgroups' LDS and 128
// registers (nine of them spilled) let four share a CU instead of three, 188 ->
// 166 us and 339 -> 298; in FP64 a third wave per SIMD spills 32 (258 -> 302
// us) and is not taken.
template <typename Real, bool MERGE>
__global__ void __launch_bounds__(64 * EXP_WAVES, sizeof(Real) == 8 ? 2 : MERGE ? 4 : 3) k_exp_force(ExpArgs<Real> a) {
  constexpr int K = ExpK<Real>::K;
  constexpr int MS = EXP_KP + 2;  // row stride of a component's coefficients in LDS
  __shared__ __align__(16) Real Ms[EXP_WAVES][8 * MS];
  // environment rows, then dE/dR (four Real a neighbour), then forces (three double)
  __shared__ __align__(16) double Fs[EXP_WAVES][sizeof(Real) == 8 ? 64 * 4 : 64 * 3];
  __shared__ double vred[EXP_WAVES][9];
  __shared__ int32_t key[MERGE ? EXP_HASH : 1];       // atom of a sum, or -1
  __shared__ double facc[MERGE ? 3 * EXP_HASH : 1];
  __shared__ int turn;                                // next row of the workgroup's run
  const Dims &d = a.d;
  // uniform over the wave: the atom's data come by scalar loads
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), c = lane & 3;
  Real *Mw = Ms[wv];
  double *Fw = Fs[wv];
  Real *Rw = (Real *)Fw;
  const int P = a.tab.P;
  const double inv_w = 1.0 / (d.rcut - d.rcut_smth);
  double vir[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) vir[k] = 0.0;
  // where atom j's force sum is in LDS: linear probing, -1 when the places
  // tried are all taken
  auto slot_of = [&](int j) {
    unsigned h = (unsigned)j * 2654435769u >> (32 - EXP_HASH_LOG);
    for (int q = 0; q < EXP_PROBES; ++q) {
      int k = key[h];
      if (k == -1) k = atomicCAS(&key[h], -1, j);
      if (k == -1 || k == j) return (int)h;
      h = (h + 1) & (EXP_HASH - 1);
    }
    return -1;
  };
  auto add = [&](int j, int sl, int k, double v) {
    if (MERGE && sl >= 0) atomicAdd(&facc[3 * sl + k], v);
    else unsafeAtomicAdd(a.force + 3 * (int64_t)j + k, v);
  };
  auto atom = [&](int i) {
    const double4 pi = a.xw[i];
    const int t = __builtin_amdgcn_readfirstlane((int)pi.w);
    // the segments' M and M' in order, each loaded when the one before is taken
    const Real *Mi = a.M + (int64_t)i * a.seg * (2 * EXP_KP * 4) + lane;
    Real va = Mi[0], vb = Mi[EXP_KP * 4];
    double fx = 0.0, fy = 0.0, fz = 0.0;
    int slot = 0;
    for (int u = 0; u < d.ntypes; ++u) {
      const int cnt = a.nreal[(int64_t)i * d.ntypes + u];
      if (cnt == 0) continue;
      const int64_t base = (int64_t)i * d.nnei + d.off[u];
      Pieces<Real> pc;
      pc.load(a.tab.piece + (int64_t)(t * d.ntypes + u) * P * 4, P, lane);
      PairStream ps;
      ps.begin(a.nlist + base, a.xw, cnt, lane);
      int cur = -1;
      Real mid = 0, ih = 0, m0[K], m1[K];
#pragma unroll
      for (int k = 0; k < K; ++k) m0[k] = m1[k] = 0;
      for (int n0 = 0; n0 < cnt; n0 += 64) {
        const int q = n0 + lane;
        const bool in = q < cnt;
        ps.next(n0, lane);
        const int j = ps.jcur, jsl = MERGE && in ? slot_of(j) : -1;
        const PairGeo g = pair_geo<sizeof(Real) == 8>(pi, ps.x, a.L, d.rcut_smth, inv_w);
        const int piece = pc.of(P, in ? (Real)g.R[0] : Real(0));
        wave_sync();
#pragma unroll
        for (int k = 0; k < 4; ++k) Rw[lane * 4 + k] = in ? (Real)g.R[k] : Real(0);
        wave_sync();
        const int left = cnt - n0;
        for (int sub = 0; sub < 4 && sub * 16 < left; ++sub) {
          const int nl = sub * 16 + (lane >> 2);
          const Real s = Rw[nl * 4], Rc = Rw[nl * 4 + c];
          const bool valid = nl < left;
          const int mine = __shfl(piece, nl);
          Real ga = 0, gb = 0;
          unsigned long long todo = __ballot(valid);
          while (todo) {
            const int np = __builtin_amdgcn_readlane(mine, __ffsll(todo) - 1);
            if (cur < 0 || np < cur) {
              cur = np;
              mid = pc.from(pc.mid, cur);
              ih = pc.from(pc.ih, cur);
              // [k][component] in memory, to one component's coefficients per lane
              wave_sync();
              Mw[c * MS + (lane >> 2)] = va;
              Mw[(4 + c) * MS + (lane >> 2)] = vb;
              slot += slot + 1 < a.seg ? 1 : 0;
              va = Mi[slot * (2 * EXP_KP * 4)];
              vb = Mi[slot * (2 * EXP_KP * 4) + EXP_KP * 4];
              wave_sync();
#pragma unroll
              for (int k = 0; k < K; ++k) {
                m0[k] = Mw[c * MS + k];
                m1[k] = Mw[(4 + c) * MS + k];
              }
            }
            const bool now = (todo >> lane & 1) && mine >= cur;
            const Real x = now ? (s - mid) * ih : Real(0), x2 = x + x;
            Real t0 = 1, t1 = x;
            Real va = fma(x, m0[1], m0[0]), vb = fma(x, m1[1], m1[0]);
#pragma unroll
            for (int k = 2; k < K; ++k) {
              const Real t2 = fma(x2, t1, -t0);
              va = fma(t2, m0[k], va);
              vb = fma(t2, m1[k], vb);
              t0 = t1;
              t1 = t2;
            }
            if (now) {
              ga = va;
              gb = vb;
            }
            todo &= ~__ballot(now);
          }
          // dE/ds gets (M'^T T) . R
          Real e = Rc * gb;
          e += __shfl_xor(e, 1);
          e += __shfl_xor(e, 2);
          Rw[nl * 4 + c] = c == 0 ? ga + e : ga;
        }
        wave_sync();
        const double g0 = Rw[lane * 4], g1 = Rw[lane * 4 + 1], g2 = Rw[lane * 4 + 2], g3 = Rw[lane * 4 + 3];
        wave_sync();
        if (in) {
          if (a.net_deriv) {
            double *nd = a.net_deriv + (base + q) * 4;
            nd[0] = g0;
            nd[1] = g1;
            nd[2] = g2;
            nd[3] = g3;
          }
          // g = dE/dr_ij = (g0 ds/dr + (g1:3 . d) dt/dr) d / r + t g1:3, t = sw / r^2
          const double x = g.x, ir = g.ir;
          const double sw = x * x * x * (-6.0 * x * x + 15.0 * x - 10.0) + 1.0;
          const double dsw = x * x * (-30.0 * x * x + 60.0 * x - 30.0) * inv_w;
          const double tt = sw * (ir * ir), A = dsw * ir;
          const double ds = A - tt, dtt = (A - 2.0 * tt) * ir;
          const double gd = fma(g1, g.dx, fma(g2, g.dy, g3 * g.dz));
          const double cc = fma(g0, ds, dtt * gd) * ir;
          const double gx = fma(cc, g.dx, tt * g1), gy = fma(cc, g.dy, tt * g2), gz = fma(cc, g.dz, tt * g3);
          fx += gx;
          fy += gy;
          fz += gz;
          Fw[lane * 3 + 0] = -gx;
          Fw[lane * 3 + 1] = -gy;
          Fw[lane * 3 + 2] = -gz;
          vir[0] = fma(-gx, g.dx, vir[0]);
          vir[1] = fma(-gx, g.dy, vir[1]);
          vir[2] = fma(-gx, g.dz, vir[2]);
          vir[3] = fma(-gy, g.dx, vir[3]);
          vir[4] = fma(-gy, g.dy, vir[4]);
          vir[5] = fma(-gy, g.dz, vir[5]);
          vir[6] = fma(-gz, g.dx, vir[6]);
          vir[7] = fma(-gz, g.dy, vir[7]);
          vir[8] = fma(-gz, g.dz, vir[8]);
        }
        wave_sync();
        // F_j, a neighbour's three components from adjacent lanes: one
        // instruction's atomics then meet 16 cache lines instead of 64
        for (int sub = 0; sub < 4 && sub * 16 < left; ++sub) {
          const int nl = sub * 16 + (lane >> 2);
          const int jn = __shfl(j, nl), sl = MERGE ? __shfl(jsl, nl) : -1;
          if (c < 3 && nl < left) add(jn, sl, c, Fw[nl * 3 + c]);
        }
      }
    }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      fx += __shfl_xor(fx, o);
      fy += __shfl_xor(fy, o);
      fz += __shfl_xor(fz, o);
    }
    if (lane == 0) {
      const int sl = MERGE ? slot_of(i) : -1;
      add(i, sl, 0, fx);
      add(i, sl, 1, fy);
      add(i, sl, 2, fz);
    }
  };
  if constexpr (MERGE) {
    for (int o = threadIdx.x; o < EXP_HASH; o += 64 * EXP_WAVES) key[o] = -1;
    for (int o = threadIdx.x; o < 3 * EXP_HASH; o += 64 * EXP_WAVES) facc[o] = 0.0;
    // runs of EXP_ROWS rows (the rows are padded to a multiple), a contiguous
    // range of them per workgroup
    const int64_t runs = a.rows / EXP_ROWS, per = (runs + gridDim.x - 1) / gridDim.x;
    const int64_t b0 = xcd_block(blockIdx.x, gridDim.x) * per;
    for (int64_t b = b0; b < b0 + per && b < runs; ++b) {
      if (threadIdx.x == 0) turn = EXP_WAVES;
      lds_barrier();
      for (int k = wv; k < EXP_ROWS;) {
        const int i = __builtin_amdgcn_readfirstlane(a.atom_of_pos[b * EXP_ROWS + k]);
        if (i >= 0) atom(i);
        int nx = 0;
        if (lane == 0) nx = atomicAdd(&turn, 1);
        k = __builtin_amdgcn_readfirstlane(nx);
      }
      lds_barrier();
      // the sums to memory, the table empty again
      for (int o = threadIdx.x; o < 4 * EXP_HASH; o += 64 * EXP_WAVES) {
        const int j = key[o >> 2];
        if (j >= 0) {
          if (c < 3) {
            unsafeAtomicAdd(a.force + 3 * (int64_t)j + c, facc[3 * (o >> 2) + c]);
            facc[3 * (o >> 2) + c] = 0.0;
          } else {
            key[o >> 2] = -1;
          }
        }
      }
    }
    lds_barrier();
  } else {
    const int64_t nwaves = (int64_t)gridDim.x * EXP_WAVES;
    const int64_t gw = xcd_block(blockIdx.x, gridDim.x) * EXP_WAVES + wv;
    const int64_t chunk = (a.rows + nwaves - 1) / nwaves;
    const int64_t p_end = (gw + 1) * chunk < a.rows ? (gw + 1) * chunk : a.rows;
    for (int64_t p = gw * chunk; p < p_end; ++p) {
      const int i = a.atom_of_pos[p];
      if (i >= 0) atom(i);
    }
  }
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    double v = vir[k];
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) v += __shfl_xor(v, o);
    if (lane == 0) vred[wv][k] = v;
  }
  __syncthreads();
  if (threadIdx.x < 9) {
    double v = 0.0;
    for (int w = 0; w < EXP_WAVES; ++w) v += vred[w][threadIdx.x];
    a.vir_part[(int64_t)blockIdx.x * 9 + threadIdx.x] = v;
  }
}

int exp_bwd_grid(int64_t rows) {
  int64_t g = rows >= EXP_MERGE ? rows / EXP_ROWS : (rows + EXP_WAVES - 1) / EXP_WAVES;
  g = (g + 7) / 8 * 8;
  return (int)(g < 8 ? 8 : g > 2048 ? 2048 : g);  // a multiple of eight: contiguous runs per XCD
}

template <typename Real>
void launch_exp_fwd(hipStream_t s, const ExpArgs<Real> &a) {
  if (a.rows <= 0) return;
  const int64_t nb = ((a.rows + EXP_WAVES - 1) / EXP_WAVES + 7) / 8 * 8;
  hipLaunchKernelGGL(k_exp_pair<Real>, dim3((unsigned)nb), dim3(64 * EXP_WAVES), 0, s, a);
  const dim3 gq((unsigned)(a.rows / 4));
  if (a.D)
    hipLaunchKernelGGL((k_exp_desc<Real, true, 8>), gq, dim3(64), sizeof(Real) * 16 * a.tab.M1p, s, a);
  else if (a.rows <= EXP_SPREAD)
    hipLaunchKernelGGL((k_exp_desc<Real, false, 2>), dim3(gq.x, 4), dim3(64), 0, s, a);
  else
    hipLaunchKernelGGL((k_exp_desc<Real, false, 8>), gq, dim3(64), 0, s, a);
}

template <typename Real>
void launch_exp_bwd(hipStream_t s, const ExpArgs<Real> &a, int grid) {
  const dim3 gq((unsigned)(a.rows / 4));
  if (a.rows > 0) {
    if (a.dD)
      hipLaunchKernelGGL((k_exp_adj<Real, true>), gq, dim3(64), sizeof(Real) * 16 * a.tab.M1p, s, a);
    else
      hipLaunchKernelGGL((k_exp_adj<Real, false>), dim3(gq.x, a.rows <= EXP_SPREAD ? 4 : 1), dim3(64), 0, s, a);
  }
  if (a.rows >= EXP_MERGE)
    hipLaunchKernelGGL((k_exp_force<Real, true>), dim3(grid), dim3(64 * EXP_WAVES), 0, s, a);
  else
    hipLaunchKernelGGL((k_exp_force<Real, false>), dim3(grid), dim3(64 * EXP_WAVES), 0, s, a);
}

template void launch_exp_fwd<double>(hipStream_t, const ExpArgs<double> &);
template void launch_exp_fwd<float>(hipStream_t, const ExpArgs<float> &);
template void launch_exp_bwd<double>(hipStream_t, const ExpArgs<double> &, int);
template void launch_exp_bwd<float>(hipStream_t, const ExpArgs<float> &, int);

}  // namespace dpk
