// Host side of the embedding nets' Chebyshev expansions (dp_expand.h): the
// nets evaluated with their tangents at Chebyshev nodes, the coefficients
// by the discrete cosine sum, the pieces by halving.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <thread>

#include "dp_expand.h"

namespace dpk {
namespace {

// What the interpolation in double can still tell from its rounding: enough to
// find the pieces, not for their coefficients in double kernels.  Many
// neighbours of an atom share a piece, so the errors of its coefficients add up
// (coefficients left at this accuracy beyond s = 2: NVE runs of hot water,
// whose closest pair passes through s = 5 to 8, ended 2 to 400 times further
// from the FP64 reference than by the layers; beyond s = 8: G there 3e-15 of
// the largest feature off, the layers 5e-16).
constexpr double EXP_PRE = 0x1p-48;

// A net's weights with the inputs of an output contiguous.
struct NetT {
  const ExpNetIn *n;
  std::vector<double> W[MAXL];
  explicit NetT(const ExpNetIn &net) : n(&net) {
    for (int l = 0; l < net.n_layers; ++l) {
      const size_t in = net.w[l], out = net.w[l + 1];
      W[l].resize(in * out);
      for (size_t i = 0; i < in; ++i)
        for (size_t o = 0; o < out; ++o) W[l][o * in + i] = net.W[l][i * out + o];
    }
  }
  // a point's time in ns: products (value and tangent), then tanh
  double ns(bool extended) const {
    double s = 0.0;
    for (int l = 0; l < n->n_layers; ++l)
      s += 2.0 * (double)W[l].size() * (extended ? 2.0 : 0.3) + n->w[l + 1] * (extended ? 100.0 : 30.0);
    return s;
  }
};

template <typename F>
struct Buffers {
  std::vector<F> h, hd, z, zd;
};

// The layers' products for J points at once (feature-major, [feature][J]): the
// sums of one output's J points stay in registers.
template <int J>
void products(const double *__restrict__ w, double b, int in, const double *__restrict__ h, double *__restrict__ z) {
  double a[J];
  for (int j = 0; j < J; ++j) a[j] = b;
  for (int i = 0; i < in; ++i)
    for (int j = 0; j < J; ++j) a[j] += w[i] * h[(size_t)i * J + j];
  for (int j = 0; j < J; ++j) z[j] = a[j];
}

// Two outputs of one point, value and tangent: in extended precision a sum
// kept in memory costs a 10-byte store and load per term, and four fit the
// register stack.
inline void products2(const double *__restrict__ wa, const double *__restrict__ wb, int in,
                      const long double *__restrict__ h, const long double *__restrict__ hd, long double (&s)[4]) {
  long double a = s[0], ad = s[1], b = s[2], bd = s[3];
  for (int i = 0; i < in; ++i) {
    const long double x = h[i], xd = hd[i];
    a += x * wa[i];
    ad += xd * wa[i];
    b += x * wb[i];
    bd += xd * wb[i];
  }
  s[0] = a;
  s[1] = ad;
  s[2] = b;
  s[3] = bd;
}

// tanh and the skips of layer l over J points, z and zd in place
template <typename F>
void layer_end(const ExpNetIn &n, int l, int J, Buffers<F> &u) {
  const int in = n.w[l], out = n.w[l + 1];
  if (!(n.lin && l + 1 == n.n_layers))
    for (int o = 0; o < out; ++o)
      for (int j = 0; j < J; ++j) {
        const size_t e = (size_t)o * J + j;
        const F t = std::tanh(u.z[e]);
        u.z[e] = t;
        u.zd[e] *= F(1) - t * t;
        if (out == in || out == 2 * in) {
          const size_t k = (size_t)(o >= in ? o - in : o) * J + j;
          u.z[e] += u.h[k];
          u.zd[e] += u.hd[k];
        }
      }
  u.h.swap(u.z);
  u.hd.swap(u.zd);
}

// u.h, u.hd = G[m][J], dG[m][J] of a net at s[J], forward mode through its layers
template <int J>
void net_eval(const NetT &t, const double *s, Buffers<double> &u) {
  const ExpNetIn &n = *t.n;
  u.h.assign(s, s + J);
  u.hd.assign(J, 1.0);
  for (int l = 0; l < n.n_layers; ++l) {
    const int in = n.w[l], out = n.w[l + 1];
    u.z.resize((size_t)out * J);
    u.zd.resize((size_t)out * J);
    for (int o = 0; o < out; ++o) {
      const double *w = t.W[l].data() + (size_t)o * in;
      products<J>(w, n.b[l][o], in, u.h.data(), u.z.data() + (size_t)o * J);
      products<J>(w, 0.0, in, u.hd.data(), u.zd.data() + (size_t)o * J);
    }
    layer_end(n, l, J, u);
  }
}

template <int J>
void net_eval(const NetT &t, const long double *s, Buffers<long double> &u) {
  const ExpNetIn &n = *t.n;
  std::vector<long double> G, D;
  for (int j = 0; j < J; ++j) {
    u.h.assign(1, s[j]);
    u.hd.assign(1, 1.0L);
    for (int l = 0; l < n.n_layers; ++l) {
      const int in = n.w[l], out = n.w[l + 1];
      u.z.resize(out);
      u.zd.resize(out);
      for (int o = 0; o < out; o += 2) {
        const int o1 = o + 1 < out ? o + 1 : o;
        const double *w = t.W[l].data();
        long double a[4] = {n.b[l][o], 0.0L, n.b[l][o1], 0.0L};
        products2(w + (size_t)o * in, w + (size_t)o1 * in, in, u.h.data(), u.hd.data(), a);
        u.z[o] = a[0];
        u.zd[o] = a[1];
        u.z[o1] = a[2];
        u.zd[o1] = a[3];
      }
      layer_end(n, l, 1, u);
    }
    const size_t m1 = u.h.size();
    G.resize(m1 * J);
    D.resize(m1 * J);
    for (size_t m = 0; m < m1; ++m) {
      G[m * J + j] = u.h[m];
      D[m * J + j] = u.hd[m];
    }
  }
  u.h.swap(G);
  u.hd.swap(D);
}

struct Piece {
  int net;
  double lo, hi;
  bool ok = false;
  std::vector<double> C;  // [2][EXP_KP][M1p]
};

// f(k) for k < n on up to nthreads threads; false if one of them threw (out
// of memory).
template <class Fn>
bool parallel_for(size_t n, size_t nthreads, Fn f) {
  std::atomic<size_t> next{0};
  std::atomic<bool> good{true};
  auto work = [&]() {
    try {
      for (size_t k; (k = next.fetch_add(1)) < n;) f(k);
    } catch (...) {
      good = false;
    }
  };
  std::vector<std::thread> pool;
  nthreads = std::min<size_t>({nthreads, (size_t)std::max(1u, std::thread::hardware_concurrency()), n});
  try {
    for (size_t k = 1; k < nthreads; ++k) pool.emplace_back(work);
  } catch (...) {
    // no more threads to be had: those there are do the rest
  }
  work();
  for (auto &th : pool) th.join();
  return good;
}

// Interpolates the pieces' nets in the real type F at J nodes and sets ok where
// the last two coefficients of every feature are within tol.
template <typename F, int J>
bool fit_pieces(const std::vector<NetT> &nets, int M1p, double tol, std::vector<Piece> &pieces) {
  const F pi = (F)3.14159265358979323846264338327950288L;
  F ct[J][J], node[J];
  for (int k = 0; k < J; ++k) {
    node[k] = std::cos(pi * ((F)k + F(0.5)) / J);
    for (int j = 0; j < J; ++j) ct[k][j] = std::cos(pi * (F)k * ((F)j + F(0.5)) / J) * (k == 0 ? F(1) : F(2)) / J;
  }
  // as many threads as have a millisecond of work each, four at most: a caller's
  // own threads may be spinning on the same CPUs (eight, from 0.3 ms, took a
  // water model's FP16 load from 26 to 35 ms just after a numpy least squares)
  double ns = 0.0;
  for (auto &p : pieces) ns += nets[p.net].ns(sizeof(F) > sizeof(double)) * J;
  const size_t nth = (size_t)std::min(4.0, 1.0 + ns / 1e6);
  return parallel_for(pieces.size(), nth, [&](size_t q) {
    Piece &p = pieces[q];
    Buffers<F> u;
    F s[J];
    for (int j = 0; j < J; ++j) s[j] = ((F)p.lo + (F)p.hi) / 2 + ((F)p.hi - (F)p.lo) / 2 * node[j];
    net_eval<J>(nets[p.net], s, u);
    p.C.assign((size_t)2 * EXP_KP * M1p, 0.0);
    p.ok = true;
    for (int w = 0; w < 2; ++w) {
      const std::vector<F> &g = w ? u.hd : u.h;
      F big = 0, tail = 0;
      for (const F &v : g) {
        big = std::max(big, std::fabs(v));
        if (!std::isfinite((double)v)) p.ok = false;
      }
      for (size_t m = 0; m < g.size() / J; ++m)
        for (int k = 0; k < J; ++k) {
          F a = 0;
          for (int j = 0; j < J; ++j) a += ct[k][j] * g[m * J + j];
          p.C[(size_t)(w * EXP_KP + k) * M1p + m] = (double)a;
          if (k >= J - 2) tail = std::max(tail, std::fabs(a));
        }
      if (!(tail <= (F)tol * big)) p.ok = false;
    }
  });
}

}  // namespace

ExpTables exp_build(const std::vector<ExpNetIn> &nets, int ntypes, int M1p, bool f64) {
  const int K = f64 ? EXP_K64 : EXP_K32;
  const double tol = f64 ? 0x1p-52 : 0x1p-25;
  ExpTables t;
  t.K = K;
  t.M1p = M1p;
  const int nn = (int)nets.size();
  std::vector<NetT> nt(nets.begin(), nets.end());
  const int pmax = std::min(EXP_PMAX, EXP_BITS / ntypes);
  std::vector<std::vector<Piece>> done(nn);
  std::vector<Piece> todo;
  // Pieces below s = 1 of a centre type's nets, so far or at least: most of an
  // atom's neighbours lie beyond 1 A, and nets so rough that they lie in more
  // pieces than the atom's rows hold have no expansion.
  auto rough = [&]() {
    for (int c = 0; c < ntypes; ++c) {
      int bulk = 0;
      for (int u = 0; u < ntypes; ++u) {
        for (auto &p : done[c * ntypes + u]) bulk += p.lo < 1.0 ? 1 : 0;
        for (auto &p : todo) bulk += p.net == c * ntypes + u && p.lo < 1.0 ? 1 : 0;
      }
      if (bulk > EXP_SEG - 4) return true;
    }
    return false;
  };
  // Halve until every interval is within tol; intervals past a net's pmax-th
  // from the left can never be used.  False: no expansion.
  auto halve = [&](bool extended, double tl) {
    for (int level = 0; level < 10 && !todo.empty(); ++level) {
      const bool good = extended ? fit_pieces<long double, EXP_K64>(nt, M1p, tl, todo)
                        : f64    ? fit_pieces<double, EXP_K64>(nt, M1p, tl, todo)
                                 : fit_pieces<double, EXP_K32>(nt, M1p, tl, todo);
      if (!good) return false;
      std::vector<Piece> rest;
      for (auto &p : todo) {
        if (p.ok) {
          done[p.net].push_back(std::move(p));
        } else {
          Piece a, b;
          a.net = b.net = p.net;
          a.lo = p.lo;
          a.hi = b.lo = 0.5 * (p.lo + p.hi);
          b.hi = p.hi;
          rest.push_back(a);
          rest.push_back(b);
        }
      }
      for (int k = 0; k < nn; ++k) {
        std::vector<double> lo;
        for (auto &p : done[k]) lo.push_back(p.lo);
        for (auto &p : rest)
          if (p.net == k) lo.push_back(p.lo);
        if ((int)lo.size() <= pmax) continue;
        std::sort(lo.begin(), lo.end());
        const double cut = lo[pmax];
        auto past = [&](const Piece &p) { return p.net == k && p.lo >= cut; };
        done[k].erase(std::remove_if(done[k].begin(), done[k].end(), past), done[k].end());
        rest.erase(std::remove_if(rest.begin(), rest.end(), past), rest.end());
      }
      todo.swap(rest);
      if (rough()) return false;
    }
    return true;
  };
  // For the extended precision, double finds the intervals first, to above its
  // own rounding; [0, 2] before the rest, which says of rough nets that they
  // are (four and more types in double: 60 ms and more of work for nothing).
  for (int far = 0; far < 2; ++far) {
    todo.clear();
    for (int k = 0; k < nn; ++k)
      for (double hi = far ? 2.0 * EXP_SMIN : EXP_SMIN; hi <= (far ? EXP_SMAX : EXP_SMIN); hi *= 2.0) {
        Piece p;
        p.net = k;
        p.lo = far ? 0.5 * hi : 0.0;
        p.hi = hi;
        todo.push_back(p);
      }
    if (!halve(false, f64 ? EXP_PRE : tol)) return t;
  }
  for (int far = 0; f64 && far < 2; ++far) {
    todo.clear();
    for (auto &v : done) {
      std::vector<Piece> rest;
      for (auto &p : v) ((p.lo >= EXP_SMIN) == (far != 0) ? todo : rest).push_back(std::move(p));
      v.swap(rest);
    }
    if (!halve(true, tol)) return t;
  }
  // the contiguous run of pieces from 0
  double smax = EXP_SMAX;
  for (int k = 0; k < nn; ++k) {
    auto &v = done[k];
    std::sort(v.begin(), v.end(), [](const Piece &a, const Piece &b) { return a.lo < b.lo; });
    double hi = 0.0;
    size_t q = 0;
    while (q < v.size() && v[q].lo == hi) hi = v[q++].hi;
    v.resize(q);
    smax = std::min(smax, hi);
    t.P = std::max(t.P, (int)q);
  }
  if (smax < EXP_SMIN) return t;
  todo.clear();
  if (rough()) return t;
  t.smax = smax;
  const size_t row = (size_t)2 * EXP_KP * M1p;
  t.lo.assign((size_t)nn * t.P, HUGE_VAL);
  t.mid.assign((size_t)nn * t.P, 0.0);
  t.ih.assign((size_t)nn * t.P, 0.0);
  t.C.assign((size_t)nn * t.P * row, 0.0);
  for (int k = 0; k < nn; ++k)
    for (size_t q = 0; q < done[k].size(); ++q) {
      const size_t at = (size_t)k * t.P + q;
      t.lo[at] = done[k][q].lo;
      t.mid[at] = 0.5 * (done[k][q].lo + done[k][q].hi);
      t.ih[at] = 2.0 / (done[k][q].hi - done[k][q].lo);
      std::copy(done[k][q].C.begin(), done[k][q].C.end(), t.C.begin() + at * row);
    }
  t.ok = true;
  return t;
}

}  // namespace dpk
