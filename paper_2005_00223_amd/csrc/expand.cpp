// Host side of the embedding nets' Chebyshev expansions (dp_expand.h): the
// nets evaluated with their tangents at Chebyshev nodes, the coefficients
// by the discrete cosine sum, the pieces by halving.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <iterator>
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

// G[m], dG[m] of a net at s, forward mode through its layers.  Two outputs
// at a time, their four sums in registers: in extended precision a sum kept
// in memory costs a 10-byte store and load per term.
template <typename F>
void net_eval(const ExpNetIn &n, F s, std::vector<F> &h, std::vector<F> &hd, std::vector<F> &z, std::vector<F> &zd) {
  h.assign(1, s);
  hd.assign(1, F(1));
  for (int l = 0; l < n.n_layers; ++l) {
    const int in = n.w[l], out = n.w[l + 1];
    z.resize(out);
    zd.resize(out);
    const double *W = n.W[l].data();
    for (int o = 0; o < out; o += 2) {
      const int o1 = o + 1 < out ? o + 1 : o;
      F a = (F)n.b[l][o], b = (F)n.b[l][o1], ad = 0, bd = 0;
      for (int i = 0; i < in; ++i) {
        const F x = h[i], xd = hd[i], wa = (F)W[(size_t)i * out + o], wb = (F)W[(size_t)i * out + o1];
        a += x * wa;
        ad += xd * wa;
        b += x * wb;
        bd += xd * wb;
      }
      z[o] = a;
      zd[o] = ad;
      z[o1] = b;
      zd[o1] = bd;
    }
    if (!(n.lin && l + 1 == n.n_layers))
      for (int o = 0; o < out; ++o) {
        const F t = std::tanh(z[o]);
        z[o] = t;
        zd[o] *= F(1) - t * t;
        if (out == in || out == 2 * in) {
          const int k = o >= in ? o - in : o;
          z[o] += h[k];
          zd[o] += hd[k];
        }
      }
    h.swap(z);
    hd.swap(zd);
  }
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

// Interpolates the pieces' nets in the real type F and sets ok where the
// last two coefficients of every feature are within tol.
template <typename F>
bool fit_pieces(const std::vector<ExpNetIn> &nets, int M1p, int K, double tol, std::vector<Piece> &pieces) {
  const F pi = (F)3.14159265358979323846264338327950288L;
  const int M1 = pieces.empty() ? 0 : nets[0].w[nets[0].n_layers];
  const size_t blk = (size_t)K * M1;
  // threads only where the work outweighs starting them
  const size_t nth = sizeof(F) > sizeof(double) ? 4 : 1;
  std::vector<F> val(pieces.size() * 2 * blk), ct((size_t)K * K);
  for (int k = 0; k < K; ++k)
    for (int j = 0; j < K; ++j)
      ct[k * K + j] = std::cos(pi * (F)k * ((F)j + F(0.5)) / K) * (k == 0 ? F(1) : F(2)) / K;
  bool good = parallel_for(pieces.size() * K, nth, [&](size_t q) {
    const Piece &p = pieces[q / K];
    const int j = (int)(q % K);
    std::vector<F> h, hd, z, zd;
    net_eval<F>(nets[p.net], ((F)p.lo + (F)p.hi) / 2 + ((F)p.hi - (F)p.lo) / 2 * std::cos(pi * ((F)j + F(0.5)) / K), h,
                hd, z, zd);
    std::copy(h.begin(), h.end(), val.begin() + q / K * 2 * blk + (size_t)j * M1);
    std::copy(hd.begin(), hd.end(), val.begin() + (q / K * 2 + 1) * blk + (size_t)j * M1);
  });
  good = good && parallel_for(pieces.size(), nth, [&](size_t q) {
    Piece &p = pieces[q];
    p.C.assign((size_t)2 * EXP_KP * M1p, 0.0);
    p.ok = true;
    std::vector<F> acc(M1);
    for (int w = 0; w < 2; ++w) {
      const F *g = val.data() + (q * 2 + w) * blk;
      F big = 0, tail = 0;
      for (size_t e = 0; e < blk; ++e) {
        big = std::max(big, std::fabs(g[e]));
        if (!std::isfinite((double)g[e])) p.ok = false;
      }
      for (int k = 0; k < K; ++k) {
        std::fill(acc.begin(), acc.end(), F(0));
        for (int j = 0; j < K; ++j)
          for (int m = 0; m < M1; ++m) acc[m] += ct[k * K + j] * g[(size_t)j * M1 + m];
        for (int m = 0; m < M1; ++m) {
          p.C[(size_t)(w * EXP_KP + k) * M1p + m] = (double)acc[m];
          if (k >= K - 2) tail = std::max(tail, std::fabs(acc[m]));
        }
      }
      if (!(tail <= (F)tol * big)) p.ok = false;
    }
  });
  return good;
}

}  // namespace

ExpTables exp_build(const std::vector<ExpNetIn> &nets, int ntypes, int M1p, bool f64) {
  const int K = f64 ? EXP_K64 : EXP_K32;
  const double tol = f64 ? 0x1p-52 : 0x1p-25;
  ExpTables t;
  t.K = K;
  t.M1p = M1p;
  const int nn = (int)nets.size();
  const int pmax = std::min(EXP_PMAX, EXP_BITS / ntypes);
  std::vector<std::vector<Piece>> done(nn);
  std::vector<Piece> todo;
  for (int k = 0; k < nn; ++k)
    for (double hi = 2.0; hi <= EXP_SMAX; hi *= 2.0) {
      Piece p;
      p.net = k;
      p.lo = hi > 2.0 ? 0.5 * hi : 0.0;
      p.hi = hi;
      todo.push_back(p);
    }
  // Halve until every interval is within tol; intervals past a net's pmax-th
  // from the left can never be used.  For the extended precision, double
  // finds the intervals first, to above its own rounding.
  auto halve = [&](bool extended, double tl) {
    for (int level = 0; level < 10 && !todo.empty(); ++level) {
      if (!(extended ? fit_pieces<long double>(nets, M1p, K, tl, todo) : fit_pieces<double>(nets, M1p, K, tl, todo)))
        return false;
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
    }
    return true;
  };
  if (!halve(false, f64 ? EXP_PRE : tol)) return t;
  if (f64) {
    todo.clear();
    for (auto &v : done) {
      std::move(v.begin(), v.end(), std::back_inserter(todo));
      v.clear();
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
  // rough nets: an atom's neighbours, most of them beyond 1 A, would lie in
  // more pieces than its rows hold
  for (int c = 0; c < ntypes; ++c) {
    int bulk = 0;
    for (int u = 0; u < ntypes; ++u)
      for (auto &p : done[c * ntypes + u]) bulk += p.lo < 1.0 ? 1 : 0;
    if (bulk > EXP_SEG - 4) return t;
  }
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
