// C entry to the host side of the net expansions, for tests/test_expand_host.py.
#include <cstring>

#include "dp_expand.h"

// weights: net after net, layer after layer, W [in][out] then b.  Returns 0
// where the nets have no expansion; else the tables of nets x P pieces.
extern "C" int expand_host(int ntypes, int nl, const int *w, int lin, const double *weights, int f64, int *P,
                           double *smax, double *lo, double *mid, double *ih, double *C) {
  std::vector<dpk::ExpNetIn> nets((size_t)ntypes * ntypes);
  for (auto &n : nets) {
    n.n_layers = nl;
    n.lin = lin != 0;
    for (int l = 0; l <= nl; ++l) n.w[l] = w[l];
    for (int l = 0; l < nl; ++l) {
      n.W[l].assign(weights, weights + w[l] * w[l + 1]);
      weights += w[l] * w[l + 1];
      n.b[l].assign(weights, weights + w[l + 1]);
      weights += w[l + 1];
    }
  }
  const dpk::ExpTables t = dpk::exp_build(nets, ntypes, (w[nl] + 15) / 16 * 16, f64 != 0);
  if (!t.ok) return 0;
  *P = t.P;
  *smax = t.smax;
  std::memcpy(lo, t.lo.data(), sizeof(double) * t.lo.size());
  std::memcpy(mid, t.mid.data(), sizeof(double) * t.mid.size());
  std::memcpy(ih, t.ih.data(), sizeof(double) * t.ih.size());
  std::memcpy(C, t.C.data(), sizeof(double) * t.C.size());
  return 1;
}
