// Host tables of the visibility-route (FX) image (declared in fx_tables.h).
// Pure C++17, no HIP.
#include "fx_tables.h"

#include <algorithm>
#include <complex>
#include <numeric>

namespace moff {

void build_fx_tables(const HostPlan& hp, bool keep_autos, FxTables* t) {
  const int na = hp.n_ant, L = hp.L, NL = 2 * L - 1, nt = hp.n_ktypes;
  int kmax = 1;
  for (int p = 0; p < nt; ++p) kmax = std::max(kmax, static_cast<int>(hp.ktype_k[p]));
  t->NL = NL;
  t->xs = 2 * kmax - 1;
  // pair responses: cross-correlation of two tables placed at the same cell
  const int xs = t->xs;
  t->xcorr.assign(static_cast<size_t>(nt) * nt * xs * xs * 2, 0.f);
  for (int p = 0; p < nt; ++p)
    for (int q = 0; q < nt; ++q) {
      const int ka = hp.ktype_k[p], kb = hp.ktype_k[q], side = ka + kb - 1;
      const float* Ka = hp.kvals.data() + 2 * static_cast<size_t>(hp.ktype_off[p]);
      const float* Kb = hp.kvals.data() + 2 * static_cast<size_t>(hp.ktype_off[q]);
      std::vector<std::complex<double>> X(static_cast<size_t>(side) * side);
      for (int s0 = 0; s0 < ka; ++s0)
        for (int s1 = 0; s1 < ka; ++s1) {
          const std::complex<double> x(Ka[2 * (s0 * ka + s1)], Ka[2 * (s0 * ka + s1) + 1]);
          for (int r0 = 0; r0 < kb; ++r0)
            for (int r1 = 0; r1 < kb; ++r1) {
              const std::complex<double> y(Kb[2 * (r0 * kb + r1)], -Kb[2 * (r0 * kb + r1) + 1]);
              X[static_cast<size_t>(s0 - r0 + kb - 1) * side + (s1 - r1 + kb - 1)] += x * y;
            }
        }
      float* dst = t->xcorr.data() + static_cast<size_t>(p * nt + q) * xs * xs * 2;
      for (int u = 0; u < side; ++u)
        for (int v = 0; v < side; ++v) {
          dst[2 * (u * xs + v)] = static_cast<float>(X[static_cast<size_t>(u) * side + v].real());
          dst[2 * (u * xs + v) + 1] = static_cast<float>(X[static_cast<size_t>(u) * side + v].imag());
        }
    }
  // antennas by footprint cell
  t->order.resize(na);
  std::iota(t->order.begin(), t->order.end(), 0);
  std::stable_sort(t->order.begin(), t->order.end(), [&](int x, int y) {
    return hp.iy0[x] != hp.iy0[y] ? hp.iy0[x] < hp.iy0[y] : hp.ix0[x] < hp.ix0[y];
  });
  // lag rows that are summed, and the entries of each, by counting sort
  std::vector<int32_t> base(static_cast<size_t>(nt) * nt, -1);
  for (int p = 0; p < nt; ++p)
    for (int q = p; q < nt; ++q) {
      base[p * nt + q] = static_cast<int32_t>(t->rows.size());
      for (int dy = 0; dy < (p == q ? L : NL); ++dy) t->rows.push_back((p * nt + q) * NL + dy);
    }
  auto row_of = [&](int a, int b, int* dx) {   // antennas; -1: the mirror is summed
    const int p = hp.ant_ktype[a], q = hp.ant_ktype[b];
    const int dy = hp.iy0[a] - hp.iy0[b] + L - 1;
    *dx = hp.ix0[a] - hp.ix0[b] + L - 1;
    if (p > q || (p == q && (dy > L - 1 || (dy == L - 1 && *dx > L - 1)))) return -1;
    return base[p * nt + q] + dy;
  };
  auto each = [&](auto&& f) {
    for (int i = 0; i < na; ++i)
      for (int j = 0; j < na; ++j) {
        if (i == j && !keep_autos) continue;
        int dx = 0;
        const int r = row_of(t->order[i], t->order[j], &dx);
        if (r >= 0) f(i, j, r, dx);
      }
  };
  t->ptr.assign(t->rows.size() + 1, 0);
  each([&](int, int, int r, int) { ++t->ptr[r + 1]; });
  for (size_t r = 0; r < t->rows.size(); ++r) t->ptr[r + 1] += t->ptr[r];
  t->ab.assign(static_cast<size_t>(t->ptr.back()), 0);
  t->dx.assign(t->ab.size(), 0);
  std::vector<int32_t> fill(t->ptr.begin(), t->ptr.end() - 1);
  each([&](int i, int j, int r, int dx) {
    const uint32_t upper = static_cast<uint32_t>(std::min(i, j)) * na + std::max(i, j);
    const size_t at = static_cast<size_t>(fill[r]++);
    t->ab[at] = static_cast<int32_t>(upper | (i > j ? kFxConjBit : 0u));
    t->dx[at] = static_cast<uint16_t>(dx);
  });
}

}  // namespace moff
