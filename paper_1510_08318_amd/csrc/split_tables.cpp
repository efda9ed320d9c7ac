// Host tables of the matrix-core float32 frame transform (split.hip).  Built
// with -ffp-contract=off, as plan.cpp.
#include <algorithm>
#include <cmath>
#include <numeric>

#include "plan.h"
#include "split_shape.h"

namespace moff {

void build_split_tables(HostPlan& P) {
  HostPlan::Split& T = P.split;
  T = HostPlan::Split{};
  if (!split_grid(P.N)) return;
  const SplitShape S = split_shape(P.N);
  const int L = S.L, K = S.K, NW = S.NW;
  if (split_layout(P.N, P.n_ant).end > kMfmaLdsMax) return;

  // ---- phase factors, [block of 16 base outputs][cos, sin][part, high first][lane][8]
  const int parts = kSplitParts;
  T.coef.assign(static_cast<size_t>(NW) * 2 * parts * 64 * 8, 0);
  for (int b = 0; b < NW; ++b)
    for (int part = 0; part < 2; ++part)
      for (int lane = 0; lane < 64; ++lane)
        for (int i = 0; i < K; ++i) {
          const int base = 16 * b + lane % 16;
          const int p = (part == 1 && base == 0) ? L : base;
          // angle pi (2 i - L + 1) p / N, reduced modulo 2 N units of pi / N
          const long long u = (static_cast<long long>(2 * i - L + 1) * p) % (2 * P.N);
          const double a = 3.14159265358979323846264338327950288 * static_cast<double>(u) / P.N;
          double left = std::ldexp(part == 0 ? std::cos(a) : std::sin(a), split_coef(P.N));
          for (int q = 0; q < parts; ++q) {
            const uint16_t bits = to_binary16(left);
            left -= from_binary16(bits);
            for (int copy = 0; copy < (K == 16 ? 2 : 1); ++copy) {
              // K = 16: both halves of the data meet the same factor
              const int pos = split_pos(K, i, copy) - (K == 32 ? 32 * copy : 0);
              if (pos / 8 != lane / 16) continue;
              T.coef[(((static_cast<size_t>(b) * 2 + part) * parts + q) * 64 + lane) * 8 + pos % 8] = bits;
            }
          }
        }

  // ---- gather programs, one per wave: the non-empty cells of its row pairs,
  // longest first, 64 cells (one per lane) at a time; a group of cells takes as
  // many steps as its longest one.
  T.real = true;
  for (size_t i = 1; i < P.kvals.size(); i += 2) T.real = T.real && P.kvals[i] == 0.f;
  const uint32_t zero_slot = static_cast<uint32_t>(8 * P.n_ant);
  struct Step {
    uint32_t x[64];
    float wr[64], wi[64];
    bool end;
  };
  std::vector<std::vector<Step>> prog(NW);
  for (int w = 0; w < NW; ++w) {
    struct Cell {
      int at, n, dst;
    };
    std::vector<Cell> cells;
    for (int j = 0; j < S.RP; ++j)
      for (int up = 0; up < 2; ++up) {
        const int i = w + NW * j, iy = up ? L - 1 - i : i, lr = up * S.RP + j;
        for (int ix = 0; ix < L; ++ix) {
          const int at = iy * L + ix, n = P.csr_ptr[at + 1] - P.csr_ptr[at];
          if (n > 0) cells.push_back({at, n, (lr * S.GP + ix) * 8});
        }
      }
    std::stable_sort(cells.begin(), cells.end(), [](const Cell& a, const Cell& b) { return a.n > b.n; });
    const uint32_t pad_dst = static_cast<uint32_t>(L * 8);   // the pad column of the wave's first row: never read
    for (size_t c0 = 0; c0 < cells.size(); c0 += 64) {
      for (int s = 0; s < cells[c0].n; ++s) {
        Step st{};
        st.end = s + 1 == cells[c0].n;
        for (int lane = 0; lane < 64; ++lane) {
          const bool has = c0 + lane < cells.size();
          const uint32_t dst = has ? static_cast<uint32_t>(cells[c0 + lane].dst) : pad_dst;
          uint32_t e = zero_slot;
          if (has && s < cells[c0 + lane].n) {
            const int k = P.csr_ptr[cells[c0 + lane].at] + s;
            e = static_cast<uint32_t>(8 * P.csr_ant[k]);
            st.wr[lane] = P.kvals[2 * P.csr_tap[k]];
            st.wi[lane] = P.kvals[2 * P.csr_tap[k] + 1];
          }
          st.x[lane] = e | (dst << 16);
        }
        prog[w].push_back(st);
      }
    }
    while (prog[w].size() % kSplitBatch) {
      Step st{};
      for (int lane = 0; lane < 64; ++lane) st.x[lane] = zero_slot | (pad_dst << 16);
      prog[w].push_back(st);
    }
    T.steps = std::max(T.steps, static_cast<int>(prog[w].size()));
  }
  T.steps = std::max(T.steps, kSplitBatch);   // (all-zero tables have no steps: the first batch is still read)
  const int SP = T.steps / 2;   // pairs of steps
  T.prog.assign(static_cast<size_t>(NW) * SP * 64 * 4, 0);
  if (!T.real) T.progi.assign(static_cast<size_t>(NW) * SP * 64 * 2, 0.f);
  const int FW = (T.steps + 31) / 32;
  T.ends.assign(static_cast<size_t>(NW) * FW, 0);
  T.n_steps.assign(NW, 0);
  for (int w = 0; w < NW; ++w) {
    T.n_steps[w] = static_cast<int>(prog[w].size());
    for (size_t s = 0; s < prog[w].size(); ++s) {
      if (prog[w][s].end) T.ends[static_cast<size_t>(w) * FW + s / 32] |= 1u << (s % 32);
      for (int lane = 0; lane < 64; ++lane) {
        const size_t at = ((static_cast<size_t>(w) * SP + s / 2) * 64 + lane);
        T.prog[at * 4 + 2 * (s % 2)] = prog[w][s].x[lane];
        T.prog[at * 4 + 2 * (s % 2) + 1] = float_bits(prog[w][s].wr[lane]);
        if (!T.real) T.progi[at * 2 + s % 2] = prog[w][s].wi[lane];
      }
    }
  }

  // ---- the largest folded value per unit of the largest sample component
  double wmax = 0.0;
  for (int iy = 0; iy < K; ++iy)
    for (int ix = 0; ix < K; ++ix) {
      double sum = 0.0;
      for (int q = 0; q < 4; ++q) {
        const int at = (q & 1 ? L - 1 - iy : iy) * L + (q & 2 ? L - 1 - ix : ix);
        for (int k = P.csr_ptr[at]; k < P.csr_ptr[at + 1]; ++k)
          sum += std::fabs(static_cast<double>(P.kvals[2 * P.csr_tap[k]])) +
                 std::fabs(static_cast<double>(P.kvals[2 * P.csr_tap[k] + 1]));
      }
      wmax = std::max(wmax, sum);
    }
  T.wmax = wmax > 0.0 ? wmax : 1.0;
  T.on = true;
}

}  // namespace moff
