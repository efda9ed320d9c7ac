// Host tables of the visibility-route (FX) image (fx.hip), built on first use
// by fx_tables.cpp.  Pure C++17, no HIP.
#pragma once

#include <cstdint>
#include <vector>

#include "plan.h"

namespace moff {

// Tables of the visibility-route image (Sec. 2, eq. dirty-image-FX with
// eq. e-field-conv), built on first use:
//   order    : antennas in the order of their footprint cells (row, column); the
//              visibilities are formed in this order, so that the pairs of a
//              lag row lie close together.  Positions below are in this order.
//   rows     : lag rows that are summed, (p * n_types + q) * NL + dy, footprint
//              offset dy - (L - 1) = iy0_a - iy0_b of pairs (a of type p, b of
//              type q): p == q, dy up to L - 1 (row L - 1: columns up to L - 1),
//              and p < q, every dy.  The others are mirrors (types swapped,
//              offset negated) and hold the conjugate sums.
//   ptr      : [rows + 1] the rows' entries, in ascending (a, b) position
//   ab / dx  : per entry, min(a, b) * n_ant + max(a, b) (positions), the
//              upper-triangle visibility, with kFxConjBit set when a > b (read
//              it conjugated), and the column ix0_a - ix0_b + L - 1.  a == b
//              only when the zero-spacing terms are kept.
//   xcorr    : per type pair, X[u][v] = sum K_p[s][t] conj(K_q[s - u + k_q - 1][t - v + k_q - 1])
//              on a (k_p + k_q - 1)^2 support, stored [pair][xs][xs] as float32 (re, im).
constexpr uint32_t kFxConjBit = 0x80000000u;

struct FxTables {
  int NL = 0, xs = 0;
  std::vector<int32_t> order, rows, ptr, ab;
  std::vector<uint16_t> dx;
  std::vector<float> xcorr;
};
void build_fx_tables(const HostPlan& hp, bool keep_autos, FxTables* t);

}  // namespace moff
