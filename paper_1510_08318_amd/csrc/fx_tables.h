// Host tables of the visibility-route (FX) image (fx.hip), built on first use
// by fx_tables.cpp.  Pure C++17, no HIP.
#pragma once

#include <algorithm>
#include <cstddef>
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

// Staged blocks: 4+4-bit samples as int8 planes (re, im) of 64 samples;
// complex64 samples, calibrated, as three bfloat16 levels of x and of y, of 32.
constexpr int kFxTile = 64;
constexpr int fx_step(bool ci4) { return ci4 ? 64 : 32; }
constexpr size_t fx_block_bytes(bool ci4) { return static_cast<size_t>(kFxTile) * (ci4 ? 64 * 2 : 32 * 2 * 6); }
inline size_t fx_plane_bytes(bool ci4, int n_ant, int64_t n_time) {   // of one channel
  return fx_block_bytes(ci4) * ((n_ant + kFxTile - 1) / kFxTile) *
         static_cast<size_t>((n_time + fx_step(ci4) - 1) / fx_step(ci4));
}

// How a call is cut into launches: channels in chunks whose workspace keeps within
// 2 GiB, but of eight where there are eight (one per XCD: with fewer, XCDs idle), and
// the samples in passes over time where they leave no room for eight channels.
// Between passes the visibilities are summed in float64: 16 bytes per pair, read and
// written once per pass.  A pass therefore holds at least as many bytes of samples
// as a channel has of visibilities (8 bytes per pair; 2600 complex64 or 16000
// 4+4-bit samples at 4000 antennas), also where that takes the eight channels
// beyond 2 GiB: from 2900 antennas on, 4 GiB at 4000.  (With what was left of 2 GiB a
// pass was a single step from 3340 antennas on: 8 channels of 4000 antennas took 69
// ms for 3000 complex64 samples and 224 ms for 20000 of 4+4 bits, 10.6 and 9.0 here.)
struct FxChunks {
  int channels;              // per launch
  int64_t pass;              // time samples per pass
  size_t samples, sums;      // staged samples and running sums (0: one pass), bytes per channel
  size_t per_channel;        // all of a channel's workspace, bytes
};
// fixed: the workspace per channel beside the samples and the running sums
inline FxChunks fx_chunks(bool ci4, int n_ant, int n_chan, int64_t n_time, size_t fixed) {
  const size_t budget = size_t(2) << 30, pairs = static_cast<size_t>(n_ant) * n_ant;
  const size_t few = static_cast<size_t>(std::min(n_chan, 8));
  const size_t step = fx_plane_bytes(ci4, n_ant, 1), whole = fx_plane_bytes(ci4, n_ant, n_time);
  const size_t least = std::max<size_t>(1, 8 * pairs / step) * step;
  FxChunks f{};
  f.pass = n_time;
  f.samples = whole;
  if ((fixed + whole) * few > budget && whole > least) {
    f.sums = 16 * pairs;
    const size_t room = budget / few > fixed + f.sums ? budget / few - fixed - f.sums : 0;
    f.samples = std::max(least, room / step * step);
    f.pass = static_cast<int64_t>(f.samples / step) * fx_step(ci4);
  }
  f.per_channel = (fixed + f.sums + f.samples + 255) / 256 * 256;
  f.channels = static_cast<int>(
      std::min<size_t>({static_cast<size_t>(n_chan), std::max(few, budget / f.per_channel), size_t(65535)}));
  return f;
}

}  // namespace moff
