// Shapes of the matrix-core float32 frame transform (split.hip), shared by the
// host tables (split_tables.cpp) and the kernel.
//
// The aperture is taken about its centre: with theta_i(p) = pi (2 i - L + 1) p / N
// (a unit phase per output away from the image transform, which |Y|^2 does not
// see), cells i and L - 1 - i have opposite phase angles, so a line x[L] of the
// aperture enters only as its sums s_i = x_i + x_{L-1-i} and differences
// d_i = x_i - x_{L-1-i}, i < K = L / 2:
//   C(p) = sum_i s_i cos theta_i(p),  S(p) = sum_i d_i sin theta_i(p),
//   Y(p) = C(p) + i S(p),  Y(-p) = C(p) - i S(p),  p = q - L.
// Outputs p = 0 .. L-1 are the base half, the others follow as partners.  At
// p = 0 only C is needed and at p = -L only S, so the two share base slot 0
// (cosines of p = 0, sines of p = L).
#pragma once

#include "shape.h"

namespace moff {

constexpr bool split_grid(int N) { return N == 64 || N == 128; }

struct SplitShape {
  int N, L, K;          // grid, aperture side, folded length
  int NW;               // waves per workgroup: one 16-wide block of base columns each
  int RP;               // row pairs each wave grids (iy = i and L - 1 - i, i = wave + NW j)
  int GP;               // gathered grid: row pitch, complex float32 elements
  int FP;               // folded grid: row pitch, bytes
};

constexpr SplitShape split_shape(int N) {
  const int L = N / 2, K = L / 2, NW = L / 16;
  // folded row: {sum, difference along x} x {re, im} x {high, low half} x K sixteen-bit values, plus 16 bytes
  // (16 consecutive rows then start 16 bytes apart modulo the LDS width)
  return SplitShape{N, L, K, NW, K / NW, L + 2, 8 * K * 2 + 16};
}

// Position of folded index i in a folded row or a phase-factor operand, in
// sixteen-bit elements, so that lane group g of an operand read holds just the
// indices whose row-stage results it receives (accumulator rows 4 g + j).
// K = 32: [8 g + t] is i = 4 g + t (t < 4) or 16 + 4 g + t - 4; the high and
// the low half are separate arrays.  K = 16: [8 g + t] is the high half of
// i = 4 g + t (t < 4) or the low half of i = 4 g + t - 4.
constexpr int split_pos(int K, int i, int lo) {
  return K == 32 ? 32 * lo + 8 * ((i % 16) / 4) + 4 * (i / 16) + i % 4 : 8 * (i / 4) + 4 * lo + i % 4;
}

// Dynamic LDS, byte offsets: gathered grid, folded grid, calibrated samples
// e[n_ant + 1] (last slot zero), gains, self power.
struct SplitLayout {
  int g, f, e, gl, pw, end;
};
constexpr SplitLayout split_layout(int N, int n_ant) {
  const SplitShape s = split_shape(N);
  SplitLayout m{};
  m.g = 0;
  m.f = s.L * s.GP * 8;
  m.e = m.f + 2 * s.K * s.FP;
  m.pw = align_up(m.e + 8 * (n_ant + 1), 16);
  m.gl = m.pw + 8 * n_ant;
  m.end = m.gl + 8 * n_ant;
  return m;
}

// Phase factors are scaled by 2^split_coef and folded grid values kept at or
// below 2^kSplitField, so that a row-stage result, at most
// 2 K 2^kSplitField 2^split_coef = 2^15, fits binary16.  The bound on the folded
// values is that of the cell with the most table weight and of every sample at its
// largest, so they lie far below it, the more so where a few antennas or frames are
// loud; their low halves meet the floor of binary16 (2^-25) first, and take what
// the phase factors can spare (2^8 and 2^1: an antenna 1e4 times as loud as 203
// others, seven samples, N = 64: relative error 3.8e-7 with 2^5 and 2^4, 1.1e-7).
constexpr int kSplitField = 8;
constexpr int split_coef(int N) { return N == 64 ? 2 : 1; }

// binary16 numbers per phase factor.  Two keep 22 bits or more, but their rounding
// is the same in every frame and does not average out as the samples' does: with
// two the error of an image under the uv-plane rule, which takes out the part
// proportional to the image, came to 1.1 times the FFT kernel's at N = 64 and 0.9
// to 1.05 at N = 128 (203 antennas of dense complex tables; without that rule to
// 0.5 to 0.7).  Images under that rule take a third (33 bits): at N = 64 in both
// stages (0.65 of the FFT's error, for 3 to 19 % more time), at N = 128 in the row
// stage only (0.8 to 1.0, 5 %), whose column stage has 4 times as many products and
// no registers left.
constexpr int kSplitParts = 3;
constexpr bool split_third_in_columns(int N) { return N == 64; }

}  // namespace moff
