// Visibility-route (FX) imaging of one integration on the device, for
// cross-checks of the MOFF image by the paper's other method (Sec. 2: the
// time-averaged cross-products of the calibrated antenna fields, eq. cc-vis,
// gridded with each pair's power response, the cross-correlation of the two
// aperture illuminations, eq. e-field-conv, and transformed once, eq.
// dirty-image-FX, give the MOFF image; with the zero-spacing a == b terms left
// out it equals the image with the antennas' self power removed).
//
//   fx_correlate_kernel  V[c][a][b] = sum_t e_a conj(e_b), e = g E, for a <= b
//                        (the upper triangle; V is Hermitian): float32 as three
//                        bfloat16 levels on the matrix cores over 32-sample
//                        chunks, chunks summed in float64 (complex64 samples);
//                        fx_correlate_i8_kernel: exact integer products on the
//                        matrix cores (4+4-bit samples)
//   one table type:
//   fx_bin_cells_kernel  H[c][k] = sum of V[c][a][b] over the pairs whose
//                        footprints are offset by that of the k-th cell with
//                        pairs (half the cells: the others are conjugates)
//   fx_row_kernel        Z[c][ly][q] = sum_lx H[c][ly][lx] w^((lx - L + 1)(q - N/2))
//                        (rows up to the zero lag; the others are conjugates)
//   fx_col_kernel        I[c][r][q] = scale P[r][q] Re sum_ly w^((ly - L + 1)(r - N/2)) Z[c][ly][q],
//                        P the table's power pattern, the transform of its
//                        autocorrelation (real, two columns per complex transform)
//   several types:
//   fx_bin_kernel        H[c][pq][dy][dx] the same per ordered pair of table
//                        types (p, q), a dense grid of offsets (dy, dx) - (L - 1)
//                        (plan-time CSR, fixed order); half the cells are
//                        summed, their mirrors H[qp][-dy][-dx] written as the
//                        conjugates
//   fx_lag_kernel        R[c][ly][lx] = sum_pq sum_(u,v) X_pq[u][v]
//                        H[c][pq][ly - u + k_q - 1][lx - v + k_q - 1]  (LDS-tiled;
//                        rows up to the zero lag)
//   fx_row_kernel, fx_col_kernel   as above, of R and without P
//
// w = exp(+2 pi i / N); lags span -(L - 1) .. L - 1, so the image comes out in
// the same pixel order as the MOFF image.  Every sum runs in a fixed order
// (no atomics); the correlator and the binning accumulate in float64, each
// pair response's lag sum in float32 (the pairs in float64), and the two
// transform passes run in float32; intermediate arrays are float32.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "dft.h"
#include "fx.h"
#include "fx_tables.h"
#include "ingest.h"

namespace moff {

namespace {

constexpr int kFxChunk = 32;   // time samples staged per step
constexpr unsigned kFxXcds = 8;  // accelerator dies (XCDs), each with its own L2

// Workgroups go to the XCDs round-robin by linear index.  For a 1-D grid of
// kFxXcds * ceil(n / kFxXcds) * per blocks over n channels of `per` blocks
// each, the channel of block b and its index within the channel: all blocks of
// a channel share one residue mod kFxXcds, so one XCD's L2 serves the data of
// that channel.  Returns false for the padding blocks.
__device__ __forceinline__ bool xcd_channel(unsigned b, unsigned per, int n, int* ch, unsigned* j) {
  const unsigned xcd = b % kFxXcds, s = b / kFxXcds;
  *ch = static_cast<int>(xcd + kFxXcds * (s / per));
  *j = s % per;
  return *ch < n;
}
inline size_t xcd_grid(size_t per, int n) { return per * kFxXcds * ((static_cast<size_t>(n) + kFxXcds - 1) / kFxXcds); }

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

}  // namespace

// Complex64 samples, on the matrix cores (v_mfma_f32_16x16x32_bf16): every
// calibrated float32 component is held as three bfloat16 numbers, high, middle
// and low, 8 bits each and so all 24 of it at float32's own range, and a
// product takes the six terms above 2^-24 (hh, hm, mh, mm, hl, lh) with float32
// accumulation: the accuracy of the float32 matrix instruction at 2.7 times its
// rate (64 channels x 128 samples of 1024 antennas: 438 us with that
// instruction, 294 here, of which the products take 87 at their peak rate and
// the conversions, repeated for every tile an antenna is in, most of the rest;
// relative error of the image 2.05e-7 and 2.02e-7).  The visibility matrix is Hermitian, V_ba = conj(V_ab), and the binning
// reads its upper triangle only, so only the tiles on and above the diagonal
// are formed.  One workgroup per (64 x 64 antenna tile, channel), four waves
// of a 32 x 32 sub-tile each (2 x 2 blocks of 16 x 16).  With e = x + i y,
//   Re V_ab = sum x_a x_b + y_a y_b,   Im V_ab = sum y_a x_b - sum x_a y_b.
// A and B take their samples in the same lane order, so each is summed once
// whatever order the instruction gives its contraction index; the accumulators
// hold D[4 (l / 16) + v][l % 16].  Each 32-sample chunk is summed in float32
// and the chunks in float64.
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 b16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 b16x8 __attribute__((ext_vector_type(8)));
constexpr int kC64Tile = 64;                // antennas per side of a tile
constexpr int kC64Pitch = kFxChunk + 8;     // LDS row, bfloat16: 16-byte operand reads of 16 rows hit distinct banks

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void fx_correlate_kernel(FxArgs a) {
  // [block a, b][x, y][high, middle, low][antenna][sample]
  __shared__ __attribute__((aligned(16))) __bf16 pl[2][2][3][kC64Tile][kC64Pitch];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wa = wave >> 1, wb = wave & 1, r16 = lane & 15, kk = lane >> 4;
  const int na = a.n_ant, n_tiles = (na + kC64Tile - 1) / kC64Tile;
  int cl;
  unsigned tri;
  if (!xcd_channel(blockIdx.x, static_cast<unsigned>(n_tiles * (n_tiles + 1) / 2), a.n_launch, &cl, &tri)) return;
  int t = static_cast<int>(tri), ta = 0;      // upper-triangle tile (ta, tb), tb >= ta
  while (ta < n_tiles && t >= n_tiles - ta) {
    t -= n_tiles - ta;
    ++ta;
  }
  if (ta >= n_tiles) return;                  // beyond the triangle (the launch has none)
  const int tb = ta + t;
  const int a0 = ta * kC64Tile, b0 = tb * kC64Tile, c = a.c0 + cl;
  const float2* E = reinterpret_cast<const float2*>(a.E);
  double acc[2][2][4][2] = {};
  // staging: thread = (antenna an, samples kC64Per sg ..), so each thread keeps
  // its two antennas' gains for the whole integration
  constexpr int kC64Per = kFxChunk * kC64Tile / 256;
  static_assert(kC64Per == 8, "one 16-byte row segment per thread, part and level");
  const int an = tid % kC64Tile, sg = tid / kC64Tile;
  const int ia = a0 + an, ib = b0 + an;
  // antennas past the last one read the last one with a zero gain (their rows
  // are not stored)
  auto gain_of = [&](int ant) {
    if (ant >= na) return make_float2(0.f, 0.f);
    return a.gains ? a.gains[static_cast<size_t>(c) * na + ant] : make_float2(1.f, 0.f);
  };
  const float2 gg[2] = {gain_of(ia), gain_of(ib)};
  const size_t stride = static_cast<size_t>(a.n_chan) * na;   // samples of consecutive times
  const float2* src[2];
#pragma unroll
  for (int blk = 0; blk < 2; ++blk) {
    const int ant = blk ? ib : ia;
    src[blk] = E + static_cast<size_t>(kC64Per * sg) * stride + static_cast<size_t>(c) * na + (ant < na ? ant : na - 1);
  }
  float2 raw[2][kC64Per];
  auto load_chunk = [&](int64_t t0) {   // all of a chunk's loads in flight at once
    const size_t at = static_cast<size_t>(t0) * stride;
    if (t0 + kFxChunk <= a.n_time) {    // uniform
#pragma unroll
      for (int i = 0; i < kC64Per; ++i)
#pragma unroll
        for (int blk = 0; blk < 2; ++blk) raw[blk][i] = src[blk][at + i * stride];
    } else {
#pragma unroll
      for (int i = 0; i < kC64Per; ++i)
#pragma unroll
        for (int blk = 0; blk < 2; ++blk) {
          raw[blk][i] = make_float2(0.f, 0.f);
          if (t0 + kC64Per * sg + i < a.n_time) raw[blk][i] = src[blk][at + i * stride];
        }
    }
  };
  load_chunk(0);
  for (int64_t t0 = 0; t0 < a.n_time; t0 += kFxChunk) {
#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
      b16x8 lv[2][3];
#pragma unroll
      for (int i = 0; i < kC64Per; i += 2) {
        const float2 v0 = cmul(gg[blk], raw[blk][i]), v1 = cmul(gg[blk], raw[blk][i + 1]);
#pragma unroll
        for (int part = 0; part < 2; ++part) {
          f32x2 x = part ? f32x2{v0.y, v1.y} : f32x2{v0.x, v1.x};
#pragma unroll
          for (int l = 0; l < 3; ++l) {
            const b16x2 h = __builtin_convertvector(x, b16x2);
            lv[part][l][i] = h[0];
            lv[part][l][i + 1] = h[1];
            if (l < 2) x -= __builtin_convertvector(h, f32x2);
          }
        }
      }
#pragma unroll
      for (int part = 0; part < 2; ++part)
#pragma unroll
        for (int l = 0; l < 3; ++l) *reinterpret_cast<b16x8*>(&pl[blk][part][l][an][kC64Per * sg]) = lv[part][l];
    }
    __syncthreads();
    if (t0 + kFxChunk < a.n_time) load_chunk(t0 + kFxChunk);   // in flight during the products
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      b16x8 A[2][3];
#pragma unroll
      for (int part = 0; part < 2; ++part)
#pragma unroll
        for (int l = 0; l < 3; ++l)
          A[part][l] = *reinterpret_cast<const b16x8*>(&pl[0][part][l][32 * wa + 16 * i + r16][8 * kk]);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        b16x8 B[2][3];
#pragma unroll
        for (int part = 0; part < 2; ++part)
#pragma unroll
          for (int l = 0; l < 3; ++l)
            B[part][l] = *reinterpret_cast<const b16x8*>(&pl[1][part][l][32 * wb + 16 * j + r16][8 * kk]);
        // x_a x_b + y_a y_b and y_a x_b - x_a y_b: the small terms of both
        // products first, so that a chunk's sum rounds twice at full size
        auto terms = [&](const b16x8 (&x)[3], const b16x8 (&y)[3], f32x4 r) {
          r = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[2], y[0], r, 0, 0, 0);
          r = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[0], y[2], r, 0, 0, 0);
          r = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[1], y[1], r, 0, 0, 0);
          r = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[1], y[0], r, 0, 0, 0);
          return __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[0], y[1], r, 0, 0, 0);
        };
        b16x8 N[3];   // - y_b
#pragma unroll
        for (int l = 0; l < 3; ++l) N[l] = -B[1][l];
        f32x4 re = {0.f, 0.f, 0.f, 0.f}, im = {0.f, 0.f, 0.f, 0.f};
        re = terms(A[0], B[0], re);
        im = terms(A[1], B[0], im);
        re = terms(A[1], B[1], re);
        im = terms(A[0], N, im);
        re = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[0][0], B[0][0], re, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[1][0], B[0][0], im, 0, 0, 0);
        re = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[1][0], B[1][0], re, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[0][0], N[0], im, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          acc[i][j][v][0] += re[v];
          acc[i][j][v][1] += im[v];
        }
      }
    }
    __syncthreads();
  }
  float2* V = a.V + static_cast<size_t>(cl) * na * na;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int ia = a0 + 32 * wa + 16 * i + 4 * kk + v, ib = b0 + 32 * wb + 16 * j + r16;
        if (ia >= na || ib >= na) continue;
        const float x = static_cast<float>(acc[i][j][v][0]), y = static_cast<float>(acc[i][j][v][1]);
        V[static_cast<size_t>(ia) * na + ib] = make_float2(x, y);
      }
}

// 4+4-bit samples: the cross-products are exact integer sums, formed on the
// matrix cores (v_mfma_i32_16x16x64_i8, int32 accumulation) from the raw
// samples; the gains are constant over the integration and are applied once,
// V_ab = g_a conj(g_b) sum_t E_a conj(E_b), in float64.  One workgroup per
// (64 x 64 antenna tile on or above the diagonal, channel), four waves of a
// 32 x 32 sub-tile each (2 x 2 blocks of 16 x 16).  Per 64-sample step the
// real and imaginary parts of both antenna blocks are staged in LDS as int8
// rows [antenna][sample], and each wave runs four products (re.re, im.im,
// im.re, re.im) per block; the next step's samples are loaded into registers
// while the current step's products run.  Samples are loaded four antennas at a
// time (unaligned 4-byte loads) for four samples, widened as packed bytes and
// transposed 4 x 4 in registers.  Bound by the vector work of the staging and
// the latency of its loads, not by the products (6 % of the matrix rate): byte
// by byte, with a bounds check and a 64-bit address per byte, it took 132 us at
// 256 channels x 256 samples of 350 antennas, this form takes 88 (the V it
// writes, 126 MB, about 30).  A and B take their samples in the
// same lane order, so the sum covers each sample once whatever order the
// instruction gives its contraction index; the accumulators hold
// D[4 (l / 16) + j][l % 16].
typedef int i32x4 __attribute__((ext_vector_type(4)));
constexpr int kI8Step = 64;                 // samples per step
constexpr int kI8Pitch = kI8Step + 16;      // LDS row bytes: 16-byte operand reads of 16 rows hit distinct banks

constexpr int kI8Blocks = 2;                          // 16 x 16 blocks per wave and side
constexpr int kI8Tile = 32 * kI8Blocks;               // antennas per side of a tile

__global__ __launch_bounds__(256) void fx_correlate_i8_kernel(FxArgs a) {
  __shared__ __attribute__((aligned(16))) int8_t pl[4][kI8Tile][kI8Pitch];   // re A, im A, re B, im B
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int na = a.n_ant, n_tiles = (na + kI8Tile - 1) / kI8Tile;
  int cl;
  unsigned tri;
  if (!xcd_channel(blockIdx.x, static_cast<unsigned>(n_tiles * (n_tiles + 1) / 2), a.n_launch, &cl, &tri)) return;
  int t = static_cast<int>(tri), ta = 0;      // upper-triangle tile (ta, tb), tb >= ta
  while (ta < n_tiles && t >= n_tiles - ta) {
    t -= n_tiles - ta;
    ++ta;
  }
  if (ta >= n_tiles) return;                  // beyond the triangle (the launch has none)
  const int a0 = ta * kI8Tile, b0 = (ta + t) * kI8Tile, c = a.c0 + cl;
  const int8_t* E = reinterpret_cast<const int8_t*>(a.E);
  const size_t tstride = static_cast<size_t>(a.n_chan) * na;
  // staging: thread = (antennas 4 ag .., samples 4 sg ..) of both blocks
  const int ag = tid % (kI8Tile / 4), sg = tid / (kI8Tile / 4);
  // a load of four antennas' bytes ends with the row at the latest; what it
  // shifts out are antennas of the group before, what it shifts in is zero
  const int8_t* src[2];
  unsigned down[2];
  bool none[2];
#pragma unroll
  for (int blk = 0; blk < 2; ++blk) {
    const int ant = (blk ? b0 : a0) + 4 * ag, from = ant <= na - 4 ? ant : na >= 4 ? na - 4 : 0;
    none[blk] = ant >= na;
    down[blk] = none[blk] ? 0u : 8u * static_cast<unsigned>(ant - from);
    src[blk] = E + static_cast<size_t>(4 * sg) * tstride + static_cast<size_t>(c) * na + from;
  }
  // this wave's sub-tile and its operand rows
  const int ah = w >> 1, bh = w & 1, l16 = lane & 15, g = lane >> 4;
  i32x4 acc[kI8Blocks][kI8Blocks][4];
#pragma unroll
  for (int i = 0; i < kI8Blocks; ++i)
#pragma unroll
    for (int j = 0; j < kI8Blocks; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[i][j][q] = i32x4{0, 0, 0, 0};
  uint32_t nxt[2][4];   // [block][sample], a byte per antenna
  auto load_step = [&](int64_t t0) {
    const size_t at = static_cast<size_t>(t0) * tstride;
    const bool full = t0 + kI8Step <= a.n_time && na >= 4;   // uniform
#pragma unroll
    for (int blk = 0; blk < 2; ++blk)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int8_t* from = src[blk] + at + i * tstride;
        uint32_t v = 0;
        if (full) {
          __builtin_memcpy(&v, from, 4);
        } else if (t0 + 4 * sg + i < a.n_time) {
          if (na >= 4) __builtin_memcpy(&v, from, 4);
          else
            for (int k = 0; k < na; ++k) v |= static_cast<uint32_t>(static_cast<uint8_t>(from[k])) << (8 * k);
        }
        nxt[blk][i] = none[blk] ? 0u : v >> down[blk];
      }
  };
  // four 4-bit two's complement values in the low nibbles, widened to bytes
  auto widen = [](uint32_t v) {
    v &= 0x0F0F0F0Fu;
    const uint32_t neg = v & 0x08080808u;
    return v | ((neg << 5) - (neg << 1));
  };
  // byte transpose: d[k] takes byte k of x[0..3]
  auto transpose = [](const uint32_t (&x)[4], uint32_t (&d)[4]) {
    const uint32_t p0 = __builtin_amdgcn_perm(x[1], x[0], 0x05010400u), p1 = __builtin_amdgcn_perm(x[1], x[0], 0x07030602u);
    const uint32_t q0 = __builtin_amdgcn_perm(x[3], x[2], 0x05010400u), q1 = __builtin_amdgcn_perm(x[3], x[2], 0x07030602u);
    d[0] = __builtin_amdgcn_perm(q0, p0, 0x05040100u);
    d[1] = __builtin_amdgcn_perm(q0, p0, 0x07060302u);
    d[2] = __builtin_amdgcn_perm(q1, p1, 0x05040100u);
    d[3] = __builtin_amdgcn_perm(q1, p1, 0x07060302u);
  };
  load_step(0);
  for (int64_t t0 = 0; t0 < a.n_time; t0 += kI8Step) {
#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
      uint32_t re[4], im[4], dr[4], di[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        re[i] = widen(nxt[blk][i] >> 4);
        im[i] = widen(nxt[blk][i]);
      }
      transpose(re, dr);
      transpose(im, di);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        *reinterpret_cast<uint32_t*>(&pl[2 * blk][4 * ag + k][4 * sg]) = dr[k];
        *reinterpret_cast<uint32_t*>(&pl[2 * blk + 1][4 * ag + k][4 * sg]) = di[k];
      }
    }
    __syncthreads();
    if (t0 + kI8Step < a.n_time) load_step(t0 + kI8Step);   // in flight during the products
    i32x4 ar[kI8Blocks], ai[kI8Blocks], br[kI8Blocks], bi[kI8Blocks];
#pragma unroll
    for (int i = 0; i < kI8Blocks; ++i) {
      ar[i] = *reinterpret_cast<const i32x4*>(&pl[0][16 * kI8Blocks * ah + 16 * i + l16][16 * g]);
      ai[i] = *reinterpret_cast<const i32x4*>(&pl[1][16 * kI8Blocks * ah + 16 * i + l16][16 * g]);
      br[i] = *reinterpret_cast<const i32x4*>(&pl[2][16 * kI8Blocks * bh + 16 * i + l16][16 * g]);
      bi[i] = *reinterpret_cast<const i32x4*>(&pl[3][16 * kI8Blocks * bh + 16 * i + l16][16 * g]);
    }
#pragma unroll
    for (int i = 0; i < kI8Blocks; ++i)
#pragma unroll
      for (int j = 0; j < kI8Blocks; ++j) {
        acc[i][j][0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ar[i], br[j], acc[i][j][0], 0, 0, 0);
        acc[i][j][1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ai[i], bi[j], acc[i][j][1], 0, 0, 0);
        acc[i][j][2] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ai[i], br[j], acc[i][j][2], 0, 0, 0);
        acc[i][j][3] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ar[i], bi[j], acc[i][j][3], 0, 0, 0);
      }
    __syncthreads();
  }
  float2* V = a.V + static_cast<size_t>(cl) * na * na;
#pragma unroll
  for (int i = 0; i < kI8Blocks; ++i)
#pragma unroll
    for (int j = 0; j < kI8Blocks; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int ia = a0 + 16 * kI8Blocks * ah + 16 * i + 4 * g + e, ib = b0 + 16 * kI8Blocks * bh + 16 * j + l16;
        if (ia >= na || ib >= na) continue;
        // E_a conj(E_b) = (xa xb + ya yb) + i (ya xb - xa yb)
        const double vr = static_cast<double>(acc[i][j][0][e]) + acc[i][j][1][e];
        const double vi = static_cast<double>(acc[i][j][2][e]) - acc[i][j][3][e];
        double zr = vr, zi = vi;
        if (a.gains) {
          const float2 ga = a.gains[static_cast<size_t>(c) * na + ia], gb = a.gains[static_cast<size_t>(c) * na + ib];
          // g_a conj(g_b)
          const double gr = static_cast<double>(ga.x) * gb.x + static_cast<double>(ga.y) * gb.y;
          const double gi = static_cast<double>(ga.y) * gb.x - static_cast<double>(ga.x) * gb.y;
          zr = gr * vr - gi * vi;
          zi = gr * vi + gi * vr;
        }
        V[static_cast<size_t>(ia) * na + ib] = make_float2(static_cast<float>(zr), static_cast<float>(zi));
      }
}

constexpr int kFxBinBatch = 8;   // pair loads in flight per thread of the binning

// One thread per (channel, type pair, offset cell).  The thread of a cell at
// or before its mirror (types swapped, offset negated) sums the cell's pairs
// and writes the mirror cell as the conjugate; the thread of a later cell has
// nothing to do.
__global__ __launch_bounds__(256) void fx_bin_kernel(FxArgs a) {
  const int nl2 = a.NL * a.NL;
  const size_t cells = static_cast<size_t>(a.n_types) * a.n_types * nl2;
  int c;
  unsigned blk;
  if (!xcd_channel(blockIdx.x, static_cast<unsigned>((cells + 255) / 256), a.n_launch, &c, &blk)) return;
  const size_t i = static_cast<size_t>(blk) * 256 + threadIdx.x;
  if (i >= cells) return;
  const int tp = static_cast<int>(i / nl2), off = static_cast<int>(i % nl2);
  const size_t m = static_cast<size_t>((tp % a.n_types) * a.n_types + tp / a.n_types) * nl2 + (nl2 - 1 - off);
  if (m < i) return;
  const float2* V = a.V + static_cast<size_t>(c) * a.n_ant * a.n_ant;
  double x = 0.0, y = 0.0;
  // Rows of short, redundant baselines hold hundreds of pairs: loads go out
  // kFxBinBatch at a time (indices, then visibilities) and are summed in the
  // same order as one at a time.
  int k = a.pair_ptr[i];
  const int k1 = a.pair_ptr[i + 1];
  for (; k + kFxBinBatch <= k1; k += kFxBinBatch) {
    uint32_t e[kFxBinBatch];
    float2 v[kFxBinBatch];
#pragma unroll
    for (int j = 0; j < kFxBinBatch; ++j) e[j] = static_cast<uint32_t>(a.pair_ab[k + j]);
#pragma unroll
    for (int j = 0; j < kFxBinBatch; ++j) v[j] = V[e[j] & ~kFxConjBit];
#pragma unroll
    for (int j = 0; j < kFxBinBatch; ++j) {
      x += v[j].x;
      y += (e[j] & kFxConjBit) ? -v[j].y : v[j].y;
    }
  }
  for (; k < k1; ++k) {
    const uint32_t e = static_cast<uint32_t>(a.pair_ab[k]);
    const float2 v = V[e & ~kFxConjBit];
    x += v.x;
    y += (e & kFxConjBit) ? -v.y : v.y;
  }
  float2* H = a.H + static_cast<size_t>(c) * cells;
  H[i] = make_float2(static_cast<float>(x), static_cast<float>(y));
  if (m != i) H[m] = make_float2(static_cast<float>(x), static_cast<float>(-y));
}

// One workgroup per (16 x 64 block of lag cells, channel); each thread owns
// four horizontally adjacent cells.  Per type pair the block's window of H
// (with a halo of the pair response's side) and the response itself are
// staged in LDS; cells of H outside the lag grid read as zero.  Along a
// response row the four cells' window values slide by one column per tap, so
// a row of `side` taps reads side + 3 window values instead of 4 side.  The
// pair responses obey X_qp(-u) = conj X_pq(u) and the binned sums
// H_qp(-d) = conj H_pq(d) (centred offsets), so the lag grid obeys
// R(-l) = conj R(l): only rows up to the zero lag are formed, its own row from
// the cells before the zero lag.  Four taps at a time, so that the window
// slides by naming its columns anew and not by moving them (64 channels of 1024
// antennas with 3 x 3 and 7 x 7 tables: 132 us one tap at a time, with complex
// responses and all rows, 110 here).
constexpr int kLagRows = 16, kLagCols = 64, kLagCells = 4;   // block of lag cells; cells per thread

template <bool REAL>   // real tables have real pair responses: half the multiply-adds
__global__ __launch_bounds__(256) void fx_lag_kernel(FxArgs a) {
  extern __shared__ float2 fx_lds[];
  const int NL = a.NL, nt = a.n_types, c = blockIdx.z;
  // window rows (of the widest window) as kLagCells planes, column x at
  // [x % kLagCells][x / kLagCells]: the threads' reads of one column each,
  // kLagCells apart, are then consecutive
  const int hp = (kLagCols + a.xs - 1 + kLagCells - 1) / kLagCells, hw = kLagCells * hp;
  float2* Ht = fx_lds;                            // [kLagRows + xs - 1][hw]
  float2* Xt = fx_lds + (kLagRows + a.xs - 1) * hw;   // [side][side]
  const int tyl = threadIdx.x / (kLagCols / kLagCells), txg = threadIdx.x % (kLagCols / kLagCells);
  const int ty0 = blockIdx.y * kLagRows, tx0 = blockIdx.x * kLagCols;
  const int mid = NL / 2;                         // the zero lag, L - 1
  if (ty0 > mid || (ty0 == mid && tx0 > mid)) return;   // no cell at or before its mirror
  const size_t plane = static_cast<size_t>(NL) * NL;
  double x[kLagCells] = {}, y[kLagCells] = {};
  for (int tp = 0; tp < nt * nt; ++tp) {
    const int kb = a.ktype_k[tp % nt], side = a.ktype_k[tp / nt] + kb - 1;
    const int ey = kLagRows + side - 1, ex = kLagCols + side - 1;
    const int hy0 = ty0 + kb - side, hx0 = tx0 + kb - side;
    const float2* H = a.H + (static_cast<size_t>(c) * nt * nt + tp) * plane;
    const float2* X = a.xcorr + static_cast<size_t>(tp) * a.xs * a.xs;
    __syncthreads();   // the previous pair's windows are no longer read
    for (int i = threadIdx.x; i < ey * ex; i += blockDim.x) {
      const int hy = hy0 + i / ex, hx = hx0 + i % ex;
      const int x = i % ex;
      Ht[(i / ex) * hw + (x % kLagCells) * hp + x / kLagCells] =
          (hy >= 0 && hy < NL && hx >= 0 && hx < NL) ? H[static_cast<size_t>(hy) * NL + hx] : make_float2(0.f, 0.f);
    }
    for (int i = threadIdx.x; i < side * side; i += blockDim.x) Xt[i] = X[(i / side) * a.xs + i % side];
    __syncthreads();
    // cell (tyl, 4 txg + j) at response tap (u, v) reads window cell
    // (tyl - u + side - 1, 4 txg + j - v + side - 1); one pair's response sum
    // in float32, the pairs combined in float64
    float px[kLagCells] = {}, py[kLagCells] = {};
    for (int u = 0; u < side; ++u) {
      const float2* hrow = Ht + (tyl - u + side - 1) * hw + txg;
      auto col = [&](int x) { return hrow[(x % kLagCells) * hp + x / kLagCells]; };   // column kLagCells txg + x
      auto tap = [&](float2 w, const float2& h0, const float2& h1, const float2& h2, const float2& h3) {
        const float2 h[kLagCells] = {h0, h1, h2, h3};
#pragma unroll
        for (int j = 0; j < kLagCells; ++j) {
          if constexpr (REAL) {
            px[j] = fmaf(w.x, h[j].x, px[j]);
            py[j] = fmaf(w.x, h[j].y, py[j]);
          } else {
            px[j] = fmaf(w.x, h[j].x, fmaf(-w.y, h[j].y, px[j]));
            py[j] = fmaf(w.x, h[j].y, fmaf(w.y, h[j].x, py[j]));
          }
        }
      };
      const float2* X = Xt + u * side;
      float2 h0 = col(side - 1), h1 = col(side), h2 = col(side + 1), h3 = col(side + 2);
      int v = 0;
      for (; v + 4 < side; v += 4) {   // four taps, four new columns
        const float2 g1 = col(side - 2 - v), g2 = col(side - 3 - v), g3 = col(side - 4 - v), g4 = col(side - 5 - v);
        tap(X[v], h0, h1, h2, h3);
        tap(X[v + 1], g1, h0, h1, h2);
        tap(X[v + 2], g2, g1, h0, h1);
        tap(X[v + 3], g3, g2, g1, h0);
        h0 = g4, h1 = g3, h2 = g2, h3 = g1;
      }
      for (; v < side; ++v) {
        tap(X[v], h0, h1, h2, h3);
        h3 = h2;
        h2 = h1;
        h1 = h0;
        if (v + 1 < side) h0 = col(side - 2 - v);
      }
    }
#pragma unroll
    for (int j = 0; j < kLagCells; ++j) {
      x[j] += px[j];
      y[j] += py[j];
    }
  }
  const int ly = ty0 + tyl;
  float2* R = a.R + static_cast<size_t>(c) * plane;
#pragma unroll
  for (int j = 0; j < kLagCells; ++j) {
    const int lx = tx0 + kLagCells * txg + j;
    const bool canonical = ly < mid || (ly == mid && lx <= mid);
    if (ly >= NL || lx >= NL || !canonical) continue;
    R[static_cast<size_t>(ly) * NL + lx] = make_float2(static_cast<float>(x[j]), static_cast<float>(y[j]));
    if (ly == mid && lx != mid)
      R[static_cast<size_t>(ly) * NL + (NL - 1 - lx)] = make_float2(static_cast<float>(x[j]), static_cast<float>(-y[j]));
  }
}

// One table type: only the cells that hold pairs are summed, and the pair
// response is applied to the image (its transform is the table's power
// pattern), so no lag grid is formed.  Cells are listed in cell order, those
// at or before their mirror; LANES lanes share a cell and take its pairs in
// turn, their float64 sums meeting in a fixed order.  (A dense lag grid of one
// thread per cell left most threads without pairs and the others with up to
// hundreds: 158 us for the binning, 195 for the lag convolution at 256 channels
// of 350 redundant antennas, N = 256, where this kernel takes 84, bound by the
// scattered 8-byte reads of V.)
template <int LANES>
__global__ __launch_bounds__(256) void fx_bin_cells_kernel(FxArgs a) {
  int c;
  unsigned blk;
  constexpr int PER = 256 / LANES;   // cells per workgroup
  if (!xcd_channel(blockIdx.x, static_cast<unsigned>((a.n_cells + PER - 1) / PER), a.n_launch, &c, &blk)) return;
  const int cell = static_cast<int>(blk) * PER + threadIdx.x / LANES, sub = threadIdx.x % LANES;
  double x = 0.0, y = 0.0;
  if (cell < a.n_cells) {
    const float2* V = a.V + static_cast<size_t>(c) * a.n_ant * a.n_ant;
    const int i = a.cell_at[cell];
    const int k1 = a.pair_ptr[i + 1];
    int k = a.pair_ptr[i] + sub;
    auto add = [&](uint32_t e, float2 v) {
      x += v.x;
      y += (e & kFxConjBit) ? -v.y : v.y;
    };
    for (; k + 3 * LANES < k1; k += 4 * LANES) {
      uint32_t e[4];
      float2 v[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) e[j] = static_cast<uint32_t>(a.pair_ab[k + j * LANES]);
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = V[e[j] & ~kFxConjBit];
#pragma unroll
      for (int j = 0; j < 4; ++j) add(e[j], v[j]);
    }
    for (; k < k1; k += LANES) {
      const uint32_t e = static_cast<uint32_t>(a.pair_ab[k]);
      add(e, V[e & ~kFxConjBit]);
    }
  }
#pragma unroll
  for (int off = LANES / 2; off >= 1; off >>= 1) {
    x += __shfl_down(x, off, LANES);
    y += __shfl_down(y, off, LANES);
  }
  if (cell < a.n_cells && sub == 0)
    a.H[static_cast<size_t>(c) * a.n_cells + cell] = make_float2(static_cast<float>(x), static_cast<float>(y));
}

// The lag grid's transform, N-point lines as PA x QB: pass A (job n2) takes the
// PA-point transform of points QB n1 + n2 in registers, pass B (job q1) the
// QB-point transform over n2 of its outputs q1 times w^(n2 q1), output
// q1 + PA q2; one exchange through LDS in between.  (Radix-2 stages in LDS, a
// barrier each, took 60 and 97 us for the row and the column pass at 256
// channels, N = 256; these take 17 and 34.)
//
// Lag d = j - (L - 1) of a lag-grid line is point n = d mod N with the factor
// (-1)^d, so that the transform's output index is the pixel index:
// w^(d (q - N/2)) = (-1)^d w^(d q).  Point N/2 (d = -L) is zero.
template <int N>
struct FxLine {
  static constexpr int PA = N >= 128 ? 16 : N >= 32 ? 8 : 4, QB = N / PA;
  static constexpr int L = N / 2, NL = N - 1;
};
constexpr int kFxLines = 16;   // lines per workgroup

__device__ __forceinline__ float2 odd_sign(int n, float2 v) { return (n & 1) ? make_float2(-v.x, -v.y) : v; }

// Row pass: one workgroup per (block of lag rows, channel).  With
// R(-l) = conj R(l), the transform of lag row NL - 1 - ly is the conjugate of
// that of row ly, so only rows up to the zero lag, L - 1, are transformed.
// CELLS: a row comes from the list of cells (row L - 1: its other half is the
// mirror), else from the lag grid.
template <int N, bool CELLS>
__global__ __launch_bounds__(256) void fx_row_kernel(FxArgs a) {
  using F = FxLine<N>;
  constexpr int PA = F::PA, QB = F::QB, L = F::L, NL = F::NL, PITCH = PA * (QB + 1);
  __shared__ float2 X[kFxLines * (PITCH > N ? PITCH : N)];
  __shared__ float2 tw[N];
  const int c = blockIdx.y, ly0 = blockIdx.x * kFxLines;
  for (int i = threadIdx.x; i < N; i += 256) tw[i] = a.tw[i];
  if constexpr (CELLS) {
    for (int i = threadIdx.x; i < kFxLines * N; i += 256) X[i] = make_float2(0.f, 0.f);
    __syncthreads();
    const int last = ly0 + kFxLines < L ? ly0 + kFxLines : L;
    const float2* H = a.H + static_cast<size_t>(c) * a.n_cells;
    for (int i = a.row_ptr[ly0] + threadIdx.x; i < a.row_ptr[last]; i += 256) {
      const int at = a.cell_at[i], ly = at / NL, n = (at % NL - (L - 1)) & (N - 1);
      const float2 v = odd_sign(n, H[i]);
      X[(ly - ly0) * N + n] = v;
      if (ly == L - 1 && n != 0) X[(ly - ly0) * N + (N - n)] = make_float2(v.x, -v.y);
    }
  }
  __syncthreads();
  constexpr int JA = (kFxLines * QB + 255) / 256;   // pass-A jobs per thread
  float2 x[JA][PA];
  const float2* R = CELLS ? nullptr : a.R + static_cast<size_t>(c) * NL * NL;
#pragma unroll
  for (int j = 0; j < JA; ++j) {
    const int job = threadIdx.x + 256 * j, k = job / QB, n2 = job % QB, ly = ly0 + k;
    if (k >= kFxLines) continue;
#pragma unroll
    for (int n1 = 0; n1 < PA; ++n1) {
      const int n = QB * n1 + n2;
      if constexpr (CELLS) {
        x[j][n1] = X[k * N + n];
      } else {
        const int d = n < L ? n : n - N;
        x[j][n1] = (ly < L && d >= -(L - 1))
                       ? odd_sign(n, R[static_cast<size_t>(ly) * NL + d + L - 1]) : make_float2(0.f, 0.f);
      }
    }
    Dft<PA>::run(x[j]);
#pragma unroll
    for (int q1 = 1; q1 < PA; ++q1) x[j][q1] = c_mul(x[j][q1], tw[n2 * q1]);
  }
  if constexpr (CELLS) __syncthreads();   // every line is read before it is overwritten
#pragma unroll
  for (int j = 0; j < JA; ++j) {
    const int job = threadIdx.x + 256 * j, k = job / QB, n2 = job % QB;
    if (k >= kFxLines) continue;
#pragma unroll
    for (int q1 = 0; q1 < PA; ++q1) X[k * PITCH + q1 * (QB + 1) + n2] = x[j][q1];
  }
  __syncthreads();
  float2* Z = a.Z + static_cast<size_t>(c) * L * N;
  for (int job = threadIdx.x; job < kFxLines * PA; job += 256) {
    const int k = job / PA, q1 = job % PA, ly = ly0 + k;
    if (ly >= L) continue;
    float2 y[QB];
#pragma unroll
    for (int n2 = 0; n2 < QB; ++n2) y[n2] = X[k * PITCH + q1 * (QB + 1) + n2];
    Dft<QB>::run(y);
#pragma unroll
    for (int q2 = 0; q2 < QB; ++q2) Z[static_cast<size_t>(ly) * N + q1 + PA * q2] = y[q2];
  }
}

// Column pass: one workgroup per (block of 2 CW image columns, channel).  Each
// column of Z is Hermitian in the lag (Z(-l, q) = conj Z(l, q)), so its
// transform is real and the rows up to the zero lag hold all of it: columns q
// and q + CW go through one complex transform as Z(., q) + i Z(., q + CW), and
// the real and imaginary parts of the result are the two image columns.
// CELLS: times the one table's power pattern (its pair response).
template <int N, bool CELLS>
__global__ __launch_bounds__(256) void fx_col_kernel(FxArgs a) {
  using F = FxLine<N>;
  constexpr int PA = F::PA, QB = F::QB, L = F::L, CW = N / 2 < kFxLines ? N / 2 : kFxLines;
  __shared__ float2 X[N * CW];   // [q1 QB + n2][line]
  __shared__ float2 tw[N];
  const int c = blockIdx.y, q0 = blockIdx.x * 2 * CW;   // c: channel within the launch
  for (int i = threadIdx.x; i < N; i += 256) tw[i] = a.tw[i];
  __syncthreads();
  const float2* Z = a.Z + static_cast<size_t>(c) * L * N;
  for (int job = threadIdx.x; job < CW * QB; job += 256) {
    const int k = job % CW, n2 = job / CW;
    float2 x[PA];
#pragma unroll
    for (int n1 = 0; n1 < PA; ++n1) {
      const int n = QB * n1 + n2;
      const int l = n < L ? n : N - n;        // |d|; rows hold d = -l
      float2 v = make_float2(0.f, 0.f);
      if (l < L) {
        const float2 z1 = Z[static_cast<size_t>(L - 1 - l) * N + q0 + k];
        const float2 z2 = Z[static_cast<size_t>(L - 1 - l) * N + q0 + CW + k];
        // z1 + i z2, of the conjugates where d > 0
        v = n < L ? make_float2(z1.x + z2.y, z2.x - z1.y) : make_float2(z1.x - z2.y, z1.y + z2.x);
      }
      x[n1] = odd_sign(n, v);
    }
    Dft<PA>::run(x);
#pragma unroll
    for (int q1 = 0; q1 < PA; ++q1) X[(q1 * QB + n2) * CW + k] = q1 ? c_mul(x[q1], tw[n2 * q1]) : x[0];
  }
  __syncthreads();
  float* out = a.out + static_cast<size_t>(a.c0 + c) * N * N;
  for (int job = threadIdx.x; job < CW * PA; job += 256) {
    const int k = job % CW, q1 = job / CW;
    float2 y[QB];
#pragma unroll
    for (int n2 = 0; n2 < QB; ++n2) y[n2] = X[(q1 * QB + n2) * CW + k];
    Dft<QB>::run(y);
#pragma unroll
    for (int q2 = 0; q2 < QB; ++q2) {
      const size_t pix = static_cast<size_t>(q1 + PA * q2) * N + q0 + k;
      double s1 = a.scale, s2 = a.scale;
      if constexpr (CELLS) {
        s1 *= a.Pp[pix];
        s2 *= a.Pp[pix + CW];
      }
      out[pix] = static_cast<float>(y[q2].x * s1);
      out[pix + CW] = static_cast<float>(y[q2].y * s2);
    }
  }
}

namespace {

template <int N, bool CELLS>
hipError_t launch_fx_transform(const FxArgs& a, hipStream_t st) {
  constexpr int CW = N / 2 < kFxLines ? N / 2 : kFxLines;
  hipLaunchKernelGGL((fx_row_kernel<N, CELLS>), dim3((N / 2 + kFxLines - 1) / kFxLines, a.n_launch), dim3(256), 0, st, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((fx_col_kernel<N, CELLS>), dim3(N / (2 * CW), a.n_launch), dim3(256), 0, st, a);
  return hipGetLastError();
}

template <bool CELLS>
hipError_t launch_fx_transform_n(const FxArgs& a, hipStream_t st) {
  switch (a.N) {
    case 8: return launch_fx_transform<8, CELLS>(a, st);
    case 16: return launch_fx_transform<16, CELLS>(a, st);
    case 32: return launch_fx_transform<32, CELLS>(a, st);
    case 64: return launch_fx_transform<64, CELLS>(a, st);
    case 128: return launch_fx_transform<128, CELLS>(a, st);
    case 256: return launch_fx_transform<256, CELLS>(a, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_fx(const FxArgs& a, bool ci4, hipStream_t st) {
  if (a.n_ant < 1 || a.n_launch < 1 || a.n_launch > 65535 || a.c0 < 0 || a.c0 + a.n_launch > a.n_chan || a.N < 8 ||
      a.N > 256 || a.NL != 2 * a.L - 1 || a.n_types < 1 || a.n_types > kMaxTypesDev)
    return hipErrorInvalidValue;
  if (ci4) {
    const size_t nt = static_cast<size_t>((a.n_ant + kI8Tile - 1) / kI8Tile);
    const size_t blocks = xcd_grid(nt * (nt + 1) / 2, a.n_launch);
    if (blocks > 0x7FFFFFFFu) return hipErrorInvalidValue;
    hipLaunchKernelGGL(fx_correlate_i8_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, a);
  } else {
    const size_t nt = static_cast<size_t>((a.n_ant + kC64Tile - 1) / kC64Tile);
    const size_t blocks = xcd_grid(nt * (nt + 1) / 2, a.n_launch);
    if (blocks > 0x7FFFFFFFu) return hipErrorInvalidValue;
    hipLaunchKernelGGL(fx_correlate_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, a);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (a.n_types == 1) {
    if (a.n_cells > 0) {
      // sixteen lanes per cell where cells hold several pairs each (redundant
      // arrays), else one
      const bool many = a.n_pairs >= 8 * static_cast<int64_t>(a.n_cells);
      const size_t per = many ? 16 : 256;
      const size_t blocks = xcd_grid((static_cast<size_t>(a.n_cells) + per - 1) / per, a.n_launch);
      if (blocks > 0x7FFFFFFFu) return hipErrorInvalidValue;
      if (many) hipLaunchKernelGGL(fx_bin_cells_kernel<16>, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, a);
      else hipLaunchKernelGGL(fx_bin_cells_kernel<1>, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, a);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return launch_fx_transform_n<true>(a, st);
  }
  const size_t cells = static_cast<size_t>(a.n_types) * a.n_types * a.NL * a.NL;
  const size_t bin_blocks = xcd_grid((cells + 255) / 256, a.n_launch);
  if (bin_blocks > 0x7FFFFFFFu) return hipErrorInvalidValue;
  hipLaunchKernelGGL(fx_bin_kernel, dim3(static_cast<unsigned>(bin_blocks)), dim3(256), 0, st, a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const unsigned lag_bx = static_cast<unsigned>((a.NL + kLagCols - 1) / kLagCols);
  const unsigned lag_by = static_cast<unsigned>((a.L + kLagRows - 1) / kLagRows);   // rows 0 .. L - 1
  const size_t lag_lds =
      sizeof(float2) * static_cast<size_t>((kLagRows + a.xs - 1) * ((kLagCols + a.xs - 1 + kLagCells - 1) / kLagCells * kLagCells) +
                                           a.xs * a.xs);
  const dim3 lag_grid(lag_bx, lag_by, a.n_launch), lag_block(kLagRows * kLagCols / kLagCells);
  if (a.real_tables) hipLaunchKernelGGL(fx_lag_kernel<true>, lag_grid, lag_block, lag_lds, st, a);
  else hipLaunchKernelGGL(fx_lag_kernel<false>, lag_grid, lag_block, lag_lds, st, a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  return launch_fx_transform_n<false>(a, st);
}

}  // namespace moff
