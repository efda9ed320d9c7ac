// Visibility-route (FX) imaging of one integration on the device, for
// cross-checks of the MOFF image by the paper's other method (Sec. 2: the
// time-averaged cross-products of the calibrated antenna fields, eq. cc-vis,
// gridded with each pair's power response, the cross-correlation of the two
// aperture illuminations, eq. e-field-conv, and transformed once, eq.
// dirty-image-FX, give the MOFF image; with the zero-spacing a == b terms left
// out it equals the image with the antennas' self power removed).
//
//   fx_stage_*_kernel    the samples as the correlators read them, antennas in
//                        the order of their cells
//   fx_correlate_kernel  V[c][a][b] = sum_t e_a conj(e_b), e = g E, for a <= b
//                        (the upper triangle; V is Hermitian): float32 as three
//                        bfloat16 levels on the matrix cores, summed in float64
//                        over steps of 32 samples (complex64 samples);
//                        fx_correlate_i8_kernel: exact integer products on the
//                        matrix cores (4+4-bit samples)
//   fx_bin_kernel        H[c][pq][dy][dx] = sum of V[c][a][b] over the pairs of
//                        table types (p, q) whose footprints are offset by
//                        (dy, dx) - (L - 1) cells (fixed order); half the rows
//                        are summed, their mirrors H[qp][-dy][-dx] are the
//                        conjugates
//   fx_lag_kernel        R[c][ly][lx] = sum_pq sum_(u,v) X_pq[u][v]
//                        H[c][pq][ly - u + k_q - 1][lx - v + k_q - 1]  (LDS-tiled;
//                        rows up to the zero lag; several table types)
//   fx_row_kernel        Z[c][ly][q] = sum_lx R[c][ly][lx] w^((lx - L + 1)(q - N/2))
//                        (rows up to the zero lag; the others are conjugates)
//   fx_col_kernel        I[c][r][q] = scale Re sum_ly w^((ly - L + 1)(r - N/2)) Z[c][ly][q]
//                        (real, two columns per complex transform)
//   With one table type the last two take H for R and multiply the image by the
//   table's power pattern, the transform of its autocorrelation X.
//
// w = exp(+2 pi i / N); lags span -(L - 1) .. L - 1, so the image comes out in
// the same pixel order as the MOFF image.  The sums run in a fixed order, but for
// the binning's: lanes of one instruction whose pairs share a lag cell add to it with
// LDS atomics, in the order in which the hardware takes them (results have repeated
// bit for bit wherever that was checked, regular arrays among them; nothing
// guarantees it).  The correlator and the binning accumulate in float64, each
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

// Staging: a workgroup takes 64 antennas x one step of samples of a channel and
// writes them in the form the correlators read, antennas at their places in the
// order of the visibilities (four lanes to an antenna: 64-byte row segments).  Every block is then read by all tiles of its antennas
// (one per 64 other antennas), which earlier converted it each for itself.
//
// Complex64 samples: e = g E, each component as three bfloat16 numbers, high,
// middle and low (8 bits each, all 24 of it, at float32's own range):
// [x, y][level][antenna][sample].
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 b16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 b16x8 __attribute__((ext_vector_type(8)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
constexpr int kC64Step = fx_step(false), kI8Step = fx_step(true);

__global__ __launch_bounds__(256) void fx_stage_c64_kernel(FxArgs a) {
  constexpr int PER = kC64Step * kFxTile / 256;   // samples per thread
  static_assert(PER == 8, "one 16-byte row segment per thread, part and level");
  const int na = a.n_ant, tiles = (na + kFxTile - 1) / kFxTile;
  const int cl = blockIdx.z, sg = threadIdx.x % 4, ant = blockIdx.y * kFxTile + threadIdx.x / 4;
  const int c = a.c0 + cl, pos = ant < na ? a.place[ant] : ant;
  const int64_t t = a.t0 + static_cast<int64_t>(blockIdx.x) * kC64Step + PER * sg;
  float2 v[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) v[i] = make_float2(0.f, 0.f);
  if (ant < na) {
    const float2 g = a.gains ? a.gains[static_cast<size_t>(c) * na + ant] : make_float2(1.f, 0.f);
    const float2* E = reinterpret_cast<const float2*>(a.E) + (static_cast<size_t>(t) * a.n_chan + c) * na + ant;
    const size_t stride = static_cast<size_t>(a.n_chan) * na;
#pragma unroll
    for (int i = 0; i < PER; ++i)
      if (t + i < a.t1) v[i] = E[i * stride];
#pragma unroll
    for (int i = 0; i < PER; ++i) v[i] = t + i < a.t1 ? cmul(g, v[i]) : make_float2(0.f, 0.f);
  }
  b16x8 lv[2][3];
#pragma unroll
  for (int i = 0; i < PER; i += 2)
#pragma unroll
    for (int part = 0; part < 2; ++part) {
      f32x2 x = part ? f32x2{v[i].y, v[i + 1].y} : f32x2{v[i].x, v[i + 1].x};
#pragma unroll
      for (int l = 0; l < 3; ++l) {
        const b16x2 h = __builtin_convertvector(x, b16x2);
        lv[part][l][i] = h[0];
        lv[part][l][i + 1] = h[1];
        if (l < 2) x -= __builtin_convertvector(h, f32x2);
      }
    }
  __bf16* dst = reinterpret_cast<__bf16*>(a.planes + ((static_cast<size_t>(cl) * tiles + pos / kFxTile) * gridDim.x + blockIdx.x) *
                                                         fx_block_bytes(false)) +
                pos % kFxTile * kC64Step + PER * sg;
#pragma unroll
  for (int part = 0; part < 2; ++part)
#pragma unroll
    for (int l = 0; l < 3; ++l) *reinterpret_cast<b16x8*>(dst + (part * 3 + l) * kFxTile * kC64Step) = lv[part][l];
}

// 4+4-bit samples: the raw samples as int8, [re, im][antenna][sample]; the gains,
// constant over the integration, are applied to the sums.  Sixteen samples of
// one antenna per thread.
__global__ __launch_bounds__(256) void fx_stage_i8_kernel(FxArgs a) {
  constexpr int PER = kI8Step * kFxTile / 256;
  static_assert(PER == 16, "one 16-byte row segment per thread and part");
  const int na = a.n_ant, tiles = (na + kFxTile - 1) / kFxTile;
  const int cl = blockIdx.z, sg = threadIdx.x % 4, ant = blockIdx.y * kFxTile + threadIdx.x / 4;
  const int c = a.c0 + cl, pos = ant < na ? a.place[ant] : ant;
  const int64_t t = a.t0 + static_cast<int64_t>(blockIdx.x) * kI8Step + PER * sg;
  int8_t b[PER] = {};
  if (ant < na) {
    const int8_t* E = reinterpret_cast<const int8_t*>(a.E) + (static_cast<size_t>(t) * a.n_chan + c) * na + ant;
    const size_t stride = static_cast<size_t>(a.n_chan) * na;
#pragma unroll
    for (int i = 0; i < PER; ++i)
      if (t + i < a.t1) b[i] = E[i * stride];
  }
  uint32_t re[PER / 4] = {}, im[PER / 4] = {};
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    re[i / 4] |= static_cast<uint32_t>(static_cast<uint8_t>(b[i] >> 4)) << (8 * (i % 4));
    im[i / 4] |= static_cast<uint32_t>(static_cast<uint8_t>(static_cast<int8_t>(b[i] << 4) >> 4)) << (8 * (i % 4));
  }
  char* dst = a.planes + ((static_cast<size_t>(cl) * tiles + pos / kFxTile) * gridDim.x + blockIdx.x) * fx_block_bytes(true) +
              pos % kFxTile * kI8Step + PER * sg;
  *reinterpret_cast<uint4*>(dst) = make_uint4(re[0], re[1], re[2], re[3]);
  *reinterpret_cast<uint4*>(dst + kFxTile * kI8Step) = make_uint4(im[0], im[1], im[2], im[3]);
}

// The correlators: V_ab for a <= b (V_ba = conj V_ab, and the binning reads the
// upper triangle only), one workgroup per (64 x 64 antenna tile on or above the
// diagonal, channel), four waves of a 32 x 32 sub-tile each, or eight of 32 x 16
// (blocks of 16 x 16).  Per step both antenna blocks are copied into LDS, the next step's
// copies in flight meanwhile.  A and B take their samples in the same lane
// order, so each is summed once whatever order the instruction gives its
// contraction index; accumulators hold D[4 (l / 16) + v][l % 16].

// Tile (ta, tb) and channel of a workgroup; false for the padding ones.
__device__ __forceinline__ bool corr_tile(const FxArgs& a, int* cl, int* ta, int* tb) {
  const int n_tiles = (a.n_ant + kFxTile - 1) / kFxTile;
  unsigned tri;
  if (!xcd_channel(blockIdx.x, static_cast<unsigned>(n_tiles * (n_tiles + 1) / 2), a.n_launch, cl, &tri)) return false;
  int t = static_cast<int>(tri);
  *ta = 0;
  while (*ta < n_tiles && t >= n_tiles - *ta) {
    t -= n_tiles - *ta;
    ++*ta;
  }
  *tb = *ta + t;
  return *ta < n_tiles;
}

// Copies of one step: 16 bytes per thread and round, both blocks, into LDS rows
// of ROW bytes at a pitch 16 bytes longer (operand reads of 16 rows then hit
// distinct banks).
template <int NT, int ROUNDS>
__device__ __forceinline__ void load_step(const char* a, const char* b, i32x4 (&v)[2][ROUNDS]) {
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    v[0][r] = reinterpret_cast<const i32x4*>(a)[r * NT + threadIdx.x];
    v[1][r] = reinterpret_cast<const i32x4*>(b)[r * NT + threadIdx.x];
  }
}
template <int NT, int ROW, int ROUNDS>
__device__ __forceinline__ void store_step(char* lds, const i32x4 (&v)[2][ROUNDS]) {   // [block][row]
#pragma unroll
  for (int blk = 0; blk < 2; ++blk)
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      const int at = (r * NT + threadIdx.x) * 16;
      *reinterpret_cast<i32x4*>(lds + (blk * (ROUNDS * NT * 16 / ROW) + at / ROW) * (ROW + 16) + at % ROW) = v[blk][r];
    }
}

// Sum of a pass, or of all: the running sums of passes before the last in Vd.
__device__ __forceinline__ void put_visibility(const FxArgs& a, int cl, int ia, int ib, double x, double y) {
  const size_t at = (static_cast<size_t>(cl) * a.n_ant + ia) * a.n_ant + ib;
  if (a.Vd) {
    if (!a.first) {
      const double2 s = a.Vd[at];
      x += s.x;
      y += s.y;
    }
    if (!a.last) {
      a.Vd[at] = make_double2(x, y);
      return;
    }
  }
  a.V[at] = make_float2(static_cast<float>(x), static_cast<float>(y));
}

// Complex64 samples: v_mfma_f32_16x16x32_bf16 on the levels, a product taking the
// six terms above 2^-24 (hh, hm, mh, mm, hl, lh) with float32 accumulation: the
// accuracy of the float32 matrix instruction at 2.7 times its rate.  With
// e = x + i y,
//   Re V_ab = sum x_a x_b + y_a y_b,   Im V_ab = sum y_a x_b - x_a y_b;
// each 32-sample step is summed in float32 and the steps in float64.  At 64
// channels x 128 samples of 1024 antennas: 438 us with the float32 instruction,
// 294 with the levels made by every tile, 235-258 here (eight waves; 268 with
// four of 32 x 32) and 40 for the staging.  The products take 87 at their peak
// rate, the LDS 109, the vector work 75, hardly overlapped.
constexpr int kC64Threads = 512;

__global__ __launch_bounds__(kC64Threads) __attribute__((amdgpu_waves_per_eu(4))) void fx_correlate_kernel(FxArgs a) {
  constexpr int NT = kC64Threads, ROW = kC64Step * 2, PITCH = ROW + 16;
  __shared__ __attribute__((aligned(16))) char pl[2 * 6 * kFxTile * PITCH];   // [block][x, y][level][antenna]
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wa = wave >> 2, wb = wave & 3, r16 = lane & 15, kk = lane >> 4;
  const int na = a.n_ant, tiles = (na + kFxTile - 1) / kFxTile;
  int cl, ta, tb;
  if (!corr_tile(a, &cl, &ta, &tb)) return;
  const int64_t steps = (a.t1 - a.t0 + kC64Step - 1) / kC64Step;
  const char* pa = a.planes + (static_cast<size_t>(cl) * tiles + ta) * steps * fx_block_bytes(false);
  const char* pb = a.planes + (static_cast<size_t>(cl) * tiles + tb) * steps * fx_block_bytes(false);
  double acc[2][4][2] = {};
  i32x4 next[2][3];
  load_step<NT>(pa, pb, next);
  for (int64_t st = 0; st < steps; ++st) {
    store_step<NT, ROW>(pl, next);
    __syncthreads();
    pa += fx_block_bytes(false);
    pb += fx_block_bytes(false);
    if (st + 1 < steps) load_step<NT>(pa, pb, next);   // in flight during the products
    auto operand = [&](int blk, int part, int l, int row) {
      return *reinterpret_cast<const b16x8*>(pl + (((blk * 2 + part) * 3 + l) * kFxTile + row) * PITCH + 16 * kk);
    };
    b16x8 B[2][3];
#pragma unroll
    for (int part = 0; part < 2; ++part)
#pragma unroll
      for (int l = 0; l < 3; ++l) B[part][l] = operand(1, part, l, 16 * wb + r16);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      // the small terms of both products first, so that a step's sum rounds
      // twice at full size
      f32x4 re = {0.f, 0.f, 0.f, 0.f}, im = {0.f, 0.f, 0.f, 0.f};
      b16x8 hi[2];
#pragma unroll
      for (int part = 0; part < 2; ++part) {
        b16x8 A[3];
#pragma unroll
        for (int l = 0; l < 3; ++l) A[l] = operand(0, part, l, 32 * wa + 16 * i + r16);
        hi[part] = A[0];
        const b16x8(&X)[3] = B[part];       // x_a x_b, y_a y_b
        const b16x8(&Y)[3] = B[1 - part];   // - x_a y_b, y_a x_b
        auto sign = [&](b16x8 v) { return part == 0 ? -v : v; };
        auto mm = [](b16x8 x, b16x8 y, f32x4 r) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, y, r, 0, 0, 0); };
        re = mm(A[2], X[0], re);
        im = mm(A[2], sign(Y[0]), im);
        re = mm(A[0], X[2], re);
        im = mm(A[0], sign(Y[2]), im);
        re = mm(A[1], X[1], re);
        im = mm(A[1], sign(Y[1]), im);
        re = mm(A[1], X[0], re);
        im = mm(A[1], sign(Y[0]), im);
        re = mm(A[0], X[1], re);
        im = mm(A[0], sign(Y[1]), im);
      }
      re = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi[0], B[0][0], re, 0, 0, 0);
      im = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi[1], B[0][0], im, 0, 0, 0);
      re = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi[1], B[1][0], re, 0, 0, 0);
      im = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi[0], -B[1][0], im, 0, 0, 0);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        acc[i][v][0] += re[v];
        acc[i][v][1] += im[v];
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int ia = ta * kFxTile + 32 * wa + 16 * i + 4 * kk + v, ib = tb * kFxTile + 16 * wb + r16;
      if (ia < na && ib < na) put_visibility(a, cl, ia, ib, acc[i][v][0], acc[i][v][1]);
    }
}

// 4+4-bit samples: the cross-products are exact integer sums, formed on the
// matrix cores (v_mfma_i32_16x16x64_i8, int32 accumulation) from the raw
// samples, four products (re.re, im.im, im.re, re.im) per block; the gains are
// applied once, V_ab = g_a conj(g_b) sum_t E_a conj(E_b), in float64.  Bound by
// what surrounds the products (6 % of the matrix rate): at 256 channels x 256
// samples of 350 antennas 132 us with samples unpacked byte by byte for every
// tile, 55 here and 31 for the staging (the V it writes, 126 MB, about 30).
__global__ __launch_bounds__(256) void fx_correlate_i8_kernel(FxArgs a) {
  constexpr int ROW = kI8Step, PITCH = ROW + 16;
  __shared__ __attribute__((aligned(16))) char pl[2 * 2 * kFxTile * PITCH];   // [block][re, im][antenna]
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int ah = w >> 1, bh = w & 1, l16 = lane & 15, g = lane >> 4;
  const int na = a.n_ant, tiles = (na + kFxTile - 1) / kFxTile;
  int cl, ta, tb;
  if (!corr_tile(a, &cl, &ta, &tb)) return;
  const int c = a.c0 + cl;
  const int64_t steps = (a.t1 - a.t0 + kI8Step - 1) / kI8Step;
  const char* pa = a.planes + (static_cast<size_t>(cl) * tiles + ta) * steps * fx_block_bytes(true);
  const char* pb = a.planes + (static_cast<size_t>(cl) * tiles + tb) * steps * fx_block_bytes(true);
  i32x4 acc[2][2][4];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[i][j][q] = i32x4{0, 0, 0, 0};
  i32x4 next[2][2];
  load_step<256>(pa, pb, next);
  for (int64_t st = 0; st < steps; ++st) {
    store_step<256, ROW>(pl, next);
    __syncthreads();
    pa += fx_block_bytes(true);
    pb += fx_block_bytes(true);
    if (st + 1 < steps) load_step<256>(pa, pb, next);   // in flight during the products
    auto operand = [&](int blk, int part, int row) {
      return *reinterpret_cast<const i32x4*>(pl + ((blk * 2 + part) * kFxTile + row) * PITCH + 16 * g);
    };
    i32x4 ar[2], ai[2], br[2], bi[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      ar[i] = operand(0, 0, 32 * ah + 16 * i + l16);
      ai[i] = operand(0, 1, 32 * ah + 16 * i + l16);
      br[i] = operand(1, 0, 32 * bh + 16 * i + l16);
      bi[i] = operand(1, 1, 32 * bh + 16 * i + l16);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        acc[i][j][0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ar[i], br[j], acc[i][j][0], 0, 0, 0);
        acc[i][j][1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ai[i], bi[j], acc[i][j][1], 0, 0, 0);
        acc[i][j][2] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ai[i], br[j], acc[i][j][2], 0, 0, 0);
        acc[i][j][3] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ar[i], bi[j], acc[i][j][3], 0, 0, 0);
      }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int ia = ta * kFxTile + 32 * ah + 16 * i + 4 * g + e, ib = tb * kFxTile + 32 * bh + 16 * j + l16;
        if (ia >= na || ib >= na) continue;
        // E_a conj(E_b) = (xa xb + ya yb) + i (ya xb - xa yb)
        const double vr = static_cast<double>(acc[i][j][0][e]) + acc[i][j][1][e];
        const double vi = static_cast<double>(acc[i][j][2][e]) - acc[i][j][3][e];
        double zr = vr, zi = vi;
        if (a.gains) {
          const float2 ga = a.gains[static_cast<size_t>(c) * na + a.order[ia]];
          const float2 gb = a.gains[static_cast<size_t>(c) * na + a.order[ib]];
          // g_a conj(g_b)
          const double gr = static_cast<double>(ga.x) * gb.x + static_cast<double>(ga.y) * gb.y;
          const double gi = static_cast<double>(ga.y) * gb.x - static_cast<double>(ga.x) * gb.y;
          zr = gr * vr - gi * vi;
          zi = gr * vi + gi * vr;
        }
        put_visibility(a, cl, ia, ib, zr, zi);
      }
}

// Copies of a lag row's sums per wave of the binning, where the longest row has 64
// pairs or more to a cell: as many as keep the four waves' near 16 KB.  Lanes take
// them in turn, so that pairs that share a cell meet less often: 322 antennas in a
// line on 15 lags, 1762 channels, 2.8 ms with a thread per cell, 4.1 with one copy,
// 1.2 here; 616 on 31 lags, 97 channels, 2.4, 3.3, 0.63; 200 on 7 x 7 lags, 500
// channels, 503 us, 217, 76.  Fewer pairs to a cell only pay for clearing and adding the copies
// (96 against 94 us at 256 channels of 324 antennas).
//
// Longer rows (256 pairs or more to a cell, which lines of antennas reach) pay for more:
// near 32 KB, and near 64 KB where the launch has too few of them to share a unit's
// LDS.  A line of 1088 antennas, 285 channels: 9.0 ms with 16 KB, 4.5 with 32 and 2.7
// with 64 at N = 256 (143 long rows to a pass), 9.4, 3.7 and 2.5 at N = 128; 600 at N = 64, 3.3, 2.1
// and 2.6 at 1000 channels, 1.12, 0.36 and 0.20 at 97.  (900 antennas
// in one cell of N = 64, 32 channels, lose by it: 110, 113 and 121 us.)
int fx_copies(int NL, int longest, int64_t groups) {
  if (longest < 64 * NL) return 1;
  const int lds = longest < 256 * NL ? 16384 : groups > 512 ? 32768 : 65536;
  int c = 1;
  while (c < 16 && 4 * 2 * 8 * NL * c * 2 <= lds) c *= 2;
  return c;
}
// Doubles from copy to copy: neighbouring lanes' copies then lie apart in the banks
// (32 of 8 bytes) whether their cells are adjacent or every other one.
__host__ __device__ constexpr int fx_copy_pitch(int NL, int copies) {
  return copies == 1 ? 2 * NL : 2 * NL + (32 / copies + 32 - 2 * NL % 32) % 32;
}

// The sums of one lag row per workgroup (row, channel) and, where no row has more than
// kFxShortRow pairs, of four rows, one per wave.  The waves of a row add contiguous
// parts of its pairs into float64 rows of their own in LDS, which are then summed
// in order.  The row's entries are in the order of the
// visibilities, whose antennas are sorted by cell, so that neighbouring lanes
// read neighbouring elements of V (a thread per lag cell, with pairs scattered
// over V, was bound by those reads: 302 us at 64 channels of 1024 antennas, 148
// here; 84 and 48 at 256 channels of 350).  Short rows are bound by starting,
// clearing and adding up: 1052 channels of 51 antennas of two types at N = 64, with a
// thread per cell, a workgroup per row and a wave per row, take 46, 132 and 45 us; the
// call of 256 channels of 128 antennas at N = 128 (rows to 1024) 58 and 50 us with four
// waves and one to a row, of 128 antennas at N = 16 (rows to 4096) 45 and 74.  Mirrors
// (types swapped, offset negated) get the conjugates where the lag convolution reads them.
constexpr int kFxShortRow = 1024;
__host__ __device__ constexpr unsigned fx_bin_groups(int n_rows, int rows) {
  return static_cast<unsigned>((n_rows + rows - 1) / rows);
}

template <bool SPREAD, int ROWS>   // several copies; rows per workgroup (1 or 4)
__global__ __launch_bounds__(256) void fx_bin_kernel(FxArgs a) {
  extern __shared__ double fx_sums[];   // [4][copies][pitch], real and imaginary rows
  const int NL = a.NL, nt = a.n_types, mid = NL / 2;
  constexpr int W = 4 / ROWS;   // waves of a row
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, copies = SPREAD ? a.copies : 1;
  int c;
  unsigned r;
  if (!xcd_channel(blockIdx.x, fx_bin_groups(a.n_rows, ROWS), a.n_launch, &c, &r)) return;
  if (ROWS > 1) r = r * ROWS + wave;
  const bool in = ROWS == 1 || r < static_cast<unsigned>(a.n_rows);   // (a wave beyond the last row adds nothing)
  const int k0 = in ? a.row_ptr[r] : 0, n = in ? a.row_ptr[r + 1] - k0 : 0;
  const bool empty = n == 0 && nt == 1;   // (the row pass knows that it is zero)
  if (ROWS == 1 && empty) return;
  const int pitch = SPREAD ? fx_copy_pitch(NL, copies) : 2 * NL;
  for (int i = threadIdx.x; i < 4 * copies * pitch; i += 256) fx_sums[i] = 0.0;
  __syncthreads();
  const float2* V = a.V + static_cast<size_t>(c) * a.n_ant * a.n_ant;
  double* sum = fx_sums + (wave * copies + (lane & (copies - 1))) * pitch;
  const int part = ROWS > 1 ? 0 : wave;
  const int k1 = k0 + static_cast<int>((part + 1) * static_cast<int64_t>(n) / W);
  int k = k0 + static_cast<int>(part * static_cast<int64_t>(n) / W) + lane;
  auto add = [&](uint32_t e, int dx, float2 v) {
    unsafeAtomicAdd(sum + dx, static_cast<double>(v.x));
    unsafeAtomicAdd(sum + NL + dx, static_cast<double>((e & kFxConjBit) ? -v.y : v.y));
  };
  constexpr int B = 4;   // entries in flight per lane
  for (; k + (B - 1) * 64 < k1; k += B * 64) {
    uint32_t e[B];
    int dx[B];
    float2 v[B];
#pragma unroll
    for (int j = 0; j < B; ++j) {
      e[j] = a.pair_ab[k + j * 64];
      dx[j] = a.pair_dx[k + j * 64];
    }
#pragma unroll
    for (int j = 0; j < B; ++j) v[j] = V[e[j] & ~kFxConjBit];
#pragma unroll
    for (int j = 0; j < B; ++j) add(e[j], dx[j], v[j]);
  }
  for (; k < k1; k += 64) {
    const uint32_t e = a.pair_ab[k];
    add(e, a.pair_dx[k], V[e & ~kFxConjBit]);
  }
  __syncthreads();
  if (ROWS > 1 && (!in || empty)) return;
  const int tp = a.rows[r] / NL, dy = a.rows[r] % NL, p = tp / nt, q = tp % nt;
  const bool half_row = p == q && dy == mid;   // only columns up to the zero lag were summed
  const size_t plane = static_cast<size_t>(nt == 1 ? a.L : NL) * NL;
  float2* H = a.H + static_cast<size_t>(c) * nt * nt * plane;
  // rows that the lag convolution reads: up to the zero lag and the responses' reach
  const int reach = mid + a.xs;
  const double* row = fx_sums + (ROWS > 1 ? wave * pitch : 0);
  for (int x = ROWS > 1 ? lane : threadIdx.x; x < NL; x += 64 * W) {
    const int from = half_row && x > mid ? NL - 1 - x : x;
    double re = 0.0, im = 0.0;
#pragma unroll 4
    for (int w = 0; w < W * copies; ++w) {
      re += row[w * pitch + from];
      im += row[w * pitch + NL + from];
    }
    const float2 v = make_float2(static_cast<float>(re), static_cast<float>(from == x ? im : -im));
    if (dy <= reach) H[static_cast<size_t>(tp) * plane + static_cast<size_t>(dy) * NL + x] = v;
    if (nt > 1 && NL - 1 - dy <= reach && !half_row)
      H[static_cast<size_t>(q * nt + p) * plane + static_cast<size_t>(NL - 1 - dy) * NL + (NL - 1 - x)] =
          make_float2(v.x, -v.y);
  }
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

// The lag grid's transform, N-point lines as PA x QB: pass A (job n2) takes the
// PA-point transform of points QB n1 + n2 in registers, pass B (job q1) the
// QB-point transform over n2 of its outputs q1 times w^(n2 q1), output
// q1 + PA q2; one exchange through LDS in between.  (Radix-2 stages in LDS, a
// barrier each, took 60 and 97 us for the row and the column pass at 256
// channels, N = 256; these take 26 and 33.)
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
// ONE: one table type, rows of pair sums (a row without pairs is not written and
// reads as zero); else rows of the lag grid.
template <int N, bool ONE>
__global__ __launch_bounds__(256) void fx_row_kernel(FxArgs a) {
  using F = FxLine<N>;
  constexpr int PA = F::PA, QB = F::QB, L = F::L, NL = F::NL, PITCH = PA * (QB + 1);
  __shared__ float2 X[kFxLines * PITCH];
  __shared__ float2 tw[N];
  const int c = blockIdx.y, ly0 = blockIdx.x * kFxLines;
  for (int i = threadIdx.x; i < N; i += 256) tw[i] = a.tw[i];
  __syncthreads();
  constexpr int JA = (kFxLines * QB + 255) / 256;   // pass-A jobs per thread
  float2 x[JA][PA];
  const float2* R = ONE ? a.H + static_cast<size_t>(c) * L * NL : a.R + static_cast<size_t>(c) * NL * NL;
#pragma unroll
  for (int j = 0; j < JA; ++j) {
    const int job = threadIdx.x + 256 * j, k = job / QB, n2 = job % QB, ly = ly0 + k;
    if (k >= kFxLines) continue;
    bool row = ly < L;
    if constexpr (ONE) row = row && a.row_ptr[ly + 1] > a.row_ptr[ly];
#pragma unroll
    for (int n1 = 0; n1 < PA; ++n1) {
      const int n = QB * n1 + n2, d = n < L ? n : n - N;
      x[j][n1] = (row && d >= -(L - 1)) ? odd_sign(n, R[static_cast<size_t>(ly) * NL + d + L - 1]) : make_float2(0.f, 0.f);
    }
    Dft<PA>::run(x[j]);
#pragma unroll
    for (int q1 = 1; q1 < PA; ++q1) x[j][q1] = c_mul(x[j][q1], tw[n2 * q1]);
  }
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
// ONE: times the one table's power pattern, the transform of its pair response
// (no lag grid is formed: its convolution took 195 us at 256 channels, N = 256).
template <int N, bool ONE>
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
      if constexpr (ONE) {
        s1 *= a.Pp[pix];
        s2 *= a.Pp[pix + CW];
      }
      out[pix] = static_cast<float>(y[q2].x * s1);
      out[pix + CW] = static_cast<float>(y[q2].y * s2);
    }
  }
}

namespace {

template <int N, bool ONE>
hipError_t launch_fx_transform(const FxArgs& a, hipStream_t st) {
  constexpr int CW = N / 2 < kFxLines ? N / 2 : kFxLines;
  hipLaunchKernelGGL((fx_row_kernel<N, ONE>), dim3((N / 2 + kFxLines - 1) / kFxLines, a.n_launch), dim3(256), 0, st, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((fx_col_kernel<N, ONE>), dim3(N / (2 * CW), a.n_launch), dim3(256), 0, st, a);
  return hipGetLastError();
}

template <bool ONE>
hipError_t launch_fx_transform_n(const FxArgs& a, hipStream_t st) {
  switch (a.N) {
    case 8: return launch_fx_transform<8, ONE>(a, st);
    case 16: return launch_fx_transform<16, ONE>(a, st);
    case 32: return launch_fx_transform<32, ONE>(a, st);
    case 64: return launch_fx_transform<64, ONE>(a, st);
    case 128: return launch_fx_transform<128, ONE>(a, st);
    case 256: return launch_fx_transform<256, ONE>(a, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_fx(const FxArgs& a, bool ci4, hipStream_t st) {
  if (a.n_ant < 1 || a.n_launch < 1 || a.n_launch > 65535 || a.c0 < 0 || a.c0 + a.n_launch > a.n_chan || a.N < 8 ||
      a.N > 256 || a.NL != 2 * a.L - 1 || a.n_types < 1 || a.n_types > kMaxTypesDev)
    return hipErrorInvalidValue;
  const size_t nt = static_cast<size_t>((a.n_ant + kFxTile - 1) / kFxTile);
  const int64_t steps = (a.t1 - a.t0 + fx_step(ci4) - 1) / fx_step(ci4);
  const size_t blocks = xcd_grid(nt * (nt + 1) / 2, a.n_launch);
  FxArgs b = a;
  // (rows as long as the longest that the pairs would fill)
  const int64_t full_rows = (static_cast<int64_t>(a.n_ant) * a.n_ant / 2 + a.longest) / std::max(a.longest, 1);
  b.copies = fx_copies(a.NL, a.longest, full_rows * a.n_launch);
  const int bin_rows = b.copies == 1 && a.longest <= kFxShortRow ? 4 : 1;
  const size_t bin_blocks = xcd_grid(fx_bin_groups(a.n_rows, bin_rows), a.n_launch);
  if (steps < 1 || steps > 0x7FFFFFFF || blocks > 0x7FFFFFFFu || bin_blocks > 0x7FFFFFFFu) return hipErrorInvalidValue;
  const dim3 stage(static_cast<unsigned>(steps), static_cast<unsigned>(nt), a.n_launch);
  hipError_t e;
  if (ci4) {
    hipLaunchKernelGGL(fx_stage_i8_kernel, stage, dim3(256), 0, st, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(fx_correlate_i8_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, a);
  } else {
    hipLaunchKernelGGL(fx_stage_c64_kernel, stage, dim3(256), 0, st, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(fx_correlate_kernel, dim3(static_cast<unsigned>(blocks)), dim3(kC64Threads), 0, st, a);
  }
  if ((e = hipGetLastError()) != hipSuccess || !a.last) return e;
  const dim3 bins(static_cast<unsigned>(bin_blocks));
  const size_t bin_lds = sizeof(double) * 4 * b.copies * fx_copy_pitch(a.NL, b.copies);
  if (bin_rows > 1) hipLaunchKernelGGL((fx_bin_kernel<false, 4>), bins, dim3(256), bin_lds, st, b);
  else if (b.copies > 1) {
    auto k = fx_bin_kernel<true, 1>;
    if ((e = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize,
                                 static_cast<int>(bin_lds))) != hipSuccess)
      return e;
    hipLaunchKernelGGL(k, bins, dim3(256), bin_lds, st, b);
  } else hipLaunchKernelGGL((fx_bin_kernel<false, 1>), bins, dim3(256), bin_lds, st, b);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (a.n_types == 1) return launch_fx_transform_n<true>(a, st);
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
