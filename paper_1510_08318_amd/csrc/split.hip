// Float32 MOFF frames on the gfx950 matrix cores (grids of 64 and 128).
//
// The padded 2-D DFT of Sec. 3 as matrix products whose operands are pairs of
// binary16 numbers: every float32 value x is held as hi + lo with
// hi = binary16(x), lo = binary16(x - hi), which keeps 22 bits or more of it
// (absolute floor 2^-25 below operands of up to 2^15), and a product takes
// hi.hi + hi.lo + lo.hi with float32 accumulation (v_mfma_f32_16x16x32_f16); at
// N = 64 also lo.lo, and under the uv-plane rule the phase factors are three
// numbers (kSplitParts).
// The 16-bit matrix rate is 16 times the float32 vector rate.  Relative 2-norm
// error against 64 bits, FFT kernel -> this one, 5 channels x 257 samples of 203
// antennas: dense complex tables 2.5e-7 -> 0.5e-7 at N = 64, 3.3e-7 -> 1.5e-7 at
// 128; under the uv-plane rule 1.5e-7 -> 1.0e-7 and 1.6e-7 -> 1.4e-7; 3 x 3 real
// tables 1.2e-7 -> 0.3e-7 and 1.8e-7 -> 0.8e-7.
//
// Time: 128 channels x 1000 samples of 256 antennas at N = 128 2.22 -> 1.22 ms,
// 33 x 257 of 203 at N = 64 148 -> 67 us (launch and merge included).  Bound by
// issue: the matrix products take 0.48 ms of the 1.22 at their peak rate, the
// vector instructions (fold and split, pair combinations, |Y|^2, gather) 0.6,
// and little of the two runs side by side with two waves per SIMD.
//
// Three identities cut the matrix work (split_shape.h): the aperture folded
// about its centre halves both contractions, and conjugate output pairs halve
// the outputs.  With the cosine and sine factors of the base half, the row
// stage forms P1 = Re s cos, P2 = Im d sin, P3 = Re d sin, P4 = Im s cos; base
// column (P1 - P2) + i (P3 + P4), partner (P1 + P2) + i (P4 - P3); the column
// stage does the same along y.  Base slot 0 carries p = 0 (cosines) and p = -L
// (sines); there the factor 0 in place of 1 separates the two (its partner
// comes out times a unit phase).
//
// One workgroup owns one (channel, time slice).  Each wave owns 16 base
// columns, their 16 partners and all rows; a row-stage result sits in its
// lane exactly where the column stage wants its operand (accumulator row
// 4 g + j of lane group g is contraction index 4 g + j of that lane group,
// split_pos), so the half-transformed grid never leaves the registers.  Only
// the folded grid goes through LDS.  Per frame:
//   gather   each wave grids its own row pairs (iy and L - 1 - iy, interleaved
//            between waves for balance) into its own part of LDS, walking a
//            program of 64 cells at a time, one per lane, sorted by length:
//            steps and cell ends are wave-uniform, no lane waits for another;
//   fold     sums and differences along both axes, split into halves -> LDS;
//   row stage, column stage, |Y|^2 into float32 registers.
// Two workgroup barriers per frame.
//
// Scale: samples are scaled by a power of two so that folded values stay at or
// below 2^kSplitField.  4+4-bit samples have a fixed bound, 8 times the largest
// gain among the antennas with a sample other than zero in the slice (looked up
// beyond its first frame only where that leaves out a larger gain: a bound on all
// gains followed a dead antenna's, whatever it was, and at a gain of 1e6 the
// relative error of the others' image came to 1e-2); for complex64 the scale
// follows the largest sample component seen so far (a frame that exceeds it
// rescales the running sums, a rare uniform branch).
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "frame.h"
#include "ingest.h"
#include "kernels.h"
#include "split_shape.h"

namespace moff {

namespace {

typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f4 mm(h8 a, h8 b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0); }

// Two float32 values as binary16 pairs.  m1 is -1 passed at run time: the
// remainder then compiles to one mixed-precision multiply-add per value.
__device__ __forceinline__ void split2(float x, float y, float m1, h2& hi, h2& lo) {
  const f2 v = {x, y};
  hi = __builtin_convertvector(v, h2);
  const f2 r = {__builtin_fmaf(static_cast<float>(hi[0]), m1, x), __builtin_fmaf(static_cast<float>(hi[1]), m1, y)};
  lo = __builtin_convertvector(r, h2);
}

// An operand of one contraction of K folded indices: K = 32 as two operands
// (high, low), K = 16 as one operand with both halves (see split_pos).
template <int K>
struct Data {
  h8 v[K == 32 ? 2 : 1];
};
struct Coef {
  h8 hi, lo;
};

// data . coef over K, data as the A operand (rows) or the B operand (columns);
// the small products first.  `third` is the phase factors' third number, if any.
template <int K, bool DataIsA>
__device__ __forceinline__ f4 contract(const Data<K>& d, const Coef& c, const h8* third) {
  auto mul = [](h8 x, h8 y, f4 z) { return DataIsA ? mm(x, y, z) : mm(y, x, z); };
  f4 r = {0.f, 0.f, 0.f, 0.f};
  if (third) r = mul(d.v[0], *third, r);
  r = mul(d.v[0], c.lo, r);
  if constexpr (K == 32) r = mul(d.v[1], c.hi, r);
  return mul(d.v[0], c.hi, r);
}

// One wave's gather program: 64 cells at a time, steps and cell ends uniform.
template <bool CW>
__device__ __forceinline__ void gather_wave(const uint4* __restrict__ prog, const float2* __restrict__ progi,
                                            const uint32_t* __restrict__ ends, int n_steps,
                                            const char* __restrict__ e, char* __restrict__ G) {
  constexpr int B = kSplitBatch;
  float2 s = make_float2(0.f, 0.f);
  uint4 nxt[B / 2];
#pragma unroll
  for (int i = 0; i < B / 2; ++i) nxt[i] = prog[static_cast<size_t>(i) * 64];
  for (int s0 = 0; s0 < n_steps; s0 += B) {
    uint4 q[B / 2];
    float2 wi[CW ? B / 2 : 1];
#pragma unroll
    for (int i = 0; i < B / 2; ++i) {
      q[i] = nxt[i];
      if constexpr (CW) wi[i] = progi[static_cast<size_t>(s0 / 2 + i) * 64];
    }
    const int n0 = s0 + B < n_steps ? s0 + B : 0;   // (the last batch loads the first again)
#pragma unroll
    for (int i = 0; i < B / 2; ++i) nxt[i] = prog[static_cast<size_t>(n0 / 2 + i) * 64];
    const uint32_t end = ends[s0 / 32] >> (s0 % 32);
    float2 ev[B];
#pragma unroll
    for (int i = 0; i < B; ++i)
      ev[i] = *reinterpret_cast<const float2*>(e + ((i % 2 ? q[i / 2].z : q[i / 2].x) & 0xFFFFu));
#pragma unroll
    for (int i = 0; i < B; ++i) {
      const uint32_t x = i % 2 ? q[i / 2].z : q[i / 2].x;
      const float wr = __uint_as_float(i % 2 ? q[i / 2].w : q[i / 2].y);
      if constexpr (CW) {
        const float w2 = i % 2 ? wi[i / 2].y : wi[i / 2].x;
        s.x = fmaf(ev[i].x, wr, fmaf(-ev[i].y, w2, s.x));
        s.y = fmaf(ev[i].x, w2, fmaf(ev[i].y, wr, s.y));
      } else {
        s.x = fmaf(ev[i].x, wr, s.x);
        s.y = fmaf(ev[i].y, wr, s.y);
      }
      if (end & (1u << i)) {   // uniform
        *reinterpret_cast<float2*>(G + (x >> 16)) = s;
        s = make_float2(0.f, 0.f);
      }
    }
  }
}

}  // namespace

// Waves per SIMD the registers are sized for: at N = 128 the accumulators,
// phase factors and half-transformed columns take 192 registers, two waves; at
// N = 64 half of that, three.
constexpr int split_waves_per_simd(int N) { return N == 128 ? 2 : 3; }

// RT: the row stage takes the phase factors' third number, at N = 64 both stages.
template <int N, bool CI4, bool CW, bool RT>
__global__ __launch_bounds__((split_shape(N).NW * 64)) __attribute__((amdgpu_waves_per_eu(split_waves_per_simd(N))))
void split_kernel(SplitArgs a) {
  constexpr SplitShape S = split_shape(N);
  constexpr int L = S.L, K = S.K, NW = S.NW, NT = NW * 64, RP = S.RP, GP = S.GP, FP = S.FP;
  constexpr int PN = K / 16;            // 16-row panels per parity
  constexpr int QX = RP * K / 64;       // folded cells per lane, adjacent along x
  constexpr int NACC = NW * 2 * 4 * 2;  // accumulators per lane: row block, base / partner column, row, base / partner row
  extern __shared__ uint4 lds_split[];
  __shared__ double Atot[kMaxTypesDev];
  __shared__ float2 wave_max[NW];
  __shared__ int exceeded;
  char* lds = reinterpret_cast<char*>(lds_split);
  const SplitLayout lay = split_layout(N, a.n_ant);
  char* F = lds + lay.f;
  float2* e = reinterpret_cast<float2*>(lds + lay.e);
  float2* gl = reinterpret_cast<float2*>(lds + lay.gl);
  double* pw = reinterpret_cast<double*>(lds + lay.pw);

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  // workgroups are dealt to the XCDs round-robin: each gets a contiguous range
  // of (channel, slice) items
  const int per_xcd = gridDim.x / kXcds;
  const int item = (blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
  if (item >= a.n_chan * a.slices) return;
  const int c = item % a.n_chan, slice = item / a.n_chan;

  const int64_t T = a.n_time;
  const int64_t t0 = slice * T / a.slices, t1 = (slice + 1) * T / a.slices;
  const size_t frame_stride = static_cast<size_t>(a.n_chan) * a.n_ant;
  const size_t chan0 = static_cast<size_t>(c) * a.n_ant;

  // the samples of the first kPre antennas per lane are loaded a frame ahead
  constexpr int kPre = 2;
  float2 raw[kPre];
  auto load_raw = [&](int64_t t) {
    const size_t base = static_cast<size_t>(t) * frame_stride + chan0;
#pragma unroll
    for (int q = 0; q < kPre; ++q)
      if (tid + q * NT < a.n_ant) raw[q] = load_sample(a.E, base + tid + q * NT, CI4);
  };
  if (CI4 && t0 < t1) load_raw(t0);

  for (int i = tid; i < L * GP * 8 / 16; i += NT) lds_split[i] = make_uint4(0u, 0u, 0u, 0u);
  for (int i = tid; i < a.n_ant; i += NT) {
    const float2 gv = a.gains ? a.gains[static_cast<size_t>(c) * a.n_ant + i] : make_float2(1.f, 0.f);
    gl[i] = gv;
    pw[i] = 0.0;
  }
  if (tid == 0) {
    e[a.n_ant] = make_float2(0.f, 0.f);
    exceeded = 0;
  }

  // phase factors, row blocks in the order this wave takes them (its own first:
  // those are the row stage's factors too)
  constexpr bool CT = RT && split_third_in_columns(N);
  Coef cs[NW], sn[NW];
  h8 cs3[CT ? NW : 1], sn3[CT ? NW : 1];   // third numbers
  {
    const h8* src = reinterpret_cast<const h8*>(a.coef);
#pragma unroll
    for (int s = 0; s < NW; ++s) {
      const int rb = (w + s) % NW;
      auto part = [&](int trig, int q) { return src[((rb * 2 + trig) * kSplitParts + q) * 64 + lane]; };
      cs[s].hi = part(0, 0);
      cs[s].lo = part(0, 1);
      sn[s].hi = part(1, 0);
      sn[s].lo = part(1, 1);
      if constexpr (CT) {
        cs3[s] = part(0, 2);
        sn3[s] = part(1, 2);
      }
    }
  }
  const float m1 = a.minus_one;
  const float sc = (w == 0 && l16 == 0) ? 0.f : 1.f;   // base column 0 is the shared slot
  const float sr = g == 0 ? 0.f : 1.f;                 // row 0 of row block 0 likewise

  float acc[NW][2][4][2];
#pragma unroll
  for (int s = 0; s < NW; ++s)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[s][i >> 3][(i >> 1) & 3][i & 1] = 0.f;

  // scale 2^sk; `limit` is the largest sample component it allows
  int sk = 0;
  float scale = 1.f, limit = 0.f;
  auto set_scale = [&](float mx) {   // uniform; mx >= 0 finite
    int ex = 0;
    (void)frexpf(mx, &ex);           // mx < 2^ex
    sk = kSplitField - a.wexp - ex;  // wmax <= 2^wexp
    sk = sk > 126 ? 126 : sk < -126 ? -126 : sk;
    scale = ldexpf(1.f, sk);
    limit = ldexpf(1.f, ex);
  };
  auto wg_max = [&](float u, float v) {   // largest values over the workgroup (contains barriers); v: 4+4-bit only
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      u = fmaxf(u, __shfl_xor(u, off, 64));
      if constexpr (CI4) v = fmaxf(v, __shfl_xor(v, off, 64));
    }
    if (lane == 0) wave_max[w] = make_float2(u, v);
    __syncthreads();
    u = wave_max[0].x, v = wave_max[0].y;
#pragma unroll
    for (int i = 1; i < NW; ++i) {
      u = fmaxf(u, wave_max[i].x);
      if constexpr (CI4) v = fmaxf(v, wave_max[i].y);
    }
    __syncthreads();
    auto uniform = [](float x) { return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(x))); };
    return make_float2(uniform(u), CI4 ? uniform(v) : 0.f);
  };
  if constexpr (CI4) {
    // |Re g| + |Im g| of antenna i, zero where it is not finite
    auto gain = [&](int i) {
      const float m = fabsf(gl[i].x) + fabsf(gl[i].y);
      return m < __builtin_huge_valf() ? m : 0.f;
    };
    auto sample = [&](int64_t t, int i) {
      return reinterpret_cast<const uint8_t*>(a.E)[static_cast<size_t>(t) * frame_stride + chan0 + i];
    };
    auto use = [&](float m) {
      if (m > 0.f && m < __builtin_huge_valf()) set_scale(m);
    };
    float seen = 0.f, all = 0.f;   // largest gain where the first frame has a sample, and of all
    auto see = [&](int i, bool on) {
      const float m = gain(i);
      all = fmaxf(all, m);
      if (on) seen = fmaxf(seen, m);
    };
    if (t0 < t1) {
#pragma unroll
      for (int q = 0; q < kPre; ++q)
        if (tid + q * NT < a.n_ant) see(tid + q * NT, raw[q].x != 0.f || raw[q].y != 0.f);
      for (int i = tid + kPre * NT; i < a.n_ant; i += NT) see(i, sample(t0, i) != 0);
    }
    const float2 most = wg_max(seen, all);
    use(8.f * most.x);
    if (8.f * most.y > limit) {
      for (int i = tid; i < a.n_ant; i += NT) {
        const float m = gain(i);
        if (!(m > most.x)) continue;
        uint32_t any = 0;
        for (int64_t t = t0; t < t1 && any == 0; t += 8)
#pragma unroll
          for (int k = 0; k < 8; ++k) any |= sample(t + k < t1 ? t + k : t1 - 1, i);
        if (any != 0) seen = fmaxf(seen, m);
      }
      use(8.f * wg_max(seen, 0.f).x);
    }
  }

  // ingest of frame t: e = g E scaled, self power per antenna in float64
  auto ingest = [&](int64_t t) {
    bool over = false;
    auto take = [&](int i, float2 r) {
      const float2 v = c_mul(gl[i], r);
      unsafeAtomicAdd(pw + i, static_cast<double>(v.x) * v.x + static_cast<double>(v.y) * v.y);   // this lane alone writes pw[i]
      if constexpr (!CI4) {
        const float m = fmaxf(fabsf(v.x), fabsf(v.y));
        over = over || (m > limit && m < __builtin_huge_valf());
      }
      e[i] = make_float2(v.x * scale, v.y * scale);
    };
#pragma unroll
    for (int q = 0; q < kPre; ++q)
      if (tid + q * NT < a.n_ant) take(tid + q * NT, raw[q]);
    const size_t base = static_cast<size_t>(t) * frame_stride + chan0;
    for (int i = tid + kPre * NT; i < a.n_ant; i += NT) take(i, load_sample(a.E, base + i, CI4));
    if constexpr (!CI4)
      if (over) exceeded = 1;
  };
  // after the barrier that follows ingest(t): a larger scale limit if frame t needs it
  auto rescale = [&](int64_t t) {
    if constexpr (!CI4) {
      if (__builtin_amdgcn_readfirstlane(exceeded) == 0) return;
      const size_t base = static_cast<size_t>(t) * frame_stride + chan0;
      float mx = 0.f;
      for (int i = tid; i < a.n_ant; i += NT) {
        const float2 v = c_mul(gl[i], load_sample(a.E, base + i, CI4));
        const float m = fmaxf(fabsf(v.x), fabsf(v.y));
        if (m < __builtin_huge_valf()) mx = fmaxf(mx, m);
      }
      mx = wg_max(mx, 0.f).x;
      const int old = sk;
      set_scale(fminf(2.f * mx, 3.0e38f));   // with headroom: later frames seldom exceed it
      for (int i = tid; i < a.n_ant; i += NT) {
        const float2 v = c_mul(gl[i], load_sample(a.E, base + i, CI4));
        e[i] = make_float2(v.x * scale, v.y * scale);
      }
      // (the sums are still zero at the first scale; later ones are smaller)
      const int df = 2 * (sk - old);
      const float f = df >= 0 ? 1.f : ldexpf(1.f, df < -252 ? -252 : df);
#pragma unroll
      for (int s = 0; s < NW; ++s)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[s][i >> 3][(i >> 1) & 3][i & 1] *= f;
      if (tid == 0) exceeded = 0;
      __syncthreads();
    }
  };

  const uint4* prog = a.prog + static_cast<size_t>(w) * (a.steps / 2) * 64 + lane;
  const float2* progi = CW ? a.progi + static_cast<size_t>(w) * (a.steps / 2) * 64 + lane : nullptr;
  const uint32_t* ends = a.ends + w * ((a.steps + 31) / 32);
  const int n_steps = a.n_steps[w];
  char* Gw = lds + w * (2 * RP * GP * 8);

  double* run64 = a.acc64 ? a.acc64 + static_cast<size_t>(item) * NACC * NT : nullptr;
  bool flushed = false;
  int in_block = 0;

  if (t0 < t1) {
    if constexpr (!CI4) load_raw(t0);
    __syncthreads();
    ingest(t0);
    if (t0 + 1 < t1) load_raw(t0 + 1);
  }
  __syncthreads();
  if (t0 < t1) rescale(t0);

  for (int64_t t = t0; t < t1; ++t) {
    // The two workgroups of a SIMD drift apart: the one whose phase waits for
    // memory and LDS issues first, the one in the long column stage fills the
    // gaps (at 128 channels x 1000 samples of 256 antennas, N = 128: 1.31 ms
    // without priorities, 1.22 with).
    __builtin_amdgcn_s_setprio(2);
    if constexpr (RT && !CT) {
      // (requested anew each frame: held through the loop, these 8 registers were
      // spilled with 15 more, 1.41 ms instead of 1.28 at the shape above)
      int zero;
      asm volatile("s_mov_b32 %0, 0" : "=s"(zero));
      const h8* src = reinterpret_cast<const h8*>(a.coef) + zero + w * 2 * kSplitParts * 64 + lane;
      cs3[0] = src[2 * 64];
      sn3[0] = src[(kSplitParts + 2) * 64];
    }
    gather_wave<CW>(prog, progi, ends, n_steps, reinterpret_cast<const char*>(e), Gw);
    wave_sync();
    {
      // fold QX adjacent cells of row pair j, split, store
      const int j = lane >> 3, x0 = QX * (lane & 7), i = w + NW * j;
      const float2* up = reinterpret_cast<const float2*>(Gw) + j * GP;
      const float2* dn = up + RP * GP;
      float2 A[QX], B[QX], C[QX], D[QX];
#pragma unroll
      for (int q = 0; q < QX; q += 2) {
        const float4 va = *reinterpret_cast<const float4*>(up + x0 + q);
        const float4 vb = *reinterpret_cast<const float4*>(up + L - 2 - x0 - q);
        const float4 vc = *reinterpret_cast<const float4*>(dn + x0 + q);
        const float4 vd = *reinterpret_cast<const float4*>(dn + L - 2 - x0 - q);
        A[q] = make_float2(va.x, va.y), A[q + 1] = make_float2(va.z, va.w);
        B[q] = make_float2(vb.z, vb.w), B[q + 1] = make_float2(vb.x, vb.y);
        C[q] = make_float2(vc.x, vc.y), C[q + 1] = make_float2(vc.z, vc.w);
        D[q] = make_float2(vd.z, vd.w), D[q + 1] = make_float2(vd.x, vd.y);
      }
#pragma unroll
      for (int y = 0; y < 2; ++y) {
        float v[4][QX];   // {sum, difference along x} x {re, im}
#pragma unroll
        for (int q = 0; q < QX; ++q) {
          const float2 l = y ? c_sub(A[q], C[q]) : c_add(A[q], C[q]), r = y ? c_sub(B[q], D[q]) : c_add(B[q], D[q]);
          v[0][q] = l.x + r.x;
          v[1][q] = l.y + r.y;
          v[2][q] = l.x - r.x;
          v[3][q] = l.y - r.y;
        }
        _Float16* row = reinterpret_cast<_Float16*>(F + (y * K + i) * FP);
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          _Float16* hi = row + p * 2 * K + split_pos(K, x0, 0);
          _Float16* lo = row + p * 2 * K + split_pos(K, x0, 1);
          if constexpr (QX == 4) {
            h2 a0, b0, a1, b1;
            split2(v[p][0], v[p][1], m1, a0, b0);
            split2(v[p][2], v[p][3], m1, a1, b1);
            *reinterpret_cast<h4*>(hi) = __builtin_shufflevector(a0, a1, 0, 1, 2, 3);
            *reinterpret_cast<h4*>(lo) = __builtin_shufflevector(b0, b1, 0, 1, 2, 3);
          } else {
            h2 a0, b0;
            split2(v[p][0], v[p][1], m1, a0, b0);
            *reinterpret_cast<h2*>(hi) = a0;
            *reinterpret_cast<h2*>(lo) = b0;
          }
        }
      }
    }
    __syncthreads();

    // row stage: this wave's 16 base columns and their partners, all rows
    h4 z[2][2][2][2][PN];   // [y sum, difference][base, partner][re, im][high, low][panel]
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int pn = 0; pn < PN; ++pn) {
        const _Float16* row = reinterpret_cast<const _Float16*>(F + (y * K + 16 * pn + l16) * FP) + 8 * g;
        auto operand = [&](int p) {
          Data<K> d;
          d.v[0] = *reinterpret_cast<const h8*>(row + p * 2 * K);
          if constexpr (K == 32) d.v[1] = *reinterpret_cast<const h8*>(row + p * 2 * K + K);
          return d;
        };
        const h8 *c3 = RT ? cs3 : nullptr, *s3 = RT ? sn3 : nullptr;
        const f4 P1 = contract<K, true>(operand(0), cs[0], c3), P4 = contract<K, true>(operand(1), cs[0], c3);
        const f4 P3 = contract<K, true>(operand(2), sn[0], s3), P2 = contract<K, true>(operand(3), sn[0], s3);
        float v[2][2][4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          v[0][0][q] = fmaf(-sc, P2[q], P1[q]);
          v[0][1][q] = fmaf(sc, P3[q], P4[q]);
          v[1][0][q] = fmaf(sc, P1[q], P2[q]);
          v[1][1][q] = fmaf(sc, P4[q], -P3[q]);
        }
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int r = 0; r < 2; ++r) {
            h2 a0, b0, a1, b1;
            split2(v[b][r][0], v[b][r][1], m1, a0, b0);
            split2(v[b][r][2], v[b][r][3], m1, a1, b1);
            z[y][b][r][0][pn] = __builtin_shufflevector(a0, a1, 0, 1, 2, 3);
            z[y][b][r][1][pn] = __builtin_shufflevector(b0, b1, 0, 1, 2, 3);
          }
      }
    if (t + 1 < t1) {
      ingest(t + 1);
      if (t + 2 < t1) load_raw(t + 2);
    }
    __syncthreads();

    // column stage and |Y|^2: all row blocks of both column sets
    __builtin_amdgcn_s_setprio(0);
    auto column = [&](int y, int b, int r) {
      Data<K> d;
      if constexpr (K == 32) {
        d.v[0] = __builtin_shufflevector(z[y][b][r][0][0], z[y][b][r][0][PN - 1], 0, 1, 2, 3, 4, 5, 6, 7);
        d.v[1] = __builtin_shufflevector(z[y][b][r][1][0], z[y][b][r][1][PN - 1], 0, 1, 2, 3, 4, 5, 6, 7);
      } else {
        d.v[0] = __builtin_shufflevector(z[y][b][r][0][0], z[y][b][r][1][0], 0, 1, 2, 3, 4, 5, 6, 7);
      }
      return d;
    };
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const Data<K> sre = column(0, b, 0), sim = column(0, b, 1), dre = column(1, b, 0), dim = column(1, b, 1);
#pragma unroll
      for (int s = 0; s < NW; ++s) {
        const h8 *c3 = CT ? cs3 + s : nullptr, *s3 = CT ? sn3 + s : nullptr;
        const f4 P1 = contract<K, false>(sre, cs[s], c3), P4 = contract<K, false>(sim, cs[s], c3);
        const f4 P3 = contract<K, false>(dre, sn[s], s3), P2 = contract<K, false>(dim, sn[s], s3);
        const float s0 = (w + s) % NW == 0 ? sr : 1.f;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float br, bi, pr, pi;
          if (q == 0) {
            br = fmaf(-s0, P2[0], P1[0]), bi = fmaf(s0, P3[0], P4[0]);
            pr = fmaf(s0, P1[0], P2[0]), pi = fmaf(s0, P4[0], -P3[0]);
          } else {
            br = P1[q] - P2[q], bi = P3[q] + P4[q];
            pr = P1[q] + P2[q], pi = P4[q] - P3[q];
          }
          if constexpr (N == 64) {
            // (one rounding of the running sum per frame instead of two; the
            // gather bounds this grid, so the extra instruction is free)
            acc[s][b][q][0] += fmaf(br, br, bi * bi);
            acc[s][b][q][1] += fmaf(pr, pr, pi * pi);
          } else {
            acc[s][b][q][0] = fmaf(br, br, fmaf(bi, bi, acc[s][b][q][0]));
            acc[s][b][q][1] = fmaf(pr, pr, fmaf(pi, pi, acc[s][b][q][1]));
          }
        }
      }
    }
    // blocked accumulation: fold the block's float32 sums into float64 (as in
    // the FFT kernel: first block stored, later ones added, one writer each)
    if (a.acc64 && ++in_block == kBlockFrames && t + 1 < t1) {   // uniform
      int zero;
      asm volatile("s_mov_b32 %0, 0" : "=s"(zero));
      double* blk = run64 + zero + tid;
      const double un = ldexp(1.0, -2 * sk);
#pragma unroll
      for (int s = 0; s < NW; ++s)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          float& v = acc[s][i >> 3][(i >> 1) & 3][i & 1];
          if (!flushed) blk[(s * 16 + i) * NT] = static_cast<double>(v) * un;
          else unsafeAtomicAdd(blk + (s * 16 + i) * NT, static_cast<double>(v) * un);
          v = 0.f;
        }
      flushed = true;
      in_block = 0;
    }
    if (t + 1 < t1) rescale(t + 1);
  }

  // ---- epilogue: self power per type, then the pixels
  {
    double p[kMaxTypesDev] = {0.0, 0.0, 0.0, 0.0};
    for (int i = tid; i < a.n_ant; i += NT) {
      const int tp = a.ant_type[i];
#pragma unroll
      for (int q = 0; q < kMaxTypesDev; ++q) p[q] += (tp == q) ? pw[i] : 0.0;
    }
    block_sum4<NT>(p, Atot);   // (its barriers also end every use of the grids)
  }
  const double un = ldexp(1.0, -2 * sk), unc = ldexp(1.0, -4 * split_coef(N));
  const size_t img_stride = static_cast<size_t>(N) * N;
  float* stage = reinterpret_cast<float*>(lds);   // [N][N], groups of 16 columns XORed by row / 4
  static_assert(N * N * 4 <= L * GP * 8 + 2 * K * FP, "staging must fit in the grids");
#pragma unroll
  for (int s = 0; s < NW; ++s) {
    const int rb = (w + s) % NW;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int b = i >> 3, q = (i >> 1) & 3, pr = i & 1;
      const int row = 16 * rb + 4 * g + q, col = 16 * w + l16;   // base indices
      const int r = pr ? (row == 0 ? 0 : L - row) : L + row, x = b ? (col == 0 ? 0 : L - col) : L + col;
      const size_t pix = static_cast<size_t>(r) * N + x;
      double sum = static_cast<double>(acc[s][b][q][pr]) * un;
      if (flushed)
        sum += __hip_atomic_load(run64 + (s * 16 + i) * NT + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      sum *= unc;
      float* at = stage + r * N + (x ^ (((r >> 2) & 3) << 4));
      if (a.mode == kModePartial) {
        *at = static_cast<float>(sum);
      } else if (a.mode == kModeAccum) {
        float& o = a.out[static_cast<size_t>(c) * img_stride + pix];
        o = static_cast<float>(static_cast<double>(o) + sum);
      } else {
        double v = sum;
        if (a.subtract)
          for (int p = 0; p < a.n_types; ++p) v -= Atot[p] * a.Pp[p * img_stride + pix];
        *at = static_cast<float>(v * a.scale);
      }
    }
  }
  if (a.mode != kModeAccum) {
    __syncthreads();
    float* dst = a.out + (a.mode == kModePartial ? static_cast<size_t>(item) : static_cast<size_t>(c)) * img_stride;
    for (int i = tid; i < N * N / 4; i += NT) {
      const int r = i / (N / 4), x = 4 * (i % (N / 4));
      const float4 v = *reinterpret_cast<const float4*>(stage + r * N + (x ^ (((r >> 2) & 3) << 4)));
      *reinterpret_cast<float4*>(dst + static_cast<size_t>(r) * N + x) = v;
    }
  }
  if (tid < a.n_types) {
    if (a.mode == kModePartial) a.outA[static_cast<size_t>(item) * a.n_types + tid] = Atot[tid];
    else if (a.mode == kModeAccum) a.outA[static_cast<size_t>(c) * a.n_types + tid] += Atot[tid];
  }
}

namespace {

template <int N, bool RT>
const void* split_symbol_n(bool ci4, bool cw) {
  return ci4 ? (cw ? reinterpret_cast<const void*>(split_kernel<N, true, true, RT>)
                   : reinterpret_cast<const void*>(split_kernel<N, true, false, RT>))
             : (cw ? reinterpret_cast<const void*>(split_kernel<N, false, true, RT>)
                   : reinterpret_cast<const void*>(split_kernel<N, false, false, RT>));
}

const void* split_symbol(int N, bool ci4, bool cw, bool third) {
  if (N == 64) return third ? split_symbol_n<64, true>(ci4, cw) : split_symbol_n<64, false>(ci4, cw);
  if (N == 128) return third ? split_symbol_n<128, true>(ci4, cw) : split_symbol_n<128, false>(ci4, cw);
  return nullptr;
}

}  // namespace

hipError_t launch_split(const SplitArgs& a, int N, bool ci4, int grid, hipStream_t st) {
  const void* k = split_symbol(N, ci4, a.progi != nullptr, a.third != 0);
  if (!k || grid <= 0 || grid % kXcds != 0 || static_cast<int64_t>(grid) < static_cast<int64_t>(a.n_chan) * a.slices)
    return hipErrorInvalidValue;
  const int lds = split_layout(N, a.n_ant).end;
  hipError_t err = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (err != hipSuccess) return err;
  void* args[] = {const_cast<SplitArgs*>(&a)};
  return hipLaunchKernel(k, dim3(grid), dim3(split_shape(N).NW * 64), args, lds, st);
}

int split_blocks_per_cu(int N, bool ci4, bool cw, bool third, int n_ant) {
  const void* k = split_symbol(N, ci4, cw, third);
  return k ? blocks_held(k, split_shape(N).NW * 64, split_layout(N, n_ant).end) : 0;
}

}  // namespace moff
