// In-register complex DFTs for the gfx950 frame transform.
//
// All transforms use the positive exponent, X[k] = sum_n x[n] exp(+2 pi i n k / R),
// unnormalised, natural order in and out (Sec. 3: the image is the Fourier
// transform of the gridded field with the fringe sign of Sec. 2).  Twiddles of
// the in-register stages are compile-time constants; multiplications by 1,
// +-i and the eighth roots are strength-reduced.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

namespace moff {

__device__ __forceinline__ float2 c_add(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 c_sub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 c_mul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
// a * conj(b)
__device__ __forceinline__ float2 c_mul_conj(float2 a, float2 b) {
  return make_float2(a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y);
}
__device__ __forceinline__ float2 c_mul_i(float2 a) { return make_float2(-a.y, a.x); }
__device__ __forceinline__ float2 c_mul_mi(float2 a) { return make_float2(a.y, -a.x); }
__device__ __forceinline__ float2 c_neg(float2 a) { return make_float2(-a.x, -a.y); }

template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

// cos / sin of 2 pi k / 16 (k < 16), exact decimal expansions of the
// sixteenth roots of unity.
struct Root16 {
  static constexpr float c1 = 0.92387953251128675613f;  // cos(pi / 8)
  static constexpr float s1 = 0.38268343236508977173f;  // sin(pi / 8)
  static constexpr float r2 = 0.70710678118654752440f;  // sqrt(2) / 2
  static constexpr float re(int k) {
    constexpr float t[16] = {1.f, c1, r2, s1, 0.f, -s1, -r2, -c1, -1.f, -c1, -r2, -s1, 0.f, s1, r2, c1};
    return t[k & 15];
  }
  static constexpr float im(int k) {
    constexpr float t[16] = {0.f, s1, r2, c1, 1.f, c1, r2, s1, 0.f, -s1, -r2, -c1, -1.f, -c1, -r2, -s1};
    return t[k & 15];
  }
};

// a * exp(+2 pi i K16 / 16), 0 <= K16 < 16.
template <int k16>
__device__ __forceinline__ float2 rot16(float2 a) {
  if constexpr (k16 == 0) {
    return a;
  } else if constexpr (k16 == 4) {
    return c_mul_i(a);
  } else if constexpr (k16 == 8) {
    return c_neg(a);
  } else if constexpr (k16 == 12) {
    return c_mul_mi(a);
  } else if constexpr (k16 == 2) {  // (1 + i) / sqrt 2
    return make_float2((a.x - a.y) * Root16::r2, (a.x + a.y) * Root16::r2);
  } else if constexpr (k16 == 6) {  // (-1 + i) / sqrt 2
    return make_float2((-a.x - a.y) * Root16::r2, (a.x - a.y) * Root16::r2);
  } else if constexpr (k16 == 10) {  // (-1 - i) / sqrt 2
    return make_float2((a.y - a.x) * Root16::r2, (-a.x - a.y) * Root16::r2);
  } else if constexpr (k16 == 14) {  // (1 - i) / sqrt 2
    return make_float2((a.x + a.y) * Root16::r2, (a.y - a.x) * Root16::r2);
  } else {
    constexpr float c = Root16::re(k16), s = Root16::im(k16);
    return make_float2(a.x * c - a.y * s, a.x * s + a.y * c);
  }
}

// cos / sin of 2 pi k / 32 (k < 32), exact decimal expansions of the
// thirty-second roots of unity; sin(2 pi k / 32) = cos(2 pi (k - 8) / 32).
struct Root32 {
  static constexpr float c1 = 0.98078528040323044913f;  // cos(pi / 16)
  static constexpr float s1 = 0.19509032201612826785f;  // sin(pi / 16)
  static constexpr float c3 = 0.83146961230254523708f;  // cos(3 pi / 16)
  static constexpr float s3 = 0.55557023301960222474f;  // sin(3 pi / 16)
  static constexpr float re(int k) {
    constexpr float t[32] = {1.f,       c1,  Root16::c1,  c3,  Root16::r2,  s3,  Root16::s1,  s1,
                             0.f,       -s1, -Root16::s1, -s3, -Root16::r2, -c3, -Root16::c1, -c1,
                             -1.f,      -c1, -Root16::c1, -c3, -Root16::r2, -s3, -Root16::s1, -s1,
                             0.f,       s1,  Root16::s1,  s3,  Root16::r2,  c3,  Root16::c1,  c1};
    return t[k & 31];
  }
  static constexpr float im(int k) { return re((k - 8) & 31); }
};

// a * exp(+2 pi i K / R), R dividing 32.
template <int R, int K>
__device__ __forceinline__ float2 rot(float2 a) {
  static_assert(32 % R == 0, "rotation order must divide 32");
  constexpr int k = ((K % R) + R) % R;
  constexpr int k32 = k * (32 / R);
  if constexpr (k32 % 2 != 0) {     // an odd thirty-second root
    constexpr float c = Root32::re(k32), s = Root32::im(k32);
    return make_float2(a.x * c - a.y * s, a.x * s + a.y * c);
  } else {
    return rot16<k32 / 2>(a);
  }
}

// Butterflies with the multiplication folded into their additions: with
// w = c (1 + i t), t = tan(arg w), e +- w o = e +- c p for p = o + i t o, six
// fused multiply-adds instead of the eight operations of a product and two sums
// (Linzer and Feig, "Implementation of efficient FFT algorithms on fused
// multiply-add architectures", 1993).  Past 45 degrees w = s (u + i) with the
// cotangent u.  Each output is rounded once and p once.
__device__ __forceinline__ float2 lf_tan(float2 o, float t) { return make_float2(fmaf(-o.y, t, o.x), fmaf(o.x, t, o.y)); }
__device__ __forceinline__ float2 lf_cot(float2 o, float u) { return make_float2(fmaf(o.x, u, -o.y), fmaf(o.y, u, o.x)); }
__device__ __forceinline__ float2 c_fma(float m, float2 p, float2 e) { return make_float2(fmaf(m, p.x, e.x), fmaf(m, p.y, e.y)); }

// a = e + exp(2 pi i K / 32) o, b = e - exp(2 pi i K / 32) o.
template <int K>
__device__ __forceinline__ void butterfly(float2 e, float2 o, float2& a, float2& b) {
  if constexpr (K % 8 == 0) {
    const float2 t = rot16<K / 2>(o);
    a = c_add(e, t);
    b = c_sub(e, t);
  } else {
    constexpr float c = Root32::re(K), s = Root32::im(K);
    constexpr bool cot = (c < 0 ? -c : c) < (s < 0 ? -s : s);
    constexpr float m = cot ? s : c;
    constexpr float q = static_cast<float>(cot ? static_cast<double>(c) / s : static_cast<double>(s) / c);
    const float2 p = cot ? lf_cot(o, q) : lf_tan(o, q);
    a = c_fma(m, p, e);
    b = c_fma(-m, p, e);
  }
}

// Dense R-point DFT in registers (R = 1, 2, 4, 8, 16) of x[n] exp(2 pi i n T / 32)
// (T = 0: the plain DFT): radix-2 decimation in time, each level's butterflies
// taking the twist of their own sub-sequence.
template <int R, int T = 0>
struct Dft {
  __device__ __forceinline__ static void run(float2* x) {
    if constexpr (R > 1) {
      float2 e[R / 2], o[R / 2];
#pragma unroll
      for (int m = 0; m < R / 2; ++m) {
        e[m] = x[2 * m];
        o[m] = x[2 * m + 1];
      }
      Dft<R / 2, 2 * T % 32>::run(e);
      Dft<R / 2, 2 * T % 32>::run(o);
      static_for<0, R / 2>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        butterfly<(T + k * (32 / R)) % 32>(e[k], o[k], x[k], x[k + R / 2]);
      });
    }
  }
};

// R-point DFT of x[n] exp(2 pi i n T / 32) whose inputs are zero for n >= NZ (NZ a
// power of two <= R).  Decimation in frequency removes the zero half: the even
// outputs are the R/2-point DFT of the same inputs, the odd ones that of the
// inputs twisted by one more R-th root.  Only x[0 .. NZ-1] is read.
template <int R, int NZ, int T = 0>
__device__ __forceinline__ void dft_pruned(float2* x) {
  static_assert(NZ >= 1 && NZ <= R && (NZ & (NZ - 1)) == 0, "NZ must be a power of two <= R");
  if constexpr (NZ == R) {
    Dft<R, T>::run(x);
  } else {
    float2 e[R / 2], o[R / 2];
#pragma unroll
    for (int n = 0; n < NZ; ++n) e[n] = o[n] = x[n];
    dft_pruned<R / 2, NZ, T>(e);
    dft_pruned<R / 2, NZ, (T + 32 / R) % 32>(o);
#pragma unroll
    for (int k = 0; k < R / 2; ++k) {
      x[2 * k] = e[k];
      x[2 * k + 1] = o[k];
    }
  }
}

// A twisted DFT, X[k] = sum_n x[n] w_N^{n b} exp(2 pi i n k / R), with a twist b
// known only at run time, 0 <= b R < N: six operations for every butterfly and none
// for the twiddles, 192 at R = 16 where 15 twiddles and a plain DFT take 208 (at R = 8
// 72 and 80).  Against 64 bits the power of a pruned 256-point column (16 x 16) comes
// out at 1.20e-7 with it and 1.23e-7 with twiddles, but that of a 128-point one
// (16 x 8) at 1.14e-7 and 1.09e-7: it is used at R = 16 only.
// It takes R/2 factors, the level that joins sub-transforms to S points S/4 of them
// (k and k + S/4 differ by a factor of i), one at S = 2.  Their angles lie below
// 2 pi (k + 1) / S, so whether a factor is kept as (cosine, tangent) or (sine,
// cotangent) is known beforehand (twist_cot); S = 2 reaches both ends and keeps
// (cosine, sine).
constexpr int twist_level(int R, int i) {
  int S = R, off = 0;
  while (S >= 4 && i >= off + S / 4) {
    off += S / 4;
    S /= 2;
  }
  return S;
}
constexpr int twist_offset(int R, int S) { return S == 2 ? R / 2 - 1 : R / 2 - S / 2; }
constexpr bool twist_cot(int S, int k) { return 8 * k >= S && S > 4; }
// Factor i of the R-point DFT twisted by b, from the table of w_N^k.
template <int N>
__device__ __forceinline__ float2 twist_factor(const float2* __restrict__ tw, int R, int i, int b) {
  const int S = twist_level(R, i), k = i - twist_offset(R, S);
  const float2 w = tw[(b * (R / S) + k * (N / S)) & (N - 1)];
  if (S == 2) return w;
  if (twist_cot(S, k)) return make_float2(w.y, static_cast<float>(static_cast<double>(w.x) / w.y));
  return make_float2(w.x, static_cast<float>(static_cast<double>(w.y) / w.x));
}

template <int R, int TOP = R>
struct TwistedDft {
  __device__ __forceinline__ static void run(float2* x, const float2* f) {
    if constexpr (R > 1) {
      float2 e[R / 2], o[R / 2];
#pragma unroll
      for (int m = 0; m < R / 2; ++m) {
        e[m] = x[2 * m];
        o[m] = x[2 * m + 1];
      }
      TwistedDft<R / 2, TOP>::run(e, f);
      TwistedDft<R / 2, TOP>::run(o, f);
      if constexpr (R == 2) {   // (no tangent holds over a half turn: the difference from the sum)
        const float2 w = f[twist_offset(TOP, 2)];
        x[0] = make_float2(fmaf(o[0].x, w.x, fmaf(-o[0].y, w.y, e[0].x)), fmaf(o[0].x, w.y, fmaf(o[0].y, w.x, e[0].y)));
        x[1] = make_float2(fmaf(2.f, e[0].x, -x[0].x), fmaf(2.f, e[0].y, -x[0].y));
      } else {
#pragma unroll
        for (int k = 0; k < R / 2; ++k) {
          const int kq = k % (R / 4);
          const float2 w = f[twist_offset(TOP, R) + kq];
          const float2 oi = k < R / 4 ? o[k] : c_mul_i(o[k]);
          const float2 p = twist_cot(R, kq) ? lf_cot(oi, w.y) : lf_tan(oi, w.y);
          x[k] = c_fma(w.x, p, e[k]);
          x[k + R / 2] = c_fma(-w.x, p, e[k]);
        }
      }
    }
  }
};

// Inverse-direction R-point DFT, X[k] = sum_n x[n] exp(-2 pi i n k / R), through
// conjugation: conj(DFT(conj(x))).
template <int R>
__device__ __forceinline__ void idft(float2* x) {
#pragma unroll
  for (int i = 0; i < R; ++i) x[i].y = -x[i].y;
  Dft<R>::run(x);
#pragma unroll
  for (int i = 0; i < R; ++i) x[i].y = -x[i].y;
}

}  // namespace moff
