// One-dimensional transforms of a compile-time length held in registers,
// with the twiddle factors as compile-time constants (instruction literals
// in complex64: no table loads and no scalar registers).
#pragma once

#include "common.h"

// exp(-2 pi i k / N), k < N, in double: octant-reduced Taylor series, exact
// at the multiples of a quarter turn.
namespace twiddle {
constexpr double kTwoPi = 6.283185307179586476925286766559;
struct CS {
  double c, s;
};
constexpr CS cos_sin(long q, long D) {  // of 2 pi q / D, 0 <= q < D, D a multiple of 8
  if (2 * q > D) {
    CS r = cos_sin(D - q, D);
    return CS{r.c, -r.s};
  }
  if (4 * q > D) {
    CS r = cos_sin(D / 2 - q, D);
    return CS{-r.c, r.s};
  }
  if (8 * q > D) {
    CS r = cos_sin(D / 4 - q, D);
    return CS{r.s, r.c};
  }
  const double x = kTwoPi * (double)q / (double)D, x2 = x * x;
  double c = 0, s = 0;
  for (int k = 11; k >= 0; --k) {  // Horner, terms to x^23
    c = 1.0 - c * x2 / (double)((2 * k + 1) * (2 * k + 2));
    s = 1.0 - s * x2 / (double)((2 * k + 2) * (2 * k + 3));
  }
  return CS{c, s * x};
}
template <int N>
struct Table {
  double re[N], im[N];
  constexpr Table() : re(), im() {
    for (int k = 0; k < N; ++k) {
      const CS r = cos_sin(8L * k, 8L * N);
      re[k] = r.c;
      im[k] = -r.s;
    }
  }
};
template <int N> __device__ constexpr Table<N> table{};
}  // namespace twiddle

// x exp(sign 2 pi i k / N), k a constant once the caller's loops are unrolled
template <typename T, int N, int SIGN>
__device__ __forceinline__ cplx<T> mul_tw(cplx<T> x, int k) {
  const double c = twiddle::table<N>.re[k], s = SIGN < 0 ? twiddle::table<N>.im[k] : -twiddle::table<N>.im[k];
  if (s == 0.0) return c > 0 ? x : -x;
  if (c == 0.0) return s > 0 ? mk(-x.im, x.re) : mk(x.im, -x.re);
  const T cr = (T)c, ci = (T)s;
  return mk(x.re * cr - x.im * ci, x.re * ci + x.im * cr);
}

template <typename T, int R, int SIGN>
__device__ __forceinline__ void butterfly(cplx<T>* v) {
  if constexpr (R == 2) {
    const cplx<T> a = v[0], b = v[1];
    v[0] = a + b;
    v[1] = a - b;
  } else if constexpr (R == 3) {
    const T h = (T)0.86602540378443864676372317075294;
    const cplx<T> t = v[1] + v[2], d = v[1] - v[2];
    const cplx<T> m = mk(v[0].re - (T)0.5 * t.re, v[0].im - (T)0.5 * t.im);
    const cplx<T> js = SIGN < 0 ? mk(h * d.im, -h * d.re) : mk(-h * d.im, h * d.re);  // sign i h d
    v[0] = v[0] + t;
    v[1] = m + js;
    v[2] = m - js;
  } else if constexpr (R == 4) {
    const cplx<T> s0 = v[0] + v[2], s1 = v[0] - v[2], s2 = v[1] + v[3], s3 = v[1] - v[3];
    const cplx<T> js = SIGN < 0 ? mk(s3.im, -s3.re) : mk(-s3.im, s3.re);
    v[0] = s0 + s2;
    v[1] = s1 + js;
    v[2] = s0 - s2;
    v[3] = s1 - js;
  } else {
    cplx<T> in[R];
#pragma unroll
    for (int r = 0; r < R; ++r) in[r] = v[r];
#pragma unroll
    for (int s = 0; s < R; ++s) {
      cplx<T> acc = in[0];
#pragma unroll
      for (int r = 1; r < R; ++r) acc = acc + mul_tw<T, R, SIGN>(in[r], (r * s) % R);
      v[s] = acc;
    }
  }
}

template <typename T, int N, int Ns, int SIGN>
__device__ __forceinline__ void line_fft_stages(cplx<T>* a, cplx<T>* b) {
  if constexpr (Ns < N) {
    constexpr int R = pick_radix(N / Ns);
    constexpr int per = N / R;
    constexpr int tstep = N / (Ns * R);
#pragma unroll
    for (int j = 0; j < per; ++j) {
      const int k = j % Ns;
      cplx<T> v[R];
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = r ? mul_tw<T, N, SIGN>(a[j + r * per], (r * k * tstep) % N) : a[j];
      butterfly<T, R, SIGN>(v);
      const int o = (j / Ns) * Ns * R + k;
#pragma unroll
      for (int r = 0; r < R; ++r) b[o + r * Ns] = v[r];
    }
    line_fft_stages<T, N, Ns * R, SIGN>(b, a);
  }
}

// x <- DFT_N(x), SIGN -1 forward / +1 inverse (unnormalised)
template <typename T, int N, int SIGN>
__device__ __forceinline__ void line_fft(cplx<T>* x) {
  cplx<T> y[N];
  line_fft_stages<T, N, 1, SIGN>(x, y);
  if constexpr (count_stages(N) % 2 == 1) {
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = y[i];
  }
}
