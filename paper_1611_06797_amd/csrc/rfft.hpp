// Register-resident transforms of real lines, built on the complex ones of
// fft.hpp: X[k] = sum_n x[n] exp(-2 pi i k n / N) for k = 0 .. N / 2 (the
// other half is the complex conjugate and is never computed).  One thread
// owns one line.  All loops unroll at compile time, so outputs that the
// caller does not use cost nothing.
//
// Coprime factors N = N1 N2 use the prime-factor index maps of fft.hpp: real
// N1-point transforms, of which only k1 <= N1 / 2 is kept (the partner
// N1 - k1 is the conjugate), then a complex N2-point transform per k1, or a
// real one where k1 is its own partner.  Prime powers use decimation in time
// N = R M on half spectra: the columns k' = 0 .. M / 2 give every output once.
#pragma once
#include "fft.hpp"

namespace ltmp2 {

template <class T, int N>
struct RFft {
  // X[0 .. N/2]; the imaginary parts of X[0] and (N even) X[N/2] are zero
  static LT_HD void run(const T* x, cplx<T>* X) {
    constexpr int R = lead_radix(N);
    constexpr int N1 = pfa_first(N);
    if constexpr (N1 > 0) {
      constexpr int N2 = N / N1;
      constexpr int T1 = inv_mod(N2 % N1, N1), T2 = inv_mod(N1 % N2, N2);
      cplx<T> z[N1 / 2 + 1][N2];
#pragma unroll
      for (int i2 = 0; i2 < N2; ++i2) {
        T a[N1];
        cplx<T> A[N1 / 2 + 1];
#pragma unroll
        for (int i1 = 0; i1 < N1; ++i1) a[i1] = x[(N2 * i1 + N1 * i2) % N];
        RFft<T, N1>::run(a, A);
#pragma unroll
        for (int k1 = 0; k1 <= N1 / 2; ++k1) z[k1][i2] = A[k1];
      }
#pragma unroll
      for (int k1 = 0; k1 <= N1 / 2; ++k1) {
        if (k1 == 0 || 2 * k1 == N1) {
          T a[N2];
          cplx<T> A[N2 / 2 + 1];
#pragma unroll
          for (int i2 = 0; i2 < N2; ++i2) a[i2] = z[k1][i2].x;
          RFft<T, N2>::run(a, A);
#pragma unroll
          for (int k2 = 0; k2 <= N2 / 2; ++k2) put(X, N2 * T1 * k1 + N1 * T2 * k2, A[k2]);
        } else {
          Fft<T, -1, N2>::run(z[k1]);
#pragma unroll
          for (int k2 = 0; k2 < N2; ++k2) put(X, N2 * T1 * k1 + N1 * T2 * k2, z[k1][k2]);
        }
      }
    } else if constexpr (N == 1) {
      X[0] = {x[0], T(0)};
    } else if constexpr (N == 2) {
      X[0] = {x[0] + x[1], T(0)};
      X[1] = {x[0] - x[1], T(0)};
    } else if constexpr (N == 3) {
      constexpr T s = T(0.866025403784438646763723170752936183);
      const T t = x[1] + x[2];
      X[0] = {x[0] + t, T(0)};
      X[1] = {x[0] - T(0.5) * t, -s * (x[1] - x[2])};
    } else if constexpr (N == 4) {
      const T t0 = x[0] + x[2], t2 = x[1] + x[3];
      X[0] = {t0 + t2, T(0)};
      X[1] = {x[0] - x[2], x[3] - x[1]};
      X[2] = {t0 - t2, T(0)};
    } else if constexpr (N == 5) {
      constexpr cs w1 = unit_root(1, 5);
      constexpr cs w2 = unit_root(2, 5);
      constexpr T c1 = T(w1.c), c2 = T(w2.c), s1 = T(w1.s), s2 = T(w2.s);
      const T b1 = x[1] + x[4], d1 = x[1] - x[4], b2 = x[2] + x[3], d2 = x[2] - x[3];
      X[0] = {x[0] + b1 + b2, T(0)};
      X[1] = {x[0] + c1 * b1 + c2 * b2, -(s1 * d1 + s2 * d2)};
      X[2] = {x[0] + c2 * b1 + c1 * b2, s1 * d2 - s2 * d1};
    } else {
      constexpr int M = N / R;
      cplx<T> y[R][M / 2 + 1];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        T a[M];
#pragma unroll
        for (int m = 0; m < M; ++m) a[m] = x[m * R + r];
        RFft<T, M>::run(a, y[r]);
      }
      {  // k' = 0: a real R-point transform
        T a[R];
        cplx<T> A[R / 2 + 1];
#pragma unroll
        for (int r = 0; r < R; ++r) a[r] = y[r][0].x;
        RFft<T, R>::run(a, A);
#pragma unroll
        for (int q = 0; q <= R / 2; ++q) X[M * q] = A[q];
      }
#pragma unroll
      for (int k = 1; k <= M / 2; ++k) {
        cplx<T> t[R];
        t[0] = y[0][k];
#pragma unroll
        for (int r = 1; r < R; ++r) {
          const cplx<T> w = twiddle<T, -1>(long(r) * k, N);
          // the Nyquist column of an even M is real
          t[r] = (2 * k == M) ? cplx<T>{y[r][k].x * w.x, y[r][k].x * w.y} : cmul_tw(y[r][k], w);
        }
        Dft<T, -1, R>::run(t);
        // 2 k = M pairs output q with R - 1 - q: the first half suffices
#pragma unroll
        for (int q = 0; q < ((2 * k == M) ? (R + 1) / 2 : R); ++q) put(X, k + M * q, t[q]);
      }
    }
  }

 private:
  // output k (mod N) or, above N / 2, its conjugate at N - k
  static LT_HD void put(cplx<T>* X, int k, cplx<T> v) {
    k %= N;
    if (2 * k <= N)
      X[k] = v;
    else
      X[N - k] = {v.x, -v.y};
  }
};

}  // namespace ltmp2
