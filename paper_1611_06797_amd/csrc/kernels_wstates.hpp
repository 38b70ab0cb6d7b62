// Transformed states on the grid (step (iii)):
//   w_j^{(G')}(r) = Omega^-1/2 sum_G W_j(G) e^{iG.r},
// from the real-basis product P = C Psi_v,
//   P[(g, j, 0)][q] = sum_a Re C_ja B[a][q],  P[(g, j, 1)][q] = sum_a Im C_ja B[a][q],
// where B[a] holds c_a(0), then Re c_a(G_k), Im c_a(G_k) for the half sphere.
// The orbitals are real, so the rows of P are the half-sphere coefficients of
// two real fields, the real and the imaginary part of w: each row is
// transformed by itself, from kz >= 0 only, and stored as a field of its own,
// w [item][2][ld], in the plane order of the pair transforms
// (r = (z N + x) N + y).
//
// Bound by the stores of w (24 grid: 1.94 GB per launch of 17538 states) and
// the vector ALUs.  A workgroup keeps its rows of P and the whole field (all
// kz >= 0 of all x planes, or of a slab of them) in shared memory: P is read
// once and in order, each stage is one pass of independent lines, and the
// last transform, along z, stores whole runs of (x, y).  That one packs two
// real lines into each complex transform.  The former kernel, one complex
// transform of both fields by groups of planes x2 + M xs, gathered every
// coefficient from global memory once per group through index tables: 24 grid
// 1151 -> 534 us per launch (3.6 TB/s stored), 27 grid 22144 states 4488 ->
// 1835 us, 36 grid 12320 states 4958 -> 1750, 15 grid 5450 states 113 -> 40.
// A row of P is fetched by eight independent loads a thread (27 grid 2352 ->
// 1835 us).
#pragma once
#include "transforms.hpp"

namespace ltmp2 {

// Vectors of the largest sphere whose largest index is k: |m|^2 < (k + 1)^2, a
// quarter more than the sphere of radius k at the sizes here.
__host__ __device__ constexpr int sphere_max(int k) {
  int c = 0;
  for (int x = 0; x <= k; ++x)
    for (int y = 0; y <= k; ++y) {
      int z = k;
      while (z >= 0 && x * x + y * y + z * z >= (k + 1) * (k + 1)) --z;
      c += (x ? 2 : 1) * (y ? 2 : 1) * (z >= 0 ? 2 * z + 1 : 0);
    }
  return c;
}

// Fields per workgroup, slabs of x planes per field and threads.  Two fields
// while three workgroups still fit a CU, else one.  One slab where the whole
// field fits a CU (27 grid, FP64: 716 us for 12160 states, three slabs and two
// workgroups 801), else the fewest that leave room for two workgroups (36 grid,
// FP32: 1750 us for 12320 states with three, 1911 with two slabs and one
// workgroup).  That is judged at a sphere of radius K.  Where the largest sphere
// of the window would not fit then, those that do not run in the WIDE form, in
// more slabs (40 grid, FP64, K = 13: 10059 vectors 0.97 ms for 1200 states in
// eight slabs, 3.6 by the general kernel; 9939 vectors 0.61 in five slabs).
template <class T, int N, int K, bool WIDE = false>
struct WstShape {
  static constexpr int R = slab_row(N);
  static constexpr size_t bytes(int f, int s, int npw) {
    return sizeof(cplx<T>) * f * (size_t(N / s) * (K + 1) * R + (npw + 1) / 2 + 1);
  }
  static constexpr int radius_k = 21 * K * K * K / 5;  // vectors of a sphere of radius K
  static constexpr int F = bytes(2, 1, radius_k) <= 52 * 1024 ? 2 : 1;
  static constexpr bool fits(int s, size_t cap) {
    return bytes(F, s, radius_k) <= cap && (!WIDE || bytes(F, s, sphere_max(K)) <= 150 * 1024);
  }
  static constexpr int slabs() {
    if (fits(1, 148 * 1024)) return 1;
    for (size_t cap : {size_t(78) * 1024, size_t(148) * 1024})
      for (int s = 2; s < N; ++s)
        if (N % s == 0 && fits(s, cap)) return s;
    return N;
  }
  static constexpr int S = slabs(), SP = N / S;
  static constexpr int nk = 2 * K + 1, NSLOT = (K + 1) * nk;
  static constexpr int zlines = (F * SP * N + 1) / 2;
  static constexpr int NT = zlines <= 128 ? 128 : zlines >= 512 ? 512 : (zlines + 63) / 64 * 64;
  // waves per SIMD: registers for a complex line and its transform
  static constexpr int MINW = sizeof(T) == 4 ? (N <= 20 ? 4 : N <= 27 ? 3 : 2) : 2;
  static constexpr size_t lds(int npw) { return bytes(F, S, npw); }
  static constexpr bool holds_all = bytes(F, S, sphere_max(K)) <= 150 * 1024;
};

// wx [2 kt + 1][kt + 1][2 kt + 1] + one entry: for (kx, kz, ky), the index of the
// coefficient pair in a row of P (0: G = 0; (npw + 1) / 2: none, as the last entry
// says), bit 15 set where its conjugate is meant (sets that fit shared memory
// have fewer than 2^15 pairs).  kt = K, or the set's own largest index below it
// (SMALL: contexts under a workspace cap; its range checks take 1 to 8 % of the
// kernel's time, on the 30 grid in FP32 a quarter).
template <class T, int N, int K, bool WIDE, bool SMALL>
__global__ __launch_bounds__((WstShape<T, N, K, WIDE>::NT), (WstShape<T, N, K, WIDE>::MINW))
void k_wstates_real(const T* __restrict__ P, int npw, const unsigned short* __restrict__ wx, int kt,
                    double scale, T* __restrict__ w, long ld) {
  using W = WstShape<T, N, K, WIDE>;
  constexpr int F = W::F, SP = W::SP, R = W::R, NT = W::NT, nk = W::nk;
  extern __shared__ __align__(16) char smem[];
  cplx<T>* t = reinterpret_cast<cplx<T>*>(smem);  // [F][SP][K + 1][R]
  const int nce = (npw + 1) / 2 + 1;
  cplx<T>* co = t + F * SP * (K + 1) * R;  // [F][nce]
  const int tid = threadIdx.x;
  const long f0 = long(blockIdx.x) * F;
  T* out = w + f0 * ld;
#pragma unroll
  for (int f = 0; f < F; ++f) {
    const T* row = P + (f0 + f) * npw;
    T* c = reinterpret_cast<T*>(co + f * nce);
    for (int q0 = tid; q0 < npw; q0 += 8 * NT) {
      T x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) x[u] = row[min(q0 + u * NT, npw - 1)];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int q = q0 + u * NT;
        if (q < npw) c[q ? q + 1 : 0] = T(scale) * x[u];
      }
    }
    if (tid == 0) {
      c[1] = T(0);
      co[f * nce + nce - 1] = {T(0), T(0)};
    }
  }
  __syncthreads();
  for (int s = 0; s < W::S; ++s) {
    // x: slot (kz, ky) of a field, all planes from registers
    for (int l = tid; l < F * W::NSLOT; l += NT) {
      const int f = l / W::NSLOT, sl = l - f * W::NSLOT;
      const int kz = sl / nk, ky = sl - kz * nk - K;
      const int k = SMALL ? kt : K, plane = (k + 1) * (2 * k + 1);
      const int row = k * plane + kz * (2 * k + 1) + ky + k;
      const bool in = !SMALL || (kz <= k && ky >= -k && ky <= k);
      cplx<T> v[N];
#pragma unroll
      for (int x = 0; x < N; ++x) {
        const int kx = x <= N / 2 ? x : x - N;
        v[x] = {T(0), T(0)};
        if (kx >= -K && kx <= K) {
          const int at = row + kx * plane;
          const int code = wx[!SMALL || (in && kx >= -k && kx <= k) ? at : (2 * k + 1) * plane];
          v[x] = co[f * nce + (code & 0x7fff)];
          v[x].y = code & 0x8000 ? -v[x].y : v[x].y;
        }
      }
      Fft<T, 1, N>::run(v);
      cplx<T>* d = t + (f * SP * (K + 1) + kz) * R + ky + K;
      if constexpr (W::S == 1) {
#pragma unroll
        for (int x = 0; x < N; ++x) d[x * (K + 1) * R] = v[x];
      } else {
#pragma unroll
        for (int q = 0; q < W::S; ++q)
          if (q == s)
#pragma unroll
            for (int x = 0; x < SP; ++x) d[x * (K + 1) * R] = v[q * SP + x];
      }
    }
    __syncthreads();
    // y: row (f, x, kz), expanded in place from nk to N values
    for (int l = tid; l < F * SP * (K + 1); l += NT) {
      cplx<T>* row = t + l * R;
      cplx<T> v[N];
#pragma unroll
      for (int y = 0; y < N; ++y) {
        const int ky = y <= N / 2 ? y : y - N;
        v[y] = (ky >= -K && ky <= K) ? row[ky + K] : cplx<T>{T(0), T(0)};
      }
      Fft<T, 1, N>::run(v);
#pragma unroll
      for (int y = 0; y < N; ++y) row[y] = v[y];
    }
    __syncthreads();
    // z: real lines p and p + H of the (f, x, y) order in one transform, of
    // the spectrum A + i B with A(-k) = conj A(k), B(-k) = conj B(k)
    constexpr int L = F * SP * N, H = (L + 1) / 2;
    for (int p = tid; p < H; p += NT) {
      const int p2 = p + H < L ? p + H : p;
      const int xa = p / N, ya = p - xa * N, xb = p2 / N, yb = p2 - xb * N;
      const cplx<T>*a = t + xa * (K + 1) * R + ya, *b = t + xb * (K + 1) * R + yb;
      cplx<T> v[N];
      v[0] = {a[0].x, b[0].x};
#pragma unroll
      for (int z = 1; z < N; ++z) v[z] = {T(0), T(0)};
#pragma unroll
      for (int k = 1; k <= K; ++k) {
        const cplx<T> A = a[k * R], B = b[k * R];
        v[k] = {A.x - B.y, A.y + B.x};
        v[N - k] = {A.x + B.y, B.x - A.y};
      }
      Fft<T, 1, N>::run(v);
      const int fa = xa / SP, fb = xb / SP;
      T* oa = out + fa * ld + (s * SP + xa - fa * SP) * N + ya;
      T* ob = out + fb * ld + (s * SP + xb - fb * SP) * N + yb;
#pragma unroll
      for (int z = 0; z < N; ++z) {
        oa[z * N * N] = v[z].x;
        if (L % 2 == 0 || p2 != p) ob[z * N * N] = v[z].y;
      }
    }
    if constexpr (W::S > 1) __syncthreads();  // the next x stage overwrites the rows
  }
}

}  // namespace ltmp2
