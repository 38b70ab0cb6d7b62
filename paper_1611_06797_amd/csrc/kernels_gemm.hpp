// Dense contractions of the LTMP2 path on CDNA matrix cores, FP64 and FP32.
//
//   k_gf_chi:  chi(r, r') = G_occ(r, r') * G_vir(r, r') for one pair of tiles
//              (tile and its transpose; chi is symmetric for real orbitals;
//              added to chi when accumulating the spin channels), with
//                G_occ = sum_i psi_i(r) exp((e_i - mu) tau) psi_i(r')
//                G_vir = sum_a psi_a(r) exp(-(e_a - mu) tau) psi_a(r')
//              both accumulated in the same kernel and multiplied in the
//              epilogue (G_vir(r', r) = G_vir(r, r') needs no transpose).
//   k_gemm_kmajor: C[m][n] = rs(m) sum_k A[k][m] s_k B[k][n], used for the
//              transformed-state product W = C Psi_v and for exporting
//              Green's-function rows.
//
// Arithmetic modes (template MODE; the split-BF16 products have kernels of
// their own, kernels_gemm3.hpp):
//   kF64    v_mfma_f64_16x16x4f64, FP64 operands and accumulation
//   kF32    v_mfma_f32_16x16x4f32, FP32 operands and accumulation
// Operand lanes: lane l supplies A[l % 16][k] and B[k][l % 16] for the
// k-slice (l / 16) of the instruction.  Accumulator element v of lane l is
// D[(l / 16) + 4 v][l % 16] for the FP64 instruction and D[4 (l / 16) + v]
// [l % 16] for the FP32 one (measured on gfx950 with single-instruction
// probes).
//
// Bound by the matrix cores (a plain library product of 8192^3 reaches 72.6
// TFLOP/s in FP64 and 152 in FP32 on this card): M x N x K = 12160 x 3959 x
// 1984 in FP64 3.12 ms, 61 TFLOP/s (5.28 ms with one buffer and two barriers a
// slice); 35076 x 1743 x 1706 in FP32 1.90 ms, 110 TFLOP/s (3.29 ms); chi of
// 13824 points and 1743 orbitals in FP32 2.87 ms, 116 TFLOP/s (3.24 ms).  Tiles
// of 128 measured no more in FP32 (88 TFLOP/s) and spill in FP64.  K slices alternate between
// two shared-memory buffers: the next slice is fetched into registers and
// stored into the idle buffer while the matrix cores work, one barrier per
// slice.  Rows of the buffers are padded by 16 elements, so that the four k
// rows of an instruction's operand lie in different banks.
#pragma once
#include <hip/hip_runtime.h>

#include "modes.h"

namespace ltmp2 {

typedef double d4v __attribute__((ext_vector_type(4)));
typedef float f4v __attribute__((ext_vector_type(4)));

template <int MODE>
struct Mma;

template <>
struct Mma<kF64> {
  using T = double;
  using Acc = d4v;
  static __device__ __forceinline__ int row(int l, int v) { return (l >> 4) + 4 * v; }
  static __device__ __forceinline__ Acc zero() { return Acc{0, 0, 0, 0}; }
  static __device__ __forceinline__ Acc mma(T a, T b, Acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
};
template <>
struct Mma<kF32> {
  using T = float;
  using Acc = f4v;
  static __device__ __forceinline__ int row(int l, int v) { return 4 * (l >> 4) + v; }
  static __device__ __forceinline__ Acc zero() { return Acc{0, 0, 0, 0}; }
  static __device__ __forceinline__ Acc mma(T a, T b, Acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};

// Tile of B x B outputs for 256 threads: WAVES x WAVES waves in the plane,
// each P x P blocks of 16 x 16, and KS = 4 / WAVES^2 waves per block that
// share the k rows of a slice (BK rows, BK / KS per wave).
template <int MODE, int B_>
struct GemmTile {
  using T = typename Mma<MODE>::T;
  static constexpr int B = B_, WAVES = B > 32 ? 2 : 1, KS = 4 / (WAVES * WAVES);
  static constexpr int P = B / (16 * WAVES), BK = KS > 1 ? 32 : 16, PAD = 16;
  static constexpr int PER = BK * B / 256;  // elements of one operand per thread and slice
  struct Buf {
    T a[BK][B + PAD], b[BK][B + PAD];
  };
};

template <int MODE, int B>
using GemmAcc = typename Mma<MODE>::Acc[GemmTile<MODE, B>::P][GemmTile<MODE, B>::P];

// Buffer over everything from p on (p the same in all lanes), and one element
// of it at a lane's offset plus a uniform one, in bytes.
template <class V>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const V* p) {
  const unsigned long long u = reinterpret_cast<unsigned long long>(p);
  const unsigned lo = __builtin_amdgcn_readfirstlane(unsigned(u));
  const unsigned hi = __builtin_amdgcn_readfirstlane(unsigned(u >> 32));
  void* q = reinterpret_cast<void*>((static_cast<unsigned long long>(hi) << 32) | lo);
  return __builtin_amdgcn_make_buffer_rsrc(q, short(0), -1, 0x00020000);
}
__device__ __forceinline__ float row_load(const float*, __amdgpu_buffer_rsrc_t rs, unsigned lane,
                                          unsigned row) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, lane, row, 0));
}
__device__ __forceinline__ double row_load(const double*, __amdgpu_buffer_rsrc_t rs,
                                           unsigned lane, unsigned row) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rs, lane, row, 0));
}

// acc += sum_{k < K} A[k][m0 + .] s_k B[k][n0 + .] over one tile.  Columns
// beyond M (N) repeat the last one: their outputs are never stored.  A slice's
// rows are addressed from the slice's first row in scalar registers, the lane's
// column and the row's step being the two 32-bit offsets of a buffer load:
// vector instructions cost FP32 matrix time, which the same ALUs execute.  The
// last slice, if short, and operands whose BK rows span 4 GiB or more are
// addressed with 64 bits.
template <int MODE, int B>
__device__ __forceinline__ void tile_phase(const typename Mma<MODE>::T* __restrict__ A, long lda,
                                           int M, long m0,
                                           const typename Mma<MODE>::T* __restrict__ Bp, long ldb,
                                           int N, long n0, int K, const double* __restrict__ sk,
                                           typename GemmTile<MODE, B>::Buf (&buf)[2],
                                           GemmAcc<MODE, B>& acc) {
  using G = GemmTile<MODE, B>;
  using T = typename G::T;
  constexpr int STEP = 256 / B;  // k rows per pass of the workgroup
  constexpr bool kRow = B >= 64;  // a wave's row is the same for all its lanes
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wk = wave / (G::WAVES * G::WAVES), wp = wave % (G::WAVES * G::WAVES);
  const int wr = wp / G::WAVES * (B / G::WAVES), wc = wp % G::WAVES * (B / G::WAVES);
  const int cc = tid % B;
  const int kr = kRow ? __builtin_amdgcn_readfirstlane(tid / B) : tid / B;
  const unsigned es = sizeof(T);
  // rows inside the slice: uniform part in `row`, the rest in the lane offset
  const unsigned la = unsigned(min(m0 + cc, long(M) - 1) + (kRow ? 0 : long(kr) * lda)) * es;
  const unsigned lb = unsigned(min(n0 + cc, long(N) - 1) + (kRow ? 0 : long(kr) * ldb)) * es;
  const unsigned sa = __builtin_amdgcn_readfirstlane(unsigned(STEP * lda) * es);
  const unsigned sb = __builtin_amdgcn_readfirstlane(unsigned(STEP * ldb) * es);
  const bool narrow = G::BK * max(lda, ldb) * long(es) < (1L << 32);
  T av[G::PER], bv[G::PER];
  auto fetch = [&](int k0) {
    if (narrow && k0 + G::BK <= K) {
      const long k1 = k0 + (kRow ? kr : 0);
      const auto ra = row_rsrc(A + k1 * lda), rb = row_rsrc(Bp + k1 * ldb);
#pragma unroll
      for (int u = 0; u < G::PER; ++u) {
        av[u] = row_load(A, ra, la, unsigned(u) * sa);
        bv[u] = row_load(Bp, rb, lb, unsigned(u) * sb);
      }
      if (sk)
#pragma unroll
        for (int u = 0; u < G::PER; ++u) av[u] *= T(sk[k0 + kr + u * STEP]);
    } else {
#pragma unroll
      for (int u = 0; u < G::PER; ++u) {
        const int k = k0 + kr + u * STEP;
        av[u] = bv[u] = T(0);
        if (k < K) {
          av[u] = A[long(k) * lda + min(m0 + cc, long(M) - 1)] * (sk ? T(sk[k]) : T(1));
          bv[u] = Bp[long(k) * ldb + min(n0 + cc, long(N) - 1)];
        }
      }
    }
  };
  auto store = [&](typename G::Buf& s) {
#pragma unroll
    for (int u = 0; u < G::PER; ++u) {
      s.a[tid / B + u * STEP][cc] = av[u];
      s.b[tid / B + u * STEP][cc] = bv[u];
    }
  };
  auto mma = [&](const typename G::Buf& s) {
#pragma unroll
    for (int ks = 0; ks < G::BK / (4 * G::KS); ++ks) {
      const int k = (wk * (G::BK / (4 * G::KS)) + ks) * 4 + (lane >> 4);
      T a[G::P], b[G::P];
#pragma unroll
      for (int p = 0; p < G::P; ++p) {
        a[p] = s.a[k][wr + 16 * p + (lane & 15)];
        b[p] = s.b[k][wc + 16 * p + (lane & 15)];
      }
#pragma unroll
      for (int p = 0; p < G::P; ++p)
#pragma unroll
        for (int q = 0; q < G::P; ++q) acc[p][q] = Mma<MODE>::mma(a[p], b[q], acc[p][q]);
    }
  };
  if (K <= 0) return;
  fetch(0);
  store(buf[0]);
  __syncthreads();
  // two slices per turn: the buffer of each is known at compile time
  for (int k0 = 0; k0 < K; k0 += 2 * G::BK) {
    const bool m1 = k0 + G::BK < K, m2 = k0 + 2 * G::BK < K;
    if (m1) fetch(k0 + G::BK);
    mma(buf[0]);
    if (m1) store(buf[1]);
    __syncthreads();
    if (!m1) break;
    if (m2) fetch(k0 + 2 * G::BK);
    mma(buf[1]);
    if (m2) store(buf[0]);
    __syncthreads();
  }
}

template <int MODE, int B>
__device__ __forceinline__ void tile_zero(GemmAcc<MODE, B>& acc) {
#pragma unroll
  for (int p = 0; p < GemmTile<MODE, B>::P; ++p)
#pragma unroll
    for (int q = 0; q < GemmTile<MODE, B>::P; ++q) acc[p][q] = Mma<MODE>::zero();
}

// Sum of the KS waves' accumulators in wave 0 (fixed order); red is scratch of
// at least 3 P^2 x 64 accumulators.
template <int MODE, int B>
__device__ __forceinline__ void tile_ksum(GemmAcc<MODE, B>& acc, typename Mma<MODE>::Acc* red) {
  using G = GemmTile<MODE, B>;
  if constexpr (G::KS > 1) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (wave > 0)
#pragma unroll
      for (int p = 0; p < G::P; ++p)
#pragma unroll
        for (int q = 0; q < G::P; ++q)
          red[((wave - 1) * G::P * G::P + p * G::P + q) * 64 + lane] = acc[p][q];
    __syncthreads();
    if (wave == 0)
#pragma unroll
      for (int w = 0; w < G::KS - 1; ++w)
#pragma unroll
        for (int p = 0; p < G::P; ++p)
#pragma unroll
          for (int q = 0; q < G::P; ++q) acc[p][q] += red[(w * G::P * G::P + p * G::P + q) * 64 + lane];
    __syncthreads();
  }
}

// Upper-triangular tile index t -> (bi <= bj) of nt x nt tiles: groups of
// eight columns, each by rows, so that tiles in flight together share their
// strips (eight columns and as many rows as there are eights in flight).
__device__ inline void tri_tile(long t, int nt, int& bi, int& bj) {
  // first tile of group g: sum over h < g of 64 h + 36 = 32 g^2 + 4 g
  long g = long((sqrt(16.0 + 128.0 * double(t)) - 4.0) / 64.0);
  while (32 * g * g + 4 * g > t) --g;
  while (32 * (g + 1) * (g + 1) + 4 * (g + 1) <= t) ++g;
  const int c0 = int(8 * g), w = min(8, nt - c0);
  long r = t - (32 * g * g + 4 * g);
  if (r < long(c0) * w) {  // full rows above the diagonal block
    bi = int(r / w);
    bj = c0 + int(r % w);
    return;
  }
  r -= long(c0) * w;
  int q = 0;
  while (r >= w - q) r -= w - q++;
  bi = c0 + q;
  bj = c0 + q + int(r);
}

// psi: [n_states][ld] real orbitals on the grid (occupied rows first).
// fo[i] = exp((e_i - mu) tau), fv[a] = exp(-(e_a - mu) tau).
// chi: [n][ldc], n a multiple of B; tiles of each XCD are contiguous in the
// triangular order, so neighbours share their row strips in its L2.
template <int MODE, int B>
__global__ __launch_bounds__(256, 2) void k_gf_chi(const typename Mma<MODE>::T* __restrict__ psi,
                                                  long ld, int no, int nv, long n,
                                                  const double* __restrict__ fo,
                                                  const double* __restrict__ fv,
                                                  typename Mma<MODE>::T* __restrict__ chi,
                                                  long ldc, int accumulate) {
  using G = GemmTile<MODE, B>;
  using T = typename G::T;
  __shared__ typename G::Buf buf[2];
  const long t = n / B, total = t * (t + 1) / 2, per = (total + 7) / 8;
  const long tile = long(blockIdx.x % 8) * per + blockIdx.x / 8;
  if (tile >= total) return;
  int bi, bj;
  tri_tile(tile, int(t), bi, bj);
  const long m0 = long(bi) * B, n0 = long(bj) * B;
  GemmAcc<MODE, B> ao, av;
  tile_zero<MODE, B>(ao);
  tile_zero<MODE, B>(av);
  const T* psv = psi + long(no) * ld;
  tile_phase<MODE, B>(psi, ld, int(n), m0, psi, ld, int(n), n0, no, fo, buf, ao);
  tile_phase<MODE, B>(psv, ld, int(n), m0, psv, ld, int(n), n0, nv, fv, buf, av);
  auto* red = reinterpret_cast<typename Mma<MODE>::Acc*>(buf);
  tile_ksum<MODE, B>(ao, red);
  tile_ksum<MODE, B>(av, red);
  // through LDS, so that both the tile and its transpose are written by rows
  using Out = T[B][B + 1];
  static_assert(sizeof(Out) <= sizeof(buf));
  Out& cs = *reinterpret_cast<Out*>(buf);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (wave < G::WAVES * G::WAVES) {
    const int wr = wave / G::WAVES * (B / G::WAVES), wc = wave % G::WAVES * (B / G::WAVES);
#pragma unroll
    for (int p = 0; p < G::P; ++p)
#pragma unroll
      for (int q = 0; q < G::P; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          cs[wr + 16 * p + Mma<MODE>::row(lane, v)][wc + 16 * q + (lane & 15)] =
              ao[p][q][v] * av[p][q][v];
  }
  __syncthreads();
  for (int e = tid; e < B * B; e += 256) {
    const int r = e / B, c = e % B;
    T* d = &chi[(m0 + r) * ldc + n0 + c];
    *d = accumulate ? *d + cs[r][c] : cs[r][c];
    if (bi != bj) {
      T* dt = &chi[(n0 + r) * ldc + m0 + c];
      *dt = accumulate ? *dt + cs[c][r] : cs[c][r];
    }
  }
}

// C[m][n] = rs(m) sum_k A[k][m] s_k B[k][n] for m < M, n < N;
// rs(m) = rowscale[(m / rdiv) % rmod] (or 1 if rowscale is null).
// XCD x takes a contiguous range of the row-major tiles.
template <int MODE, int B>
__global__ __launch_bounds__(256, 2) void k_gemm_kmajor(const typename Mma<MODE>::T* __restrict__ A,
                                                       long lda,
                                                       const typename Mma<MODE>::T* __restrict__ Bp,
                                                       long ldb,
                                                       typename Mma<MODE>::T* __restrict__ C,
                                                       long ldc, int M, int N, int K,
                                                       const double* __restrict__ sk,
                                                       const double* __restrict__ rowscale,
                                                       int rdiv, int rmod) {
  using G = GemmTile<MODE, B>;
  using T = typename G::T;
  __shared__ typename G::Buf buf[2];
  const int tn = (N + B - 1) / B;
  const long total = long((M + B - 1) / B) * tn, per = (total + 7) / 8;
  const long tile = long(blockIdx.x % 8) * per + blockIdx.x / 8;
  if (tile >= total) return;
  const long m0 = tile / tn * B, n0 = tile % tn * B;
  GemmAcc<MODE, B> acc;
  tile_zero<MODE, B>(acc);
  tile_phase<MODE, B>(A, lda, M, m0, Bp, ldb, N, n0, K, sk, buf, acc);
  tile_ksum<MODE, B>(acc, reinterpret_cast<typename Mma<MODE>::Acc*>(buf));
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (wave >= G::WAVES * G::WAVES) return;
  const int wr = wave / G::WAVES * (B / G::WAVES), wc = wave % G::WAVES * (B / G::WAVES);
#pragma unroll
  for (int p = 0; p < G::P; ++p)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const long m = m0 + wr + 16 * p + Mma<MODE>::row(lane, v);
      if (m >= M) continue;
      const T s = rowscale ? T(rowscale[(m / rdiv) % rmod]) : T(1);
#pragma unroll
      for (int q = 0; q < G::P; ++q) {
        const long n = n0 + wc + 16 * q + (lane & 15);
        if (n < N) C[m * ldc + n] = s * acc[p][q][v];
      }
    }
}

}  // namespace ltmp2
