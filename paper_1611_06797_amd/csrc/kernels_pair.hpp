// Fock-like contraction (step (iv.b)) on real lines.
//
// For one outer G' and one occupied pair i <= j, with real orbitals psi and
// complex transformed states w (their real and imaginary parts stored as
// separate real fields):
//   A_ij(G) = dV sum_r psi_i(r) w_j(r) e^{-iG.r},  G in the auxiliary set,
//   xpart = sum_G v(G) [A_ij conj(A_ji) + A_ji conj(A_ij)]   (i < j)
//         = sum_G v(G) |A_ii|^2                               (i = j).
// Summed over pairs this is S_x(G') = sum_G v(G) sum_ij A_ij(G) A^{(-G')}_ji(-G),
// using A^{(-G')}_ji(-G) = conj A^{(G')}_ji(G) for real orbitals.
//
// The auxiliary set contains -G with G and v depends on |G| only, so in the
// sum over G the products of a real-part field with an imaginary-part field
// cancel between G and -G: the two parts of w contribute separately, each
// through the real fields f = psi_i u_j and g = psi_j u_i.  For real fields
// the sum over the signs of (kx, ky, kz) turns into a sum over products of
// cosines and sines per axis,
//   sum_{signs} Re f^(G) conj g^(G) = m(kx) m(ky) m(kz) sum_{rows} F G,
// m(0) = 1, m(k) = 2, where F is the real trigonometric transform of f: every
// axis is a real transform of real lines (RFft) whose real and imaginary
// parts become separate real rows, and no spectrum is ever unfolded.  Half
// the registers of complex lines of the same length, and half the transform
// work per part.
//
// What bounds it (counters and timing variants on the 27 and 36 grids): the
// vector ALUs, the L1 reads (8 bytes per point and field at 64 B per clock)
// and shared memory cost about the same, and only independent workgroups
// overlap them, so the work is cut into small workgroups, as many per CU as
// shared memory holds, with as few barriers per field as possible.  Complex
// lines in 256-thread workgroups against this form, ns per item (one G', one
// pair) of launches of 30 000 to 100 000 items: in FP32 12 grid 5.0 -> 3.0, 15:
// 10.7 -> 5.5, 16: 9.5 -> 6.2, 18: 14.3 -> 10.6, 20: 24.6 -> 14.2, 24: 32 -> 23,
// 25: 97 -> 35, 27: 85 -> 39, 30: 91 -> 50, 32: 98 -> 62, 36: 112 -> 99, 40: 219
// -> 136; in FP64 12: 8.9 -> 8.6, 15: 19.6 -> 14.8, 16: 18.6 -> 16.4, 18: 24.7 ->
// 25.7 (the one grid that did not gain), 20: 42 -> 39, 24: 61 -> 60, 25: 240 ->
// 99, 27: 196 -> 100, 30: 336 -> 165, 32: 308 -> 199, 36: 516 -> 290, 40: 575 ->
// 390.  The figures at the rules below are of a stand-alone launch of 31 200
// items whose transformed states do not fit the caches.
#pragma once
#include "launch_items.hpp"
#include "rfft.hpp"
#include "transforms.hpp"

namespace ltmp2 {

// Everything one cell contributes to a pair launch.  Grid fields of the pair
// transforms are stored z plane by z plane, r = (z N + x) N + y, so that the
// z lines of consecutive (x, y) are consecutive in memory at every z: a wave
// reads 256 contiguous bytes per z instead of pieces of several rows.
struct PairCell {
  const void* psi;     // [nocc][ld] orbitals (T)
  const void* w;       // [gb][nocc][2][ld] real and imaginary parts of w (T)
  const int* pairs;    // [npairs] i | j << 16
  const int* cols;     // [ncol] kept (ky, kz) columns: row index ry | rz << 8
  double* xpart;       // [gb][npairs] partial sums of this block
  long ld;
  // v(G) by m^2 = (|G| / b)^2 < nm2: 4 pi / (vden m^2) up to m2lim, else 0
  int nocc, npairs, gb, kmax, ncol, nm2, m2lim;
  double dV2, vden;
  // optional split by auxiliary cutoff shell (ShellBins): number of spheres
  // by m^2 <= m2lim (beyond, v = 0), the shells of the outer vectors
  // from the block's first one on, and xbins [gb][npairs][nb]
  const signed char* shm2 = nullptr;   // nullptr: no split
  const signed char* shell = nullptr;  // shell of G' = shell[g0 + gl]
  double* xbins = nullptr;
  int nb = 0, g0 = 0;
};

// Rows of an axis: row 0 is k = 0, rows 2k - 1 and 2k are the cosine and sine
// (real and imaginary) parts of k.
__host__ __device__ constexpr int row_k(int r) { return (r + 1) / 2; }

// Largest kept index of any auxiliary set the library takes (its vectors fit
// the register outputs of the chi transforms: |m|^2 <= 101).
constexpr int kAuxMax = 10, kAuxM2 = 101;

// Kept-set instances compiled for a grid: the alias-free window kwin(N), one
// below it, and everything the grid can hold.  A smaller kept set runs the
// smallest instance that holds it (its extra rows are not among the columns).
__host__ __device__ constexpr int pair_kw(int n) { return kwin(n) < kAuxMax ? kwin(n) : kAuxMax; }
__host__ __device__ constexpr int pair_kf(int n) {
  return (n - 1) / 2 < kAuxMax ? (n - 1) / 2 : kAuxMax;
}

// Most (ky, kz) columns a kept set with largest index k can have.
__host__ __device__ constexpr int pair_cols_max(int k) {
  int lim = (k + 1) * (k + 1) - 1, c = 0;
  if (lim > kAuxM2) lim = kAuxM2;
  for (int a = 0; a <= 2 * k; ++a)
    for (int b = 0; b <= 2 * k; ++b)
      c += row_k(a) * row_k(a) + row_k(b) * row_k(b) <= lim ? 1 : 0;
  return c;
}

// Row stride of the line buffer: odd, against bank conflicts.
__host__ __device__ constexpr int line_row(int n) { return n | 1; }

// Shared memory: z-transformed lines of one slab of n / ns planes, and the
// (ky, kz) columns of the planes of the earlier slabs.
__host__ __device__ constexpr size_t pair_lds_bytes(size_t es, int n, int k, int ns, int ncol) {
  return es * (size_t(n / ns) * (2 * k + 1) * line_row(n) + size_t(n - n / ns) * ncol);
}

// Threads per workgroup: at least one per column; beyond that the smallest
// workgroups that still fill the CU's wave slots from its shared memory, FP64
// lines, which fill them with fewer, one size up from the 18 grid on (ns per
// item, FP32: 18 grid 128 threads 10.3 and with the split by cutoff shell 12.5,
// 192 threads 9.8 and 12.7; 24 grid, |k| <= 6, 192 threads 20.0, 320 22.1; 27 grid
// 256 threads 42.6, 384 54; 36 grid 512 threads 108, 384 116; FP64: 18 grid 192
// threads 26.9, 128 27.4.  The 12 grid would run 64 threads 5 % faster when the
// card is full, and loses 20 % to latency when it is not).
// pair_threads has the last word: workgroups alone on their CU take 512.
__host__ __device__ constexpr int pair_threads_shared(size_t es, int n, int k) {
  const int cols = (pair_cols_max(k) + 63) / 64 * 64;
  const int nt = n <= (es == 8 ? 16 : 18) ? 128 : n <= 24 ? 192 : n <= 27 ? 256 : 512;
  return cols > nt ? cols : nt;
}

// Static shared memory of a pair kernel of nt threads, at most: v(G) and the
// shells by m^2, the row table, one or nine FP64 slots per wave, and their
// alignment.
__host__ __device__ constexpr size_t pair_static(int k, int nt, bool bins) {
  const size_t nm2 = 2 * size_t(k) * k + 2 * k + 1;
  return 8 * nm2 + (bins ? nm2 : 1) + 4 * (2 * k + 1) + nt / 64 * 8 * (bins ? 1 + kMaxShells : 1) +
         64;
}

// The z lines of a slab in percent of what their rounds could hold.
__host__ __device__ constexpr int slab_fill(int n, int ns, int nt) {
  const int lines = n / ns * n;
  return 100 * lines / ((lines + nt - 1) / nt * nt);
}

// Slabs per field.  One where the whole field fits next to a second workgroup
// (each slab costs two more barriers; a third or fourth workgroup gains nothing
// in FP32: 27 grid, one slab and three slabs 42.6 ns per item), else the fewest
// that leave room for two workgroups and whose z lines fill more than 60 % of
// their rounds (FP64: 25 grid 110 ns in five slabs of 125 lines for 256
// threads, 101 in one slab; 27 grid, |k| <= 10, nine slabs of 81 lines 346,
// one slab 134; 30 grid, |k| <= 9, fifteen slabs 451, one 164), else the fewest
// that fit at all.  The long lines of FP64 leave few waves per workgroup, so
// there a third workgroup comes first, if its slabs are one round each (24
// grid, three slabs of 192 lines 60 ns, one slab 66, two slabs 75).  The split
// by cutoff shell needs 700 bytes more and so, on the 36 grid in FP32, three
// slabs where two are enough without it (115 ns per item; two slabs are then
// one workgroup per CU, 170).  On the 32 grid (|k| <= 9, FP32) the exact count
// lets one slab pass where a rounded one took two (68 -> 63 ns).
__host__ __device__ constexpr int pair_slabs(size_t es, int n, int k, bool bins = false) {
  const int nt = pair_threads_shared(es, n, k), cols = pair_cols_max(k);
  const size_t stat = pair_static(k, nt, bins);
  for (int wgs = es == 8 ? 3 : 2; wgs >= 2; --wgs)
    for (int ns = 1; ns <= n; ++ns)
      if (n % ns == 0 && (ns == 1 || slab_fill(n, ns, nt) >= 60) &&
          (ns == 1 || wgs == 2 || n / ns * n <= nt) &&
          pair_lds_bytes(es, n, k, ns, cols) + stat <= size_t(160) * 1024 / wgs)
        return ns;
  for (int ns = 1; ns <= n; ++ns)
    if (n % ns == 0 && pair_lds_bytes(es, n, k, ns, cols) <= size_t(150) * 1024) return ns;
  return n;
}

// A workgroup that has its CU to itself brings all the waves its registers
// allow (FP64: 24 grid, |k| <= 10, 384 threads 95 ns, 512 threads 90; 25 grid 256
// threads 125, 512 threads 101).
__host__ __device__ constexpr int pair_threads(size_t es, int n, int k) {
  const int nt = pair_threads_shared(es, n, k);
  const size_t lds = pair_lds_bytes(es, n, k, pair_slabs(es, n, k), pair_cols_max(k));
  return es == 8 && lds + pair_static(k, nt, false) > size_t(80) * 1024 && nt < 512 ? 512 : nt;
}

// Waves per SIMD the launch bounds ask for: the register need is about three
// line lengths (six in FP64).  The split by cutoff shell adds its bins to the
// epilogue: one wave fewer on the small grids, whose instances spill otherwise
// (15 grid, |k| <= 7, FP32: 16.0 ns per item with eight, 14.2 with seven; 12
// grid, |k| <= 5, FP64: 11.9 with six, 11.1 with five).
__host__ __device__ constexpr int pair_minw(size_t es, int n, bool bins = false) {
  if (es == 8) return n <= 12 ? (bins ? 5 : 6) : n <= 18 ? 4 : n <= 24 ? 3 : 2;
  return n <= 15 ? (bins ? 7 : 8) : n <= 20 ? 6 : n <= 24 ? 5 : 4;
}

// Barrier that orders shared memory only: global loads stay in flight.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Grid fields through buffer resources: the base in scalar registers, a
// 32-bit lane offset, no 64-bit address arithmetic.  The field's address is
// the same for every lane; taking it from the first lane tells the compiler
// so.  Word 3 holds the gfx9-family default format; num_records bounds every
// access to the field (reads past it return zero).
template <class V>
__device__ inline __amdgpu_buffer_rsrc_t field_rsrc(const V* p, unsigned n) {
  const unsigned long long u = reinterpret_cast<unsigned long long>(p);
  const unsigned lo = __builtin_amdgcn_readfirstlane(unsigned(u));
  const unsigned hi = __builtin_amdgcn_readfirstlane(unsigned(u >> 32));
  void* q = reinterpret_cast<void*>((static_cast<unsigned long long>(hi) << 32) | lo);
  return __builtin_amdgcn_make_buffer_rsrc(q, short(0), int(n * sizeof(V)), 0x00020000);
}
template <class V>
__device__ inline V field_load(__amdgpu_buffer_rsrc_t rs, unsigned off);
template <>
__device__ inline float field_load<float>(__amdgpu_buffer_rsrc_t rs, unsigned off) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0));
}
template <>
__device__ inline double field_load<double>(__amdgpu_buffer_rsrc_t rs, unsigned off) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rs, off, 0, 0));
}

// First column and number of columns << 16 of each row rz (columns come in
// ascending (rz, ry) order, ry without gaps).
template <int NK, int NT>
__device__ __forceinline__ void row_table(const int* cols, int ncol, int* rows) {
  for (int r = threadIdx.x; r < NK; r += NT) rows[r] = 0;
  __syncthreads();
  for (int c = threadIdx.x; c < ncol; c += NT) {
    const int rz = cols[c] >> 8;
    if (c + 1 == ncol || (cols[c + 1] >> 8) != rz) {
      const int cnt = (cols[c] & 0xff) + 1;
      rows[rz] = (c + 1 - cnt) | (cnt << 16);
    }
  }
  __syncthreads();
}

// Trigonometric transform of the real field pa pu (pa alone without PROD) onto
// the columns: out[rx] of column threadIdx.x.  Slab by slab, z lines (x, y) into the line buffer
// t1 [SP][nk][R], y lines (x, rz) in place or, in all slabs but the last,
// into the column buffer t2 [x][ncol]; then x lines per column.  Ends without
// a barrier: t1 and t2 may be refilled after the caller's next one.
template <class T, int N, int KM, int NT, int NS, bool PROD = true>
__device__ __forceinline__ void line_transform(const T* pa, const T* pu, const int* cols, int ncol,
                                               T* t1, T* t2, const int* rows,
                                               T (&out)[2 * KM + 1]) {
  constexpr int R = line_row(N), nk = 2 * KM + 1, SP = N / NS, P = N * N;
  const int tid = threadIdx.x;
  const auto ra = field_rsrc(pa, P * N), ru = field_rsrc(pu, P * N);
#pragma unroll 1
  for (int s = 0; s < NS; ++s) {
#pragma unroll 1
    for (int l = tid; l < SP * N; l += NT) {
      const unsigned r0 = unsigned(s * SP * N + l) * unsigned(sizeof(T));
      T v[N], a[N], u[N];
      cplx<T> X[N / 2 + 1];
#pragma unroll
      for (int z = 0; z < N; ++z) a[z] = field_load<T>(ra, r0 + unsigned(z * P * sizeof(T)));
      if constexpr (PROD)
#pragma unroll
        for (int z = 0; z < N; ++z) u[z] = field_load<T>(ru, r0 + unsigned(z * P * sizeof(T)));
      // all loads of the line are issued before the first product waits: in FP32
      // calls on the 24 and 40 grids are 1 to 1.6 % faster with it, chi on the 36
      // grid 2 % (its exchange 1.6 % slower); in FP64 15 to 25 grids are 1 % faster
      // without
      if constexpr (sizeof(T) == 4) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int z = 0; z < N; ++z) v[z] = PROD ? a[z] * u[z] : a[z];
      RFft<T, N>::run(v, X);
      const int xs = l / N;
      T* o = t1 + xs * (nk * R) + (l - xs * N);
      o[0] = X[0].x;
#pragma unroll
      for (int k = 1; k <= KM; ++k) {
        o[(2 * k - 1) * R] = X[k].x;
        o[(2 * k) * R] = X[k].y;
      }
    }
    lds_barrier();
#pragma unroll 1
    for (int l = tid; l < SP * nk; l += NT) {
      T* row = t1 + l * R;
      T v[N];
      cplx<T> X[N / 2 + 1];
#pragma unroll
      for (int y = 0; y < N; ++y) v[y] = row[y];
      RFft<T, N>::run(v, X);
      if (NS > 1 && s + 1 < NS) {
        const int xs = l / nk, m = rows[l - xs * nk], cnt = m >> 16;
        T* d = t2 + (s * SP + xs) * ncol + (m & 0xffff);
        if (cnt > 0) d[0] = X[0].x;
#pragma unroll
        for (int k = 1; k <= KM; ++k)
          if (2 * k < cnt) {
            d[2 * k - 1] = X[k].x;
            d[2 * k] = X[k].y;
          }
      } else {
        row[0] = X[0].x;
#pragma unroll
        for (int k = 1; k <= KM; ++k) {
          row[2 * k - 1] = X[k].x;
          row[2 * k] = X[k].y;
        }
      }
    }
    lds_barrier();
  }
  if (tid < ncol) {
    const int cd = cols[tid];
    const T* c1 = t1 + (cd >> 8) * R + (cd & 0xff);
    T v[N];
    cplx<T> X[N / 2 + 1];
#pragma unroll
    for (int x = 0; x < N; ++x)
      v[x] = (x < N - SP) ? t2[x * ncol + tid] : c1[(x - (N - SP)) * (nk * R)];
    RFft<T, N>::run(v, X);
    out[0] = X[0].x;
#pragma unroll
    for (int k = 1; k <= KM; ++k) {
      out[2 * k - 1] = X[k].x;
      out[2 * k] = X[k].y;
    }
  }
}

// One (G', pair) item.  BINS: the per-shell split of the cutoff extrapolation
// is compiled in (taken when pc.shm2 is set).  A thread's eight bins live in
// registers for the epilogue of one part only; kept across the transforms of
// both parts they spilled (15 grid, |k| <= 7, FP32: 23.7 ns per item against
// 14.2; 20 grid, |k| <= 9: 41.8 and 32.3; 12 grid, |k| <= 3, FP64: 12.3 and 9.0).
template <class T, int N, int KM, bool BINS>
__device__ __forceinline__ void pair_item(const PairCell& pc, int gl, int p, T* t1) {
  constexpr int NT = pair_threads(sizeof(T), N, KM), NS = pair_slabs(sizeof(T), N, KM, BINS);
  constexpr int nk = 2 * KM + 1, SP = N / NS;
  constexpr int kM2 = 2 * KM * KM + 2 * KM + 1;  // m^2 of any row triple lies below
  __shared__ double vm[kM2];
  __shared__ signed char sh[BINS ? kM2 : 1];
  __shared__ int rows[NS > 1 ? nk : 1];
  __shared__ double red[NT / 64];
  __shared__ double binw[BINS ? NT / 64 * kMaxShells : 1];
  const int tid = threadIdx.x;
  const int i = pc.pairs[p] & 0xffff, j = pc.pairs[p] >> 16;
  const T* psi = static_cast<const T*>(pc.psi);
  const T* w = static_cast<const T*>(pc.w);
  T* t2 = t1 + SP * nk * line_row(N);
  const bool split = BINS && pc.shm2;
  // tables by m^2 in shared memory: read one column at a time in the
  // epilogue, a chain of dependent global reads otherwise (a fifth of the 36
  // grid's time)
  for (int k = tid; k < pc.nm2; k += NT) {
    vm[k] = k >= 1 && k <= pc.m2lim ? 4.0 * M_PI / (pc.vden * double(k)) : 0.0;
    if constexpr (BINS)
      if (split) sh[k] = k <= pc.m2lim ? pc.shm2[k] : 1;
  }
  if constexpr (NS > 1) row_table<nk, NT>(pc.cols, pc.ncol, rows);
  double s = 0.0;
  const int sg = split ? pc.shell[pc.g0 + gl] : 0;
#pragma unroll 1
  for (int part = 0; part < 2; ++part) {  // real, imaginary part of w
    const T* ui = w + ((long(gl) * pc.nocc + i) * 2 + part) * pc.ld;
    const T* uj = w + ((long(gl) * pc.nocc + j) * 2 + part) * pc.ld;
    T xf[nk] = {}, xg[nk] = {};
    line_transform<T, N, KM, NT, NS>(psi + long(i) * pc.ld, uj, pc.cols, pc.ncol,
                                      t1, t2, rows, xf);
    lds_barrier();
    if (i != j) {
      line_transform<T, N, KM, NT, NS>(psi + long(j) * pc.ld, ui, pc.cols, pc.ncol,
                                        t1, t2, rows, xg);
      lds_barrier();
    } else {
#pragma unroll
      for (int k = 0; k < nk; ++k) xg[k] = xf[k];
    }
    double sb[BINS ? kMaxShells : 1] = {};
    if (tid < pc.ncol) {
      const int cd = pc.cols[tid];
      const int ky = row_k(cd & 0xff), kz = row_k(cd >> 8), r2 = ky * ky + kz * kz;
      const double m = double((ky ? 2 : 1) * (kz ? 2 : 1));
      const double* vt = vm + r2;
      const double q0 = vt[0] * (double(xf[0]) * double(xg[0]));
      if constexpr (BINS)
        if (split) bin_add(sb, min(int(sh[r2]), sg) - 1, m * q0);
      double q = 0.0;
#pragma unroll
      for (int k = 1; k <= KM; ++k) {
        const double t = vt[k * k] * (double(xf[2 * k - 1]) * double(xg[2 * k - 1]) +
                                      double(xf[2 * k]) * double(xg[2 * k]));
        q += t;
        if constexpr (BINS)
          if (split) bin_add(sb, min(int(sh[r2 + k * k]), sg) - 1, 2.0 * m * t);
      }
      s += m * (q0 + 2.0 * q);
    }
    if constexpr (BINS) {
      // bins leave the registers before the next part's transforms: each wave's
      // sum into its own slots
#pragma unroll
      for (int b = 0; b < kMaxShells; ++b)
        if (b < pc.nb) {
          double v = sb[b];
          for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
          double* slot = binw + (tid >> 6) * kMaxShells + b;
          if ((tid & 63) == 0) *slot = part ? *slot + v : v;
        }
    }
  }
  const double scale = (i == j ? 1.0 : 2.0) * pc.dV2;
  s = block_sum(s, red);
  if (tid == 0) pc.xpart[long(gl) * pc.npairs + p] = scale * s;
  if constexpr (BINS) {
    if (split && tid < pc.nb) {  // block_sum's barriers order the slots
      double b = 0.0;
      for (int w = 0; w < NT / 64; ++w) b += binw[w * kMaxShells + tid];
      pc.xbins[(long(gl) * pc.npairs + p) * pc.nb + tid] = scale * b;
    }
  }
}

// One cell, items [first, first + count) of its (G', pair) list: the pairs come
// in blocks of (i, j) and each XCD takes a contiguous range, so the workgroups
// resident on one XCD share a handful of psi_i and w_j^{(G')} in its L2.
template <class T, int N, int KM, bool BINS>
__global__ __launch_bounds__(pair_threads(sizeof(T), N, KM), pair_minw(sizeof(T), N, BINS)) void k_pair(
    PairCell pc, long first, long count) {
  extern __shared__ __align__(16) char smem[];
  const long b = block_item(blockIdx.x, count);
  if (b < 0) return;
  const long t = first + b;
  const int gl = int(t / pc.npairs);
  pair_item<T, N, KM, BINS>(pc, gl, int(t - long(gl) * pc.npairs), reinterpret_cast<T*>(smem));
}

// Several cells of the same grid and kept-set instance in one launch: the
// work list is the concatenation of every cell's (G', pair) items (prefix[c] =
// first item of cell c), of which it takes [first, first + count), one item per
// workgroup, in XCD-contiguous ranges.
template <class T, int N, int KM>
__global__ __launch_bounds__(pair_threads(sizeof(T), N, KM),
                             pair_minw(sizeof(T), N)) void k_pair_multi(const PairCell* __restrict__ cells,
                                                                        const long* __restrict__ prefix,
                                                                        int ncells, long first,
                                                                        long count) {
  extern __shared__ __align__(16) char smem[];
  const long b = block_item(blockIdx.x, count);
  if (b < 0) return;
  const long t = first + b;
  int lo = 0, hi = ncells - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) / 2;
    if (prefix[mid] <= t) lo = mid; else hi = mid - 1;
  }
  const PairCell pc = cells[lo];
  const long u = t - prefix[lo];
  const int gl = int(u / pc.npairs);
  pair_item<T, N, KM, false>(pc, gl, int(u - long(gl) * pc.npairs), reinterpret_cast<T*>(smem));
}

// Transforms of real fields to the half set H of auxiliary vectors, with the
// same line transforms:
//   OVERLAP = false, first pass of the double transform of chi: item r,
//     out[o * ld + r] = scale sum_r' chi(r, r') e^{+iG_o.r'}   (a = chi)
//   OVERLAP = true, overlap densities (step (i)): item (a, j),
//     out[(a nh + o) nocc + j] = scale sum_r psi_a(r) psi_j(r) e^{-iG_o.r}
//     (a = all orbitals, the nocc occupied ones first)
// The fields come in the order r = (x N + z) N + y: the first transform runs
// along x (consecutive lanes read consecutive (z, y)), the last along z; the
// kept set is the same in every order of the axes.  The trigonometric
// coefficients of all columns then meet in shared memory, where each output
// combines its (up to) eight:
//   sum f e^{i s G.r} = prod over axes of (C - i s sgn(k) S),  S = -sum f sin.
// Bound by the line transforms and by reading the rows of chi; consecutive
// items run on one XCD, so the 8-byte outputs of neighbouring rows fill
// lines in its L2.  Against complex transforms of two rows (four products) per
// workgroup, dispatched round-robin: rows of chi on the 36 grid 4136 -> 2169 us
// (8.7 GB read), 24 grid 243 -> 180, 15 grid 35 -> 15, 18 grid FP64 129 -> 69;
// overlap densities on the 36 grid 55 -> 15.5 ms.
template <class T, int N, int KM, bool OVERLAP>
__global__ __launch_bounds__(pair_threads(sizeof(T), N, KM), pair_minw(sizeof(T), N))
void k_real_forward(const T* __restrict__ a, long ld, int nocc, long first, long count,
                    const int* __restrict__ cols, int ncol, const int* __restrict__ gdesc, int nh,
                    int kmax, double scale, cplx<T>* __restrict__ out) {
  constexpr int NT = pair_threads(sizeof(T), N, KM), NS = pair_slabs(sizeof(T), N, KM);
  constexpr int nk = 2 * KM + 1, SP = N / NS;
  extern __shared__ __align__(16) char smem[];
  __shared__ int rows[nk];
  const long b = block_item(blockIdx.x, count);
  if (b < 0) return;
  const long it = first + b;
  T* t1 = reinterpret_cast<T*>(smem);
  T* t2 = t1 + SP * nk * line_row(N);
  const int tid = threadIdx.x;
  row_table<nk, NT>(cols, ncol, rows);
  T x[nk] = {};
  long o0, step;
  if constexpr (OVERLAP) {
    const long av = it / nocc, j = it - av * nocc;
    line_transform<T, N, KM, NT, NS>(a + (nocc + av) * ld, a + j * ld, cols, ncol, t1, t2, rows,
                                     x);
    o0 = av * nh * nocc + j;
    step = nocc;
  } else {
    line_transform<T, N, KM, NT, NS, false>(a + it * ld, a + it * ld, cols, ncol, t1, t2, rows, x);
    o0 = it;
    step = ld;
  }
  __syncthreads();
  if (tid < ncol)
#pragma unroll
    for (int k = 0; k < nk; ++k) t1[k * ncol + tid] = x[k];
  __syncthreads();
  for (int o = tid; o < nh; o += NT) {
    const int g = gdesc[o];
    int kx = g & 0xff, ky = ((g >> 8) & 0xff) - kmax, kz = (g >> 16) - kmax;
    if (kx > N / 2) kx -= N;
    const int ax = kx < 0 ? -kx : kx, ay = ky < 0 ? -ky : ky, az = kz < 0 ? -kz : kz;
    // cosine rows and, where the index is not 0, sine rows one further
    const T* c0 = t1 + (az ? 2 * az - 1 : 0) * ncol + (rows[ax ? 2 * ax - 1 : 0] & 0xffff) +
                  (ay ? 2 * ay - 1 : 0);
    const int dz = ncol;  // to the sine row of z, x and y
    const int dx = ax ? (rows[2 * ax] & 0xffff) - (rows[2 * ax - 1] & 0xffff) : 0;
    T re = c0[0], im = T(0);
    const T sx = kx > 0 ? T(1) : T(-1), sy = ky > 0 ? T(1) : T(-1), sz = kz > 0 ? T(1) : T(-1);
    if (ax) im -= sx * c0[dx];
    if (ay) im -= sy * c0[1];
    if (az) im -= sz * c0[dz];
    if (ax && ay) re -= sx * sy * c0[dx + 1];
    if (ax && az) re -= sx * sz * c0[dx + dz];
    if (ay && az) re -= sy * sz * c0[1 + dz];
    if (ax && ay && az) im += sx * sy * sz * c0[dx + 1 + dz];
    out[o0 + o * step] = {T(scale) * re, OVERLAP ? -T(scale) * im : T(scale) * im};
  }
}

// Occupied orbitals into the plane order of the pair transforms:
// out[(z N + x) N + y] = in[(x N + z) N + y].  Grid (ceil(n^3 / 256), nocc).
template <class T>
__global__ __launch_bounds__(256) void k_plane_order(const T* __restrict__ in, long ld, int n,
                                                     T* __restrict__ out) {
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r >= n * n * n) return;
  const int y = r % n, x = (r / n) % n, z = r / (n * n);
  out[long(blockIdx.y) * ld + r] = in[long(blockIdx.y) * ld + (x * n + z) * n + y];
}

}  // namespace ltmp2
