// Transform kernels of the LTMP2 path (templated on precision T and grid n).
#pragma once
#include "transforms.hpp"

namespace ltmp2 {

struct SphereCols {
  int ncol;
  int kmax;
  const int* cdesc;   // [ncol]
  const int* cstart;  // [ncol + 1]
  const int* ckx;     // [n_pw]
};

// ---------------------------------------------------------------------------
// Orbitals on the grid: psi_p(r) = Omega^-1/2 sum_G c_p(G) e^{iG.r}, real for
// time-reversal-invariant coefficients (Gamma point).
//   coef: [n_items][n_pw] complex, entries in column order of the sphere
//   psi:  [n_items][ld] real
template <class T, int N>
__global__ __launch_bounds__(kThreads) void k_orbitals(const cplx<double>* __restrict__ coef, int npw,
                                                       SphereCols sc, int sx, double scale,
                                                       T* __restrict__ psi, long ld) {
  extern __shared__ __align__(16) char smem[];
  const int nk = 2 * sc.kmax + 1;
  SlabLds<T> L = inv_lds<T>(smem, N, nk, sx);
  fill_twiddles<T, 1, N>(L.tw);
  const long p = blockIdx.x;
  const cplx<double>* c = coef + p * npw;
  T* out = psi + p * ld;
  auto cf = [&](int e) { return cplx<T>{T(c[e].x), T(c[e].y)}; };
  auto st = [&](int x, int y, int z, cplx<T> v) { out[(x * N + z) * N + y] = T(scale) * v.x; };
  inverse_sphere<T, N>(cf, st, sc.kmax, sx, sc.ncol, sc.cdesc, sc.cstart, sc.ckx, L);
}

// ---------------------------------------------------------------------------
// Second pass (columns) and the Coulomb trace: for G' = H[g],
//   chi(G, G') = dV sum_r e^{-iG.r} chihat(r, G'),  G in the full set,
//   pd[g] = v(G') sum_G v(G) |chi(G, G')|^2,
// v and the shells of the bins given for H (those of -H are the same).
// Optionally stores chi(G, G') for G' in H and, by chi(-G, -G') =
// conj chi(G, G') (real chi(r, r')), for G' in -H:  out[G][G'] (ng x ng),
// and the same sum split by auxiliary cutoff shell (bins.out [n_h][nb]).
template <class T, int N, int OPT>
__global__ __launch_bounds__(kThreads) void k_chi_cols(const cplx<T>* __restrict__ chihat, long ld,
                                                       const int* __restrict__ gdesc_all, int ng,
                                                       int nh, const double* __restrict__ v,
                                                       int kmax, int sx, double dV,
                                                       double* __restrict__ pd,
                                                       cplx<double>* __restrict__ chi_out,
                                                       ShellBins bins) {
  extern __shared__ __align__(16) char smem[];
  __shared__ double red[kThreads / 64];
  __shared__ double redb[kThreads / 64 * kMaxShells];
  const int nk = 2 * kmax + 1;
  SlabLds<T> L = fwd_lds<T>(smem, N, nk, sx);
  fill_twiddles<T, -1, N>(L.tw);
  const int g = blockIdx.x;
  const cplx<T>* col = chihat + long(g) * ld;
  int gd[OPT];
  cplx<T> acc[OPT];
#pragma unroll
  for (int t = 0; t < OPT; ++t) {
    const int o = threadIdx.x + t * kThreads;
    gd[t] = (o < ng) ? gdesc_all[o] : 0;
    acc[t] = {T(0), T(0)};
  }
  __syncthreads();
  auto ld_ = [&](int x, int y, int z) { return col[(x * N + z) * N + y]; };
  forward_pruned<T, -1, N, OPT>(ld_, kmax, sx, gd, ng, acc, L);
  double s = 0.0;
  double sb[kMaxShells] = {};
  const int sg = bins.shell ? bins.shell[g] : 0;
#pragma unroll
  for (int t = 0; t < OPT; ++t) {
    const int o = threadIdx.x + t * kThreads;
    if (o < ng) {
      const double re = dV * double(acc[t].x), im = dV * double(acc[t].y);
      const int oh = o < nh ? o : o - nh;
      const double term = v[oh] * (re * re + im * im);
      s += term;
      if (bins.shell) bin_add(sb, min(int(bins.shell[oh]), sg) - 1, term);
      if (chi_out) {
        const int on = (o < nh) ? o + nh : o - nh;
        chi_out[long(o) * ng + g] = {re, im};
        chi_out[long(on) * ng + g + nh] = {re, -im};
      }
    }
  }
  s = block_sum(s, red);
  if (threadIdx.x == 0) pd[g] = v[g] * s;
  if (bins.shell) {
    block_sum_bins(sb, redb);
    if (threadIdx.x == 0)
      for (int b = 0; b < bins.nb; ++b) bins.out[long(g) * bins.nb + b] = v[g] * sb[b];
  }
}

// ---------------------------------------------------------------------------
// Hartree-like route to the direct term (Implementation section, step
// (iv.a)), a cross-check of the chi route that shares none of its kernels:
//   h^{(G')}(r)  = sum_i psi_i(r) w_i^{(G')}(r)
//   X^{(G')}(G)  = dV sum_r e^{-iG.r} h^{(G')}(r)      (= chi(G, -G'))
//   pdh[g0 + gl] = v(G') sum_G v(G) |X^{(G')}(G)|^2,   E_d(tau) = -4 sum_{H} pdh.
// k_hsum: grid (ceil(n_r / 256), gb); h [gb][ld] complex.
// psi and w in the plane order of the pair transforms, h likewise
// (r = (z N + x) N + y).
template <class T>
__global__ __launch_bounds__(256) void k_hsum(const T* __restrict__ psi, long ld,
                                              const T* __restrict__ w, int no, long nr,
                                              cplx<T>* __restrict__ h) {
  const long r = long(blockIdx.x) * 256 + threadIdx.x;
  const long gl = blockIdx.y;
  if (r >= nr) return;
  cplx<T> s = {T(0), T(0)};
  for (int i = 0; i < no; ++i) {
    const T a = psi[long(i) * ld + r];
    const T* b = w + (gl * no + i) * 2 * ld + r;
    s.x += a * b[0];
    s.y += a * b[ld];
  }
  h[gl * ld + r] = s;
}

// one block per outer vector gl of the block
template <class T, int N, int OPT>
__global__ __launch_bounds__(kThreads) void k_hartree(const cplx<T>* __restrict__ h, long ld,
                                                      const int* __restrict__ gdesc_all, int ng,
                                                      const double* __restrict__ v, int kmax,
                                                      int sx, double dV, int g0,
                                                      double* __restrict__ pdh) {
  extern __shared__ __align__(16) char smem[];
  __shared__ double red[kThreads / 64];
  const int nk = 2 * kmax + 1;
  SlabLds<T> L = fwd_lds<T>(smem, N, nk, sx);
  fill_twiddles<T, -1, N>(L.tw);
  const int gl = blockIdx.x;
  const cplx<T>* col = h + long(gl) * ld;
  int gd[OPT];
  cplx<T> acc[OPT];
#pragma unroll
  for (int t = 0; t < OPT; ++t) {
    const int o = threadIdx.x + t * kThreads;
    gd[t] = (o < ng) ? gdesc_all[o] : 0;
    acc[t] = {T(0), T(0)};
  }
  __syncthreads();
  auto ld_ = [&](int x, int y, int z) { return col[(z * N + x) * N + y]; };
  forward_pruned<T, -1, N, OPT>(ld_, kmax, sx, gd, ng, acc, L);
  double s = 0.0;
#pragma unroll
  for (int t = 0; t < OPT; ++t) {
    const int o = threadIdx.x + t * kThreads;
    if (o < ng) {
      const double re = dV * double(acc[t].x), im = dV * double(acc[t].y);
      s += v[o < ng / 2 ? o : o - ng / 2] * (re * re + im * im);
    }
  }
  s = block_sum(s, red);
  if (threadIdx.x == 0) pdh[g0 + gl] = v[g0 + gl] * s;
}

// ---------------------------------------------------------------------------
// Transformed states on the grid where the orbital sphere is beyond the window
// of kernels_wstates.hpp (the caller's grid aliases; see there for P and w):
// both fields as one complex transform, W_j(G) gathered from P where the x
// stage needs it.
// Entry e of the sphere (column order) uses wq[e] = q, the place of Re c(G_k) in
// a row of P (Im c(G_k) follows it; 0 for G = 0, which has none), bit 31 set for
// -G_k.  With s = +1 for G_k and -1 for -G_k (c_a(-G) = conj c_a(G)):
//   W(G) = (P_re[q] - s P_im[q + 1]) + i (P_im[q] + s P_re[q + 1]).
template <class T, int N>
__global__ __launch_bounds__(kThreads) void k_wstates(const T* __restrict__ P, int npw,
                                                      const int* __restrict__ wq,
                                                      SphereCols sc, int sx, double scale,
                                                      T* __restrict__ w, long ld) {
  extern __shared__ __align__(16) char smem[];
  const int nk = 2 * sc.kmax + 1;
  SlabLds<T> L = inv_lds<T>(smem, N, nk, sx);
  fill_twiddles<T, 1, N>(L.tw);
  const long item = blockIdx.x;
  const T* pre = P + (2 * item) * long(npw);
  const T* pim = pre + npw;
  T* out = w + 2 * item * ld;
  // W_j(G) of sphere entry e, gathered from the real basis (each entry is
  // used once per slab group)
  auto cf = [&](int e) {
    const int q = wq[e] & 0xffff;
    T re = pre[q], im = pim[q];
    if (q > 0) {
      const T s = wq[e] < 0 ? T(-1) : T(1);
      re -= s * pim[q + 1];
      im += s * pre[q + 1];
    }
    return cplx<T>{re, im};
  };
  auto st = [&](int x, int y, int z, cplx<T> v) {
    T* o = out + (z * N + x) * N + y;
    o[0] = T(scale) * v.x;
    o[ld] = T(scale) * v.y;
  };
  inverse_sphere<T, N>(cf, st, sc.kmax, sx, sc.ncol, sc.cdesc, sc.cstart, sc.ckx, L);
}

}  // namespace ltmp2
