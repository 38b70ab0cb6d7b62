// Transform kernels instantiated for one grid size n = LTMP2_N.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <map>
#include <mutex>
#include <type_traits>

#include "dispatch.h"

#ifndef LTMP2_N
#error "LTMP2_N must be defined"
#endif

namespace ltmp2 {
namespace {

constexpr int N = LTMP2_N;
constexpr size_t kLdsCap = 150 * 1024;
constexpr size_t kLdsHalf = 78 * 1024;
constexpr size_t kLdsQuarter = 39 * 1024;

template <class T>
int choose_sx(int nk, int cap = 10) {
  int sx = slab_tile_at_most(N, cap);
  while (sx > 1 && inv_lds_bytes<T>(N, nk, sx) > kLdsCap) sx = slab_tile_at_most(N, sx - 1);
  return sx;
}

// The same for the forward transforms (z-pass buffer only, see fwd_lds).
template <class T>
int choose_sx_fwd(int nk, int cap = 10) {
  int sx = slab_tile_at_most(N, cap);
  while (sx > 1 && fwd_lds_bytes<T>(N, nk, sx) > kLdsCap) sx = slab_tile_at_most(N, sx - 1);
  return sx;
}

// Dynamic shared memory above the default needs a per-kernel attribute; set
// it once per kernel (never while a stream is being captured into a graph).
bool ensure_lds(const void* kern, size_t lds) {
  static std::mutex mu;
  static std::map<const void*, size_t> done;
  std::lock_guard<std::mutex> lk(mu);
  auto it = done.find(kern);
  if (it != done.end() && it->second >= lds) return true;
  if (hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, int(lds)) !=
      hipSuccess)
    return false;
  done[kern] = lds;
  return true;
}

template <class K>
ltmp2_status launch_nt(K kern, dim3 grid, int nt, size_t lds, hipStream_t st, auto... args) {
  if (lds > kLdsCap) return LTMP2_EINVAL;
  if (grid.x == 0 || grid.y == 0) return LTMP2_OK;
  if (!ensure_lds(reinterpret_cast<const void*>(kern), lds)) return LTMP2_EDEVICE;
  hipLaunchKernelGGL(kern, grid, dim3(nt), lds, st, args...);
  return hipGetLastError() == hipSuccess ? LTMP2_OK : LTMP2_EDEVICE;
}

template <class K>
ltmp2_status launch(K kern, dim3 grid, size_t lds, hipStream_t st, auto... args) {
  return launch_nt(kern, grid, kThreads, lds, st, args...);
}

template <template <int> class F>
ltmp2_status by_opt(int nout, auto&&... a) {
  const int need = (nout + kThreads - 1) / kThreads;
  if (need <= 1) return F<1>::go(a...);
  if (need <= 3) return F<3>::go(a...);
  if (need <= 9) return F<9>::go(a...);
  if (need <= 17) return F<17>::go(a...);
  return LTMP2_EINVAL;
}

template <class T>
ltmp2_status orbitals(const cplx<double>* coef, int nstates, int npw, SphereCols sc, double scale,
                      T* psi, long ld, hipStream_t st) {
  const int nk = 2 * sc.kmax + 1, sx = choose_sx<T>(nk);
  return launch(k_orbitals<T, N>, dim3(nstates), inv_lds_bytes<T>(N, nk, sx), st, coef, npw, sc,
                sx, scale, psi, ld);
}

template <class T>
struct ChiColsF {
  template <int OPT>
  struct F {
    static ltmp2_status go(const cplx<T>* chihat, long ld, const int* gdesc, int ng, int nh,
                           const double* v, int kmax, double dV, double* pd,
                           cplx<double>* chi_out, ShellBins bins, hipStream_t st) {
      const int nk = 2 * kmax + 1, sx = choose_sx_fwd<T>(nk);
      return launch(k_chi_cols<T, N, OPT>, dim3(nh), fwd_lds_bytes<T>(N, nk, sx), st, chihat, ld,
                    gdesc, ng, nh, v, kmax, sx, dV, pd, chi_out, bins);
    }
  };
};
template <class T>
ltmp2_status chi_cols(const cplx<T>* chihat, long ld, const int* gdesc, int ng, int nh,
                      const double* v, int kmax, double dV, double* pd, cplx<double>* chi_out,
                      ShellBins bins, hipStream_t st) {
  return by_opt<ChiColsF<T>::template F>(ng, chihat, ld, gdesc, ng, nh, v, kmax, dV, pd, chi_out,
                                         bins, st);
}

template <class T>
struct HartreeF {
  template <int OPT>
  struct F {
    static ltmp2_status go(const cplx<T>* h, long ld, const int* gdesc, int ng, const double* v,
                           int kmax, double dV, int g0, int gb, double* pdh, hipStream_t st) {
      const int nk = 2 * kmax + 1, sx = choose_sx_fwd<T>(nk);
      return launch(k_hartree<T, N, OPT>, dim3(gb), fwd_lds_bytes<T>(N, nk, sx), st, h, ld, gdesc,
                    ng, v, kmax, sx, dV, g0, pdh);
    }
  };
};
template <class T>
ltmp2_status hartree(const cplx<T>* h, long ld, const int* gdesc, int ng, const double* v,
                     int kmax, double dV, int g0, int gb, double* pdh, hipStream_t st) {
  return by_opt<HartreeF<T>::template F>(ng, h, ld, gdesc, ng, v, kmax, dV, g0, gb, pdh, st);
}

template <class T, int K, bool WIDE = false, bool SMALL = false>
ltmp2_status wstates_window_launch(const T* P, int npw, const void* tab, int kt, int nitems,
                                   double scale, T* w, long ld, hipStream_t st) {
  using W = WstShape<T, N, K, WIDE>;
  if constexpr (!W::holds_all)
    if (W::lds(npw) > kLdsCap)
      return wstates_window_launch<T, K, true>(P, npw, tab, kt, nitems, scale, w, ld, st);
  if constexpr (K < korb_win(N) && !SMALL)
    if (kt < K)
      return wstates_window_launch<T, K, WIDE, true>(P, npw, tab, kt, nitems, scale, w, ld, st);
  return launch_nt(k_wstates_real<T, N, K, WIDE, SMALL>, dim3(unsigned(2L * nitems / W::F)), W::NT,
                   W::lds(npw), st, P, npw, static_cast<const unsigned short*>(tab), kt, scale, w,
                   ld);
}

// Window instance of the transformed states for a cell (-1: the general kernel,
// also for a set that has so many more vectors than a sphere of its largest
// index that they leave no room next to the field, or so few that the table by
// wavevector is larger than five bytes for each)
template <class T, int K>
constexpr bool wstates_holds(int npw) {
  static_assert(WstShape<T, N, K, true>::holds_all);
  return WstShape<T, N, K>::lds(npw) <= kLdsCap || WstShape<T, N, K, true>::lds(npw) <= kLdsCap;
}
template <class T>
int wstates_kept(int kmax, int npw) {
  constexpr int ko = korb_win(N), kl = ko < 2 ? ko : ko - 1;
  const int win = wstates_window(N, kmax), nk = 2 * kmax + 1;
  if (2 * nk * nk * (kmax + 1) > 5 * npw + 4) return -1;
  return (win == ko ? wstates_holds<T, ko>(npw) : wstates_holds<T, kl>(npw)) ? win : -1;
}

template <class T>
ltmp2_status wstates(const T* P, int npw, const void* tab, int kt, SphereCols sc, int nitems,
                     double scale, T* w, long ld, hipStream_t st) {
  constexpr int ko = korb_win(N), kl = ko < 2 ? ko : ko - 1;
  const int win = wstates_kept<T>(sc.kmax, npw);
  if (win == ko)
    return wstates_window_launch<T, ko>(P, npw, tab, kt, nitems, scale, w, ld, st);
  if (win == kl)
    return wstates_window_launch<T, kl>(P, npw, tab, kt, nitems, scale, w, ld, st);
  // the largest slab tile that lets four workgroups share a CU, unless two
  // workgroups per CU would allow more than twice that tile
  const int nk = 2 * sc.kmax + 1;
  auto tile = [nk](size_t cap) {
    int sx = slab_tile_at_most(N, 10);
    while (sx > 1 && inv_lds_bytes<T>(N, nk, sx) > cap) sx = slab_tile_at_most(N, sx - 1);
    return sx;
  };
  const int s4 = tile(kLdsQuarter), s2 = tile(kLdsHalf);
  const int sx = 2 * s4 >= s2 ? s4 : s2;
  return launch(k_wstates<T, N>, dim3(nitems), inv_lds_bytes<T>(N, nk, sx), st, P, npw,
                static_cast<const int*>(tab), sc, sx, scale, w, ld);
}

// Kept-set instance of the pair kernels for a cell (-1: none holds it).
int pair_instance(int kmax) {
  constexpr int kw = pair_kw(N), kf = pair_kf(N);
  if (kw > 1 && kmax <= kw - 1) return kw - 1;
  if (kmax <= kw) return kw;
  return kmax <= kf ? kf : -1;
}

// fn(integral_constant<KM>) for the instance that holds kmax.
template <class Fn>
ltmp2_status with_instance(int kmax, Fn&& fn) {
  constexpr int kw = pair_kw(N), kf = pair_kf(N);
  const int k = pair_instance(kmax);
  if constexpr (kw > 1)
    if (k == kw - 1) return fn(std::integral_constant<int, kw - 1>{});
  if (k == kw) return fn(std::integral_constant<int, kw>{});
  if constexpr (kf > kw)
    if (k == kf) return fn(std::integral_constant<int, kf>{});
  return LTMP2_EINVAL;
}

template <class T, int KM, bool BINS = false>
size_t pair_lds(int ncol) {
  constexpr int ns = pair_slabs(sizeof(T), N, KM, BINS);
  return pair_lds_bytes(sizeof(T), N, KM, ns, ncol);
}

template <class T, bool OVERLAP>
ltmp2_status real_forward(const T* a, long ld, int nocc, long items, const int* cols, int ncol,
                          const int* gdesc, int nh, int kmax, double scale, cplx<T>* out,
                          hipStream_t st) {
  return with_instance(kmax, [&](auto km) -> ltmp2_status {
    constexpr int KM = decltype(km)::value, NT = pair_threads(sizeof(T), N, KM);
    if (ncol < 1 || ncol > pair_cols_max(KM)) return LTMP2_EINVAL;
    const size_t lds = std::max(pair_lds<T, KM>(ncol), sizeof(T) * (2 * KM + 1) * ncol);
    return launch_ranges(items, NT, [&](long first, long count) {
      return launch_nt(k_real_forward<T, N, KM, OVERLAP>, dim3(launch_blocks(count)), NT, lds, st,
                       a, ld, nocc, first, count, cols, ncol, gdesc, nh, kmax, scale, out);
    });
  });
}
template <class T>
ltmp2_status overlap(const T* psi, long ld, int no, int nv, const int* cols, int ncol,
                     const int* gdesc, int nh, int kmax, double dV, cplx<T>* nd, hipStream_t st) {
  return real_forward<T, true>(psi, ld, no, long(no) * nv, cols, ncol, gdesc, nh, kmax, dV, nd, st);
}
template <class T>
ltmp2_status chi_rows(const T* chi, long ld, int nr, const int* cols, int ncol, const int* gdesc,
                      int nh, int kmax, double dV, cplx<T>* chihat, hipStream_t st) {
  return real_forward<T, false>(chi, ld, 1, nr, cols, ncol, gdesc, nh, kmax, dV, chihat, st);
}

// Launches that split by cutoff shell run an instance with that epilogue
// compiled in; the others run one without it (fewer live registers).
template <class T>
ltmp2_status pair(const PairCell& pc, hipStream_t st) {
  return with_instance(pc.kmax, [&](auto km) -> ltmp2_status {
    constexpr int KM = decltype(km)::value, NT = pair_threads(sizeof(T), N, KM);
    if (pc.ncol < 1 || pc.ncol > pair_cols_max(KM) || pc.nm2 > 2 * KM * KM + 2 * KM + 1)
      return LTMP2_EINVAL;
    return launch_ranges(long(pc.npairs) * pc.gb, NT, [&](long first, long count) {
      const dim3 grid(launch_blocks(count));
      if (pc.shm2)
        return launch_nt(k_pair<T, N, KM, true>, grid, NT, pair_lds<T, KM, true>(pc.ncol), st, pc,
                         first, count);
      return launch_nt(k_pair<T, N, KM, false>, grid, NT, pair_lds<T, KM>(pc.ncol), st, pc, first,
                       count);
    });
  });
}

// Several cells of one kept-set instance in one launch of `total` items.
template <class T>
ltmp2_status pair_multi(const PairCell* cells, const long* prefix, int ncells, long total,
                        int kmax_max, int ncol_max, hipStream_t st) {
  return with_instance(kmax_max, [&](auto km) -> ltmp2_status {
    constexpr int KM = decltype(km)::value, NT = pair_threads(sizeof(T), N, KM);
    if (ncol_max < 1 || ncol_max > pair_cols_max(KM)) return LTMP2_EINVAL;
    return launch_ranges(total, NT, [&](long first, long count) {
      return launch_nt(k_pair_multi<T, N, KM>, dim3(launch_blocks(count)), NT,
                       pair_lds<T, KM>(ncol_max), st, cells, prefix, ncells, first, count);
    });
  });
}

// Launch shape of an instance: x planes whose z lines one round of a
// workgroup covers, and workgroups resident on a CU.
template <class T>
void pair_shape(int kmax, int ncol, int* planes, int* wg_per_cu) {
  *planes = *wg_per_cu = 1;
  (void)with_instance(kmax, [&](auto km) -> ltmp2_status {
    constexpr int KM = decltype(km)::value, NT = pair_threads(sizeof(T), N, KM);
    *planes = std::max(1, NT / N);
    int n = 0;
    const void* k = reinterpret_cast<const void*>(k_pair_multi<T, N, KM>);
    if (ensure_lds(k, pair_lds<T, KM>(ncol)) &&
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k, NT, pair_lds<T, KM>(ncol)) ==
            hipSuccess)
      *wg_per_cu = std::max(1, n);
    return LTMP2_OK;
  });
}

template <class T>
ltmp2_status plane_order(const T* in, long ld, int nocc, T* out, hipStream_t st) {
  return launch(k_plane_order<T>, dim3((N * N * N + 255) / 256, nocc), 0, st, in, ld, N, out);
}

// Explicit instantiation in both compilation passes, so the device pass
// instantiates every kernel the host launchers reference.
#define LTMP2_INST(T)                                                                          \
  template ltmp2_status orbitals<T>(const cplx<double>*, int, int, SphereCols, double, T*, long,\
                                    hipStream_t);                                              \
  template ltmp2_status overlap<T>(const T*, long, int, int, const int*, int, const int*, int, \
                                   int, double, cplx<T>*, hipStream_t);                        \
  template ltmp2_status chi_rows<T>(const T*, long, int, const int*, int, const int*, int, int,\
                                    double, cplx<T>*, hipStream_t);                            \
  template ltmp2_status chi_cols<T>(const cplx<T>*, long, const int*, int, int, const double*, \
                                    int, double, double*, cplx<double>*, ShellBins,            \
                                    hipStream_t);                                              \
  template ltmp2_status wstates<T>(const T*, int, const void*, int, SphereCols, int, double, T*,\
                                   long, hipStream_t);                                               \
  template int wstates_kept<T>(int, int);                                                      \
  template ltmp2_status pair<T>(const PairCell&, hipStream_t);                                 \
  template ltmp2_status pair_multi<T>(const PairCell*, const long*, int, long, int, int,       \
                                      hipStream_t);                                            \
  template void pair_shape<T>(int, int, int*, int*);                                           \
  template ltmp2_status plane_order<T>(const T*, long, int, T*, hipStream_t);                  \
  template ltmp2_status hartree<T>(const cplx<T>*, long, const int*, int, const double*, int,   \
                                   double, int, int, double*, hipStream_t);
LTMP2_INST(double)
LTMP2_INST(float)

}  // namespace

#define LTMP2_CAT2(a, b) a##b
#define LTMP2_CAT(a, b) LTMP2_CAT2(a, b)
#if !defined(__HIP_DEVICE_COMPILE__)
extern const GridOps<double> LTMP2_CAT(kGridOpsD_, LTMP2_N);
extern const GridOps<float> LTMP2_CAT(kGridOpsF_, LTMP2_N);
const GridOps<double> LTMP2_CAT(kGridOpsD_, LTMP2_N) = {
    orbitals<double>, overlap<double>, chi_rows<double>, chi_cols<double>, wstates<double>,
    pair<double>, pair_multi<double>, hartree<double>, pair_shape<double>, plane_order<double>,
    pair_instance, wstates_kept<double>};
const GridOps<float> LTMP2_CAT(kGridOpsF_, LTMP2_N) = {
    orbitals<float>, overlap<float>, chi_rows<float>, chi_cols<float>, wstates<float>,
    pair<float>, pair_multi<float>, hartree<float>, pair_shape<float>, plane_order<float>,
    pair_instance, wstates_kept<float>};
#endif

}  // namespace ltmp2
