// Internal state of an LTMP2 context (shared by the C ABI implementation
// files; not part of the public header).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>
#include <vector>

#include "../../include/ltmp2.h"
#include "dispatch.h"

// A second stream (default priority, not synchronised with the null stream) for
// work that is independent of the caller's: the direct terms of an energy run
// beside its exchange terms, with which they share no buffer.  Small cells are
// bound by the latency of their launches, 12^3 in FP64 eight chains of four and
// five kernels that leave most CUs idle: 865 us one after the other, 599 beside
// each other (24^3 in FP32 72.7 and 70.5 ms).
struct SideStream {
  hipStream_t st = nullptr;
  hipEvent_t fork = nullptr, join = nullptr;
  // Without it everything runs on the caller's stream `main`: where creation
  // failed, and where `main` has a priority or CUs of its own, which the caller
  // chose for all of the work (and streams of different priorities must not
  // wait for each other).
  void create(hipStream_t main) {
    const bool handle = main && main != hipStreamLegacy && main != hipStreamPerThread;
    int priority = 0;
    if ((!handle || (hipStreamGetPriority(main, &priority) == hipSuccess && priority == 0)) &&
        hipStreamCreateWithFlags(&st, hipStreamNonBlocking) == hipSuccess &&
        (!handle || same_cus(main, st)) &&
        hipEventCreateWithFlags(&fork, hipEventDisableTiming) == hipSuccess &&
        hipEventCreateWithFlags(&join, hipEventDisableTiming) == hipSuccess)
      return;
    (void)hipGetLastError();
    destroy();
  }
  static bool same_cus(hipStream_t a, hipStream_t b) {
    uint32_t ma[32] = {}, mb[32] = {};
    if (hipExtStreamGetCUMask(a, 32, ma) != hipSuccess ||
        hipExtStreamGetCUMask(b, 32, mb) != hipSuccess)
      return false;
    for (int k = 0; k < 32; ++k)
      if (ma[k] != mb[k]) return false;
    return true;
  }
  void destroy() {
    if (join) (void)hipEventDestroy(join);
    if (fork) (void)hipEventDestroy(fork);
    if (st) (void)hipStreamDestroy(st);
    st = nullptr;
    fork = join = nullptr;
  }
};

// While it lives, `side` runs behind what `main` held at its construction; its
// end makes `main` wait for `side`, on every path out of the scope.
class Beside {
 public:
  Beside(SideStream& s, hipStream_t main, bool want) : side(s), main(main) {
    on = want && s.st && hipEventRecord(s.fork, main) == hipSuccess &&
         hipStreamWaitEvent(s.st, s.fork, 0) == hipSuccess;
  }
  ~Beside() {
    if (on && (hipEventRecord(side.join, side.st) != hipSuccess ||
               hipStreamWaitEvent(main, side.join, 0) != hipSuccess))
      (void)hipStreamSynchronize(side.st);
  }
  Beside(const Beside&) = delete;
  Beside& operator=(const Beside&) = delete;
  hipStream_t stream() const { return on ? side.st : main; }

 private:
  SideStream& side;
  hipStream_t main;
  bool on;
};

struct ltmp2_ctx {
  bool own_scratch = true;  // false: chi / chihat / P / w belong to a batch or spin channel 1
  bool batched = false;     // cell of a batch
  ltmp2_params prm{};
  std::string err;
  bool failed = false;
  hipStream_t stream = nullptr;

  // sizes
  int n = 0, nr = 0, npw = 0, nst = 0, no = 0, nv = 0, ng = 0, nh = 0, ntau = 0, npairs = 0;
  int ldbpw = 0;  // row stride of d_bpw (n_pw rounded up to a multiple of 4)
  // split-BF16x3 operands (k-octet-blocked hi / lo, see kernels_gemm3.hpp):
  // orbitals scaled by sqrt of the Laplace factors (per tau), overlap
  // densities (once), virtual basis scaled by the virtual factors (per tau)
  int kpo = 0, kpv = 0;  // occupied / virtual counts rounded up to 64
  long ldnd3 = 0, ldb3 = 0;
  void *d_psi3h = nullptr, *d_psi3l = nullptr, *d_nd3h = nullptr, *d_nd3l = nullptr;
  void *d_b3h = nullptr, *d_b3l = nullptr;
  long nrp = 0;  // padded row stride of grid arrays (multiple of 64)
  int kmax_aux = 0, kmax_orb = 0, gblock = 0;
  double omega = 0, dV = 0, mu = 0, xmin = 0, xmax = 0, quad_delta = 0;
  double xmin_force = 0, xmax_force = 0;  // > 0: quadrature range of two spin channels
  double escale = 1.0;  // energies per unit cell: 1 / N for the supercell of an N-point mesh
  int n_kmesh = 1;      // k-point mesh points per axis (1: Gamma only)
  int quad_flags = 0;
  std::string mlp_path;
  std::vector<double> eps, tau, w;
  std::vector<int> aux;  // [ng][3], H first then -H

  // device tables
  ltmp2::SphereCols sc{};
  int* d_cdesc = nullptr;
  int* d_cstart = nullptr;
  int* d_ckx = nullptr;
  void* d_wtab = nullptr;         // coefficients of the transformed states (GridOps::wstates)
  int wtab_k = 0;
  int* d_gdesc = nullptr;
  int* d_pairs = nullptr;
  int* d_cols = nullptr;          // [ncol] columns of the pair transforms (PairCell)
  signed char* d_shm2 = nullptr;  // [m2lim + 1] spheres by m^2 (cutoff extrapolation)
  int ncol = 0, nm2 = 0, m2lim = 0;  // PairCell
  double vden = 0.0;
  double* d_v = nullptr;          // [nh] v(G') of H
  double* d_fo = nullptr;  // [ntau][no]
  double* d_fv = nullptr;  // [ntau][nv]

  // device data, element type double (FP64) or float (FP32, BF16X3)
  size_t esz = sizeof(double);
  void* d_psi = nullptr;       // [nst][nrp]
  void* d_psiz = nullptr;      // [no][nrp] occupied, in the plane order of the pair transforms
                               // (null: see occupied())
  void* d_nd = nullptr;        // [nv][nh][no] complex
  void* d_bpw = nullptr;       // [nv][ldbpw] real basis of virtual coefficients
  void* d_chi = nullptr;       // [nrp][nrp]
  void* d_chihat = nullptr;    // [nh][nrp] complex
  double* d_pd = nullptr;      // [nh]
  void* d_P = nullptr;         // [gblock * no * 2][npw]
  void* d_w = nullptr;         // [gblock * no][2][nrp] real and imaginary fields, plane order
  double* d_xpart = nullptr;   // [nh][npairs]
  double* d_xrow = nullptr;    // [nh] v(G') times the row sums of d_xpart
  double* d_scal = nullptr;    // [2 * ntau + 8] device scalars
  // internal cutoff extrapolation: nb nested auxiliary spheres (0 = off)
  int nb = 0;
  double alpha = 1.05;
  std::vector<double> eaux_n;    // [nb] cutoffs eaux / alpha^(n-1)
  signed char* d_shell = nullptr;  // [nh] spheres containing each vector of H
  double* d_pdb = nullptr;     // [nh][nb] direct-term bins per G'
  double* d_xb = nullptr;      // [nh][npairs][nb] exchange bins per (G', pair)
  double* d_xrowb = nullptr;   // [nh][nb]
  double* d_scalb = nullptr;   // [ntau][2][nb] per-tau bin sums (E_d, E_x)
  bool ext_valid = false;
  std::vector<double> ext_d, ext_x;  // [nb] energies per cutoff (last ltmp2_energy)
  double ext_inf[3] = {0, 0, 0};

  // spin-unrestricted cells: the second spin channel (owned; shares the
  // quadrature and the chi buffer of this context, which holds spin alpha)
  ltmp2_ctx* beta = nullptr;
  std::vector<void*> owned;
  size_t bytes = 0;

  SideStream side;  // contexts with scratch of their own

  // optional per-stage event timing
  bool timing = false;
  struct Mark {
    int stage;
    hipEvent_t a, b;
  };
  std::vector<Mark> marks;
  std::vector<hipEvent_t> pool;
  double stage_ms[8] = {0};
  long stage_n[8] = {0};
};

namespace ltmp2 {
// Host drivers of one Laplace point (ltmp2.hip); values land in d_scal.
ltmp2_status run_direct(ltmp2_ctx* c, int itau, hipStream_t st);
// Pieces of the exchange term used by batched execution.
PairCell pair_cell(const ltmp2_ctx* c, int g0, int gb);
// Occupied orbitals in the pair transforms' order: kept, or in the chi scratch.
inline void* occupied(const ltmp2_ctx* c) { return c->d_psiz ? c->d_psiz : c->d_chi; }
ltmp2_status exchange_block_prepare(ltmp2_ctx* c, int itau, int g0, int gb);
ltmp2_status exchange_reduce(ltmp2_ctx* c, int itau, int g_first, int g_count);
ltmp2_status setup_cell(ltmp2_ctx* c, const int32_t* miller, const double* eps,
                        const double* coeff, const double* tau, const double* w);
// Validation of a cell's inputs; *use receives the coefficients to pass on
// (the caller's, or their real form held in `store`).
ltmp2_status validate_inputs(const ltmp2_params* p, const int32_t* miller, const double* eps,
                             const double* coeff, const double* tau, const double* w,
                             std::vector<double>& store, const double** use);
const std::string& setup_error();
void set_setup_error(const std::string& msg);
// Orbitals real up to a phase (or degenerate blocks with a real basis) to
// real form (real_orbitals.cpp); `out` stays empty if nothing changes.
ltmp2_status unfold_kmesh(int n_k, int n_bands, int n_occ, const int32_t* n_pw_k,
                          const int32_t* miller, const double* eps, const double* coeff,
                          std::vector<int32_t>& miller_s, std::vector<double>& eps_s,
                          std::vector<double>& coeff_s, std::string& err);
ltmp2_status real_orbitals(int npw, const int32_t* miller, int nst, const double* eps, int nocc,
                           const double* coeff, std::vector<double>& out, bool* changed,
                           std::string& err);
}  // namespace ltmp2
