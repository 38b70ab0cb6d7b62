// Learned Laplace quadrature: a small MLP proposes the minimax exponents and
// weights, a few Remez steps polish them, and the plain fit is both the arbiter
// (certification by equioscillation) and the fallback.
//
// Network: 3 -> 64 (tanh) -> 64 (tanh) -> 24, FP32.
//   input   (log x_min, log R / log 1e4, N / 12),   R = x_max / x_min
//   output  slots 0..11: log alpha_n, slots 12..23: log beta_n of the
//           unit-interval fit (y = x / x_min in [1, R]); the first N of each
//           half are used, the rest are masked out of the loss.
// Loss: mean squared error over the unmasked outputs.
// Training: Adam on the GPU with the kernels below (forward, backward, Adam);
// every reduction is a fixed-order loop, so runs are reproducible.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <initializer_list>
#include <mutex>
#include <string>
#include <thread>
#include <utility>
#include <vector>

#include "../../include/ltmp2.h"
#include "quadrature.h"

namespace ltmp2 {

constexpr int kIn = 3, kH = 64, kOut = 24;
constexpr int kP = kH * kIn + kH + kH * kH + kH + kOut * kH + kOut;
static_assert(kP == LTMP2_MLP_NPARAM, "parameter count");

struct Net {
  const float *W1, *b1, *W2, *b2, *W3, *b3;
};
inline Net unpack(const float* p) {
  Net n;
  n.W1 = p;
  n.b1 = n.W1 + kH * kIn;
  n.W2 = n.b1 + kH;
  n.b2 = n.W2 + kH * kH;
  n.W3 = n.b2 + kH;
  n.b3 = n.W3 + kOut * kH;
  return n;
}

// Y[b][o] = act(sum_i X[b][i] W[o][i] + bias[o]); act 1 = tanh
__global__ void k_lin_fwd(const float* __restrict__ X, int B, int I, const float* __restrict__ W,
                          const float* __restrict__ bias, int O, int act, float* __restrict__ Y) {
  const long t = long(blockIdx.x) * blockDim.x + threadIdx.x;
  if (t >= long(B) * O) return;
  const int b = int(t / O), o = int(t - long(b) * O);
  float s = bias[o];
  for (int i = 0; i < I; ++i) s += X[long(b) * I + i] * W[o * I + i];
  Y[t] = act ? tanhf(s) : s;
}

// Loss and gradient of one minibatch in two launches.
//
// k_mlp_step: workgroups walk the batch in chunks of kS samples.  The whole
// network (24 KB) and a chunk's activations sit in shared memory; forward,
// masked squared error, backward and the chunk's weight gradients follow one
// another between barriers, and each thread keeps its share of the gradient
// in registers over all its chunks.  part [workgroups][kP], lossb
// [workgroups].  k_mlp_reduce adds the workgroups' parts in fixed order and,
// when training, applies Adam, one thread per parameter.
//
// Bound by latency (0.2 GFLOP per 1024 samples): one kernel per layer and
// direction, with the weight gradients summed over the batch by 17 workgroups
// (234 us per launch), took 800 us a step of 1024 samples.
constexpr int kS = 16, kStep = 256, kW = kH + 1;  // kW: padded row, any read order is conflict-free
constexpr int kMaxParts = 256;

__global__ __launch_bounds__(kStep) void k_mlp_step(const float* __restrict__ P,
                                                    const float* __restrict__ X,
                                                    const float* __restrict__ Y,
                                                    const float* __restrict__ M,
                                                    const int* __restrict__ idx, int B,
                                                    float inv_count, float* __restrict__ part,
                                                    float* __restrict__ lossb) {
  __shared__ float W1[kH * kIn], b1[kH], W2[kH * kW], b2[kH], W3[kOut * kW], b3[kOut];
  __shared__ float x[kS][kIn], h1[kS][kW], h2[kS][kW], d1[kS][kW], d2[kS][kW], dO[kS][kOut];
  __shared__ float red[kStep];
  const int t = threadIdx.x;
  for (int k = t; k < kP; k += kStep) {
    int q = k;
    const float v = P[k];
    if (q < kH * kIn) W1[q] = v;
    else if ((q -= kH * kIn) < kH) b1[q] = v;
    else if ((q -= kH) < kH * kH) W2[q / kH * kW + q % kH] = v;
    else if ((q -= kH * kH) < kH) b2[q] = v;
    else if ((q -= kH) < kOut * kH) W3[q / kH * kW + q % kH] = v;
    else b3[q - kOut * kH] = v;
  }
  // gradient entries of this thread: W2[o2][i2 .. i2 + 15], six of W3, one of
  // W1 and one bias
  float g2[16] = {}, g3[6] = {}, g1 = 0.f, gb = 0.f, loss = 0.f;
  const int o2 = t / 4, i2 = t % 4 * 16;
  const int o = t & 63, bq = t >> 6;  // forward / backward: output o of samples bq, bq + 4, ...
  for (int c0 = blockIdx.x * kS; c0 < B; c0 += gridDim.x * kS) {
    const int nb = min(kS, B - c0);
    __syncthreads();
    if (t < kS * kIn) {
      const int b = t / kIn;
      x[b][t % kIn] = b < nb ? X[long(idx ? idx[c0 + b] : c0 + b) * kIn + t % kIn] : 0.f;
    }
    __syncthreads();
    for (int b = bq; b < kS; b += 4) {
      float s = b1[o];
      for (int i = 0; i < kIn; ++i) s += x[b][i] * W1[o * kIn + i];
      h1[b][o] = tanhf(s);
    }
    __syncthreads();
    {
      float s[kS / 4];
#pragma unroll
      for (int u = 0; u < kS / 4; ++u) s[u] = b2[o];
#pragma unroll 8
      for (int i = 0; i < kH; ++i) {
        const float w = W2[o * kW + i];
#pragma unroll
        for (int u = 0; u < kS / 4; ++u) s[u] += h1[bq + 4 * u][i] * w;
      }
#pragma unroll
      for (int u = 0; u < kS / 4; ++u) h2[bq + 4 * u][o] = tanhf(s[u]);
    }
    __syncthreads();
    for (int e = t; e < kS * kOut; e += kStep) {
      const int b = e / kOut, k = e - b * kOut;
      float s = b3[k];
#pragma unroll 8
      for (int i = 0; i < kH; ++i) s += h2[b][i] * W3[k * kW + i];
      float d = 0.f;
      if (b < nb) {
        const long r = long(idx ? idx[c0 + b] : c0 + b) * kOut + k;
        d = (s - Y[r]) * M[r];
      }
      dO[b][k] = 2.f * d * inv_count;
      loss += d * d;
    }
    __syncthreads();
    {
      float s[kS / 4] = {};
#pragma unroll 8
      for (int k = 0; k < kOut; ++k) {
        const float w = W3[k * kW + o];
#pragma unroll
        for (int u = 0; u < kS / 4; ++u) s[u] += dO[bq + 4 * u][k] * w;
      }
#pragma unroll
      for (int u = 0; u < kS / 4; ++u) {
        const float a = h2[bq + 4 * u][o];
        d2[bq + 4 * u][o] = s[u] * (1.f - a * a);
      }
    }
    __syncthreads();
    {
      float s[kS / 4] = {};
#pragma unroll 8
      for (int k = 0; k < kH; ++k) {
        const float w = W2[k * kW + o];
#pragma unroll
        for (int u = 0; u < kS / 4; ++u) s[u] += d2[bq + 4 * u][k] * w;
      }
#pragma unroll
      for (int u = 0; u < kS / 4; ++u) {
        const float a = h1[bq + 4 * u][o];
        d1[bq + 4 * u][o] = s[u] * (1.f - a * a);
      }
    }
    __syncthreads();
#pragma unroll 4
    for (int b = 0; b < kS; ++b) {
      const float d = d2[b][o2];
#pragma unroll
      for (int u = 0; u < 16; ++u) g2[u] += d * h1[b][i2 + u];
#pragma unroll
      for (int u = 0; u < 6; ++u) {
        const int e = t + u * kStep;
        g3[u] += dO[b][e >> 6] * h2[b][e & 63];
      }
    }
    for (int b = 0; b < kS; ++b) {
      if (t < kH * kIn) g1 += d1[b][t / kIn] * x[b][t % kIn];
      if (t < kH) gb += d1[b][t];
      else if (t < 2 * kH) gb += d2[b][t - kH];
      else if (t < 2 * kH + kOut) gb += dO[b][t - 2 * kH];
    }
  }
  float* G = part + long(blockIdx.x) * kP;
  if (t < kH * kIn) G[t] = g1;
  G += kH * kIn;
  if (t < kH) G[t] = gb;
  G += kH;
#pragma unroll
  for (int u = 0; u < 16; ++u) G[o2 * kH + i2 + u] = g2[u];
  G += kH * kH;
  if (t >= kH && t < 2 * kH) G[t - kH] = gb;
  G += kH;
#pragma unroll
  for (int u = 0; u < 6; ++u) G[t + u * kStep] = g3[u];
  G += kOut * kH;
  if (t >= 2 * kH && t < 2 * kH + kOut) G[t - 2 * kH] = gb;
  red[t] = loss;
  __syncthreads();
  for (int w = kStep / 2; w > 0; w >>= 1) {
    if (t < w) red[t] += red[t + w];
    __syncthreads();
  }
  if (t == 0) lossb[blockIdx.x] = red[0];
}

struct Adam {
  float lr, b1, b2, eps, bc1, bc2;
};

// g[p] = sum_w part[w][p]; loss[0] += sum_w lossb[w]; with m: Adam step of p
__global__ __launch_bounds__(256) void k_mlp_reduce(const float* __restrict__ part, int nw,
                                                    const float* __restrict__ lossb,
                                                    float* __restrict__ g, float* __restrict__ loss,
                                                    float* __restrict__ p, float* __restrict__ m,
                                                    float* __restrict__ v, Adam ad) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (blockIdx.x == 0) {
    __shared__ float red[256];
    red[threadIdx.x] = int(threadIdx.x) < nw ? lossb[threadIdx.x] : 0.f;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
      if (int(threadIdx.x) < w) red[threadIdx.x] += red[threadIdx.x + w];
      __syncthreads();
    }
    if (threadIdx.x == 0) loss[0] += red[0];
  }
  if (i >= kP) return;
  float gi = 0.f;
#pragma unroll 16
  for (int w = 0; w < nw; ++w) gi += part[long(w) * kP + i];
  g[i] = gi;
  if (!m) return;
  const float mi = ad.b1 * m[i] + (1.f - ad.b1) * gi;
  const float vi = ad.b2 * v[i] + (1.f - ad.b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p[i] -= ad.lr * (mi / ad.bc1) / (sqrtf(vi / ad.bc2) + ad.eps);
}

namespace {

inline unsigned nblk(long n) { return unsigned((n + 255) / 256); }

// splitmix64 (Steele, Lea, Flood 2014): counter-based 64-bit generator
inline uint64_t splitmix64(uint64_t& s) {
  uint64_t z = (s += 0x9E3779B97F4A7C15ull);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
inline double uniform01(uint64_t& s) { return double(splitmix64(s) >> 11) * 0x1.0p-53; }

// Device memory of one call, one allocation cut into 256-byte aligned pieces.
struct Work {
  char* base = nullptr;
  size_t used = 0;
  ~Work() {
    if (base) (void)hipFree(base);
  }
  static size_t piece(size_t n) { return (std::max<size_t>(n, 1) * sizeof(float) + 255) / 256 * 256; }
  bool init(std::initializer_list<std::pair<float**, size_t>> want) {
    size_t total = 0;
    for (auto& w : want) total += piece(w.second);
    void* q = nullptr;
    if (hipMalloc(&q, total) != hipSuccess) return false;
    base = static_cast<char*>(q);
    for (auto& w : want) {
      *w.first = reinterpret_cast<float*>(base + used);
      used += piece(w.second);
    }
    return true;
  }
};

void forward(const float* P, const float* X, int B, float* h1, float* h2, float* O,
             hipStream_t st) {
  Net n = unpack(P);
  hipLaunchKernelGGL(k_lin_fwd, dim3(nblk(long(B) * kH)), dim3(256), 0, st, X, B, kIn, n.W1, n.b1,
                     kH, 1, h1);
  hipLaunchKernelGGL(k_lin_fwd, dim3(nblk(long(B) * kH)), dim3(256), 0, st, h1, B, kH, n.W2, n.b2,
                     kH, 1, h2);
  hipLaunchKernelGGL(k_lin_fwd, dim3(nblk(long(B) * kOut)), dim3(256), 0, st, h2, B, kH, n.W3,
                     n.b3, kOut, 0, O);
}

// workgroups (parts) of a minibatch of B samples
inline int step_parts(int B) { return std::min(kMaxParts, (B + kS - 1) / kS); }

// gradient of the masked MSE into G, summed squared error added to loss; with
// m: one Adam step of P
void step(const float* X, const float* Y, const float* M, const int* idx, int B, float inv_count,
          float* P, float* part, float* lossb, float* G, float* loss, float* m, float* v, Adam ad,
          hipStream_t st) {
  const int nw = step_parts(B);
  hipLaunchKernelGGL(k_mlp_step, dim3(nw), dim3(kStep), 0, st, P, X, Y, M, idx, B, inv_count, part,
                     lossb);
  hipLaunchKernelGGL(k_mlp_reduce, dim3((kP + 255) / 256), dim3(256), 0, st, part, nw, lossb, G,
                     loss, P, m, v, ad);
}

float mask_count(const float* M, long n) {
  double c = 0.0;
  for (long i = 0; i < n; ++i) c += M[i];
  return float(c);
}

thread_local std::string g_mlp_error;

ltmp2_status mfail(ltmp2_status s, const std::string& m) {
  g_mlp_error = m;
  return s;
}

}  // namespace

void mlp_features(double x_min, double x_max, int n_tau, float* f) {
  f[0] = float(std::log(x_min));
  f[1] = float(std::log(x_max / x_min) / std::log(1e4));
  f[2] = float(n_tau) / 12.0f;
}

const char* mlp_last_error() { return g_mlp_error.c_str(); }

}  // namespace ltmp2

using namespace ltmp2;

extern "C" ltmp2_status ltmp2_mlp_init(uint64_t seed, float* params) {
  if (!params) return mfail(LTMP2_EINVAL, "params is NULL");
  uint64_t s = seed;
  auto fill = [&](float* p, int fan_in, int fan_out, int count) {
    const double a = std::sqrt(6.0 / (fan_in + fan_out));  // Glorot uniform
    for (int k = 0; k < count; ++k) p[k] = float((2.0 * uniform01(s) - 1.0) * a);
  };
  Net n = unpack(params);
  fill(const_cast<float*>(n.W1), kIn, kH, kH * kIn);
  std::fill(const_cast<float*>(n.b1), const_cast<float*>(n.b1) + kH, 0.f);
  fill(const_cast<float*>(n.W2), kH, kH, kH * kH);
  std::fill(const_cast<float*>(n.b2), const_cast<float*>(n.b2) + kH, 0.f);
  fill(const_cast<float*>(n.W3), kH, kOut, kOut * kH);
  std::fill(const_cast<float*>(n.b3), const_cast<float*>(n.b3) + kOut, 0.f);
  return LTMP2_OK;
}

extern "C" ltmp2_status ltmp2_quadrature_table(int n_tau, int count, const double* R,
                                               double* alpha, double* beta, double* delta) {
  if ((count > 0) && (!R || !alpha || !beta)) return mfail(LTMP2_EINVAL, "NULL array");
  const int r = quadrature_table(n_tau, count, R, alpha, beta, delta);
  if (r == 1) return mfail(LTMP2_EINVAL, "need ascending R > 1 and 1 <= n_tau <= 16");
  if (r != 0) return mfail(LTMP2_ENUMERIC, "continuation failed");
  return LTMP2_OK;
}

extern "C" ltmp2_status ltmp2_mlp_dataset(int count, uint64_t seed, double dmin_lo, double dmin_hi,
                                          double ratio_lo, double ratio_hi, const int* n_taus,
                                          int n_choices, float* X, float* Y, float* M,
                                          double* xrange) {
  if (count < 1 || !n_taus || n_choices < 1 || !X || !Y || !M)
    return mfail(LTMP2_EINVAL, "bad dataset arguments");
  if (!(0 < dmin_lo && dmin_lo <= dmin_hi) || !(1 < ratio_lo && ratio_lo <= ratio_hi))
    return mfail(LTMP2_EINVAL, "bad sampling ranges");
  for (int c = 0; c < n_choices; ++c)
    if (n_taus[c] < 1 || n_taus[c] > 12) return mfail(LTMP2_EINVAL, "n_tau choices must be 1..12");
  uint64_t s = seed;
  std::vector<double> xmin(count), ratio(count);
  std::vector<int> nt(count);
  for (int k = 0; k < count; ++k) {
    nt[k] = n_taus[std::min<int>(n_choices - 1, int(uniform01(s) * n_choices))];
    xmin[k] = std::exp(std::log(dmin_lo) + uniform01(s) * std::log(dmin_hi / dmin_lo));
    ratio[k] = std::exp(std::log(ratio_lo) + uniform01(s) * std::log(ratio_hi / ratio_lo));
  }
  std::fill(Y, Y + size_t(count) * kOut, 0.f);
  std::fill(M, M + size_t(count) * kOut, 0.f);
  // one continuation sweep per n_tau choice, sweeps in parallel threads
  std::vector<int> status(n_choices, 0);
  std::vector<std::thread> pool;
  for (int c = 0; c < n_choices; ++c) {
    pool.emplace_back([&, c]() {
      const int n = n_taus[c];
      for (int c2 = 0; c2 < c; ++c2)
        if (n_taus[c2] == n) return;  // repeated choice: handled once
      std::vector<int> idx;
      for (int k = 0; k < count; ++k)
        if (nt[k] == n) idx.push_back(k);
      if (idx.empty()) return;
      std::sort(idx.begin(), idx.end(), [&](int a, int b) { return ratio[a] < ratio[b]; });
      std::vector<double> R(idx.size()), al(idx.size() * n), be(idx.size() * n);
      for (size_t q = 0; q < idx.size(); ++q) R[q] = ratio[idx[q]];
      if (quadrature_table(n, (int)idx.size(), R.data(), al.data(), be.data(), nullptr) != 0) {
        status[c] = 1;
        return;
      }
      for (size_t q = 0; q < idx.size(); ++q) {
        const int k = idx[q];
        for (int t = 0; t < n; ++t) {
          Y[size_t(k) * kOut + t] = float(std::log(al[q * n + t]));
          Y[size_t(k) * kOut + 12 + t] = float(std::log(be[q * n + t]));
          M[size_t(k) * kOut + t] = 1.f;
          M[size_t(k) * kOut + 12 + t] = 1.f;
        }
      }
    });
  }
  for (auto& t : pool) t.join();
  for (int c = 0; c < n_choices; ++c)
    if (status[c]) return mfail(LTMP2_ENUMERIC, "minimax table failed");
  for (int k = 0; k < count; ++k) {
    mlp_features(xmin[k], xmin[k] * ratio[k], nt[k], X + size_t(k) * kIn);
    if (xrange) {
      xrange[2 * k] = xmin[k];
      xrange[2 * k + 1] = xmin[k] * ratio[k];
    }
  }
  return LTMP2_OK;
}

extern "C" ltmp2_status ltmp2_mlp_forward(const float* params, const float* X, int n, float* Yout,
                                          void* stream) {
  if (!params || !X || !Yout || n < 1) return mfail(LTMP2_EINVAL, "bad arguments");
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  Work w;
  float *P, *Xd, *H1, *H2, *O;
  if (!w.init({{&P, kP}, {&Xd, size_t(n) * kIn}, {&H1, size_t(n) * kH}, {&H2, size_t(n) * kH},
               {&O, size_t(n) * kOut}}))
    return mfail(LTMP2_ENOMEM, "device allocation failed");
  if (hipMemcpyAsync(P, params, kP * sizeof(float), hipMemcpyHostToDevice, st) != hipSuccess ||
      hipMemcpyAsync(Xd, X, size_t(n) * kIn * sizeof(float), hipMemcpyHostToDevice, st) !=
          hipSuccess)
    return mfail(LTMP2_EDEVICE, "copy failed");
  forward(P, Xd, n, H1, H2, O, st);
  if (hipGetLastError() != hipSuccess) return mfail(LTMP2_EDEVICE, "launch failed");
  if (hipMemcpyAsync(Yout, O, size_t(n) * kOut * sizeof(float), hipMemcpyDeviceToHost, st) !=
          hipSuccess ||
      hipStreamSynchronize(st) != hipSuccess)
    return mfail(LTMP2_EDEVICE, "copy back failed");
  return LTMP2_OK;
}

// ---------------------------------------------------------------------------
// Allocation-free forward pass.  The hidden activations of up to
// LTMP2_MLP_NOALLOC_MAX_ROWS rows live in `scratch`, a device array of this
// file that every GPU running the library holds for the life of the process
// (8 MiB).  Host code never passes the array's name to a kernel: each
// device's own address of it comes from hipGetSymbolAddress, taken once per
// device (with that device current) on the entry point's first call there.
// Both hidden layers are written in full before they are read, so nothing
// needs clearing between calls; calls that overlap on one GPU share the
// array and race.
namespace {
constexpr int kNoAllocRows = LTMP2_MLP_NOALLOC_MAX_ROWS;
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

static __device__ __align__(256) float scratch[2 * size_t(kNoAllocRows) * kH];

namespace {
// Device address of this GPU's scratch array (nullptr on failure).
float* scratch_on_current_device(std::string& err) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    err = "no usable current device";
    return nullptr;
  }
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr) {
      err = std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e);
      return nullptr;
    }
    g_scratch_ptr[dev] = static_cast<float*>(ptr);
  }
  return g_scratch_ptr[dev];
}
}  // namespace

extern "C" ltmp2_status ltmp2_mlp_forward_noalloc(const float* params_dev, const float* X_dev,
                                                  int n, float* Y_dev, void* hip_stream) {
  if (!params_dev || !X_dev || !Y_dev) return mfail(LTMP2_EINVAL, "NULL device pointer");
  if (n < 1 || n > kNoAllocRows)
    return mfail(LTMP2_EINVAL, "n must be in [1, " + std::to_string(kNoAllocRows) +
                                   "] for the allocation-free forward pass");
  std::string err;
  float* h = scratch_on_current_device(err);
  if (!h) return mfail(LTMP2_EDEVICE, err);
  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
  forward(params_dev, X_dev, n, h, h + size_t(kNoAllocRows) * kH, Y_dev, st);
  if (hipGetLastError() != hipSuccess) return mfail(LTMP2_EDEVICE, "launch failed");
  return LTMP2_OK;
}

extern "C" ltmp2_status ltmp2_mlp_grad(const float* params, const float* X, const float* Y,
                                       const float* M, int n, float* grad, float* loss,
                                       void* stream) {
  if (!params || !X || !Y || !M || !grad || n < 1) return mfail(LTMP2_EINVAL, "bad arguments");
  const float cnt = mask_count(M, long(n) * kOut);
  if (!(cnt > 0)) return mfail(LTMP2_EINVAL, "empty mask");
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  Work w;
  float *P, *G, *Xd, *Yd, *Md, *part, *lossb, *ld;
  const int nw = step_parts(n);
  if (!w.init({{&P, kP}, {&G, kP}, {&Xd, size_t(n) * kIn}, {&Yd, size_t(n) * kOut},
               {&Md, size_t(n) * kOut}, {&part, size_t(nw) * kP}, {&lossb, nw}, {&ld, 1}}))
    return mfail(LTMP2_ENOMEM, "device allocation failed");
  const size_t bo = size_t(n) * kOut * sizeof(float);
  if (hipMemcpyAsync(P, params, kP * sizeof(float), hipMemcpyHostToDevice, st) != hipSuccess ||
      hipMemcpyAsync(Xd, X, size_t(n) * kIn * sizeof(float), hipMemcpyHostToDevice, st) ||
      hipMemcpyAsync(Yd, Y, bo, hipMemcpyHostToDevice, st) ||
      hipMemcpyAsync(Md, M, bo, hipMemcpyHostToDevice, st) ||
      hipMemsetAsync(ld, 0, sizeof(float), st))
    return mfail(LTMP2_EDEVICE, "copy failed");
  step(Xd, Yd, Md, nullptr, n, 1.f / cnt, P, part, lossb, G, ld, nullptr, nullptr, Adam{}, st);
  if (hipGetLastError() != hipSuccess) return mfail(LTMP2_EDEVICE, "launch failed");
  float l = 0.f;
  if (hipMemcpyAsync(grad, G, kP * sizeof(float), hipMemcpyDeviceToHost, st) ||
      hipMemcpyAsync(&l, ld, sizeof(float), hipMemcpyDeviceToHost, st) ||
      hipStreamSynchronize(st))
    return mfail(LTMP2_EDEVICE, "copy back failed");
  if (loss) *loss = l / cnt;
  return LTMP2_OK;
}

extern "C" ltmp2_status ltmp2_mlp_train(float* params, const float* X, const float* Y,
                                        const float* M, int n, int epochs, int batch, float lr,
                                        uint64_t seed, float* loss_hist, void* stream) {
  if (!params || !X || !Y || !M || n < 1 || epochs < 1 || batch < 1 || !(lr > 0))
    return mfail(LTMP2_EINVAL, "bad arguments");
  batch = std::min(batch, n);
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  Work w;
  float *P, *G, *dX, *dY, *dM, *m1, *m2, *part, *lossb, *dloss, *didx;
  const int nw = step_parts(batch);
  if (!w.init({{&P, kP}, {&G, kP}, {&dX, size_t(n) * kIn}, {&dY, size_t(n) * kOut},
               {&dM, size_t(n) * kOut}, {&m1, kP}, {&m2, kP}, {&part, size_t(nw) * kP},
               {&lossb, nw}, {&dloss, 1}, {&didx, n}}))
    return mfail(LTMP2_ENOMEM, "device allocation failed");
  if (hipMemcpyAsync(P, params, kP * sizeof(float), hipMemcpyHostToDevice, st) ||
      hipMemcpyAsync(dX, X, size_t(n) * kIn * sizeof(float), hipMemcpyHostToDevice, st) ||
      hipMemcpyAsync(dY, Y, size_t(n) * kOut * sizeof(float), hipMemcpyHostToDevice, st) ||
      hipMemcpyAsync(dM, M, size_t(n) * kOut * sizeof(float), hipMemcpyHostToDevice, st) ||
      hipMemsetAsync(m1, 0, kP * sizeof(float), st) || hipMemsetAsync(m2, 0, kP * sizeof(float), st))
    return mfail(LTMP2_EDEVICE, "copy failed");
  // unmasked outputs per sample (a minibatch's loss is a mean over them)
  std::vector<double> rows(n, 0.0);
  for (int b = 0; b < n; ++b)
    for (int k = 0; k < kOut; ++k) rows[b] += M[size_t(b) * kOut + k];
  uint64_t s = seed;
  std::vector<int> perm(n);
  long nstep = 0;
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  for (int ep = 0; ep < epochs; ++ep) {
    for (int k = 0; k < n; ++k) perm[k] = k;
    for (int k = n - 1; k > 0; --k) std::swap(perm[k], perm[int(uniform01(s) * (k + 1))]);
    // cosine learning-rate schedule
    const float lre = lr * 0.5f * (1.f + std::cos(float(M_PI) * ep / epochs));
    // the epoch's order in one copy; the copy back of the loss below keeps
    // perm unchanged until the stream is done with it
    if (hipMemsetAsync(dloss, 0, sizeof(float), st) ||
        hipMemcpyAsync(didx, perm.data(), size_t(n) * sizeof(int), hipMemcpyHostToDevice, st))
      return mfail(LTMP2_EDEVICE, "copy failed");
    double epoch_count = 0.0;
    for (int b0 = 0; b0 + batch <= n; b0 += batch) {
      double cnt = 0.0;
      for (int b = 0; b < batch; ++b) cnt += rows[perm[b0 + b]];
      epoch_count += cnt;
      ++nstep;
      const float bc1 = 1.f - std::pow(b1, float(nstep)), bc2 = 1.f - std::pow(b2, float(nstep));
      step(dX, dY, dM, reinterpret_cast<const int*>(didx) + b0, batch, float(1.0 / cnt), P, part,
           lossb, G, dloss, m1, m2, Adam{lre, b1, b2, eps, bc1, bc2}, st);
    }
    float l = 0.f;
    if (hipMemcpyAsync(&l, dloss, sizeof(float), hipMemcpyDeviceToHost, st) ||
        hipStreamSynchronize(st))
      return mfail(LTMP2_EDEVICE, "copy back failed");
    if (loss_hist) loss_hist[ep] = float(l / epoch_count);
  }
  if (hipGetLastError() != hipSuccess) return mfail(LTMP2_EDEVICE, "launch failed");
  if (hipMemcpyAsync(params, P, kP * sizeof(float), hipMemcpyDeviceToHost, st) ||
      hipStreamSynchronize(st))
    return mfail(LTMP2_EDEVICE, "copy back failed");
  return LTMP2_OK;
}

extern "C" ltmp2_status ltmp2_learned_quadrature(const float* params, double x_min, double x_max,
                                                 int n_tau, int polish_steps, double cert_tol,
                                                 double* tau, double* w, double* delta,
                                                 int* flags, void* stream) {
  if (!params || !tau || !w || n_tau < 1 || n_tau > 12 || !(x_min > 0) || !(x_max > x_min))
    return mfail(LTMP2_EINVAL, "bad arguments");
  float f[kIn], out[kOut];
  mlp_features(x_min, x_max, n_tau, f);
  ltmp2_status s = ltmp2_mlp_forward(params, f, 1, out, stream);
  if (s) return s;
  bool finite = true;
  for (int t = 0; t < n_tau; ++t) {
    tau[t] = std::exp(double(out[t])) / x_min;
    w[t] = std::exp(double(out[12 + t])) / x_min;
    finite = finite && std::isfinite(tau[t]) && std::isfinite(w[t]) && tau[t] > 0 && w[t] > 0;
  }
  int cert = 0;
  double d = 0.0;
  if (finite && remez_polish(x_min, x_max, n_tau, polish_steps, cert_tol, tau, w, &d, &cert) != 0)
    cert = 0;
  int fl = cert ? 1 : 0;
  if (!cert) {
    const int r = minimax_quadrature(x_min, x_max, n_tau, tau, w, &d);
    if (r != 0) return mfail(LTMP2_ENUMERIC, "fallback minimax fit failed");
    fl |= 2;
  }
  if (delta) *delta = d;
  if (flags) *flags = fl;
  return LTMP2_OK;
}

extern "C" ltmp2_status ltmp2_remez_polish(double x_min, double x_max, int n_tau, int steps,
                                           double cert_tol, double* tau, double* w, double* delta,
                                           int* certified) {
  if (!tau || !w) return mfail(LTMP2_EINVAL, "NULL array");
  if (remez_polish(x_min, x_max, n_tau, steps, cert_tol, tau, w, delta, certified) != 0)
    return mfail(LTMP2_EINVAL, "bad arguments");
  return LTMP2_OK;
}

extern "C" const char* ltmp2_mlp_last_error(void) { return mlp_last_error(); }
