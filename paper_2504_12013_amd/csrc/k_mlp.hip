// Learned temperature: a 16 -> 64 -> 64 -> 1 FP32 network (ReLU, ReLU, sigmoid) that maps level
// statistics to the temperature tau of a Jet round (the quantity the paper fixes by a schedule in
// Section 4.1 and studies in Section 7).  Inference, the backward pass and Adam run in the kernels
// below; every sum has a fixed order (no floating-point atomics), so training is reproducible.
//
// Flat parameter layout: W1[64][16] (row = hidden unit), b1[64], W2[64][64] (row = output unit),
// b2[64], w3[64], b3.  Inputs are raw features, standardised in the first kernel with the stored
// per-feature mean and standard deviation.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <string>
#include <vector>

#include "jet_internal.h"

namespace {

constexpr int kIn = 16, kH = 64;
constexpr int oW1 = 0, ob1 = oW1 + kH * kIn, oW2 = ob1 + kH, ob2 = oW2 + kH * kH, ow3 = ob2 + kH, ob3 = ow3 + kH;
constexpr int kParams = ob3 + 1;  // 5313
static_assert(kParams == JET_MLP_NPARAM, "parameter count");
constexpr int kFwdBlock = 256, kFwdWaves = kFwdBlock / 64;
constexpr unsigned kFwdGrid = 512;  // workgroups: each wave walks samples with its weights in registers

// value of `x` in lane `src` of the wave (constant src)
__device__ __forceinline__ float lane_value(float x, int src) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), src));
}

// One wave per sample, lane j = hidden unit j: forward, and with t the deltas dL/dz of every layer for
// L = mean over the batch of (y - t)^2.  A lane holds its rows of W1 and W2 in registers and takes the
// other lanes' activations by lane reads; every sum runs over its inputs in index order, as before (so
// do the batch sums below).  One thread per sample walked 5,184 products alone and left 252 of 256 CUs
// idle at a minibatch of 256; a wave per sample does both passes in 7 us.
template <bool KEEP>
__global__ __launch_bounds__(kFwdBlock) void k_mlp_forward(const float *__restrict__ theta,
                                                           const float *__restrict__ mean,
                                                           const float *__restrict__ stdv,
                                                           const float *__restrict__ X, const float *__restrict__ t,
                                                           int32_t B, float *__restrict__ xs, float *__restrict__ h1,
                                                           float *__restrict__ h2, float *__restrict__ y,
                                                           float *__restrict__ d1, float *__restrict__ d2,
                                                           float *__restrict__ d3) {
  const int j = threadIdx.x % 64;
  const int64_t waves = (int64_t)gridDim.x * kFwdWaves;
  float w1[kIn], w2[kH];
#pragma unroll
  for (int i = 0; i < kIn; i += 4) {
    const float4 q = *reinterpret_cast<const float4 *>(theta + oW1 + j * kIn + i);
    w1[i] = q.x;
    w1[i + 1] = q.y;
    w1[i + 2] = q.z;
    w1[i + 3] = q.w;
  }
#pragma unroll
  for (int i = 0; i < kH; i += 4) {
    const float4 q = *reinterpret_cast<const float4 *>(theta + oW2 + j * kH + i);
    w2[i] = q.x;
    w2[i + 1] = q.y;
    w2[i + 2] = q.z;
    w2[i + 3] = q.w;
  }
  const float b1 = theta[ob1 + j], b2 = theta[ob2 + j], w3 = theta[ow3 + j], b3 = theta[ob3];
  const float mu = j < kIn ? mean[j] : 0.0f, sd = j < kIn ? stdv[j] : 1.0f;
  for (int64_t s = (int64_t)blockIdx.x * kFwdWaves + threadIdx.x / 64; s < B; s += waves) {  // wave-uniform
    const float x = j < kIn ? (X[s * kIn + j] - mu) / sd : 0.0f;
    float z = b1;
#pragma unroll
    for (int i = 0; i < kIn; ++i) z += w1[i] * lane_value(x, i);
    const float a1 = z > 0.0f ? z : 0.0f;
    z = b2;
#pragma unroll
    for (int i = 0; i < kH; ++i) z += w2[i] * lane_value(a1, i);
    const float a2 = z > 0.0f ? z : 0.0f;
    float z3 = b3;
#pragma unroll
    for (int i = 0; i < kH; ++i) z3 += lane_value(w3, i) * lane_value(a2, i);
    const float ys = 1.0f / (1.0f + expf(-z3));
    if (j == 0) y[s] = ys;
    if (!KEEP) continue;
    if (j < kIn) xs[s * kIn + j] = x;
    h1[s * kH + j] = a1;
    h2[s * kH + j] = a2;
    const float dy = 2.0f * (ys - t[s]) / (float)B;
    const float g3 = dy * ys * (1.0f - ys);
    if (j == 0) d3[s] = g3;
    const float g2 = a2 > 0.0f ? g3 * w3 : 0.0f;
    d2[s * kH + j] = g2;
    float acc = 0.0f;
#pragma unroll
    for (int i = 0; i < kH; ++i) acc += lane_value(g2, i) * theta[oW2 + i * kH + j];
    d1[s * kH + j] = a1 > 0.0f ? acc : 0.0f;
  }
}

// sum over the batch, in sample order, of f(s, 0) * f(s, 1): the loads of kBatchU samples in flight
constexpr int kBatchU = 32;
template <typename F>
__device__ __forceinline__ float batch_sum(int32_t B, F f) {
  float acc = 0.0f;
  int32_t s = 0;
  for (; s + kBatchU <= B; s += kBatchU) {
    float a[kBatchU], b[kBatchU];
#pragma unroll
    for (int u = 0; u < kBatchU; ++u) f(s + u, a[u], b[u]);
#pragma unroll
    for (int u = 0; u < kBatchU; ++u) acc += a[u] * b[u];
  }
  for (; s < B; ++s) {
    float a, b;
    f(s, a, b);
    acc += a * b;
  }
  return acc;
}

struct AdamArgs {  // Adam (Kingma and Ba, Algorithm 1); c1 = 1/(1-beta1^t), c2 = 1/(1-beta2^t) from the host
  float *theta, *m, *v;  // theta == nullptr: gradient only
  float lr, beta1, beta2, eps, c1, c2;
};

// One thread per parameter (plus one for the loss): the batch sum in sample order, then the
// parameter's Adam step.  64-thread workgroups: 84 of them, one per CU.  Bound by the chain of
// batch-length additions, with the loads of 32 samples in flight: 13 us for 256 samples.  The whole
// training step (256 samples, loss back on the host) went from 202 to 58 us.
__global__ __launch_bounds__(64) void k_mlp_wgrad(const float *__restrict__ xs, const float *__restrict__ h1,
                                                  const float *__restrict__ h2, const float *__restrict__ y,
                                                  const float *__restrict__ t, const float *__restrict__ d1,
                                                  const float *__restrict__ d2, const float *__restrict__ d3,
                                                  int32_t B, float *__restrict__ grad, float *__restrict__ loss,
                                                  AdamArgs ad) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p > kParams) return;
  if (p == kParams) {  // the loss itself
    const float acc = batch_sum(B, [&](int32_t s, float &a, float &b) { a = b = y[s] - t[s]; });
    *loss = acc / (float)B;
    return;
  }
  // the two factors of the parameter's gradient: row lengths and columns (a bias has the factor 1)
  const float *fa, *fb = nullptr;
  int na = kH, nb = kH, ja = 0, jb = 0;
  if (p < ob1) {
    fa = d1;
    fb = xs;
    nb = kIn;
    ja = (p - oW1) / kIn;
    jb = (p - oW1) % kIn;
  } else if (p < oW2) {
    fa = d1;
    ja = p - ob1;
  } else if (p < ob2) {
    fa = d2;
    fb = h1;
    ja = (p - oW2) / kH;
    jb = (p - oW2) % kH;
  } else if (p < ow3) {
    fa = d2;
    ja = p - ob2;
  } else if (p < ob3) {
    fa = d3;
    na = 1;
    fb = h2;
    jb = p - ow3;
  } else {
    fa = d3;
    na = 1;
  }
  const float gp = batch_sum(B, [&](int32_t s, float &a, float &b) {
    a = fa[(int64_t)s * na + ja];
    b = fb ? fb[(int64_t)s * nb + jb] : 1.0f;
  });
  grad[p] = gp;
  if (!ad.theta) return;
  const float mp = ad.beta1 * ad.m[p] + (1.0f - ad.beta1) * gp;
  const float vp = ad.beta2 * ad.v[p] + (1.0f - ad.beta2) * gp * gp;
  ad.m[p] = mp;
  ad.v[p] = vp;
  ad.theta[p] = ad.theta[p] - ad.lr * (mp * ad.c1) / (sqrtf(vp * ad.c2) + ad.eps);
}

// SplitMix64 (Steele, Lea and Flood, OOPSLA 2014) for the seeded initialisation.
uint64_t splitmix(uint64_t &s) {
  uint64_t z = (s += 0x9E3779B97F4A7C15ULL);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
  return z ^ (z >> 31);
}

thread_local std::string g_mlp_error;

}  // namespace

struct jet_mlp {
  hipStream_t stream = nullptr;
  float *theta = nullptr, *m = nullptr, *v = nullptr, *grad = nullptr, *mean = nullptr, *stdv = nullptr;
  float *loss = nullptr;  // pinned host memory, written by the gradient kernel
  int64_t step = 0;
  int32_t cap = 0;  // batch capacity of the activation buffers
  float *xs = nullptr, *h1 = nullptr, *h2 = nullptr, *y = nullptr, *d1 = nullptr, *d2 = nullptr, *d3 = nullptr;
  std::string last_error;
};

namespace {

int mlp_fail(jet_mlp *net, int code, const std::string &msg) {
  if (net) net->last_error = msg;
  else g_mlp_error = msg;
  return code;
}

#define MLP_HIP(net, expr)                                                                   \
  do {                                                                                       \
    hipError_t _e = (expr);                                                                  \
    if (_e != hipSuccess) return mlp_fail(net, JET_EHIP, std::string(#expr) + ": " + hipGetErrorString(_e)); \
  } while (0)

void free_batch(jet_mlp *net) {
  float *ptrs[] = {net->xs, net->h1, net->h2, net->y, net->d1, net->d2, net->d3};
  for (float *p : ptrs)
    if (p) (void)hipFree(p);
  net->xs = net->h1 = net->h2 = net->y = net->d1 = net->d2 = net->d3 = nullptr;
  net->cap = 0;
}

int ensure_batch(jet_mlp *net, int32_t B) {
  if (B <= net->cap) return JET_OK;
  MLP_HIP(net, hipStreamSynchronize(net->stream));
  free_batch(net);
  const size_t b = (size_t)B;
  if (hipMalloc((void **)&net->xs, sizeof(float) * b * kIn) != hipSuccess ||
      hipMalloc((void **)&net->h1, sizeof(float) * b * kH) != hipSuccess ||
      hipMalloc((void **)&net->h2, sizeof(float) * b * kH) != hipSuccess ||
      hipMalloc((void **)&net->y, sizeof(float) * b) != hipSuccess ||
      hipMalloc((void **)&net->d1, sizeof(float) * b * kH) != hipSuccess ||
      hipMalloc((void **)&net->d2, sizeof(float) * b * kH) != hipSuccess ||
      hipMalloc((void **)&net->d3, sizeof(float) * b) != hipSuccess) {
    free_batch(net);
    return mlp_fail(net, JET_ENOMEM, "activation buffers");
  }
  net->cap = B;
  return JET_OK;
}

unsigned blocks_for(int64_t n, int block) { return (unsigned)((n + block - 1) / block); }
unsigned forward_grid(int32_t B) { return std::min(kFwdGrid, blocks_for(B, kFwdWaves)); }

int forward_into(jet_mlp *net, const float *X, int32_t B, float *y) {
  hipLaunchKernelGGL(k_mlp_forward<false>, dim3(forward_grid(B)), dim3(kFwdBlock), 0, net->stream, net->theta,
                     net->mean, net->stdv, X, nullptr, B, nullptr, nullptr, nullptr, y, nullptr, nullptr, nullptr);
  MLP_HIP(net, hipGetLastError());
  return JET_OK;
}

// Gradient into grad, and with ad.theta the Adam step; the loss to the host.
int grad_impl(jet_mlp *net, const float *X, const float *t, int32_t B, float *grad, float *loss, const AdamArgs &ad) {
  if (!net || !X || !t || !grad || B < 1) return mlp_fail(net, JET_EINVAL, "bad gradient arguments");
  int rc = ensure_batch(net, B);
  if (rc != JET_OK) return rc;
  hipLaunchKernelGGL(k_mlp_forward<true>, dim3(forward_grid(B)), dim3(kFwdBlock), 0, net->stream, net->theta,
                     net->mean, net->stdv, X, t, B, net->xs, net->h1, net->h2, net->y, net->d1, net->d2, net->d3);
  hipLaunchKernelGGL(k_mlp_wgrad, dim3(blocks_for(kParams + 1, 64)), dim3(64), 0, net->stream, net->xs, net->h1,
                     net->h2, net->y, t, net->d1, net->d2, net->d3, B, grad, net->loss, ad);
  MLP_HIP(net, hipGetLastError());
  if (loss) {
    MLP_HIP(net, hipStreamSynchronize(net->stream));
    *loss = *net->loss;
  }
  return JET_OK;
}

}  // namespace

namespace jet {

int mlp_infer_one(jet_mlp *net, const float *x, float *y, float *tau) {
  int rc = forward_into(net, x, 1, y);
  if (rc != JET_OK) return rc;
  MLP_HIP(net, hipMemcpyAsync(tau, y, sizeof(float), hipMemcpyDeviceToHost, net->stream));
  MLP_HIP(net, hipStreamSynchronize(net->stream));
  return JET_OK;
}

}  // namespace jet

extern "C" {

int jet_mlp_create(jet_mlp **out, uint64_t seed, void *stream) {
  if (!out) return mlp_fail(nullptr, JET_EINVAL, "out is NULL");
  *out = nullptr;
  jet_mlp *net = new jet_mlp();
  net->stream = (hipStream_t)stream;
  float **bufs[] = {&net->theta, &net->m, &net->v, &net->grad};
  for (float **b : bufs)
    if (hipMalloc((void **)b, sizeof(float) * kParams) != hipSuccess) {
      jet_mlp_free(net);
      return mlp_fail(nullptr, JET_ENOMEM, "parameter buffers");
    }
  if (hipMalloc((void **)&net->mean, sizeof(float) * kIn) != hipSuccess ||
      hipMalloc((void **)&net->stdv, sizeof(float) * kIn) != hipSuccess ||
      hipHostMalloc((void **)&net->loss, sizeof(float)) != hipSuccess) {
    jet_mlp_free(net);
    return mlp_fail(nullptr, JET_ENOMEM, "parameter buffers");
  }
  // He-uniform weights U(-sqrt(6/fan_in), sqrt(6/fan_in)), zero biases, identity standardisation
  std::vector<float> th(kParams, 0.0f), mean(kIn, 0.0f), sd(kIn, 1.0f);
  uint64_t s = seed;
  auto fill = [&](int o, int count, int fan_in) {
    const double a = sqrt(6.0 / fan_in);
    for (int i = 0; i < count; ++i) {
      const double u = (double)(splitmix(s) >> 11) * (1.0 / 9007199254740992.0);  // [0, 1)
      th[o + i] = (float)((2.0 * u - 1.0) * a);
    }
  };
  fill(oW1, kH * kIn, kIn);
  fill(oW2, kH * kH, kH);
  fill(ow3, kH, kH);
  int rc = jet_mlp_set(net, th.data(), mean.data(), sd.data());
  if (rc != JET_OK) {
    jet_mlp_free(net);
    return rc;
  }
  *out = net;
  return JET_OK;
}

int jet_mlp_set(jet_mlp *net, const float *params, const float *mean, const float *stdv) {
  if (!net) return JET_EINVAL;
  if (stdv)
    for (int i = 0; i < kIn; ++i)
      if (!(stdv[i] > 0.0f)) return mlp_fail(net, JET_EINVAL, "standard deviation must be > 0");
  MLP_HIP(net, hipStreamSynchronize(net->stream));
  if (params) {
    MLP_HIP(net, hipMemcpy(net->theta, params, sizeof(float) * kParams, hipMemcpyHostToDevice));
    MLP_HIP(net, hipMemset(net->m, 0, sizeof(float) * kParams));
    MLP_HIP(net, hipMemset(net->v, 0, sizeof(float) * kParams));
    net->step = 0;
  }
  if (mean) MLP_HIP(net, hipMemcpy(net->mean, mean, sizeof(float) * kIn, hipMemcpyHostToDevice));
  if (stdv) MLP_HIP(net, hipMemcpy(net->stdv, stdv, sizeof(float) * kIn, hipMemcpyHostToDevice));
  return JET_OK;
}

int jet_mlp_get(jet_mlp *net, float *params, float *mean, float *stdv) {
  if (!net) return JET_EINVAL;
  MLP_HIP(net, hipStreamSynchronize(net->stream));
  if (params) MLP_HIP(net, hipMemcpy(params, net->theta, sizeof(float) * kParams, hipMemcpyDeviceToHost));
  if (mean) MLP_HIP(net, hipMemcpy(mean, net->mean, sizeof(float) * kIn, hipMemcpyDeviceToHost));
  if (stdv) MLP_HIP(net, hipMemcpy(stdv, net->stdv, sizeof(float) * kIn, hipMemcpyDeviceToHost));
  return JET_OK;
}

int jet_mlp_forward(jet_mlp *net, const float *X, int32_t B, float *tau) {
  if (!net || !X || !tau || B < 1) return mlp_fail(net, JET_EINVAL, "bad forward arguments");
  return forward_into(net, X, B, tau);
}

int jet_mlp_grad(jet_mlp *net, const float *X, const float *t, int32_t B, float *grad, float *loss) {
  return grad_impl(net, X, t, B, grad, loss, AdamArgs{});
}

int jet_mlp_train_step(jet_mlp *net, const float *X, const float *t, int32_t B, float lr, float *loss) {
  if (!net) return JET_EINVAL;
  if (!(lr > 0.0f)) return mlp_fail(net, JET_EINVAL, "learning rate must be > 0");
  const double b1 = 0.9, b2 = 0.999;
  const double at = (double)(net->step + 1);
  const AdamArgs ad{net->theta, net->m,      net->v, lr, (float)b1, (float)b2, 1e-8f, (float)(1.0 / (1.0 - pow(b1, at))),
                    (float)(1.0 / (1.0 - pow(b2, at)))};
  const int rc = grad_impl(net, X, t, B, net->grad, loss, ad);
  if (rc == JET_OK) net->step += 1;
  return rc;
}

int jet_mlp_save(jet_mlp *net, const char *path) {
  if (!net || !path) return JET_EINVAL;
  std::vector<float> buf(kParams + 2 * kIn);
  int rc = jet_mlp_get(net, buf.data(), buf.data() + kParams, buf.data() + kParams + kIn);
  if (rc != JET_OK) return rc;
  FILE *f = fopen(path, "wb");
  if (!f) return mlp_fail(net, JET_EINVAL, std::string("cannot open ") + path);
  const uint32_t head[2] = {0x4d4c5054u /* "TPLM" */, (uint32_t)kParams};
  bool ok = fwrite(head, sizeof head, 1, f) == 1 && fwrite(buf.data(), sizeof(float), buf.size(), f) == buf.size();
  ok = (fclose(f) == 0) && ok;
  return ok ? JET_OK : mlp_fail(net, JET_EINVAL, std::string("cannot write ") + path);
}

int jet_mlp_load(jet_mlp *net, const char *path) {
  if (!net || !path) return JET_EINVAL;
  FILE *f = fopen(path, "rb");
  if (!f) return mlp_fail(net, JET_EINVAL, std::string("cannot open ") + path);
  uint32_t head[2] = {0, 0};
  std::vector<float> buf(kParams + 2 * kIn);
  const bool ok = fread(head, sizeof head, 1, f) == 1 && head[0] == 0x4d4c5054u && head[1] == (uint32_t)kParams &&
                  fread(buf.data(), sizeof(float), buf.size(), f) == buf.size();
  fclose(f);
  if (!ok) return mlp_fail(net, JET_EINVAL, std::string("not a temperature network file: ") + path);
  return jet_mlp_set(net, buf.data(), buf.data() + kParams, buf.data() + kParams + kIn);
}

int jet_mlp_free(jet_mlp *net) {
  if (!net) return JET_OK;
  if (net->stream) (void)hipStreamSynchronize(net->stream);
  free_batch(net);
  float *ptrs[] = {net->theta, net->m, net->v, net->grad, net->mean, net->stdv};
  for (float *p : ptrs)
    if (p) (void)hipFree(p);
  if (net->loss) (void)hipHostFree(net->loss);
  delete net;
  return JET_OK;
}

const char *jet_mlp_last_error(const jet_mlp *net) { return net ? net->last_error.c_str() : g_mlp_error.c_str(); }

}  // extern "C"
