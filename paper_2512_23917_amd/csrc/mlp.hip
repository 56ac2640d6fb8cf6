// Sketch-rank model: a 35 -> 128 -> 128 -> 1 perceptron with exact GELU that
// predicts log2 chi*(eps) of a bond from its previous spectrum, trained on
// the GPU with hand-written forward, backward (pinball loss, tau = 0.9) and
// Adam kernels.  FP32 parameters and arithmetic.
//
// Flat parameter layout: W1 (128 x 35, row-major), b1 (128), W2 (128 x 128),
// b2 (128), W3 (1 x 128), b3 (1).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "../../include/tci_c.h"
#include "common.hpp"
#include "runtime.hpp"

struct tci_sketch_model_s {
  float* params = nullptr;  // device, N_PARAMS
  float* m = nullptr;       // Adam first moment
  float* v = nullptr;       // Adam second moment
  int64_t step = 0;
  tci_allocator al{};       // allocator of the three buffers (the creating context's)
  uint32_t magic = 0x5C37C4u;
};

namespace tci {

constexpr int NI = 35, NH = 128;
constexpr int OFF_W1 = 0, OFF_B1 = NH * NI, OFF_W2 = OFF_B1 + NH, OFF_B2 = OFF_W2 + NH * NH, OFF_W3 = OFF_B2 + NH,
              OFF_B3 = OFF_W3 + NH, NPARAM = OFF_B3 + 1;
constexpr float TAU = 0.9f;

__device__ inline void philox_round_m(uint32_t c[4], const uint32_t k[2]) {
  const uint64_t p0 = (uint64_t)0xD2511F53u * c[0];
  const uint64_t p1 = (uint64_t)0xCD9E8D57u * c[2];
  const uint32_t n0 = (uint32_t)(p1 >> 32) ^ c[1] ^ k[0];
  const uint32_t n2 = (uint32_t)(p0 >> 32) ^ c[3] ^ k[1];
  c[1] = (uint32_t)p1;
  c[3] = (uint32_t)p0;
  c[0] = n0;
  c[2] = n2;
}

// He-uniform initialisation: uniform u_e = (x_e + 0.5) 2^-32 with x_e the e-th
// 32-bit output of Philox4x32-10 (key = seed, stream 7); W = (2u - 1) sqrt(6 / fan_in).
__global__ void mlp_init_kernel(float* p, uint64_t seed) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;  // index over weights only
  const int nw = NH * NI + NH * NH + NH;
  if (e >= nw) return;
  uint32_t c[4] = {(uint32_t)(e >> 2), 0u, 7u, 0u};
  uint32_t k[2] = {(uint32_t)seed, (uint32_t)(seed >> 32)};
  for (int r = 0; r < 10; ++r) {
    philox_round_m(c, k);
    k[0] += 0x9E3779B9u;
    k[1] += 0xBB67AE85u;
  }
  const double u = ((double)c[e & 3] + 0.5) * 2.3283064365386963e-10;
  if (e < NH * NI) {
    p[OFF_W1 + e] = (float)((2.0 * u - 1.0) * sqrt(6.0 / NI));
  } else if (e < NH * NI + NH * NH) {
    p[OFF_W2 + (e - NH * NI)] = (float)((2.0 * u - 1.0) * sqrt(6.0 / NH));
  } else {
    p[OFF_W3 + (e - NH * NI - NH * NH)] = (float)((2.0 * u - 1.0) * sqrt(6.0 / NH));
  }
}

__device__ inline float gelu(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }
__device__ inline float gelu_d(float x) {
  return 0.5f * (1.0f + erff(x * 0.70710678118654752f)) + x * expf(-0.5f * x * x) * 0.3989422804014327f;
}

// Forward of SPB samples per workgroup (128 threads, thread j = hidden unit j)
// and, when `grad` is set, the backward pass down to the units' derivatives:
// rows s of h1, g2, g1, h2 (n x 128) and gy, loss (n).  With few samples a
// workgroup per sample spreads them over the chip; with many, SPB samples
// share each read of the weights.  W2's row of a thread is read four at a time.
struct MlpWork {
  float *h1, *g2, *g1, *h2, *gy, *loss;
};

template <int SPB>
__global__ __launch_bounds__(128) void mlp_sample_kernel(const float* __restrict__ p, const float* __restrict__ X,
                                                         const float* __restrict__ T, int n, float* y, MlpWork w,
                                                         bool grad) {
  __shared__ float x[SPB][NI], h1[SPB][NH], g2[SPB][NH], red[SPB][2];
  const int s0 = blockIdx.x * SPB, j = threadIdx.x;
  for (int e = j; e < SPB * NI; e += NH) x[e / NI][e % NI] = s0 + e / NI < n ? X[(long long)s0 * NI + e] : 0.f;
  __syncthreads();
  float a[SPB], b[SPB], h2[SPB];
#pragma unroll
  for (int q = 0; q < SPB; ++q) a[q] = p[OFF_B1 + j];
#pragma unroll 5
  for (int i = 0; i < NI; ++i) {
    const float wv = p[OFF_W1 + j * NI + i];
#pragma unroll
    for (int q = 0; q < SPB; ++q) a[q] += wv * x[q][i];
  }
#pragma unroll
  for (int q = 0; q < SPB; ++q) {
    h1[q][j] = gelu(a[q]);
    b[q] = p[OFF_B2 + j];
  }
  __syncthreads();
  static_assert(OFF_W2 % 4 == 0 && NH % 4 == 0, "16-byte rows of W2");
  const float4* w2 = reinterpret_cast<const float4*>(p + OFF_W2 + j * NH);
#pragma unroll 8
  for (int i = 0; i < NH / 4; ++i) {
    const float4 v = w2[i];
#pragma unroll
    for (int q = 0; q < SPB; ++q) {
      b[q] += v.x * h1[q][4 * i];
      b[q] += v.y * h1[q][4 * i + 1];
      b[q] += v.z * h1[q][4 * i + 2];
      b[q] += v.w * h1[q][4 * i + 3];
    }
  }
  const float w3 = p[OFF_W3 + j];
#pragma unroll
  for (int q = 0; q < SPB; ++q) {
    h2[q] = gelu(b[q]);
    float c = w3 * h2[q];
    for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off, 64);
    if ((j & 63) == 0) red[q][j >> 6] = c;
  }
  __syncthreads();
  if (!grad) {
    if (j < SPB && s0 + j < n) y[s0 + j] = red[j][0] + red[j][1] + p[OFF_B3];
    return;
  }
  // d loss / d y of the mean pinball loss, then the units' derivatives
#pragma unroll
  for (int q = 0; q < SPB; ++q) {
    const int s = s0 + q;
    const float u = s < n ? T[s] - (red[q][0] + red[q][1] + p[OFF_B3]) : 0.f;
    const float gy = (u < 0.f ? (1.f - TAU) : -TAU) / (float)n;
    g2[q][j] = gy * w3 * gelu_d(b[q]);
    if (s < n) {
      w.h1[(long long)s * NH + j] = h1[q][j];
      w.h2[(long long)s * NH + j] = h2[q];
      w.g2[(long long)s * NH + j] = g2[q][j];
      if (j == 0) {
        w.gy[s] = gy;
        w.loss[s] = fmaxf(TAU * u, (TAU - 1.f) * u) / (float)n;
      }
    }
  }
  __syncthreads();
  float gh[SPB] = {};
#pragma unroll 8
  for (int r = 0; r < NH; ++r) {
    const float wv = p[OFF_W2 + r * NH + j];
#pragma unroll
    for (int q = 0; q < SPB; ++q) gh[q] += g2[q][r] * wv;
  }
#pragma unroll
  for (int q = 0; q < SPB; ++q)
    if (s0 + q < n) w.g1[(long long)(s0 + q) * NH + j] = gh[q] * gelu_d(a[q]);
}

// Weight gradients as products over the samples: dW2 = g2^T [h1 | 1] (its last
// column is db2), dW1 = g1^T [x | 1], dW3 = gy^T [h2 | 1], in 16 x 16 tiles, one
// element per thread; the block after the tiles sums the losses.  An element is
// summed over the samples in order, products rounded before the sum, so that
// a batch of thousands keeps the rounding of a plain loop; the bound is that
// chain and the LDS reads (one 16-byte read of each operand per four samples),
// with the next stage's loads in flight.  Gradient and prediction of 256 / 16384
// samples: 142 / 4700 us with a gradient row of 21249 values (85 KB) per sample
// summed by one thread per value, 61 / 219 us in chunks of samples with a kernel
// that adds their sums (other rounding than the loop's by 3.8e-5 of the norm at
// 16384), 55 / 329 us in order.
constexpr int MLP_STAGE = 64, MLP_TW = 16, MLP_PITCH = MLP_STAGE + 4;
constexpr int MLP_T2 = (NH / MLP_TW) * (NH / MLP_TW + 1), MLP_C1 = (NI + MLP_TW) / MLP_TW,
              MLP_T1 = (NH / MLP_TW) * MLP_C1, MLP_T3 = NH / MLP_TW + 1, MLP_TILES = MLP_T2 + MLP_T1 + MLP_T3;

__global__ __launch_bounds__(256) void mlp_grad_kernel(const float* __restrict__ X, int n, MlpWork w,
                                                       float* __restrict__ grad, float* __restrict__ loss_total) {
  __shared__ __attribute__((aligned(16))) float As[2][MLP_TW][MLP_PITCH], Bs[2][MLP_TW][MLP_PITCH];
  const int t = blockIdx.x, tid = threadIdx.x, ti = tid >> 4, tj = tid & 15;
  if (t == MLP_TILES) {
    __shared__ float red[4];
    float l = 0.f;
    for (int s = tid; s < n; s += 256) l += w.loss[s];
    l = wave_sum(l);
    if ((tid & 63) == 0) red[tid >> 6] = l;
    __syncthreads();
    if (tid == 0) *loss_total = red[0] + red[1] + red[2] + red[3];
    return;
  }
  // operands (rows = samples) with their widths, and the flat offsets of the weights and the bias
  const float *A, *B;
  int wa, wb, rt, ct, offw, offb;
  if (t < MLP_T2) {
    A = w.g2; B = w.h1; wa = NH; wb = NH; rt = t / (NH / MLP_TW + 1); ct = t % (NH / MLP_TW + 1);
    offw = OFF_W2; offb = OFF_B2;
  } else if (t < MLP_T2 + MLP_T1) {
    A = w.g1; B = X; wa = NH; wb = NI; rt = (t - MLP_T2) / MLP_C1; ct = (t - MLP_T2) % MLP_C1;
    offw = OFF_W1; offb = OFF_B1;
  } else {
    A = w.gy; B = w.h2; wa = 1; wb = NH; rt = 0; ct = t - MLP_T2 - MLP_T1; offw = OFF_W3; offb = OFF_B3;
  }
  const int r0 = MLP_TW * rt, c0 = MLP_TW * ct;
  constexpr int PER = MLP_STAGE * MLP_TW / 256;
  float la[PER], lb[PER];
  auto load = [&](int s0) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int e = tid + 256 * u, c = e & 15, s = s0 + (e >> 4), sc = min(s, n - 1);
      const float va = A[(long long)sc * wa + min(r0 + c, wa - 1)], vb = B[(long long)sc * wb + min(c0 + c, wb - 1)];
      la[u] = s < n && r0 + c < wa ? va : 0.f;
      lb[u] = s >= n || c0 + c > wb ? 0.f : c0 + c == wb ? 1.f : vb;
    }
  };
  load(0);
  float acc = 0.f;
  for (int s0 = 0, st = 0; s0 < n; s0 += MLP_STAGE, st ^= 1) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int e = tid + 256 * u;
      As[st][e & 15][e >> 4] = la[u];
      Bs[st][e & 15][e >> 4] = lb[u];
    }
    // one barrier per stage: the other buffer's readers are past theirs
    __syncthreads();
    load(s0 + MLP_STAGE);
#pragma unroll
    for (int k = 0; k < MLP_STAGE; k += 4) {
      const float4 x = *reinterpret_cast<const float4*>(&As[st][ti][k]), y = *reinterpret_cast<const float4*>(&Bs[st][tj][k]);
      acc = __fadd_rn(acc, __fmul_rn(x.x, y.x));
      acc = __fadd_rn(acc, __fmul_rn(x.y, y.y));
      acc = __fadd_rn(acc, __fmul_rn(x.z, y.z));
      acc = __fadd_rn(acc, __fmul_rn(x.w, y.w));
    }
  }
  const int r = r0 + ti, c = c0 + tj;
  if (r < wa && c < wb) grad[offw + r * wb + c] = acc;
  else if (r < wa && c == wb) grad[offb + r] = acc;
}

__global__ void adam_kernel(float* p, float* m, float* v, const float* g, float lr, float b1, float b2, float eps,
                            float c1, float c2) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= NPARAM) return;
  const float gq = g[q];
  const float mq = b1 * m[q] + (1.f - b1) * gq;
  const float vq = b2 * v[q] + (1.f - b2) * gq * gq;
  m[q] = mq;
  v[q] = vq;
  p[q] -= lr * (mq / c1) / (sqrtf(vq / c2) + eps);
}

// Features of one bond per thread: [log2 chi_max / 11, d / 4, -log10 eps / 16,
// 32 clamped log10 quantiles of the previous spectrum s (descending, length len[b])].
__global__ void features_kernel(const double* s, long long ss, const int* len, int chi_max, int d, double eps,
                                float* X, int n) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= n) return;
  const double* sb = s + b * ss;
  const int L = len[b];
  float* x = X + (long long)b * NI;
  x[0] = (float)(log2((double)chi_max) / 11.0);
  x[1] = (float)(d / 4.0);
  x[2] = (float)(-log10(eps) / 16.0);
  for (int t = 0; t < 32; ++t) {
    const int j = L > 1 ? (int)floor((t + 0.5) / 32.0 * (L - 1)) : 0;
    double q = -1.0;
    if (L > 0 && sb[0] > 0.0 && sb[j] > 0.0) q = log10(sb[j] / sb[0]) / 16.0;
    x[3 + t] = (float)fmin(0.0, fmax(-1.0, q));
  }
}

static tci_status model_check(tci_sketch_model m) {
  if (!m || m->magic != 0x5C37C4u) TCI_RET(TCI_ERR_INVALID_ARGUMENT, "invalid sketch model");
  return TCI_OK;
}

// One sample per workgroup up to two per compute unit, four above.
static void mlp_samples(const float* p, const float* X, const float* T, int n, float* y, const MlpWork& w, bool grad,
                        hipStream_t s) {
  if (n <= 512) hipLaunchKernelGGL(mlp_sample_kernel<1>, dim3(n), dim3(NH), 0, s, p, X, T, n, y, w, grad);
  else hipLaunchKernelGGL(mlp_sample_kernel<4>, dim3((n + 3) / 4), dim3(NH), 0, s, p, X, T, n, y, w, grad);
}

static tci_status grads_impl(tci_context ctx, tci_sketch_model m, const float* X, const float* T, int n, float* grad,
                             float* loss_dev) {
  hipStream_t s = ctx->stream;
  float* rows = static_cast<float*>(ctx->arena.get(sizeof(float) * (size_t)n * (4 * NH + 2)));
  if (!rows) TCI_RET(TCI_ERR_OUT_OF_MEMORY, "mlp workspace");
  const size_t nh = (size_t)n * NH;
  const MlpWork w{rows, rows + nh, rows + 2 * nh, rows + 3 * nh, rows + 4 * nh, rows + 4 * nh + n};
  mlp_samples(m->params, X, T, n, nullptr, w, true, s);
  hipLaunchKernelGGL(mlp_grad_kernel, dim3(MLP_TILES + 1), dim3(256), 0, s, X, n, w, grad, loss_dev);
  TCI_CHECK_HIP(hipGetLastError());
  return TCI_OK;
}

int sketch_model_nparams() { return NPARAM; }

tci_status sketch_predict_dev(tci_context ctx, tci_sketch_model m, const float* X, int n, float* y) {
  TCI_TRY(model_check(m));
  if (n <= 0) return TCI_OK;
  mlp_samples(m->params, X, nullptr, n, y, MlpWork{}, false, ctx->stream);
  TCI_CHECK_HIP(hipGetLastError());
  return TCI_OK;
}

tci_status sketch_features_dev(tci_context ctx, const double* s, long long ss, const int* len, int chi_max, int d,
                               double eps, float* X, int n) {
  hipLaunchKernelGGL(features_kernel, dim3((n + 63) / 64), dim3(64), 0, ctx->stream, s, ss, len, chi_max, d, eps, X, n);
  TCI_CHECK_HIP(hipGetLastError());
  return TCI_OK;
}

}  // namespace tci

using namespace tci;

extern "C" {

tci_status tci_sketch_model_create(tci_context ctx, uint64_t seed, tci_sketch_model* out) try {
  if (!ctx || !out) TCI_RET(TCI_ERR_INVALID_ARGUMENT, "null argument");
  TCI_CHECK_HIP(hipSetDevice(ctx->device));
  auto* m = new tci_sketch_model_s();
  const size_t bytes = sizeof(float) * NPARAM;
  m->al = ctx->al;
  m->params = static_cast<float*>(dev_alloc(m->al, bytes, ctx->stream));
  m->m = static_cast<float*>(dev_alloc(m->al, bytes, ctx->stream));
  m->v = static_cast<float*>(dev_alloc(m->al, bytes, ctx->stream));
  if (!m->params || !m->m || !m->v) {
    dev_free(m->al, m->params, bytes, ctx->stream);
    dev_free(m->al, m->m, bytes, ctx->stream);
    dev_free(m->al, m->v, bytes, ctx->stream);
    delete m;
    TCI_RET(TCI_ERR_OUT_OF_MEMORY, "model allocation");
  }
  TCI_CHECK_HIP(hipMemsetAsync(m->params, 0, bytes, ctx->stream));
  TCI_CHECK_HIP(hipMemsetAsync(m->m, 0, bytes, ctx->stream));
  TCI_CHECK_HIP(hipMemsetAsync(m->v, 0, bytes, ctx->stream));
  const int nw = NH * NI + NH * NH + NH;
  hipLaunchKernelGGL(mlp_init_kernel, dim3((nw + 255) / 256), dim3(256), 0, ctx->stream, m->params, seed);
  TCI_CHECK_HIP(hipGetLastError());
  TCI_CHECK_HIP(hipStreamSynchronize(ctx->stream));
  *out = m;
  return TCI_OK;
} TCI_API_CATCH

tci_status tci_sketch_model_destroy(tci_context ctx, tci_sketch_model m) try {
  if (!m) return TCI_OK;
  if (ctx) (void)hipStreamSynchronize(ctx->stream);
  const size_t bytes = sizeof(float) * NPARAM;
  hipStream_t st = ctx ? ctx->stream : nullptr;
  dev_free(m->al, m->params, bytes, st);
  dev_free(m->al, m->m, bytes, st);
  dev_free(m->al, m->v, bytes, st);
  m->magic = 0;
  delete m;
  return TCI_OK;
} TCI_API_CATCH

int64_t tci_sketch_model_nparams(void) { return NPARAM; }

tci_status tci_sketch_model_get_params(tci_context ctx, tci_sketch_model m, float* host, int64_t n) try {
  if (!ctx || !host) TCI_RET(TCI_ERR_INVALID_ARGUMENT, "null argument");
  TCI_TRY(model_check(m));
  if (n != NPARAM) TCI_RET(TCI_ERR_SHAPE, "parameter count");
  TCI_CHECK_HIP(hipMemcpyAsync(host, m->params, sizeof(float) * NPARAM, hipMemcpyDeviceToHost, ctx->stream));
  TCI_CHECK_HIP(hipStreamSynchronize(ctx->stream));
  return TCI_OK;
} TCI_API_CATCH

tci_status tci_sketch_model_set_params(tci_context ctx, tci_sketch_model m, const float* host, int64_t n) try {
  if (!ctx || !host) TCI_RET(TCI_ERR_INVALID_ARGUMENT, "null argument");
  TCI_TRY(model_check(m));
  if (n != NPARAM) TCI_RET(TCI_ERR_SHAPE, "parameter count");
  TCI_CHECK_HIP(hipMemcpyAsync(m->params, host, sizeof(float) * NPARAM, hipMemcpyHostToDevice, ctx->stream));
  TCI_CHECK_HIP(hipStreamSynchronize(ctx->stream));
  return TCI_OK;
} TCI_API_CATCH

tci_status tci_sketch_model_save(tci_context ctx, tci_sketch_model m, const char* path) try {
  if (!path) TCI_RET(TCI_ERR_INVALID_ARGUMENT, "null path");
  std::vector<float> h(NPARAM);
  TCI_TRY(tci_sketch_model_get_params(ctx, m, h.data(), NPARAM));
  FILE* f = std::fopen(path, "wb");
  if (!f) TCI_RET(TCI_ERR_INVALID_ARGUMENT, std::string("cannot open ") + path);
  const char magic[8] = {'T', 'C', 'I', 'S', 'K', 'M', '1', 0};
  const int32_t np = NPARAM;
  bool ok = std::fwrite(magic, 1, 8, f) == 8 && std::fwrite(&np, 4, 1, f) == 1 &&
            std::fwrite(h.data(), sizeof(float), NPARAM, f) == (size_t)NPARAM;
  std::fclose(f);
  if (!ok) TCI_RET(TCI_ERR_INVALID_ARGUMENT, "short write");
  return TCI_OK;
} TCI_API_CATCH

tci_status tci_sketch_model_load(tci_context ctx, const char* path, tci_sketch_model* out) try {
  if (!ctx || !path || !out) TCI_RET(TCI_ERR_INVALID_ARGUMENT, "null argument");
  FILE* f = std::fopen(path, "rb");
  if (!f) TCI_RET(TCI_ERR_INVALID_ARGUMENT, std::string("cannot open ") + path);
  char magic[8];
  int32_t np = 0;
  std::vector<float> h(NPARAM);
  bool ok = std::fread(magic, 1, 8, f) == 8 && std::memcmp(magic, "TCISKM1", 7) == 0 &&
            std::fread(&np, 4, 1, f) == 1 && np == NPARAM &&
            std::fread(h.data(), sizeof(float), NPARAM, f) == (size_t)NPARAM;
  std::fclose(f);
  if (!ok) TCI_RET(TCI_ERR_INVALID_ARGUMENT, "not a sketch-model file");
  TCI_TRY(tci_sketch_model_create(ctx, 0, out));
  return tci_sketch_model_set_params(ctx, *out, h.data(), NPARAM);
} TCI_API_CATCH

tci_status tci_sketch_predict(tci_context ctx, tci_sketch_model m, const float* X, int n, float* y) try {
  if (!ctx || (n > 0 && (!X || !y))) TCI_RET(TCI_ERR_INVALID_ARGUMENT, "null argument");
  TCI_CHECK_HIP(hipSetDevice(ctx->device));
  return sketch_predict_dev(ctx, m, X, n, y);
} TCI_API_CATCH

tci_status tci_sketch_grads(tci_context ctx, tci_sketch_model m, const float* X, const float* T, int n, float* grad,
                            float* loss) try {
  if (!ctx || !X || !T || !grad || n < 1) TCI_RET(TCI_ERR_INVALID_ARGUMENT, "bad arguments");
  TCI_TRY(model_check(m));
  TCI_CHECK_HIP(hipSetDevice(ctx->device));
  ctx->arena.reset();
  float* ld = static_cast<float*>(ctx->arena.get(sizeof(float)));
  if (!ld) TCI_RET(TCI_ERR_OUT_OF_MEMORY, "workspace");
  TCI_TRY(grads_impl(ctx, m, X, T, n, grad, ld));
  if (loss) {
    TCI_CHECK_HIP(hipMemcpyAsync(loss, ld, sizeof(float), hipMemcpyDeviceToHost, ctx->stream));
    TCI_CHECK_HIP(hipStreamSynchronize(ctx->stream));
  }
  return TCI_OK;
} TCI_API_CATCH

tci_status tci_sketch_train_step(tci_context ctx, tci_sketch_model m, const float* X, const float* T, int n, float lr,
                                 float* loss) try {
  if (!ctx || !X || !T || n < 1) TCI_RET(TCI_ERR_INVALID_ARGUMENT, "bad arguments");
  TCI_TRY(model_check(m));
  TCI_CHECK_HIP(hipSetDevice(ctx->device));
  ctx->arena.reset();
  float* grad = static_cast<float*>(ctx->arena.get(sizeof(float) * NPARAM));
  float* ld = static_cast<float*>(ctx->arena.get(sizeof(float)));
  if (!grad || !ld) TCI_RET(TCI_ERR_OUT_OF_MEMORY, "workspace");
  TCI_TRY(grads_impl(ctx, m, X, T, n, grad, ld));
  m->step += 1;
  const float b1 = 0.9f, b2 = 0.999f;
  const float c1 = (float)(1.0 - std::pow(0.9, (double)m->step));
  const float c2 = (float)(1.0 - std::pow(0.999, (double)m->step));
  hipLaunchKernelGGL(adam_kernel, dim3((NPARAM + 255) / 256), dim3(256), 0, ctx->stream, m->params, m->m, m->v, grad,
                     lr, b1, b2, 1e-8f, c1, c2);
  TCI_CHECK_HIP(hipGetLastError());
  if (loss) {
    TCI_CHECK_HIP(hipMemcpyAsync(loss, ld, sizeof(float), hipMemcpyDeviceToHost, ctx->stream));
    TCI_CHECK_HIP(hipStreamSynchronize(ctx->stream));
  }
  return TCI_OK;
} TCI_API_CATCH

tci_status tci_sketch_features(tci_context ctx, const double* s, int64_t ss, const int32_t* len, int n, int chi_max,
                               int d, double eps, float* X) try {
  if (!ctx || !s || !len || !X || n < 1 || chi_max < 1 || !(eps > 0.0)) TCI_RET(TCI_ERR_INVALID_ARGUMENT, "bad arguments");
  TCI_CHECK_HIP(hipSetDevice(ctx->device));
  return sketch_features_dev(ctx, s, ss, len, chi_max, d, eps, X, n);
} TCI_API_CATCH

}  // extern "C"
