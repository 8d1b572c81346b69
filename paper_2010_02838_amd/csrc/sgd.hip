// Fused in-place parameter updates: momentum-SGD and Adam.
//
// Momentum-SGD (paper, Algorithm 1: theta <- theta - eta * gradient; heavy-ball
// momentum in the form of the large-minibatch recipe the paper follows, Section 4.1):
//     g = grad + wd * w;  v = mu * v + g;  w -= lr * (nesterov ? g + mu * v : v)
// HBM-bound: 12 bytes read and 8 (+2 for the bf16 copy) written per parameter.
#include "common.h"
#include <math.h>

namespace cd {

// Four parameters a thread, one trip: with 4096 blocks in several trips every thread waited for its loads once a trip, and the last trip
// left blocks without work (Adam, 60.9 M parameters 400 -> 342 us).  STREAM: loads and stores of the fp32 tensors bypass the caches (342 ->
// 298 us, 6.1 TB/s) in passes that move more than twice the 256 MB of the memory-side cache.  Up to there a pass repeated on the same tensors
// finds part of them cached, and bypassing it loses: without and with, 20 to 30 bytes a parameter, SGD of 14 M 45 and 51 us, of 25.6 M without
// the 16-bit copy (511 MB) 78 and 81, with it (562 MB) 94 and 87, of 60.9 M 284 and 217; Adam of 14 M (420 MB) 68 and 70, of 25.6 M 154
// and 119.  The 16-bit copy, which the next forward pass reads, is stored through the caches always.
typedef float f32x4_v __attribute__((ext_vector_type(4)));
template <bool STREAM>
__device__ inline float4 load4(const float* p, int64_t i) {
  const f32x4_v* q = reinterpret_cast<const f32x4_v*>(p) + i;
  const f32x4_v v = STREAM ? __builtin_nontemporal_load(q) : *q;
  return make_float4(v.x, v.y, v.z, v.w);
}
template <bool STREAM>
__device__ inline void store4(float* p, int64_t i, const float (&e)[4]) {
  f32x4_v* q = reinterpret_cast<f32x4_v*>(p) + i;
  const f32x4_v v = {e[0], e[1], e[2], e[3]};
  if (STREAM) __builtin_nontemporal_store(v, q); else *q = v;
}
static bool streams(int64_t n, int bytes_each) { return n * bytes_each > (512LL << 20); }
static dim3 update_grid(int64_t n) {   // (the kernels loop where a launch would have too many threads)
  const int64_t blocks = cdiv(n >> 2 > 0 ? n >> 2 : 1, 256);
  return dim3((unsigned)(blocks < (1 << 22) ? blocks : 1 << 22));
}

template <bool LOWP, bool STREAM>
__global__ void __launch_bounds__(256) sgd_kernel(float* __restrict__ w, float* __restrict__ v,
                                                  const float* __restrict__ g, bf16_t* __restrict__ lp, int64_t n,
                                                  float lr, float mu, float wd, int nesterov) {
  const int64_t n4 = n >> 2;
  const int64_t stride = (int64_t)gridDim.x * 256;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += stride) {
    const float4 W = load4<STREAM>(w, i), V = load4<STREAM>(v, i), G = load4<STREAM>(g, i);
    float wv[4] = {W.x, W.y, W.z, W.w}, vv[4] = {V.x, V.y, V.z, V.w};
    const float gv[4] = {G.x, G.y, G.z, G.w};
#pragma unroll
    for (int k = 0; k < 4; k++) {
      const float gg = gv[k] + wd * wv[k];
      vv[k] = mu * vv[k] + gg;
      wv[k] -= lr * (nesterov ? gg + mu * vv[k] : vv[k]);
    }
    store4<STREAM>(w, i, wv);
    store4<STREAM>(v, i, vv);
    if (LOWP) {
      ushort4 o;
      o.x = f32_to_bf16(wv[0]); o.y = f32_to_bf16(wv[1]); o.z = f32_to_bf16(wv[2]); o.w = f32_to_bf16(wv[3]);
      reinterpret_cast<ushort4*>(lp)[i] = o;
    }
  }
  // ragged tail (n not a multiple of 4)
  if (blockIdx.x == 0 && threadIdx.x < (n & 3)) {
    const int64_t i = (n4 << 2) + threadIdx.x;
    const float gg = g[i] + wd * w[i];
    const float vn = mu * v[i] + gg;
    const float wn = w[i] - lr * (nesterov ? gg + mu * vn : vn);
    v[i] = vn;
    w[i] = wn;
    if (LOWP) lp[i] = f32_to_bf16(wn);
  }
}

// Adam (Kingma & Ba), the optimiser of the translation recipe the paper follows (Section 4):
//     g = grad + wd * w;  m = b1 m + (1 - b1) g;  v = b2 v + (1 - b2) g^2;
//     w -= lr * (m / c1) / (sqrt(v / c2) + eps),  c1 = 1 - b1^t, c2 = 1 - b2^t (computed on the host in double)
// The kernel takes step = lr / c1 and rs = 1 / sqrt(c2).  16 bytes read and 12 (+2) written per parameter.
__device__ inline void adam_one(float& w, float& m, float& v, float g, float b1, float b2, float step, float rs,
                                float eps, float wd) {
  const float gg = g + wd * w;
  m = b1 * m + (1.f - b1) * gg;
  v = b2 * v + (1.f - b2) * gg * gg;
  w -= step * m / (sqrtf(v) * rs + eps);
}

template <bool LOWP, bool STREAM>
__global__ void __launch_bounds__(256) adam_kernel(float* __restrict__ w, float* __restrict__ m, float* __restrict__ v,
                                                   const float* __restrict__ g, bf16_t* __restrict__ lp, int64_t n,
                                                   float b1, float b2, float step, float rs, float eps, float wd) {
  const int64_t n4 = n >> 2;
  const int64_t stride = (int64_t)gridDim.x * 256;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += stride) {
    const float4 W = load4<STREAM>(w, i), M = load4<STREAM>(m, i), V = load4<STREAM>(v, i), G = load4<STREAM>(g, i);
    float wv[4] = {W.x, W.y, W.z, W.w}, mv[4] = {M.x, M.y, M.z, M.w}, vv[4] = {V.x, V.y, V.z, V.w};
    const float gv[4] = {G.x, G.y, G.z, G.w};
#pragma unroll
    for (int k = 0; k < 4; k++) adam_one(wv[k], mv[k], vv[k], gv[k], b1, b2, step, rs, eps, wd);
    store4<STREAM>(w, i, wv);
    store4<STREAM>(m, i, mv);
    store4<STREAM>(v, i, vv);
    if (LOWP) {
      ushort4 o;
      o.x = f32_to_bf16(wv[0]); o.y = f32_to_bf16(wv[1]); o.z = f32_to_bf16(wv[2]); o.w = f32_to_bf16(wv[3]);
      reinterpret_cast<ushort4*>(lp)[i] = o;
    }
  }
  if (blockIdx.x == 0 && threadIdx.x < (n & 3)) {  // ragged tail
    const int64_t i = (n4 << 2) + threadIdx.x;
    float wn = w[i], mn = m[i], vn = v[i];
    adam_one(wn, mn, vn, g[i], b1, b2, step, rs, eps, wd);
    w[i] = wn; m[i] = mn; v[i] = vn;
    if (LOWP) lp[i] = f32_to_bf16(wn);
  }
}

}  // namespace cd

using namespace cd;

extern "C" int codistill_sgd_step(float* master_w, float* momentum_v, const float* grad, void* lowp_w_out, int64_t n,
                                  float lr, float momentum, float weight_decay, int nesterov, void* stream) {
  CD_REQUIRE(master_w && momentum_v && grad, "sgd_step: NULL pointer argument");
  CD_REQUIRE(n >= 1, "sgd_step: n=%lld must be positive", (long long)n);
  CD_REQUIRE(aligned16(master_w) && aligned16(momentum_v) && aligned16(grad) &&
                 (reinterpret_cast<uintptr_t>(lowp_w_out) & 7) == 0,
             "sgd_step: fp32 pointers must be 16-byte aligned, the bf16 pointer 8-byte aligned");
  CD_REQUIRE(lr == lr && momentum == momentum && weight_decay == weight_decay, "sgd_step: NaN hyper-parameter");
  hipStream_t s = static_cast<hipStream_t>(stream);
  ProfScope prof(CD_K_SGD, s, 6.0 * n, (lowp_w_out ? 22.0 : 20.0) * n);
  auto run = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, update_grid(n), dim3(256), 0, s, master_w, momentum_v, grad, static_cast<bf16_t*>(lowp_w_out), n, lr,
                       momentum, weight_decay, nesterov);
  };
  const bool stream_all = streams(n, lowp_w_out ? 22 : 20);
  if (lowp_w_out) { if (stream_all) run(sgd_kernel<true, true>); else run(sgd_kernel<true, false>); }
  else { if (stream_all) run(sgd_kernel<false, true>); else run(sgd_kernel<false, false>); }
  return check_launch("sgd_step");
}

extern "C" int codistill_adam_step(float* master_w, float* exp_avg, float* exp_avg_sq, const float* grad, void* lowp_w_out,
                                   int64_t n, float lr, float beta1, float beta2, float eps, float weight_decay,
                                   int64_t t, void* stream) {
  CD_REQUIRE(master_w && exp_avg && exp_avg_sq && grad, "adam_step: NULL pointer argument");
  CD_REQUIRE(n >= 1, "adam_step: n=%lld must be positive", (long long)n);
  CD_REQUIRE(t >= 1, "adam_step: the update counter t=%lld starts at 1", (long long)t);
  CD_REQUIRE(aligned16(master_w) && aligned16(exp_avg) && aligned16(exp_avg_sq) && aligned16(grad) &&
                 (reinterpret_cast<uintptr_t>(lowp_w_out) & 7) == 0,
             "adam_step: fp32 pointers must be 16-byte aligned, the bf16 pointer 8-byte aligned");
  CD_REQUIRE(lr == lr && weight_decay == weight_decay && beta1 >= 0.f && beta1 < 1.f && beta2 >= 0.f && beta2 < 1.f &&
                 eps > 0.f,
             "adam_step: need 0 <= beta1, beta2 < 1, eps > 0 and no NaN hyper-parameter");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const double c1 = 1.0 - pow((double)beta1, (double)t), c2 = 1.0 - pow((double)beta2, (double)t);
  const float step = (float)((double)lr / c1), rs = (float)(1.0 / sqrt(c2));
  ProfScope prof(CD_K_SGD, s, 12.0 * n, (lowp_w_out ? 30.0 : 28.0) * n);
  auto run = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, update_grid(n), dim3(256), 0, s, master_w, exp_avg, exp_avg_sq, grad, static_cast<bf16_t*>(lowp_w_out), n,
                       beta1, beta2, step, rs, eps, weight_decay);
  };
  const bool stream_all = streams(n, lowp_w_out ? 30 : 28);
  if (lowp_w_out) { if (stream_all) run(adam_kernel<true, true>); else run(adam_kernel<true, false>); }
  else { if (stream_all) run(adam_kernel<false, true>); else run(adam_kernel<false, false>); }
  return check_launch("adam_step");
}
