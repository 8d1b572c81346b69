// Plain layer kernels: one thread per output element, fp32 arithmetic, fp32 or bf16 storage.
// They define the layers for any shape.  Pooling and the small layers around the convolutions run on them; of the
// convolutions the weight gradients of few weights over few pixels (generic_wgrad_pays), and all with CODISTILL_FORCE_SIMPLE or
// for tensors of 2^31 elements or 2^30 pixels and more.
#include "kernels.h"
#include "conv_rules.h"

namespace cd {

#define CD_DISPATCH_T(dtype, ...)                         \
  do {                                                    \
    if ((dtype) == CD_BF16) { typedef bf16_t T; __VA_ARGS__; } \
    else { typedef float T; __VA_ARGS__; }                \
  } while (0)

static inline dim3 grid1d(int64_t n, int block = 256) { return dim3((unsigned)cdiv(n, block)); }

// ------------------------------------------------------------------------------ convolution
template <typename T>
__global__ void __launch_bounds__(256) conv_fprop_simple_k(const T* __restrict__ x, const T* __restrict__ w,
                                                           const T* __restrict__ bias, T* __restrict__ y, ConvGeom g,
                                                           int relu) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= g.M() * g.Cout) return;
  const int n = idx % g.Cout;
  int64_t m = idx / g.Cout;
  const int wo = m % g.Wo; m /= g.Wo;
  const int ho = m % g.Ho;
  const int64_t b = m / g.Ho;
  float acc = bias ? Cvt<T>::ld(bias[n]) : 0.f;
  for (int r = 0; r < g.kh; r++) {
    const int hi = ho * g.stride - g.pad + r;
    if (hi < 0 || hi >= g.H) continue;
    for (int s = 0; s < g.kw; s++) {
      const int wi = wo * g.stride - g.pad + s;
      if (wi < 0 || wi >= g.W) continue;
      const T* xp = x + ((b * g.H + hi) * g.W + wi) * g.Cin;
      const T* wp = w + (((int64_t)n * g.kh + r) * g.kw + s) * g.Cin;
      for (int c = 0; c < g.Cin; c++) acc += Cvt<T>::ld(xp[c]) * Cvt<T>::ld(wp[c]);
    }
  }
  if (relu) acc = fmaxf(acc, 0.f);
  y[idx] = Cvt<T>::st(acc);
}

template <typename T>
__global__ void __launch_bounds__(256) conv_dgrad_simple_k(const T* __restrict__ dy, const T* __restrict__ w,
                                                           T* __restrict__ dx, ConvGeom g, int accumulate) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= g.B * g.H * g.W * g.Cin) return;
  const int c = idx % g.Cin;
  int64_t p = idx / g.Cin;
  const int wi = p % g.W; p /= g.W;
  const int hi = p % g.H;
  const int64_t b = p / g.H;
  float acc = 0.f;
  for (int r = 0; r < g.kh; r++) {
    const int hn = hi + g.pad - r;
    if (hn < 0 || hn % g.stride) continue;
    const int ho = hn / g.stride;
    if (ho >= g.Ho) continue;
    for (int s = 0; s < g.kw; s++) {
      const int wn = wi + g.pad - s;
      if (wn < 0 || wn % g.stride) continue;
      const int wo = wn / g.stride;
      if (wo >= g.Wo) continue;
      const T* dp = dy + ((b * g.Ho + ho) * g.Wo + wo) * g.Cout;
      const T* wp = w + ((int64_t)r * g.kw + s) * g.Cin + c;
      const int64_t wstride = (int64_t)g.kh * g.kw * g.Cin;
      for (int n = 0; n < g.Cout; n++) acc += Cvt<T>::ld(dp[n]) * Cvt<T>::ld(wp[n * wstride]);
    }
  }
  if (accumulate) acc += Cvt<T>::ld(dx[idx]);
  dx[idx] = Cvt<T>::st(acc);
}

// one block per weight element, threads stride over the B*Ho*Wo output positions
template <typename T>
__global__ void __launch_bounds__(256) conv_wgrad_simple_k(const T* __restrict__ x, const T* __restrict__ dy,
                                                           float* __restrict__ dw, ConvGeom g) {
  __shared__ float red[4];
  int64_t e = blockIdx.x;
  const int c = e % g.Cin; e /= g.Cin;
  const int s = e % g.kw; e /= g.kw;
  const int r = e % g.kh;
  const int n = e / g.kh;
  float acc = 0.f;
  const int64_t M = g.M();
  for (int64_t m = threadIdx.x; m < M; m += 256) {
    int64_t q = m;
    const int wo = q % g.Wo; q /= g.Wo;
    const int ho = q % g.Ho;
    const int64_t b = q / g.Ho;
    const int hi = ho * g.stride - g.pad + r, wi = wo * g.stride - g.pad + s;
    if (hi < 0 || hi >= g.H || wi < 0 || wi >= g.W) continue;
    acc += Cvt<T>::ld(dy[m * g.Cout + n]) * Cvt<T>::ld(x[((b * g.H + hi) * g.W + wi) * g.Cin + c]);
  }
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) dw[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

void conv_fprop_simple(int dtype, const void* x, const void* w, const void* bias, void* y, const ConvGeom& g,
                       bool relu, hipStream_t s) {
  CD_DISPATCH_T(dtype, hipLaunchKernelGGL(conv_fprop_simple_k<T>, grid1d(g.M() * g.Cout), dim3(256), 0, s,
                                          (const T*)x, (const T*)w, (const T*)bias, (T*)y, g, (int)relu));
}
void conv_dgrad_simple(int dtype, const void* dy, const void* w, void* dx, const ConvGeom& g, bool accumulate,
                       hipStream_t s) {
  CD_DISPATCH_T(dtype, hipLaunchKernelGGL(conv_dgrad_simple_k<T>, grid1d(g.B * g.H * g.W * g.Cin), dim3(256), 0, s,
                                          (const T*)dy, (const T*)w, (T*)dx, g, (int)accumulate));
}
void conv_wgrad_simple(int dtype, const void* x, const void* dy, float* dw, const ConvGeom& g, hipStream_t s) {
  const int64_t n = (int64_t)g.Cout * g.K();
  CD_DISPATCH_T(dtype, hipLaunchKernelGGL(conv_wgrad_simple_k<T>, dim3((unsigned)n), dim3(256), 0, s, (const T*)x,
                                          (const T*)dy, dw, g));
}

// ------------------------------------------------------------------------------------- glue
template <typename T>
__global__ void __launch_bounds__(256) relu_bwd_k(T* __restrict__ dy, const T* __restrict__ y, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n && !(Cvt<T>::ld(y[i]) > 0.f)) dy[i] = Cvt<T>::st(0.f);
}
template <typename T>
__global__ void __launch_bounds__(256) channel_slice_k(const T* __restrict__ x, T* __restrict__ y, int64_t n, int Cx, int c0,
                                                       int Cy) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const int64_t m = i / Cy;
  y[i] = x[m * Cx + c0 + (int)(i - m * Cy)];
}
void channel_slice(int dtype, const void* x, void* y, int64_t M, int Cx, int c0, int Cy, hipStream_t s) {
  const int64_t n = M * Cy;
  const dim3 grid((unsigned)cdiv(n, 256));
  if (dtype == CD_BF16)
    hipLaunchKernelGGL(channel_slice_k<bf16_t>, grid, dim3(256), 0, s, static_cast<const bf16_t*>(x), static_cast<bf16_t*>(y), n, Cx, c0, Cy);
  else
    hipLaunchKernelGGL(channel_slice_k<float>, grid, dim3(256), 0, s, static_cast<const float*>(x), static_cast<float*>(y), n, Cx, c0, Cy);
}
__global__ void __launch_bounds__(256) fill_zero_f32_k(float* p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0.f;
}
void fill_zero_f32(float* p, int64_t n, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(fill_zero_f32_k, dim3((unsigned)cdiv(n, 256)), dim3(256), 0, s, p, n);
}

void relu_bwd_inplace(int dtype, void* dy, const void* y, int64_t n, hipStream_t s) {
  CD_DISPATCH_T(dtype, hipLaunchKernelGGL(relu_bwd_k<T>, grid1d(n), dim3(256), 0, s, (T*)dy, (const T*)y, n));
}

// V channels per thread (V = 8 bf16 / 4 fp32 when the channel count allows 16-byte vectors)
template <typename T, int V> struct PoolVec {
  __device__ static void ld(const T* p, float (&v)[V]) {
#pragma unroll
    for (int i = 0; i < V; i++) v[i] = Cvt<T>::ld(p[i]);
  }
  __device__ static void st(T* p, const float (&v)[V]) {
#pragma unroll
    for (int i = 0; i < V; i++) p[i] = Cvt<T>::st(v[i]);
  }
};
template <> struct PoolVec<float, 4> {
  __device__ static void ld(const float* p, float (&v)[4]) {
    const float4 t = *reinterpret_cast<const float4*>(p);
    v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
  }
  __device__ static void st(float* p, const float (&v)[4]) { *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]); }
};
template <> struct PoolVec<bf16_t, 8> {
  __device__ static void ld(const bf16_t* p, float (&v)[8]) {
    const uint4 t = *reinterpret_cast<const uint4*>(p);
    const uint32_t u[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
    for (int i = 0; i < 4; i++) { v[2 * i] = __uint_as_float(u[i] << 16); v[2 * i + 1] = __uint_as_float(u[i] & 0xffff0000u); }
  }
  __device__ static void st(bf16_t* p, const float (&v)[8]) {
    uint32_t u[4];
#pragma unroll
    for (int i = 0; i < 4; i++) u[i] = (uint32_t)f32_to_bf16(v[2 * i]) | ((uint32_t)f32_to_bf16(v[2 * i + 1]) << 16);
    *reinterpret_cast<uint4*>(p) = make_uint4(u[0], u[1], u[2], u[3]);
  }
};

template <typename T, int V>
__global__ void __launch_bounds__(256) maxpool_fwd_k(const T* __restrict__ x, T* __restrict__ y,
                                                     uint8_t* __restrict__ argmax, int64_t B, int H, int W, int C,
                                                     int Ho, int Wo, int k, int stride, int pad) {
  const int CV = C / V;
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= B * Ho * Wo * CV) return;
  const int c = (int)(idx % CV) * V;
  int64_t p = idx / CV;
  const int wo = p % Wo; p /= Wo;
  const int ho = p % Ho;
  const int64_t b = p / Ho;
  float best[V];
  uint8_t arg[V];
#pragma unroll
  for (int i = 0; i < V; i++) { best[i] = -INFINITY; arg[i] = 0; }
  for (int r = 0; r < k; r++) {
    const int hi = ho * stride - pad + r;
    if (hi < 0 || hi >= H) continue;
    for (int s = 0; s < k; s++) {
      const int wi = wo * stride - pad + s;
      if (wi < 0 || wi >= W) continue;
      float v[V];
      PoolVec<T, V>::ld(x + ((b * H + hi) * W + wi) * C + c, v);
#pragma unroll
      for (int i = 0; i < V; i++)
        if (v[i] > best[i]) { best[i] = v[i]; arg[i] = (uint8_t)(r * k + s); }  // strict: the first maximum wins
    }
  }
  const int64_t o = ((b * Ho + ho) * Wo + wo) * C + c;
  PoolVec<T, V>::st(y + o, best);
  if (argmax) {
#pragma unroll
    for (int i = 0; i < V; i++) argmax[o + i] = arg[i];
  }
}

// backward from the stored argmax: 8 channels per thread, at most ceil(k/stride)^2 windows per pixel
__global__ void __launch_bounds__(256) maxpool_bwd_idx_k(const bf16_t* __restrict__ dy, const uint8_t* __restrict__ argmax,
                                                         bf16_t* __restrict__ dx, int accumulate, int64_t B, int H,
                                                         int W, int C, int Ho, int Wo, int k, int stride, int pad) {
  const int CV = C / 8;
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= B * H * W * CV) return;
  const int c = (int)(idx % CV) * 8;
  int64_t p = idx / CV;
  const int wi = p % W; p /= W;
  const int hi = p % H;
  const int64_t b = p / H;
  float acc[8];
#pragma unroll
  for (int i = 0; i < 8; i++) acc[i] = 0.f;
  int ho0 = hi + pad - k + 1; ho0 = ho0 <= 0 ? 0 : (ho0 + stride - 1) / stride;
  int wo0 = wi + pad - k + 1; wo0 = wo0 <= 0 ? 0 : (wo0 + stride - 1) / stride;
  int ho1 = (hi + pad) / stride; if (ho1 > Ho - 1) ho1 = Ho - 1;
  int wo1 = (wi + pad) / stride; if (wo1 > Wo - 1) wo1 = Wo - 1;
  for (int ho = ho0; ho <= ho1; ho++)
    for (int wo = wo0; wo <= wo1; wo++) {
      const uint32_t tap = (uint32_t)((hi - (ho * stride - pad)) * k + (wi - (wo * stride - pad)));
      const int64_t o = ((b * Ho + ho) * Wo + wo) * C + c;
      const uint2 a = *reinterpret_cast<const uint2*>(argmax + o);
      float g[8];
      PoolVec<bf16_t, 8>::ld(dy + o, g);
#pragma unroll
      for (int i = 0; i < 8; i++) {
        const uint32_t ai = ((i < 4 ? a.x : a.y) >> (8 * (i & 3))) & 0xffu;
        acc[i] += ai == tap ? g[i] : 0.f;
      }
    }
  bf16_t* dp = dx + ((b * H + hi) * W + wi) * C + c;
  if (accumulate) {
    float o[8];
    PoolVec<bf16_t, 8>::ld(dp, o);
#pragma unroll
    for (int i = 0; i < 8; i++) acc[i] += o[i];
  }
  PoolVec<bf16_t, 8>::st(dp, acc);
}

// Gradient goes to the first maximum of each window in row-major tap order (recomputed here).
template <typename T, int V>
__global__ void __launch_bounds__(256) maxpool_bwd_k(const T* __restrict__ x, const T* __restrict__ dy,
                                                     T* __restrict__ dx, int accumulate, int64_t B, int H, int W,
                                                     int C, int Ho, int Wo, int k, int stride, int pad) {
  const int CV = C / V;
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= B * H * W * CV) return;
  const int c = (int)(idx % CV) * V;
  int64_t p = idx / CV;
  const int wi = p % W; p /= W;
  const int hi = p % H;
  const int64_t b = p / H;
  float acc[V], mine[V];
#pragma unroll
  for (int i = 0; i < V; i++) acc[i] = 0.f;
  PoolVec<T, V>::ld(x + ((b * H + hi) * W + wi) * C + c, mine);
  // output windows that contain (hi, wi): ho*stride - pad <= hi <= ho*stride - pad + k - 1
  int ho0 = hi + pad - k + 1; ho0 = ho0 <= 0 ? 0 : (ho0 + stride - 1) / stride;
  int wo0 = wi + pad - k + 1; wo0 = wo0 <= 0 ? 0 : (wo0 + stride - 1) / stride;
  int ho1 = (hi + pad) / stride; if (ho1 > Ho - 1) ho1 = Ho - 1;
  int wo1 = (wi + pad) / stride; if (wo1 > Wo - 1) wo1 = Wo - 1;
  for (int ho = ho0; ho <= ho1; ho++) {
    const int h0 = ho * stride - pad;
    for (int wo = wo0; wo <= wo1; wo++) {
      const int w0 = wo * stride - pad;
      // this position wins the window iff no earlier tap is >= it and no later tap is > it
      bool win[V];
#pragma unroll
      for (int i = 0; i < V; i++) win[i] = true;
      for (int r = 0; r < k; r++) {
        const int hh = h0 + r;
        if (hh < 0 || hh >= H) continue;
        for (int s = 0; s < k; s++) {
          const int ww = w0 + s;
          if (ww < 0 || ww >= W || (hh == hi && ww == wi)) continue;
          float v[V];
          PoolVec<T, V>::ld(x + ((b * H + hh) * W + ww) * C + c, v);
          const bool earlier = hh < hi || (hh == hi && ww < wi);
#pragma unroll
          for (int i = 0; i < V; i++) win[i] = win[i] && (earlier ? v[i] < mine[i] : v[i] <= mine[i]);
        }
      }
      float g[V];
      PoolVec<T, V>::ld(dy + ((b * Ho + ho) * Wo + wo) * C + c, g);
#pragma unroll
      for (int i = 0; i < V; i++) acc[i] += win[i] ? g[i] : 0.f;
    }
  }
  T* dp = dx + ((b * H + hi) * W + wi) * C + c;
  if (accumulate) {
    float o[V];
    PoolVec<T, V>::ld(dp, o);
#pragma unroll
    for (int i = 0; i < V; i++) acc[i] += o[i];
  }
  PoolVec<T, V>::st(dp, acc);
}

void maxpool_fwd(int dtype, const void* x, void* y, uint8_t* argmax, int64_t B, int H, int W, int C, int k, int stride,
                 int pad, hipStream_t s) {
  const int Ho = (H + 2 * pad - k) / stride + 1, Wo = (W + 2 * pad - k) / stride + 1;
  if (dtype == CD_BF16 && C % 8 == 0 && aligned16(x) && aligned16(y))
    hipLaunchKernelGGL((maxpool_fwd_k<bf16_t, 8>), grid1d(B * Ho * Wo * (C / 8)), dim3(256), 0, s, (const bf16_t*)x,
                       (bf16_t*)y, argmax, B, H, W, C, Ho, Wo, k, stride, pad);
  else
    CD_DISPATCH_T(dtype, hipLaunchKernelGGL((maxpool_fwd_k<T, 1>), grid1d(B * Ho * Wo * C), dim3(256), 0, s,
                                            (const T*)x, (T*)y, argmax, B, H, W, C, Ho, Wo, k, stride, pad));
}
void maxpool_bwd(int dtype, const void* x, const void* dy, const uint8_t* argmax, void* dx, bool accumulate, int64_t B,
                 int H, int W, int C, int k, int stride, int pad, hipStream_t s) {
  const int Ho = (H + 2 * pad - k) / stride + 1, Wo = (W + 2 * pad - k) / stride + 1;
  if (argmax && dtype == CD_BF16 && C % 8 == 0 && aligned16(dy) && aligned16(dx) && aligned16(argmax))
    hipLaunchKernelGGL(maxpool_bwd_idx_k, grid1d(B * H * W * (C / 8)), dim3(256), 0, s, (const bf16_t*)dy, argmax,
                       (bf16_t*)dx, (int)accumulate, B, H, W, C, Ho, Wo, k, stride, pad);
  else if (dtype == CD_BF16 && C % 8 == 0 && aligned16(x) && aligned16(dy) && aligned16(dx))
    hipLaunchKernelGGL((maxpool_bwd_k<bf16_t, 8>), grid1d(B * H * W * (C / 8)), dim3(256), 0, s, (const bf16_t*)x,
                       (const bf16_t*)dy, (bf16_t*)dx, (int)accumulate, B, H, W, C, Ho, Wo, k, stride, pad);
  else
    CD_DISPATCH_T(dtype, hipLaunchKernelGGL((maxpool_bwd_k<T, 1>), grid1d(B * H * W * C), dim3(256), 0, s,
                                            (const T*)x, (const T*)dy, (T*)dx, (int)accumulate, B, H, W, C, Ho, Wo, k,
                                            stride, pad));
}

// Global average pool.  A block owns one sample and up to BLOCK vectors of V channels; the rows of the image are dealt to the
// BLOCK / vectors row groups, several loads in flight per thread, and the groups are added in LDS in a fixed order.  (One
// thread per channel with a serial loop over the pixels left the chip idle: 8 samples of 32x32x32 fp32 took 227 us, one
// load latency per pixel; now 5 us.)
template <typename T, int V, int BLOCK>
__global__ void __launch_bounds__(BLOCK) gap_fwd_k(const T* __restrict__ x, T* __restrict__ y, int HW, int C) {
  __shared__ float sm[BLOCK * V];
  const int vc = C / V, v0 = blockIdx.y * BLOCK, vb = vc - v0 < BLOCK ? vc - v0 : BLOCK;
  const int rg = BLOCK / vb, tx = threadIdx.x % vb, ty = threadIdx.x / vb;
  const T* __restrict__ p = x + (int64_t)blockIdx.x * HW * C + (int64_t)(v0 + tx) * V;
  float acc[V];
#pragma unroll
  for (int k = 0; k < V; k++) acc[k] = 0.f;
  if (ty < rg) {
#pragma unroll 8
    for (int i = ty; i < HW; i += rg) {
      float v[V];
      PoolVec<T, V>::ld(p + (int64_t)i * C, v);
#pragma unroll
      for (int k = 0; k < V; k++) acc[k] += v[k];
    }
#pragma unroll
    for (int k = 0; k < V; k++) sm[threadIdx.x * V + k] = acc[k];
  }
  __syncthreads();
  // one thread per channel adds the row groups
  for (int c = threadIdx.x; c < vb * V; c += BLOCK) {
    float t = 0.f;
    for (int g = 0; g < rg; g++) t += sm[g * vb * V + c];
    y[(int64_t)blockIdx.x * C + (int64_t)v0 * V + c] = Cvt<T>::st(t / (float)HW);
  }
}
// V channels per thread
template <typename T, int V>
__global__ void __launch_bounds__(256) gap_bwd_k(const T* __restrict__ dy, T* __restrict__ dx, int accumulate, int64_t n,
                                                 int HW, int C) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= n) return;
  const int vc = C / V;
  const int64_t row = n < (1LL << 31) ? (int64_t)((unsigned)idx / (unsigned)vc) : idx / vc;
  const int c = (int)(idx - row * vc) * V;
  const int64_t b = n < (1LL << 31) ? (int64_t)((unsigned)row / (unsigned)HW) : row / HW;
  float v[V];
  PoolVec<T, V>::ld(dy + b * C + c, v);
#pragma unroll
  for (int k = 0; k < V; k++) v[k] /= (float)HW;
  if (accumulate) {
    float o[V];
    PoolVec<T, V>::ld(dx + idx * V, o);
#pragma unroll
    for (int k = 0; k < V; k++) v[k] += o[k];
  }
  PoolVec<T, V>::st(dx + idx * V, v);
}
template <typename T>
static void gap_fwd_t(const T* x, T* y, int64_t B, int HW, int C, hipStream_t s) {
  constexpr int V = sizeof(T) == 2 ? 8 : 4;
  const int vec = C % V == 0 && aligned16(x) ? V : 1, vc = C / vec;
  // long images of few channels: 1024 threads, so that a thread adds tens of pixels, not hundreds
  const bool big = (int64_t)HW * vc > 256 * 16;
  const dim3 grid((unsigned)B, (unsigned)cdiv(vc, big ? 1024 : 256));
  if (vec > 1) {
    if (big) hipLaunchKernelGGL((gap_fwd_k<T, V, 1024>), grid, dim3(1024), 0, s, x, y, HW, C);
    else hipLaunchKernelGGL((gap_fwd_k<T, V, 256>), grid, dim3(256), 0, s, x, y, HW, C);
  } else {
    if (big) hipLaunchKernelGGL((gap_fwd_k<T, 1, 1024>), grid, dim3(1024), 0, s, x, y, HW, C);
    else hipLaunchKernelGGL((gap_fwd_k<T, 1, 256>), grid, dim3(256), 0, s, x, y, HW, C);
  }
}
template <typename T>
static void gap_bwd_t(const T* dy, T* dx, bool accumulate, int64_t B, int HW, int C, hipStream_t s) {
  constexpr int V = sizeof(T) == 2 ? 8 : 4;
  if (C % V == 0 && aligned16(dy) && aligned16(dx)) {
    const int64_t n = B * HW * (C / V);
    hipLaunchKernelGGL((gap_bwd_k<T, V>), grid1d(n), dim3(256), 0, s, dy, dx, (int)accumulate, n, HW, C);
  } else {
    const int64_t n = B * HW * C;
    hipLaunchKernelGGL((gap_bwd_k<T, 1>), grid1d(n), dim3(256), 0, s, dy, dx, (int)accumulate, n, HW, C);
  }
}
void gap_fwd(int dtype, const void* x, void* y, int64_t B, int HW, int C, hipStream_t s) {
  CD_DISPATCH_T(dtype, gap_fwd_t<T>((const T*)x, (T*)y, B, HW, C, s));
}
void gap_bwd(int dtype, const void* dy, void* dx, bool accumulate, int64_t B, int HW, int C, hipStream_t s) {
  CD_DISPATCH_T(dtype, gap_bwd_t<T>((const T*)dy, (T*)dx, accumulate, B, HW, C, s));
}

// ----------------------------------------------------------------------------------- linear
// one wave per output element: lanes stride over the F input features
template <typename T>
__global__ void __launch_bounds__(256) linear_fwd_k(const T* __restrict__ x, const T* __restrict__ w,
                                                    const T* __restrict__ bias, float* __restrict__ y, int64_t B,
                                                    int F, int C) {
  const int64_t o = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (o >= B * C) return;
  const int c = o % C;
  const int64_t b = o / C;
  float acc = 0.f;
  for (int f = threadIdx.x & 63; f < F; f += 64) acc += Cvt<T>::ld(x[b * F + f]) * Cvt<T>::ld(w[(int64_t)c * F + f]);
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) y[o] = acc + (bias ? Cvt<T>::ld(bias[c]) : 0.f);
}
template <typename T>
__global__ void __launch_bounds__(256) linear_dx_k(const float* __restrict__ dy, const T* __restrict__ w,
                                                   T* __restrict__ dx, int accumulate, int64_t B, int F, int C) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= B * F) return;
  const int f = idx % F;
  const int64_t b = idx / F;
  float acc = 0.f;
#pragma unroll 8
  for (int c = 0; c < C; c++) acc += dy[b * C + c] * Cvt<T>::ld(w[(int64_t)c * F + f]);
  if (accumulate) acc += Cvt<T>::ld(dx[idx]);
  dx[idx] = Cvt<T>::st(acc);
}
// dw[c][f] = sum_b dy[b][c] x[b][f], db[c] = sum_b dy[b][c] (the column f = F, x = 1).  Block = 64 features x G row groups
// for 4 classes; the groups are added in LDS in a fixed order.  A group's rows are a chain of loads: 16 groups for up to 256 blocks, where
// every block has a compute unit to itself, otherwise 4.  fp32, 4 and 16 groups: 64 features over 128 rows, 6 blocks 11.9 and 5.5 us, 256
// blocks 11.6 and 5.2, over 1024 rows 79 and 27; from there on it depends on the rows: 2048 blocks over 32 rows 7.2 and 10.2, over 128
// 17.8 and 21.0, over 1024 232 and 227.
template <typename T, int G>
__global__ void __launch_bounds__(64 * G) linear_dw_k(const float* __restrict__ dy, const T* __restrict__ x,
                                                   float* __restrict__ dw, float* __restrict__ db, int64_t B, int F,
                                                   int C) {
  __shared__ float sm[G][4][64];
  const int fl = threadIdx.x & 63, g = threadIdx.x >> 6;
  const unsigned ft = (unsigned)(F + 64) / 64u;   // 64-column tiles of the F + 1 columns (linear_dw_grid)
  const int f = (int)(blockIdx.x % ft) * 64 + fl, c0 = (int)(blockIdx.y * (gridDim.x / ft) + blockIdx.x / ft) * 4;
  if (c0 >= C) return;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  if (f <= F) {
#pragma unroll 4
    for (int64_t b = g; b < B; b += G) {
      const float xv = f < F ? Cvt<T>::ld(x[b * F + f]) : 1.f;
#pragma unroll
      for (int k = 0; k < 4; k++)
        if (c0 + k < C) acc[k] += dy[b * C + c0 + k] * xv;
    }
  }
#pragma unroll
  for (int k = 0; k < 4; k++) sm[g][k][fl] = acc[k];
  __syncthreads();
  const int c = c0 + g;   // wave g adds class c0 + g
  if (g >= 4 || f > F || c >= C) return;
  float t = 0.f;
#pragma unroll
  for (int i = 0; i < G; i += 4) {
    const float u = (sm[i][g][fl] + sm[i + 1][g][fl]) + (sm[i + 2][g][fl] + sm[i + 3][g][fl]);
    t = i ? t + u : u;
  }
  if (f < F) dw[(int64_t)c * F + f] = t;
  else if (db) db[c] = t;
}
void linear_fwd(int dtype, const void* x, const void* w, const void* b, float* y, int64_t B, int F, int C,
                hipStream_t s) {
  CD_DISPATCH_T(dtype, hipLaunchKernelGGL(linear_fwd_k<T>, grid1d(B * C, 4), dim3(256), 0, s, (const T*)x, (const T*)w,
                                          (const T*)b, y, B, F, C));
}
void linear_bwd(int dtype, const void* x, const void* w, const float* dy, void* dx, bool accumulate, float* dw,
                float* db, int64_t B, int F, int C, hipStream_t s) {
  CD_DISPATCH_T(dtype, {
    hipLaunchKernelGGL(linear_dx_k<T>, grid1d(B * F), dim3(256), 0, s, dy, (const T*)w, (T*)dx, (int)accumulate, B, F, C);
    const LinearDwGrid g = linear_dw_grid(F, C);
    if (g.x * g.y <= 256)
      hipLaunchKernelGGL((linear_dw_k<T, 16>), dim3((unsigned)g.x, (unsigned)g.y), dim3(1024), 0, s, dy, (const T*)x, dw, db, B, F, C);
    else
      hipLaunchKernelGGL((linear_dw_k<T, 4>), dim3((unsigned)g.x, (unsigned)g.y), dim3(256), 0, s, dy, (const T*)x, dw, db, B, F, C);
  });
}

// ----------------------------------------------------------------------------- padding gaps
struct GapList { Gap g[128]; int n; };
__global__ void __launch_bounds__(64) zero_gaps_k(float* base, GapList l) {
  const int i = blockIdx.x;
  if (i < l.n && (int)threadIdx.x < l.g[i].len) base[l.g[i].off + threadIdx.x] = 0.f;
}
void zero_gaps(float* base, const Gap* gaps, int n, hipStream_t s) {
  for (int i = 0; i < n; i += 128) {
    GapList l;
    l.n = n - i < 128 ? n - i : 128;
    for (int j = 0; j < l.n; j++) l.g[j] = gaps[i + j];
    hipLaunchKernelGGL(zero_gaps_k, dim3(l.n), dim3(64), 0, s, base, l);
  }
}

}  // namespace cd
