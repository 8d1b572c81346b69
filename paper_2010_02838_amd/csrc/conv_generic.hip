// Convolutions of any channel count on the fp32 matrix instruction (v_mfma_f32_16x16x4_f32): the fp32 models, and
// the bf16 layers whose channel counts are no multiple of 8 (the bf16 kernels gather 16-byte vectors of 8 channels).
// Products and sums are fp32, as in the one-thread-per-output kernels, which stay behind CODISTILL_FORCE_SIMPLE and take
// tensors of 2^31 elements or 2^30 pixels and more.
//
//   fprop  y[m][n]  = sum_k im2col(x)[m][k]  * w[n][k]         m = (b,ho,wo), k = (r,s,c)
//   dgrad  dx[m][c] = sum_k gather(dy)[m][k] * w[n][r][s][c]   m = (b,h,w),   k = (r,s,n)
//   wgrad  dw[n][k] = sum_m dy[m][n] * im2col(x)[m][k]
//
// What bounds them: on these channel counts (3 to a few hundred) the launches are small or bound by the fp32 matrix rate
// (157 TFLOP/s, a sixteenth of the bf16 one); one thread per output spent its time on one 4-byte load per multiply-add and
// on 64-bit index divisions.  Here a tile of both operands goes through LDS, each loaded element feeds 16 to 64
// multiply-adds, and pixels are decoded once per thread.  Measured before and after: a two-block fp32 network on 32 images
// of 32x32, forward and backward, 2430 -> 389 us; the step of the channel-split Wide-ResNet, batch 96, whose second block
// reads 20 channels, 62.2 -> 8.75 ms; the two-layer fp32 network's step on 8 images 725 -> 378 us.
#include "kernels.h"
#include "conv_rules.h"
#include <type_traits>

namespace cd {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

// V consecutive elements as fp32
template <typename T, int V> struct GenVec;
template <> struct GenVec<float, 1> {
  __device__ static void ld(const float* p, float (&v)[1]) { v[0] = *p; }
};
template <> struct GenVec<float, 4> {
  __device__ static void ld(const float* p, float (&v)[4]) {
    const float4 t = *reinterpret_cast<const float4*>(p);
    v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
  }
};
template <> struct GenVec<bf16_t, 1> {
  __device__ static void ld(const bf16_t* p, float (&v)[1]) { v[0] = bf16_to_f32(*p); }
};
template <> struct GenVec<bf16_t, 4> {
  __device__ static void ld(const bf16_t* p, float (&v)[4]) {
    const uint2 t = *reinterpret_cast<const uint2*>(p);
    v[0] = __uint_as_float(t.x << 16); v[1] = __uint_as_float(t.x & 0xffff0000u);
    v[2] = __uint_as_float(t.y << 16); v[3] = __uint_as_float(t.y & 0xffff0000u);
  }
};

struct GenArgs {
  const void* src;   // fprop: x; dgrad: dy; wgrad: x
  const void* w;     // fprop, dgrad: the filter as stored; wgrad: dy
  const void* bias;  // fprop, nullable
  void* out;         // fprop: y; dgrad: dx; wgrad: fp32 [splits][N][K]
  int M, N, K;       // rows and columns of the output and the contraction (wgrad: rows = Cout, columns = K, contraction M)
  int H, W, Cin, Ho, Wo, Cout, kh, kw, stride, pad;
  int relu, accumulate;
  int m_per_split, ktiles, tiles;   // wgrad
  FastDiv by_cin, by_cout, by_kw, by_stride, by_w, by_h, by_wo, by_ho;
  float* sums;       // fprop, nullable: column sums and sums of squares of the stored values, a row block each: [blocks][stat_pitch(N)]
};
struct GenNormArgs : GenArgs { EvalNorm norm; };   // fprop with the evaluation-mode BatchNorm that follows

// an element of the output behind that BatchNorm, from the convolution's result and the residual's element
template <typename T> __device__ inline float gen_norm(const GenNormArgs& a, float v, float scale, float shift, float res) {
  v = fmaf(Cvt<T>::ld(Cvt<T>::st(v)), scale, shift);
  v = a.norm.res ? v + res : v;
  return a.norm.relu ? fmaxf(v, 0.f) : v;
}

// One output element from its definition: taps outside the image (and, in a strided data gradient, between the strides) take
// no part.  The matrix kernels multiply zeros there instead, which is the same unless the other factor is infinite or NaN
// (0 * inf = NaN): an element that comes out as NaN is computed again here.  A NaN that belongs there is found at its first
// product, so that a diverged network costs little.
template <typename T, int MODE> __device__ inline float gen_element(const GenArgs& a, int m, int n) {
  const T* __restrict__ src = static_cast<const T*>(a.src);
  const T* __restrict__ wt = static_cast<const T*>(a.w);
  const int HD = MODE == 0 ? a.Ho : a.H, WD = MODE == 0 ? a.Wo : a.W;
  const int HS = MODE == 0 ? a.H : a.Ho, WS = MODE == 0 ? a.W : a.Wo, CS = MODE == 0 ? a.Cin : a.Cout;
  const int q = m / WD, x = m - q * WD, b = q / HD, y = q - b * HD;
  float acc = MODE == 0 && a.bias ? Cvt<T>::ld(static_cast<const T*>(a.bias)[n]) : 0.f;
  for (int r = 0; r < a.kh; r++) {
    int h = MODE == 0 ? y * a.stride - a.pad + r : y + a.pad - r;
    if (h < 0 || (MODE == 1 && h % a.stride)) continue;
    if (MODE == 1) h /= a.stride;
    if (h >= HS) continue;
    for (int s = 0; s < a.kw; s++) {
      int w = MODE == 0 ? x * a.stride - a.pad + s : x + a.pad - s;
      if (w < 0 || (MODE == 1 && w % a.stride)) continue;
      if (MODE == 1) w /= a.stride;
      if (w >= WS) continue;
      const T* p = src + (unsigned)((b * HS + h) * WS + w) * (unsigned)CS;
      const unsigned tap = (unsigned)(r * a.kw + s);
      for (int c = 0; c < CS; c++) {
        const unsigned at = MODE == 0 ? (unsigned)n * (unsigned)a.K + tap * (unsigned)CS + (unsigned)c
                                      : ((unsigned)c * (unsigned)(a.kh * a.kw) + tap) * (unsigned)a.Cin + (unsigned)n;
        acc += Cvt<T>::ld(p[c]) * Cvt<T>::ld(wt[at]);
        if (acc != acc) return acc;
      }
    }
  }
  return acc;
}
// the same for element (n, k) of a weight gradient over the pixels [mbeg, mend)
template <typename T> __device__ inline float gen_wgrad_element(const GenArgs& a, int n, int k, int mbeg, int mend) {
  const T* __restrict__ x = static_cast<const T*>(a.src);
  const T* __restrict__ dy = static_cast<const T*>(a.w);
  const int tap = k / a.Cin, c = k - tap * a.Cin, r = tap / a.kw, s = tap - r * a.kw;
  float acc = 0.f;
  for (int m = mbeg; m < mend; m++) {
    const int q = m / a.Wo, b = q / a.Ho;
    const int h = (q - b * a.Ho) * a.stride - a.pad + r, w = (m - q * a.Wo) * a.stride - a.pad + s;
    if ((unsigned)h >= (unsigned)a.H || (unsigned)w >= (unsigned)a.W) continue;
    acc += Cvt<T>::ld(dy[(unsigned)m * (unsigned)a.N + (unsigned)n]) *
           Cvt<T>::ld(x[(unsigned)((b * a.H + h) * a.W + w) * (unsigned)a.Cin + (unsigned)c]);
    if (acc != acc) return acc;
  }
  return acc;
}

// the sum over the sixteen lanes of a row, in every one of them
template <int CTRL> __device__ inline float dpp_add(float v) {
  return v + __uint_as_float(__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), CTRL, 0xf, 0xf, true));
}
__device__ inline float sum16(float v) {
  v = dpp_add<0xB1>(v);    // quad_perm [1,0,3,2]
  v = dpp_add<0x4E>(v);    // quad_perm [2,3,0,1]
  v = dpp_add<0x141>(v);   // row_half_mirror
  return dpp_add<0x140>(v);   // row_mirror
}

// MODE 0: fprop, MODE 1: dgrad.  Block = 4 waves down the rows, each 16 TM rows x 16 TN columns; 32 contraction elements
// per step, two LDS buffers, the next step's elements travel in registers while the matrix cores work on this one.  The
// filter is the MFMA "A" operand, so a lane's four accumulators are four consecutive channels of one pixel.  A lane reads
// its four k of a 16-element chunk as one 16-byte LDS load; element k of a chunk lies at place 4 (k % 4) + k / 4, so that
// instruction j takes k = 4 j + lane / 16: the sums run over k in ascending order, tap by tap, as the definition and the
// plain kernels add them.  Rows are 36 floats apart: 16 rows start in 16 different 16-byte bank groups.
// A BatchNorm behind the convolution gets its column sums here (GenArgs::sums): a pass of its own over the tensor was 4 to 8 us and a launch
// (two-block fp32 network on 32 images of 32x32: six of them, 231 -> 218 us a pass; the sums add 0.5 us to a convolution).  What is left is
// added up in fp64, as the reduction pass's sums are: by the BatchNorm's own pass (bn_own_sums) or by a finalize launch, of more than
// kFinalizeChunks partial sums behind a fold.  (Folded in fp32 from 256 on, images of 250 +- 2 had a variance off by 2e-4 on 33 of 32x32.)  That
// network on 33, 65 and 128 images 285 -> 225 us, 365 -> 294, 463 -> 405
// (generic_sums_pay).
// VEC: channels per load (4 where both channel counts allow it).  NORM (fprop): the evaluation-mode BatchNorm behind it is applied
// to the values as they are stored.
template <typename T, int MODE, int VEC, int TM, int TN, bool NORM>
__global__ void __launch_bounds__(256) conv_generic_k(std::conditional_t<NORM, GenNormArgs, GenArgs> a) {
  constexpr int BM = 64 * TM, BN = 16 * TN, BK = 32, P = BK + 4;
  constexpr int KV = BK / VEC, RPP = 256 / KV, AP = BM / RPP;       // pixel rows: vectors per row, rows per pass, passes
  constexpr int FP = MODE == 0 ? (BN + RPP - 1) / RPP : (BK + 256 / (BN / VEC) - 1) / (256 / (BN / VEC));   // filter passes
  constexpr int CV = BN / VEC, FRPP = 256 / CV;                     // dgrad filter tile: vectors per k row, k rows per pass
  __shared__ __attribute__((aligned(16))) float As[2][BM * P];
  __shared__ __attribute__((aligned(16))) float Bs[2][BN * P];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int m0 = blockIdx.x * BM, n0 = blockIdx.y * BN;
  const T* __restrict__ src = static_cast<const T*>(a.src);
  const T* __restrict__ wt = static_cast<const T*>(a.w);
  const int CS = MODE == 0 ? a.Cin : a.Cout, HS = MODE == 0 ? a.H : a.Ho, WS = MODE == 0 ? a.W : a.Wo;
  const int HD = MODE == 0 ? a.Ho : a.H, WD = MODE == 0 ? a.Wo : a.W;

  const int kv = tid % KV, ar = tid / KV;
  int pb[AP], ph[AP], pw[AP];   // image base row of the gathered tensor, window origin (a row past M never reads)
#pragma unroll
  for (int j = 0; j < AP; j++) {
    const int m = m0 + ar + j * RPP;
    const unsigned mm = m < a.M ? (unsigned)m : 0u;
    const unsigned q = div_by(mm, MODE == 0 ? a.by_wo : a.by_w);
    const int x = (int)(mm - q * (unsigned)WD);
    const unsigned b = div_by(q, MODE == 0 ? a.by_ho : a.by_h);
    const int y = (int)(q - b * (unsigned)HD);
    pb[j] = (int)b * HS;
    ph[j] = MODE == 0 ? y * a.stride - a.pad : y + a.pad;
    pw[j] = MODE == 0 ? x * a.stride - a.pad : x + a.pad;
    if (m >= a.M) ph[j] = -0x10000000;
  }
  float ra[AP][VEC], rb[FP][VEC];
  auto place = [](int k) { return (k & ~15) + 4 * (k & 3) + ((k >> 2) & 3); };
  auto gload = [&](int kt) {
    {
      const int k = kt * BK + kv * VEC;
      const unsigned tap = div_by((unsigned)k, MODE == 0 ? a.by_cin : a.by_cout);
      const int c = k - (int)tap * CS, r = (int)div_by(tap, a.by_kw), s = (int)tap - r * a.kw;
#pragma unroll
      for (int j = 0; j < AP; j++) {
        int h, w;
        bool ok = k < a.K;
        if (MODE == 0) {
          h = ph[j] + r; w = pw[j] + s;
          ok = ok && h >= 0 && w >= 0;
        } else {
          h = ph[j] - r; w = pw[j] - s;
          ok = ok && h >= 0 && w >= 0;
          if (a.stride != 1) {
            const int hq = (int)div_by((unsigned)h, a.by_stride), wq = (int)div_by((unsigned)w, a.by_stride);   // (negative ones are out already)
            ok = ok && hq * a.stride == h && wq * a.stride == w;
            h = hq; w = wq;
          }
        }
        ok = ok && h < HS && w < WS;
#pragma unroll
        for (int i = 0; i < VEC; i++) ra[j][i] = 0.f;
        if (ok) GenVec<T, VEC>::ld(src + ((unsigned)((pb[j] + h) * WS + w) * (unsigned)CS + (unsigned)c), ra[j]);
      }
    }
    if (MODE == 0) {   // filter rows are contiguous along k
      const int k = kt * BK + kv * VEC;
#pragma unroll
      for (int j = 0; j < FP; j++) {
        const int n = ar + j * RPP;
#pragma unroll
        for (int i = 0; i < VEC; i++) rb[j][i] = 0.f;
        if (n < BN && n0 + n < a.N && k < a.K) GenVec<T, VEC>::ld(wt + ((unsigned)(n0 + n) * (unsigned)a.K + (unsigned)k), rb[j]);
      }
    } else {           // w[n][r][s][c]: contiguous along the output column c
      const int c = n0 + (tid % CV) * VEC;
#pragma unroll
      for (int j = 0; j < FP; j++) {
        const int kr = tid / CV + j * FRPP, k = kt * BK + kr;
        const unsigned tap = div_by((unsigned)k, a.by_cout);
        const int n = k - (int)tap * CS;
#pragma unroll
        for (int i = 0; i < VEC; i++) rb[j][i] = 0.f;
        if (kr < BK && k < a.K && c < a.N)
          GenVec<T, VEC>::ld(wt + (((unsigned)n * (unsigned)(a.kh * a.kw) + tap) * (unsigned)a.Cin + (unsigned)c), rb[j]);
      }
    }
  };
  auto lstore = [&](int buf) {
#pragma unroll
    for (int j = 0; j < AP; j++)
#pragma unroll
      for (int i = 0; i < VEC; i++) As[buf][(ar + j * RPP) * P + place(kv * VEC + i)] = ra[j][i];
#pragma unroll
    for (int j = 0; j < FP; j++) {
      if (MODE == 0) {
        const int n = ar + j * RPP;
        if (n < BN) {
#pragma unroll
          for (int i = 0; i < VEC; i++) Bs[buf][n * P + place(kv * VEC + i)] = rb[j][i];
        }
      } else {
        const int kr = tid / CV + j * FRPP;
        if (kr < BK) {
#pragma unroll
          for (int i = 0; i < VEC; i++) Bs[buf][((tid % CV) * VEC + i) * P + place(kr)] = rb[j][i];
        }
      }
    }
  };
  f32x4_t acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; i++)
#pragma unroll
    for (int j = 0; j < TM; j++) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const int fr = lane & 15, fk = (lane >> 4) * 4;
  const T* __restrict__ bias = static_cast<const T*>(a.bias);
  if (MODE == 0 && bias) {
#pragma unroll
    for (int i = 0; i < TN; i++)
#pragma unroll
      for (int q = 0; q < 4; q++) {
        const int n = n0 + i * 16 + fk + q;
        const float bv = n < a.N ? Cvt<T>::ld(bias[n]) : 0.f;
#pragma unroll
        for (int j = 0; j < TM; j++) acc[i][j][q] = bv;
      }
  }
  const int KT = (a.K + BK - 1) / BK;
  gload(0);
  lstore(0);
  __syncthreads();
  for (int kt = 0; kt < KT; kt++) {
    const int cur = kt & 1;
    if (kt + 1 < KT) gload(kt + 1);
#pragma unroll
    for (int kc = 0; kc < BK; kc += 16) {
      f32x4_t f[TN], p[TM];
#pragma unroll
      for (int i = 0; i < TN; i++) f[i] = *reinterpret_cast<const f32x4_t*>(&Bs[cur][(i * 16 + fr) * P + kc + fk]);
#pragma unroll
      for (int j = 0; j < TM; j++) p[j] = *reinterpret_cast<const f32x4_t*>(&As[cur][((wave * TM + j) * 16 + fr) * P + kc + fk]);
#pragma unroll
      for (int q = 0; q < 4; q++)
#pragma unroll
        for (int i = 0; i < TN; i++)
#pragma unroll
          for (int j = 0; j < TM; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(f[i][q], p[j][q], acc[i][j], 0, 0, 0);
    }
    if (kt + 1 < KT) lstore(cur ^ 1);
    __syncthreads();
  }
  T* __restrict__ out = static_cast<T*>(a.out);
  static_assert(TM * TN * 4 <= 32, "one bit per element of a lane");
  uint32_t again = 0;   // elements that are NaN (they count as zero until the end): bit 4 (TN j + i) + q
  float odd = 0.f;      // becomes NaN if one is, or is infinite
#pragma unroll
  for (int i = 0; i < TN; i++)
#pragma unroll
    for (int j = 0; j < TM; j++)
#pragma unroll
      for (int q = 0; q < 4; q++) odd = fmaf(acc[i][j][q], 0.f, odd);
  if (__builtin_expect(__any(odd != odd), 0)) {
#pragma unroll
    for (int i = 0; i < TN; i++)
#pragma unroll
      for (int j = 0; j < TM; j++)
#pragma unroll
        for (int q = 0; q < 4; q++)
          if (acc[i][j][q] != acc[i][j][q]) { again |= 1u << (4 * (TN * j + i) + q); acc[i][j][q] = 0.f; }
  }
  float nsc[NORM ? TN : 1][4], nsh[NORM ? TN : 1][4];   // scale and shift of this lane's channels
  if constexpr (NORM) {
#pragma unroll
    for (int i = 0; i < TN; i++)
#pragma unroll
      for (int q = 0; q < 4; q++) {
        const int n = n0 + i * 16 + fk + q;
        nsc[i][q] = nsh[i][q] = 0.f;   // (channels behind the last one are computed and not stored)
        if (n < a.N)
          running_scale_shift(a.norm.running, static_cast<const T*>(a.norm.gamma), static_cast<const T*>(a.norm.beta), a.N, n,
                              &nsc[i][q], &nsh[i][q]);
      }
  }
  constexpr bool SUMS = MODE == 0 && !NORM;
  float cs0[SUMS ? TN : 1][4], cs1[SUMS ? TN : 1][4];   // this lane's channels, summed over its rows
  if (SUMS) {
#pragma unroll
    for (int i = 0; i < TN; i++)
#pragma unroll
      for (int q = 0; q < 4; q++) { cs0[i][q] = 0.f; cs1[i][q] = 0.f; }
  }
#pragma unroll
  for (int j = 0; j < TM; j++) {
    const int m = m0 + (wave * TM + j) * 16 + fr;
    if (m >= a.M) continue;
#pragma unroll
    for (int i = 0; i < TN; i++) {
      const int n = n0 + i * 16 + fk;
      if (n >= a.N) continue;
      T* o = out + ((unsigned)m * (unsigned)a.N + (unsigned)n);
      const int nv = a.N - n < 4 ? a.N - n : 4;
      // All four elements are computed without a condition of their own (of a fourth channel that is not there: zeros, not stored).
      // Where each was changed inside `q < nv`, clang of ROCm 7.2 copied the accumulators' four registers from condition to condition and
      // wrote element 0 over 1 and 2 (v_accvgpr_write_b32 a1, v0; a2, v0) in eight of the eighteen normalising kernels, whether or not nsc and
      // nsh of the missing channels were defined.
      float v[4], old[4] = {0.f, 0.f, 0.f, 0.f};   // old: the gradient so far, or the residual
      const T* add = NORM ? nullptr : MODE == 1 && a.accumulate ? o : nullptr;
      if constexpr (NORM) {
        if (a.norm.res) add = static_cast<const T*>(a.norm.res) + ((unsigned)m * (unsigned)a.N + (unsigned)n);
      }
      if (add) {
#pragma unroll
        for (int q = 0; q < 4; q++)
          if (q < nv) old[q] = Cvt<T>::ld(add[q]);
      }
#pragma unroll
      for (int q = 0; q < 4; q++) {
        v[q] = acc[i][j][q];
        if constexpr (NORM) {
          v[q] = gen_norm<T>(a, v[q], nsc[i][q], nsh[i][q], old[q]);
        } else {
          if (MODE == 1) v[q] = a.accumulate ? v[q] + old[q] : v[q];
          if (MODE == 0) v[q] = a.relu ? fmaxf(v[q], 0.f) : v[q];
        }
      }
      if constexpr (SUMS) {
#pragma unroll
        for (int q = 0; q < 4; q++) {
          const float t = Cvt<T>::ld(Cvt<T>::st(v[q]));   // (a channel behind the last one is a sum of zeros)
          cs0[i][q] += t;
          cs1[i][q] = fmaf(t, t, cs1[i][q]);
        }
      }
      if ((a.N & 3) == 0) {   // four channels of a pixel at a 4-element boundary
        if (sizeof(T) == 4) {
          *reinterpret_cast<float4*>(o) = make_float4(v[0], v[1], v[2], v[3]);
        } else {
          *reinterpret_cast<uint2*>(o) = make_uint2((uint32_t)f32_to_bf16(v[0]) | ((uint32_t)f32_to_bf16(v[1]) << 16),
                                                    (uint32_t)f32_to_bf16(v[2]) | ((uint32_t)f32_to_bf16(v[3]) << 16));
        }
      } else {
#pragma unroll
        for (int q = 0; q < 4; q++)
          if (q < nv) o[q] = Cvt<T>::st(v[q]);
      }
    }
  }
  const int again_any = again != 0;
  if (__builtin_expect(__any(again != 0), 0)) {
    while (again) {
      const int e = __ffs(again) - 1;
      again &= again - 1;
      const int m = m0 + (wave * TM + e / (4 * TN)) * 16 + fr, n = n0 + e / 4 % TN * 16 + fk + e % 4;
      if (m >= a.M || n >= a.N) continue;
      float v = gen_element<T, MODE>(a, m, n);
      T* o = out + ((unsigned)m * (unsigned)a.N + (unsigned)n);
      if (MODE == 1 && a.accumulate) v += Cvt<T>::ld(*o);
      if (MODE == 0 && a.relu) v = fmaxf(v, 0.f);
      if constexpr (NORM) {
        float sc, sh;
        running_scale_shift(a.norm.running, static_cast<const T*>(a.norm.gamma), static_cast<const T*>(a.norm.beta), a.N, n, &sc, &sh);
        const float r = a.norm.res ? Cvt<T>::ld(static_cast<const T*>(a.norm.res)[(unsigned)m * (unsigned)a.N + (unsigned)n]) : 0.f;
        v = gen_norm<T>(a, v, sc, sh, r);
      }
      *o = Cvt<T>::st(v);
    }
  }
  if constexpr (SUMS) {
    if (a.sums) {   // uniform over the launch
      // the sixteen lanes of a channel, then the four waves, in a fixed order
      float* red = &As[0][0];   // [wave][2][BN]; (the main loop ends with a barrier)
#pragma unroll
      for (int i = 0; i < TN; i++)
#pragma unroll
        for (int q = 0; q < 4; q++) {
          const float t0 = sum16(cs0[i][q]), t1 = sum16(cs1[i][q]);
          if (fr == 0) {
            red[(wave * 2 + 0) * BN + i * 16 + fk + q] = t0;
            red[(wave * 2 + 1) * BN + i * 16 + fk + q] = t1;
          }
        }
      const bool recomputed = __syncthreads_or(again_any);
      if (__builtin_expect(recomputed, 0)) __syncthreads();   // (and what was stored is there)
      if (tid < BN && n0 + tid < a.N) {
        float t0 = 0.f, t1 = 0.f;
        if (__builtin_expect(recomputed, 0)) {   // elements were computed again behind the sums: take them from what was stored
          const int end = a.M - m0 < BM ? a.M - m0 : BM;
          for (int r = 0; r < end; r++) {
            const float t = Cvt<T>::ld(out[(unsigned)(m0 + r) * (unsigned)a.N + (unsigned)(n0 + tid)]);
            t0 += t;
            t1 = fmaf(t, t, t1);
          }
        } else {
#pragma unroll
          for (int w = 0; w < 4; w++) { t0 += red[(w * 2 + 0) * BN + tid]; t1 += red[(w * 2 + 1) * BN + tid]; }
        }
        float* o = a.sums + (int64_t)blockIdx.x * stat_pitch(a.N) + n0 + tid;
        o[0] = t0;
        o[a.N] = t1;
      }
    }
  }
}

// Weight gradient: the output is small and the contraction (pixels) long, so the four waves of a block take 16 pixels each
// of a 64-pixel step for the whole 16 TN x 16 TK tile and are added in LDS at the end; the pixel range is split over the
// grid, partial sums are added in a fixed order by a second kernel.  Tiles lie in LDS as in memory ([pixel][channel]); rows
// are 16 floats apart modulo 64, so that the four pixels an instruction reads fall into different banks.
// The bias gradient comes with it: the workgroups of the first tile column add up the dy tiles that lie in LDS, in fp32 over the 4 TN
// pixels of a step that a thread has and in fp64 over the rest.
//
// A launch takes the weight gradients of all layers of a pass (kGenWgradJobs at the most), and one more launch adds up their splits:
// nothing in the pass reads them, and a layer by itself was a launch of 5 to 9 us that filled a part of the chip, 4 us for its splits and two
// launches for its bias.  A two-block fp32 network on 32 images of 32x32: seven layers 67 -> 30 us (26 and 5), the pass 263 -> 230; the
// two-layer network on 8 images 26 -> 12 us and six launches fewer, its step 173 -> 156.
struct GenWgradJob : GenArgs {
  double* bias_part;   // [splits][N] (more than one split) or null
  float* bias_out;     // [N] (one split) or null
  uint32_t first;      // workgroups of the jobs in front of this one
  int shape;           // of the tile: see gen_wgrad_shape
};
constexpr int kGenWgradJobs = 16;
struct GenWgradBatch { GenWgradJob j[kGenWgradJobs]; int n; };
static_assert(sizeof(GenWgradBatch) <= 4096, "the table travels in the kernel arguments");
// LDS floats of a tile shape
template <int TN, int TK> constexpr int gen_wgrad_floats() {
  constexpr int BN = 16 * TN, BKK = 16 * TK, PN = TN == 1 ? 16 : BN + 16, PK = TK == 1 ? 16 : BKK + 16;
  return 64 * (PN + PK) > 4 * BN * BKK ? 64 * (PN + PK) : 4 * BN * BKK;
}

template <typename T, int VEC, int TN, int TK>
__device__ inline void gen_wgrad_tile(const GenWgradJob& a, const unsigned wg, float* sm) {
  constexpr int BN = 16 * TN, BKK = 16 * TK, MS = 64;
  constexpr int PN = TN == 1 ? 16 : BN + 16, PK = TK == 1 ? 16 : BKK + 16;
  constexpr int NV = BN / VEC, KVN = BKK / VEC;
  constexpr int DR = 256 / NV, XR = 256 / KVN;              // rows per pass
  constexpr int DP = (MS + DR - 1) / DR, XP = (MS + XR - 1) / XR;
  float* Ds = sm;
  float* Xs = sm + MS * PN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int split = wg / (unsigned)a.tiles, tile = wg % (unsigned)a.tiles;
  const int n0 = tile / a.ktiles * BN, k0 = tile % a.ktiles * BKK;
  const int mbeg = split * a.m_per_split, mend = generic_split_end(a.M, mbeg, a.m_per_split);
  const T* __restrict__ x = static_cast<const T*>(a.src);
  const T* __restrict__ dy = static_cast<const T*>(a.w);
  const int dv = tid % NV, dr = tid / NV;
  const bool dok = n0 + dv * VEC < a.N;
  const int xv = tid % KVN, xr = tid / KVN;
  const int k = k0 + xv * VEC;
  const bool kok = k < a.K;
  const int tap = kok ? (int)div_by((unsigned)k, a.by_cin) : 0;
  const int kc = k - tap * a.Cin, kr = (int)div_by((unsigned)tap, a.by_kw), ks = tap - kr * a.kw;
  int pb[XP], ph[XP], pw[XP];
#pragma unroll
  for (int j = 0; j < XP; j++) {
    const unsigned m = (unsigned)(mbeg + xr + j * XR);
    const unsigned q = div_by(m, a.by_wo);
    pw[j] = (int)(m - q * (unsigned)a.Wo);
    pb[j] = (int)div_by(q, a.by_ho);
    ph[j] = (int)(q - (unsigned)pb[j] * (unsigned)a.Ho);
  }
  // one step moves every row MS pixels on: whole images, then whole rows, then columns
  const int adv_b = MS / (a.Ho * a.Wo), adv_r = MS % (a.Ho * a.Wo), adv_h = adv_r / a.Wo, adv_w = adv_r % a.Wo;
  float rd[DP][VEC], rx[XP][VEC];
  auto gload = [&](int ms) {   // ms: first pixel of the step
#pragma unroll
    for (int j = 0; j < DP; j++) {
      const int r = dr + j * DR, m = ms + r;
#pragma unroll
      for (int i = 0; i < VEC; i++) rd[j][i] = 0.f;
      if (dok && r < MS && m < mend) GenVec<T, VEC>::ld(dy + ((unsigned)m * (unsigned)a.N + (unsigned)(n0 + dv * VEC)), rd[j]);
    }
#pragma unroll
    for (int j = 0; j < XP; j++) {
      const int r = xr + j * XR, m = ms + r;
      const int h = ph[j] * a.stride - a.pad + kr, w = pw[j] * a.stride - a.pad + ks;
#pragma unroll
      for (int i = 0; i < VEC; i++) rx[j][i] = 0.f;
      if (kok && r < MS && m < mend && (unsigned)h < (unsigned)a.H && (unsigned)w < (unsigned)a.W)
        GenVec<T, VEC>::ld(x + ((unsigned)((pb[j] * a.H + h) * a.W + w) * (unsigned)a.Cin + (unsigned)kc), rx[j]);
      pw[j] += adv_w;
      const int cw = pw[j] >= a.Wo ? 1 : 0;
      pw[j] -= cw ? a.Wo : 0;
      ph[j] += adv_h + cw;
      const int ch = ph[j] >= a.Ho ? 1 : 0;
      ph[j] -= ch ? a.Ho : 0;
      pb[j] += adv_b + ch;
    }
  };
  f32x4_t acc[TN][TK];
#pragma unroll
  for (int i = 0; i < TN; i++)
#pragma unroll
    for (int j = 0; j < TK; j++) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const int fc = lane & 15, fm = wave * 16 + (lane >> 4);
  const bool bias = k0 == 0 && (a.bias_part || a.bias_out);   // uniform over the workgroup
  double bsum = 0.0;   // of channel n0 + tid % BN, pixels tid / BN + 256 / BN i of every step
  gload(mbeg);
  for (int ms = mbeg; ms < mend; ms += MS) {
#pragma unroll
    for (int j = 0; j < DP; j++)
      if (dr + j * DR < MS) {
#pragma unroll
        for (int i = 0; i < VEC; i++) Ds[(dr + j * DR) * PN + dv * VEC + i] = rd[j][i];
      }
#pragma unroll
    for (int j = 0; j < XP; j++)
      if (xr + j * XR < MS) {
#pragma unroll
        for (int i = 0; i < VEC; i++) Xs[(xr + j * XR) * PK + xv * VEC + i] = rx[j][i];
      }
    __syncthreads();
    if (ms + MS < mend) gload(ms + MS);
    if (bias) {   // (rows past the end are zeros)
      float t = 0.f;
#pragma unroll
      for (int i = 0; i < MS * BN / 256; i++) t += Ds[(tid / BN + i * (256 / BN)) * PN + tid % BN];
      bsum += (double)t;
    }
#pragma unroll
    for (int q = 0; q < 4; q++) {
      float d[TN], v[TK];
#pragma unroll
      for (int i = 0; i < TN; i++) d[i] = Ds[(fm + 4 * q) * PN + i * 16 + fc];
#pragma unroll
      for (int j = 0; j < TK; j++) v[j] = Xs[(fm + 4 * q) * PK + j * 16 + fc];
#pragma unroll
      for (int i = 0; i < TN; i++)
#pragma unroll
        for (int j = 0; j < TK; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(d[i], v[j], acc[i][j], 0, 0, 0);
    }
    __syncthreads();
  }
  // the four waves' sums, added in order
#pragma unroll
  for (int i = 0; i < TN; i++)
#pragma unroll
    for (int j = 0; j < TK; j++)
#pragma unroll
      for (int q = 0; q < 4; q++) sm[wave * BN * BKK + (i * 16 + 4 * (lane >> 4) + q) * BKK + j * 16 + fc] = acc[i][j][q];
  __syncthreads();
  float* __restrict__ out = static_cast<float*>(a.out) + (int64_t)split * a.N * a.K;
  bool again = false;
  for (int e = tid; e < BN * BKK; e += 256) {
    const int n = n0 + e / BKK, kk = k0 + e % BKK;
    if (n < a.N && kk < a.K) {
      const float t = (sm[e] + sm[BN * BKK + e]) + (sm[2 * BN * BKK + e] + sm[3 * BN * BKK + e]);
      out[(unsigned)n * (unsigned)a.K + (unsigned)kk] = t;
      again = again || t != t;
    }
  }
  if (__builtin_expect(__any(again), 0)) {
#pragma unroll 1
    for (int e = tid; e < BN * BKK; e += 256) {
      const int n = n0 + e / BKK, kk = k0 + e % BKK;
      if (n >= a.N || kk >= a.K) continue;
      float* o = out + ((unsigned)n * (unsigned)a.K + (unsigned)kk);
      if (*o != *o) *o = gen_wgrad_element<T>(a, n, kk, mbeg, mend);
    }
  }
  if (bias) {
    __syncthreads();
    double* red = reinterpret_cast<double*>(sm);   // [256 / BN][BN]
    red[tid] = bsum;
    __syncthreads();
    if (tid < BN && n0 + tid < a.N) {
      double s = 0.0;
      for (int l = 0; l < 256 / BN; l++) s += red[l * BN + tid];
      if (a.bias_part) a.bias_part[(int64_t)split * a.N + n0 + tid] = s;
      else a.bias_out[n0 + tid] = (float)s;
    }
  }
}

template <typename T>
__global__ void __launch_bounds__(256) conv_generic_wgrad_k(GenWgradBatch b) {
  __shared__ __attribute__((aligned(16))) float sm[gen_wgrad_floats<2, 4>()];   // the largest of the shapes below
  int k = 0;
  while (k + 1 < b.n && b.j[k + 1].first <= blockIdx.x) k++;
  const GenWgradJob& a = b.j[k];
  const unsigned wg = blockIdx.x - a.first;
  switch (a.shape) {   // (gen_wgrad_shape)
    case 0: gen_wgrad_tile<T, 1, 1, 2>(a, wg, sm); break;
    case 1: gen_wgrad_tile<T, 1, 2, 2>(a, wg, sm); break;
    case 4: gen_wgrad_tile<T, 4, 1, 2>(a, wg, sm); break;
    case 5: gen_wgrad_tile<T, 4, 2, 2>(a, wg, sm); break;
    case 6: gen_wgrad_tile<T, 4, 1, 4>(a, wg, sm); break;
    default: gen_wgrad_tile<T, 4, 2, 4>(a, wg, sm); break;
  }
}
static int gen_wgrad_shape(bool v4, int tn, int tk) { return (v4 ? 4 : 0) + (tk == 4 ? 2 : 0) + (tn == 2 ? 1 : 0); }

// The splits of those layers: 64 outputs x 4 split lanes to a block, every lane adds every 4th split, fixed-order combine in LDS; of more
// than 64 splits 16 outputs x 16 lanes (a lane's chain of loads is the launch's time).  Behind a
// job's outputs a block per 16 channels adds the bias sums.
struct GenSum { const float* part; float* out; const double* bias_part; float* bias_out; uint32_t n; int splits, N; uint32_t first, bias_first; };
struct GenSums { GenSum j[kGenWgradJobs]; int n; };
static_assert(sizeof(GenSums) <= 4096, "the table travels in the kernel arguments");
__host__ __device__ inline unsigned gen_sum_lanes(int splits) { return splits > 64 ? 16u : 4u; }
__global__ void __launch_bounds__(256) gen_wgrad_sum_k(GenSums b) {
  __shared__ double bs[256];
  float* sm = reinterpret_cast<float*>(bs);
  int k = 0;
  while (k + 1 < b.n && b.j[k + 1].first <= blockIdx.x) k++;
  const GenSum& q = b.j[k];
  if (blockIdx.x >= q.bias_first) {
    const int c = (int)(blockIdx.x - q.bias_first) * 16 + (int)threadIdx.x % 16, lane = (int)threadIdx.x / 16;
    double s = 0.0;
    if (c < q.N) {
#pragma unroll 8
      for (int j = lane; j < q.splits; j += 16) s += q.bias_part[(int64_t)j * q.N + c];
    }
    bs[threadIdx.x] = s;
    __syncthreads();
    if (lane == 0 && c < q.N) {
      for (int l = 1; l < 16; l++) s += bs[l * 16 + (int)threadIdx.x];
      q.bias_out[c] = (float)s;
    }
    return;
  }
  const unsigned lanes = gen_sum_lanes(q.splits), outs = 256u / lanes;
  const unsigned ol = threadIdx.x & (outs - 1u), lane = threadIdx.x / outs;
  const uint32_t i = (blockIdx.x - q.first) * outs + ol;
  float s = 0.f;
  if (i < q.n) {
#pragma unroll 8
    for (int j = (int)lane; j < q.splits; j += (int)lanes) s += q.part[(int64_t)j * q.n + i];
  }
  sm[threadIdx.x] = s;
  __syncthreads();
  if (lane == 0 && i < q.n) {
    float t = 0.f;
    for (unsigned l = 0; l < lanes; l += 4) t += (sm[l * outs + ol] + sm[(l + 1) * outs + ol]) + (sm[(l + 2) * outs + ol] + sm[(l + 3) * outs + ol]);
    q.out[i] = t;
  }
}

bool conv_generic_supported(const ConvGeom& g) {
  return generic_conv_fits(g.B, g.H, g.W, g.Cin, g.Ho, g.Wo, g.Cout, g.kh, g.kw, g.stride, g.pad);
}

static GenArgs gen_args(const ConvGeom& g) {
  GenArgs a = {};
  a.H = g.H; a.W = g.W; a.Cin = g.Cin; a.Ho = g.Ho; a.Wo = g.Wo; a.Cout = g.Cout;
  a.kh = g.kh; a.kw = g.kw; a.stride = g.stride; a.pad = g.pad;
  a.by_cin = fast_div((uint32_t)g.Cin); a.by_cout = fast_div((uint32_t)g.Cout); a.by_kw = fast_div((uint32_t)g.kw);
  a.by_stride = fast_div((uint32_t)g.stride);
  a.by_w = fast_div((uint32_t)g.W); a.by_h = fast_div((uint32_t)g.H); a.by_wo = fast_div((uint32_t)g.Wo); a.by_ho = fast_div((uint32_t)g.Ho);
  return a;
}

template <typename T, int MODE, int VEC, bool NORM>
static void launch_generic(const std::conditional_t<NORM, GenNormArgs, GenArgs>& a, hipStream_t s) {
  const int tn = generic_column_tiles(a.N);
  const int64_t nt = cdiv(a.N, 16 * tn);
  const bool tall = generic_tall_tiles(a.M, a.N, VEC == 4);
  const dim3 grid((unsigned)cdiv(a.M, tall ? 128 : 64), (unsigned)nt);
  if (tall) {
    constexpr int TM = VEC == 4 ? 2 : 1;
    if (tn == 1) hipLaunchKernelGGL((conv_generic_k<T, MODE, VEC, TM, 1, NORM>), grid, dim3(256), 0, s, a);
    else if (tn == 2) hipLaunchKernelGGL((conv_generic_k<T, MODE, VEC, TM, 2, NORM>), grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((conv_generic_k<T, MODE, VEC, TM, 4, NORM>), grid, dim3(256), 0, s, a);
  } else {
    if (tn == 1) hipLaunchKernelGGL((conv_generic_k<T, MODE, VEC, 1, 1, NORM>), grid, dim3(256), 0, s, a);
    else if (tn == 2) hipLaunchKernelGGL((conv_generic_k<T, MODE, VEC, 1, 2, NORM>), grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((conv_generic_k<T, MODE, VEC, 1, 4, NORM>), grid, dim3(256), 0, s, a);
  }
}

// four channels per load: both channel counts are multiples of 4 and the tensors start on a vector boundary
static bool gen_vec4(int dtype, const ConvGeom& g, const void* p0, const void* p1) {
  const uintptr_t mask = dtype == CD_BF16 ? 7 : 15;
  return g.Cin % 4 == 0 && g.Cout % 4 == 0 && ((reinterpret_cast<uintptr_t>(p0) | reinterpret_cast<uintptr_t>(p1)) & mask) == 0;
}

template <typename T, bool NORM>
static void fprop_generic_t(const std::conditional_t<NORM, GenNormArgs, GenArgs>& a, bool v4, hipStream_t s) {
  if (v4) launch_generic<T, 0, 4, NORM>(a, s); else launch_generic<T, 0, 1, NORM>(a, s);
}

int conv_fprop_generic(int dtype, const void* x, const void* w, const void* bias, void* y, const ConvGeom& g, bool relu,
                       hipStream_t s, const EvalNorm* norm, float* stat_partials, size_t stat_bytes) {
  GenNormArgs a = {gen_args(g), {}};
  a.src = x; a.w = w; a.bias = bias; a.out = y; a.relu = relu;
  a.M = (int)g.M(); a.N = g.Cout; a.K = g.K();
  const bool v4 = gen_vec4(dtype, g, x, w);
  if (norm) {
    a.norm = *norm;
    if (dtype == CD_BF16) fprop_generic_t<bf16_t, true>(a, v4, s); else fprop_generic_t<float, true>(a, v4, s);
    return 0;
  }
  const int64_t chunks = cdiv(a.M, generic_tall_tiles(a.M, a.N, v4) ? 128 : 64);
  if (stat_partials && generic_sums_pay(a.M, a.N, dtype == CD_BF16 ? 2 : 4, chunks) &&
      (size_t)(chunks + 2 * kFoldChunks) * stat_pitch(a.N) * sizeof(float) <= stat_bytes)
    a.sums = stat_partials;
  if (dtype == CD_BF16) fprop_generic_t<bf16_t, false>(a, v4, s); else fprop_generic_t<float, false>(a, v4, s);
  return a.sums ? (int)chunks : 0;
}

void conv_dgrad_generic(int dtype, const void* dy, const void* w, void* dx, const ConvGeom& g, bool accumulate, hipStream_t s) {
  GenArgs a = gen_args(g);
  a.src = dy; a.w = w; a.out = dx; a.accumulate = accumulate;
  a.M = (int)(g.B * g.H * g.W); a.N = g.Cin; a.K = g.kh * g.kw * g.Cout;
  const bool v4 = gen_vec4(dtype, g, dy, w);
  if (dtype == CD_BF16) { if (v4) launch_generic<bf16_t, 1, 4, false>(a, s); else launch_generic<bf16_t, 1, 1, false>(a, s); }
  else { if (v4) launch_generic<float, 1, 4, false>(a, s); else launch_generic<float, 1, 1, false>(a, s); }
}

void conv_wgrad_generic_batch(int dtype, const GenericWgradProblem* p, int n, float* partials, size_t partials_bytes, hipStream_t s) {
  GenWgradBatch b;
  GenSums sums;
  b.n = sums.n = 0;
  uint32_t blocks = 0, sum_blocks = 0;
  char* room = reinterpret_cast<char*>(partials);
  auto run = [&]() {
    if (b.n == 0) return;
    if (dtype == CD_BF16) hipLaunchKernelGGL(conv_generic_wgrad_k<bf16_t>, dim3(blocks), dim3(256), 0, s, b);
    else hipLaunchKernelGGL(conv_generic_wgrad_k<float>, dim3(blocks), dim3(256), 0, s, b);
    if (sums.n) hipLaunchKernelGGL(gen_wgrad_sum_k, dim3(sum_blocks), dim3(256), 0, s, sums);
    b.n = sums.n = 0;
    blocks = sum_blocks = 0;
    room = reinterpret_cast<char*>(partials);
  };
  for (int k = 0; k < n; k++) {
    const ConvGeom& g = p[k].g;
    const bool v4 = gen_vec4(dtype, g, p[k].x, p[k].dy);
    const int64_t nk = (int64_t)g.Cout * g.K();
    const GenericWgradPlan plan = generic_wgrad_plan(g.M(), g.Cout, g.K(), v4, partials_bytes);
    GenericWgradRoom need = generic_wgrad_room(plan, nk, g.Cout, p[k].db != nullptr);
    // (a layer may take all of the room for its dw: the bias sums of its splits then have none, and are added up from dy by themselves)
    const bool bias = p[k].db && need.dw + need.bias <= partials_bytes;
    if (!bias) need.bias = 0;
    const int64_t wgs = plan.tiles * plan.splits;   // (each layer's fit a launch: generic_conv_fits)
    const int64_t sum_wgs = plan.splits > 1 ? cdiv(nk, 256 / gen_sum_lanes((int)plan.splits)) + (bias ? cdiv(g.Cout, 16) : 0) : 0;
    if (b.n == kGenWgradJobs || (size_t)(room - reinterpret_cast<char*>(partials)) + need.dw + need.bias > partials_bytes ||
        blocks + wgs >= (1 << 24) || sum_blocks + sum_wgs >= (1 << 24))
      run();
    if (p[k].db && !bias) colsum(dtype, p[k].dy, g.M(), g.Cout, p[k].db, reinterpret_cast<float*>(room), s);
    GenWgradJob& a = b.j[b.n++];
    static_cast<GenArgs&>(a) = gen_args(g);
    a.src = p[k].x; a.w = p[k].dy; a.bias = nullptr;
    a.M = (int)g.M(); a.N = g.Cout; a.K = g.K();
    a.ktiles = (int)plan.ktiles; a.tiles = (int)plan.tiles; a.m_per_split = plan.m_per_split;
    a.shape = gen_wgrad_shape(v4, plan.tn, plan.tk);
    a.first = blocks;
    a.out = p[k].dw; a.bias_part = nullptr; a.bias_out = bias ? p[k].db : nullptr;
    blocks += (uint32_t)wgs;
    if (plan.splits > 1) {
      GenSum& q = sums.j[sums.n++];
      q.part = reinterpret_cast<float*>(room); q.out = p[k].dw; q.n = (uint32_t)nk; q.splits = (int)plan.splits; q.N = g.Cout;
      a.out = room;
      room += need.dw;
      q.first = sum_blocks;
      q.bias_first = 0xffffffffu; q.bias_part = nullptr; q.bias_out = nullptr;
      if (bias) {
        a.bias_part = reinterpret_cast<double*>(room);
        a.bias_out = nullptr;
        room += need.bias;
        q.bias_part = a.bias_part; q.bias_out = p[k].db;
        q.bias_first = sum_blocks + (uint32_t)cdiv(nk, 256 / gen_sum_lanes(q.splits));
      }
      sum_blocks += (uint32_t)sum_wgs;
    }
  }
  run();
}

}  // namespace cd
