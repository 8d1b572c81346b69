// LayerNorm forward / backward with a fused residual add (post-LayerNorm of a Transformer sublayer:
// y = LN(a + r); the paper's translation experiments, Section 4, train the Transformer of Vaswani
// et al.).  Rows are normalised over their last axis with the biased variance, eps 1e-5.
//
// HBM-bound.  One wavefront owns a row at a time: the row (sum of the two inputs) sits in registers
// between the reductions and the output (each input element is read once, each output written
// once), lanes hold 16-byte vectors at a 64-vector stride so that a wave's loads are contiguous,
// and the two row reductions are wave shuffles.  The backward pass also needs the column sums
// dgamma = sum_rows dy*xhat and dbeta = sum_rows dy: every wave keeps running sums of its own
// columns over the rows it visits (rows are dealt round-robin), a block writes them once, and a second
// kernel adds the blocks' partials in a fixed order (deterministic, no atomics).
#include "kernels.h"
#include <algorithm>

namespace cd {

constexpr float kLnEps = 1e-5f;

template <typename T> struct LnVec;
template <> struct LnVec<float> {
  static constexpr int N = 4;
  typedef float4 Raw;
  __device__ static void unpack(const Raw& t, float (&v)[4]) { v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w; }
  __device__ static Raw pack(const float (&v)[4]) { return make_float4(v[0], v[1], v[2], v[3]); }
};
template <> struct LnVec<bf16_t> {
  static constexpr int N = 8;
  typedef uint4 Raw;
  __device__ static void unpack(const Raw& t, float (&v)[8]) {
    const uint32_t u[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
    for (int i = 0; i < 4; i++) {
      v[2 * i] = __uint_as_float(u[i] << 16);
      v[2 * i + 1] = __uint_as_float(u[i] & 0xffff0000u);
    }
  }
  __device__ static Raw pack(const float (&v)[8]) {
    uint32_t u[4];
#pragma unroll
    for (int i = 0; i < 4; i++) u[i] = (uint32_t)f32_to_bf16(v[2 * i]) | ((uint32_t)f32_to_bf16(v[2 * i + 1]) << 16);
    return make_uint4(u[0], u[1], u[2], u[3]);
  }
};

// Vector path: d is a multiple of the vector width and at most 64 * NV vectors long; a lane holds
// vectors lane, lane + 64, ... of the row.  stats: [rows][2] = mean, rstd.
template <typename T, int NV>
__global__ void __launch_bounds__(256) ln_fwd_k(const T* __restrict__ a, const T* __restrict__ r,
                                                const T* __restrict__ gamma, const T* __restrict__ beta,
                                                T* __restrict__ y, float* __restrict__ stats, int64_t rows, int d) {
  constexpr int V = LnVec<T>::N;
  typedef typename LnVec<T>::Raw Raw;
  const int lane = threadIdx.x & 63;
  const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6), nwaves = (int64_t)gridDim.x * 4;
  const int nvec = d / V;
  const float inv_d = 1.f / (float)d;
  for (int64_t row = wave; row < rows; row += nwaves) {
    const T* ap = a + row * d;
    const T* rp = r ? r + row * d : nullptr;
    float s[NV][V];
    float sum = 0.f;
#pragma unroll
    for (int j = 0; j < NV; j++) {
      const int v = lane + 64 * j;
      if (v < nvec) {
        LnVec<T>::unpack(*reinterpret_cast<const Raw*>(ap + v * V), s[j]);
        if (rp) {
          float t[V];
          LnVec<T>::unpack(*reinterpret_cast<const Raw*>(rp + v * V), t);
#pragma unroll
          for (int k = 0; k < V; k++) s[j][k] += t[k];
        }
#pragma unroll
        for (int k = 0; k < V; k++) sum += s[j][k];
      }
    }
    const float mean = wave_sum(sum) * inv_d;
    float sq = 0.f;
#pragma unroll
    for (int j = 0; j < NV; j++)
      if (lane + 64 * j < nvec) {
#pragma unroll
        for (int k = 0; k < V; k++) { const float c = s[j][k] - mean; sq += c * c; }
      }
    const float rstd = rsqrtf(wave_sum(sq) * inv_d + kLnEps);
    if (lane == 0 && stats) { stats[row * 2] = mean; stats[row * 2 + 1] = rstd; }
#pragma unroll
    for (int j = 0; j < NV; j++) {
      const int v = lane + 64 * j;
      if (v < nvec) {
        float g[V], b[V], o[V];
        LnVec<T>::unpack(*reinterpret_cast<const Raw*>(gamma + v * V), g);
        LnVec<T>::unpack(*reinterpret_cast<const Raw*>(beta + v * V), b);
#pragma unroll
        for (int k = 0; k < V; k++) o[k] = (s[j][k] - mean) * rstd * g[k] + b[k];
        *reinterpret_cast<Raw*>(y + row * d + v * V) = LnVec<T>::pack(o);
      }
    }
  }
}

// One lane's share of a row of the backward pass, as loaded.
template <typename T, int NV> struct LnBwdRow {
  typedef typename LnVec<T>::Raw Raw;
  Raw dy[NV], a[NV], r[NV], da[NV], dr[NV];
  float mean, rstd;
};

// dx = rstd * (g - mean(g) - xhat * mean(g * xhat)), g = dy * gamma, xhat = (a + r - mean) * rstd.
// dx goes to da (added to what is there if acc_a) and to dr (the residual input, likewise).
// partials: [blocks][2][d] = the block's sums of dy (dbeta) and dy * xhat (dgamma).
// A wave's rows are a serial chain of loads, two reductions and stores: the next row is requested before the current one is
// reduced.  There are at most 256 blocks, whose waves add their column sums in LDS, so that few partials are left.  Two waves per
// SIMD, one for rows of two vectors per lane: a base Transformer step of 8192 rows of 512 takes 10.01 ms so and 10.05 with one,
// one layer each with 3840 rows of 1024 1.70 and 1.68.  More, fastest where nothing else runs (512 columns: 15.8 us with one, 11.1 with
// four), wait for room beside the weight gradients of the second stream: 10.12 ms.
template <typename T, int NV, int W>
__global__ void __launch_bounds__(64 * W) ln_bwd_k(const T* __restrict__ dy, const T* __restrict__ a,
                                                const T* __restrict__ r, const T* __restrict__ gamma,
                                                const float* __restrict__ stats, T* __restrict__ da, int acc_a,
                                                T* __restrict__ dr, int acc_r, float* __restrict__ partials,
                                                int64_t rows, int d) {
  constexpr int V = LnVec<T>::N;
  typedef typename LnVec<T>::Raw Raw;
  constexpr int PLANE = 64 * NV + 64 / V;   // column c lies at (c % V) * PLANE + c / V: no two lanes on one bank, written or read
  __shared__ float sums[W / 2][2][V * PLANE];
  const int lane = threadIdx.x & 63, wib = threadIdx.x >> 6;
  const int64_t wave = (int64_t)blockIdx.x * W + wib, nwaves = (int64_t)gridDim.x * W;
  const int nvec = d / V;
  const float inv_d = 1.f / (float)d;
  float g[NV][V], sb[NV][V], sg[NV][V];
  auto load = [&](int64_t row, LnBwdRow<T, NV>& x) {
    x.mean = stats[row * 2];
    x.rstd = stats[row * 2 + 1];
#pragma unroll
    for (int j = 0; j < NV; j++) {
      const int v = lane + 64 * j;
      if (v >= nvec) continue;
      const int64_t at = row * d + v * V;
      x.a[j] = *reinterpret_cast<const Raw*>(a + at);
      x.dy[j] = *reinterpret_cast<const Raw*>(dy + at);
      if (r) x.r[j] = *reinterpret_cast<const Raw*>(r + at);
      if (da && acc_a) x.da[j] = *reinterpret_cast<const Raw*>(da + at);
      if (dr && acc_r) x.dr[j] = *reinterpret_cast<const Raw*>(dr + at);
    }
  };
  LnBwdRow<T, NV> cur, next;
  if (wave < rows) load(wave, cur);
#pragma unroll
  for (int j = 0; j < NV; j++) {
    const int v = lane + 64 * j;
#pragma unroll
    for (int k = 0; k < V; k++) { sb[j][k] = 0.f; sg[j][k] = 0.f; g[j][k] = 0.f; }
    if (v < nvec) LnVec<T>::unpack(*reinterpret_cast<const Raw*>(gamma + v * V), g[j]);
  }
  for (int64_t row = wave; row < rows; row += nwaves) {
    if (row + nwaves < rows) load(row + nwaves, next);
    const float mean = cur.mean, rstd = cur.rstd;
    float xh[NV][V], gy[NV][V];
    float s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int j = 0; j < NV; j++) {
      const int v = lane + 64 * j;
      if (v < nvec) {
        float t[V], u[V];
        LnVec<T>::unpack(cur.a[j], xh[j]);
        if (r) {
          LnVec<T>::unpack(cur.r[j], t);
#pragma unroll
          for (int k = 0; k < V; k++) xh[j][k] += t[k];
        }
        LnVec<T>::unpack(cur.dy[j], u);
#pragma unroll
        for (int k = 0; k < V; k++) {
          xh[j][k] = (xh[j][k] - mean) * rstd;
          sb[j][k] += u[k];
          sg[j][k] += u[k] * xh[j][k];
          gy[j][k] = u[k] * g[j][k];
          s1 += gy[j][k];
          s2 += gy[j][k] * xh[j][k];
        }
      }
    }
    const float m1 = wave_sum(s1) * inv_d, m2 = wave_sum(s2) * inv_d;
#pragma unroll
    for (int j = 0; j < NV; j++) {
      const int v = lane + 64 * j;
      if (v < nvec) {
        float o[V], w[V];
#pragma unroll
        for (int k = 0; k < V; k++) o[k] = rstd * (gy[j][k] - m1 - xh[j][k] * m2);
        if (da) {
#pragma unroll
          for (int k = 0; k < V; k++) w[k] = 0.f;
          if (acc_a) LnVec<T>::unpack(cur.da[j], w);
#pragma unroll
          for (int k = 0; k < V; k++) w[k] = acc_a ? w[k] + o[k] : o[k];
          *reinterpret_cast<Raw*>(da + row * d + v * V) = LnVec<T>::pack(w);
        }
        if (dr) {
#pragma unroll
          for (int k = 0; k < V; k++) w[k] = 0.f;
          if (acc_r) LnVec<T>::unpack(cur.dr[j], w);
#pragma unroll
          for (int k = 0; k < V; k++) w[k] = acc_r ? w[k] + o[k] : o[k];
          *reinterpret_cast<Raw*>(dr + row * d + v * V) = LnVec<T>::pack(w);
        }
      }
    }
    cur = next;
  }
  auto each_sum = [&](auto&& f) {
    float (&mine)[2][V * PLANE] = sums[wib & (W / 2 - 1)];
#pragma unroll
    for (int j = 0; j < NV; j++)
#pragma unroll
      for (int k = 0; k < V; k++) {
        f(mine[0][k * PLANE + lane + 64 * j], sb[j][k]);
        f(mine[1][k * PLANE + lane + 64 * j], sg[j][k]);
      }
  };
  if (wib >= W / 2) each_sum([](float& m, float v) { m = v; });
  __syncthreads();
  if (wib < W / 2) each_sum([](float& m, float v) { m += v; });
  __syncthreads();
  for (int i = threadIdx.x; i < 2 * d; i += 64 * W) {
    const int q = i >= d, c = i - q * d, at = c % V * PLANE + c / V;
    float t = sums[0][q][at];
#pragma unroll
    for (int w = 1; w < W / 2; w++) t += sums[w][q][at];
    partials[((int64_t)blockIdx.x * 2 + q) * d + c] = t;
  }
}

// Any d, any alignment: one wave per row, scalar accesses, the row re-read per pass.
template <typename T>
__global__ void __launch_bounds__(256) ln_fwd_generic_k(const T* __restrict__ a, const T* __restrict__ r,
                                                        const T* __restrict__ gamma, const T* __restrict__ beta,
                                                        T* __restrict__ y, float* __restrict__ stats, int64_t rows, int d) {
  const int lane = threadIdx.x & 63;
  const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6), nwaves = (int64_t)gridDim.x * 4;
  for (int64_t row = wave; row < rows; row += nwaves) {
    float sum = 0.f;
    for (int c = lane; c < d; c += 64) sum += Cvt<T>::ld(a[row * d + c]) + (r ? Cvt<T>::ld(r[row * d + c]) : 0.f);
    const float mean = wave_sum(sum) / (float)d;
    float sq = 0.f;
    for (int c = lane; c < d; c += 64) {
      const float v = Cvt<T>::ld(a[row * d + c]) + (r ? Cvt<T>::ld(r[row * d + c]) : 0.f) - mean;
      sq += v * v;
    }
    const float rstd = rsqrtf(wave_sum(sq) / (float)d + kLnEps);
    if (lane == 0 && stats) { stats[row * 2] = mean; stats[row * 2 + 1] = rstd; }
    for (int c = lane; c < d; c += 64) {
      const float v = Cvt<T>::ld(a[row * d + c]) + (r ? Cvt<T>::ld(r[row * d + c]) : 0.f);
      y[row * d + c] = Cvt<T>::st((v - mean) * rstd * Cvt<T>::ld(gamma[c]) + Cvt<T>::ld(beta[c]));
    }
  }
}

// Generic backward: one wave per row for dx (no column sums here; see ln_colsum_generic_k).
template <typename T>
__global__ void __launch_bounds__(256) ln_bwd_generic_k(const T* __restrict__ dy, const T* __restrict__ a,
                                                        const T* __restrict__ r, const T* __restrict__ gamma,
                                                        const float* __restrict__ stats, T* __restrict__ da, int acc_a,
                                                        T* __restrict__ dr, int acc_r, int64_t rows, int d) {
  const int lane = threadIdx.x & 63;
  const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6), nwaves = (int64_t)gridDim.x * 4;
  for (int64_t row = wave; row < rows; row += nwaves) {
    const float mean = stats[row * 2], rstd = stats[row * 2 + 1];
    float s1 = 0.f, s2 = 0.f;
    for (int c = lane; c < d; c += 64) {
      const float xh = (Cvt<T>::ld(a[row * d + c]) + (r ? Cvt<T>::ld(r[row * d + c]) : 0.f) - mean) * rstd;
      const float gy = Cvt<T>::ld(dy[row * d + c]) * Cvt<T>::ld(gamma[c]);
      s1 += gy;
      s2 += gy * xh;
    }
    const float m1 = wave_sum(s1) / (float)d, m2 = wave_sum(s2) / (float)d;
    for (int c = lane; c < d; c += 64) {
      const float xh = (Cvt<T>::ld(a[row * d + c]) + (r ? Cvt<T>::ld(r[row * d + c]) : 0.f) - mean) * rstd;
      const float gy = Cvt<T>::ld(dy[row * d + c]) * Cvt<T>::ld(gamma[c]);
      const float o = rstd * (gy - m1 - xh * m2);
      if (da) da[row * d + c] = Cvt<T>::st(o + (acc_a ? Cvt<T>::ld(da[row * d + c]) : 0.f));
      if (dr) dr[row * d + c] = Cvt<T>::st(o + (acc_r ? Cvt<T>::ld(dr[row * d + c]) : 0.f));
    }
  }
}
// Generic column sums: thread = column, block y = row slice; partials [slices][2][d].
template <typename T>
__global__ void __launch_bounds__(256) ln_colsum_generic_k(const T* __restrict__ dy, const T* __restrict__ a,
                                                           const T* __restrict__ r, const float* __restrict__ stats,
                                                           float* __restrict__ partials, int64_t rows, int d) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= d) return;
  float sb = 0.f, sg = 0.f;
  for (int64_t row = blockIdx.y; row < rows; row += gridDim.y) {
    const float xh = (Cvt<T>::ld(a[row * d + c]) + (r ? Cvt<T>::ld(r[row * d + c]) : 0.f) - stats[row * 2]) * stats[row * 2 + 1];
    const float u = Cvt<T>::ld(dy[row * d + c]);
    sb += u;
    sg += u * xh;
  }
  partials[((int64_t)blockIdx.y * 2 + 0) * d + c] = sb;
  partials[((int64_t)blockIdx.y * 2 + 1) * d + c] = sg;
}

// Adds the partials in a fixed order, for all LayerNorms of a backward pass in one launch (blockIdx.y: the LayerNorm): block =
// 16 columns x 64 lanes, every lane adds every 64th partial, the 64 lanes of a column are combined in LDS.  (Sixteen columns are one
// 64-byte piece of a row.)  256 partials of 512 columns took 6.4 us between the kernels of the pass, 30 times in a base Transformer
// step; 17 us for the 30 together.
struct LnFinalizeJobs { LnFinalizeJob job[kLnFinalizeJobs]; };
__global__ void __launch_bounds__(1024) ln_finalize_k(LnFinalizeJobs jobs) {
  const LnFinalizeJob& jb = jobs.job[blockIdx.y];
  const float* __restrict__ partials = jb.partials;
  const int chunks = jb.chunks, d = jb.d;
  float* __restrict__ dgamma = jb.dgamma;
  float* __restrict__ dbeta = jb.dbeta;
  if ((int)blockIdx.x * 16 >= d) return;
  __shared__ float sm[2][64][17];
  const int cl = threadIdx.x & 15, lane = threadIdx.x >> 4;
  const int c = blockIdx.x * 16 + cl;
  float a0 = 0.f, a1 = 0.f;
  if (c < d) {
#pragma unroll 4
    for (int j = lane; j < chunks; j += 64) {
      a0 += partials[((int64_t)j * 2 + 0) * d + c];
      a1 += partials[((int64_t)j * 2 + 1) * d + c];
    }
  }
  sm[0][lane][cl] = a0;
  sm[1][lane][cl] = a1;
  for (int half = 32; half > 0; half >>= 1) {
    __syncthreads();
    if (lane < half) {
      sm[0][lane][cl] += sm[0][lane + half][cl];
      sm[1][lane][cl] += sm[1][lane + half][cl];
    }
  }
  if (lane != 0 || c >= d) return;   // (lane 0 wrote row 0 itself)
  dbeta[c] = sm[0][0][cl];
  dgamma[c] = sm[1][0][cl];
}

// Forward: a wave per row up to 64 Ki waves (a row's load, reductions and store are serial).
static int ln_blocks(int64_t rows, int64_t max_waves) {
  int64_t waves = rows < max_waves ? rows : max_waves;
  return (int)cdiv(waves, 4);
}
// Backward: blocks of `waves` waves, at most one per compute unit (each leaves a partial sum of every column).
static int ln_bwd_blocks(int64_t rows, int waves) { return (int)std::min<int64_t>(256, cdiv(rows, waves)); }

template <typename T>
static void ln_forward_t(const T* a, const T* r, const T* gamma, const T* beta, T* y, float* stats, int64_t rows, int d,
                         hipStream_t s) {
  constexpr int V = LnVec<T>::N;
  const bool vec = d % V == 0 && aligned16(a) && aligned16(r) && aligned16(gamma) && aligned16(beta) && aligned16(y) &&
                   d <= 64 * 8 * V;
  const dim3 grid(ln_blocks(rows, 65536)), block(256);
  if (!vec) {
    hipLaunchKernelGGL((ln_fwd_generic_k<T>), grid, block, 0, s, a, r, gamma, beta, y, stats, rows, d);
    return;
  }
  const int nv = (int)cdiv(d / V, 64);
#define CD_LN_FWD(NV) hipLaunchKernelGGL((ln_fwd_k<T, NV>), grid, block, 0, s, a, r, gamma, beta, y, stats, rows, d)
  if (nv <= 1) CD_LN_FWD(1); else if (nv <= 2) CD_LN_FWD(2); else if (nv <= 4) CD_LN_FWD(4); else CD_LN_FWD(8);
#undef CD_LN_FWD
}

template <typename T>
static int ln_backward_t(const T* dy, const T* a, const T* r, const T* gamma, const float* stats, T* da, bool acc_a,
                         T* dr, bool acc_r, float* partials, int64_t rows, int d, hipStream_t s) {
  constexpr int V = LnVec<T>::N;
  const bool vec = d % V == 0 && aligned16(dy) && aligned16(a) && aligned16(r) && aligned16(gamma) && aligned16(da) &&
                   aligned16(dr) && d <= 64 * 2 * V;   // (the row, its gradient and the running sums stay in registers)
  if (vec) {
#define CD_LN_BWD(NV, W)                                                                                          \
  {                                                                                                               \
    const int blocks = ln_bwd_blocks(rows, W);                                                                    \
    hipLaunchKernelGGL((ln_bwd_k<T, NV, W>), dim3(blocks), dim3(64 * W), 0, s, dy, a, r, gamma, stats, da, (int)acc_a, dr, \
                       (int)acc_r, partials, rows, d);                                                            \
    return blocks;                                                                                                \
  }
    if (cdiv(d / V, 64) <= 1) CD_LN_BWD(1, 8)
    CD_LN_BWD(2, 4)
#undef CD_LN_BWD
  }
  const int chunks = rows < 64 ? (int)rows : 64;
  hipLaunchKernelGGL((ln_bwd_generic_k<T>), dim3(ln_blocks(rows, 1024)), dim3(256), 0, s, dy, a, r, gamma, stats, da, (int)acc_a, dr,
                     (int)acc_r, rows, d);
  hipLaunchKernelGGL((ln_colsum_generic_k<T>), dim3((unsigned)cdiv(d, 256), chunks), dim3(256), 0, s, dy, a, r, stats,
                     partials, rows, d);
  return chunks;
}

void ln_forward(int dtype, const void* a, const void* r, const void* gamma, const void* beta, void* y, float* stats,
                int64_t rows, int d, hipStream_t s) {
  if (dtype == CD_BF16)
    ln_forward_t<bf16_t>((const bf16_t*)a, (const bf16_t*)r, (const bf16_t*)gamma, (const bf16_t*)beta, (bf16_t*)y, stats,
                         rows, d, s);
  else
    ln_forward_t<float>((const float*)a, (const float*)r, (const float*)gamma, (const float*)beta, (float*)y, stats, rows,
                        d, s);
}

size_t ln_partials_bytes(int64_t rows, int d) { return (size_t)std::min<int64_t>(256, rows) * 2 * d * sizeof(float); }

int ln_backward(int dtype, const void* dy, const void* a, const void* r, const void* gamma, const float* stats, void* da,
                bool acc_a, void* dr, bool acc_r, float* partials, int64_t rows, int d, hipStream_t s) {
  if (dtype == CD_BF16)
    return ln_backward_t<bf16_t>((const bf16_t*)dy, (const bf16_t*)a, (const bf16_t*)r, (const bf16_t*)gamma, stats, (bf16_t*)da,
                                 acc_a, (bf16_t*)dr, acc_r, partials, rows, d, s);
  return ln_backward_t<float>((const float*)dy, (const float*)a, (const float*)r, (const float*)gamma, stats, (float*)da, acc_a,
                              (float*)dr, acc_r, partials, rows, d, s);
}

void ln_finalize(const LnFinalizeJob* jobs, int n, hipStream_t s) {
  for (int i0 = 0; i0 < n; i0 += kLnFinalizeJobs) {
    LnFinalizeJobs t = {};
    const int m = std::min(kLnFinalizeJobs, n - i0);
    int d = 0;
    for (int i = 0; i < m; i++) {
      t.job[i] = jobs[i0 + i];
      d = std::max(d, t.job[i].d);
    }
    hipLaunchKernelGGL(ln_finalize_k, dim3((unsigned)cdiv(d, 16), m), dim3(1024), 0, s, t);
  }
}

}  // namespace cd
