// Host rules of the convolution launches, in plain integers: no HIP header is needed, so that they can be compiled and
// checked on a machine without a GPU.  (constexpr functions are callable from device code.)
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace cd {

// ---- what conv_generic.hip takes ----------------------------------------------------------------------------------------
// 32-bit element offsets, and launches within the runtime's limits: fewer than 2^32 threads along x (256 for each 64 pixels,
// input or output, and for each tile of a weight gradient, at the least 16 x 32 elements), 65535 blocks along y (64 channels
// each).  (The runtime refused a launch of 2^32 threads, but took one of 2^33 - 2^15,
// whose count does not fit 32 bits, without an error.)  Beyond that the plain kernels run, one thread per element with 64-bit offsets.
inline bool generic_conv_fits(int64_t B, int64_t H, int64_t W, int64_t Cin, int64_t Ho, int64_t Wo, int64_t Cout, int64_t kh,
                              int64_t kw, int64_t stride, int64_t pad) {
  const int64_t lim = 1LL << 31, blocks = (1LL << 24) - 1, rows = 64 * blocks, channels = 64 * 65535LL;
  const int64_t in = B * H * W, out = B * Ho * Wo;
  return in <= rows && out <= rows && Cin <= channels && Cout <= channels && in * Cin < lim && out * Cout < lim &&
         Cout * kh * kw * Cin < lim && ((Cout + 15) / 16) * ((kh * kw * Cin + 31) / 32) + 768 <= blocks &&
         H < (1 << 24) && W < (1 << 24) && pad >= 0 && stride >= 1;
}

// Whether a weight gradient goes to conv_generic.hip.  A handful of weights over few pixels is one launch of the plain kernel,
// a block per weight, all of them resident (1024: four a compute unit); here it is a split launch and its reduction.  Both
// gradients of the two-layer network, 1 and 1 channels (9 and 27 weights): 1024 pixels 11.2 us plain, 18.9 here; 2048 15.7 and 23.8;
// 4096 23.1 and 22.1.
inline bool generic_wgrad_pays(int64_t M, int64_t weights) { return M > 2048 || weights > 1024; }

// ---- weight gradient of conv_generic.hip: a 16 tn x 16 tk tile of dw per block, the pixel range cut into splits ----
struct GenericWgradPlan {
  int tn, tk;              // 16-wide tiles of output channels and of (tap, input channel) per block
  int64_t ktiles, tiles;   // tiles along the contraction side of dw, tiles altogether
  int64_t splits;
  int m_per_split;         // pixels per split, a multiple of the 64 a step takes
};

// M pixels, N output channels, K = taps x input channels; v4: four channels per load
inline GenericWgradPlan generic_wgrad_plan(int64_t M, int N, int K, bool v4, size_t partials_bytes) {
  auto up = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
  GenericWgradPlan p;
  p.tn = N <= 16 ? 1 : 2;
  p.tk = v4 ? (K <= 32 ? 2 : 4) : 2;
  p.ktiles = up(K, 16 * p.tk);
  p.tiles = up(N, 16 * p.tn) * p.ktiles;
  // three workgroups per compute unit, but at least two 64-pixel steps each (a split costs one fp32 copy of dw), and no splits
  // of four steps or fewer, where the reduction's launch takes longer (16 and 32 channels, 256 pixels: both gradients 23.7 us
  // split, 17.4 not; 512 pixels 23.7 and 26.1)
  p.splits = M <= 256 ? 1 : up(768, p.tiles);
  if (p.splits > up(M, 128)) p.splits = up(M, 128);
  const int64_t by_mem = (int64_t)(partials_bytes / ((size_t)N * K * sizeof(float)));
  if (p.splits > by_mem) p.splits = by_mem;
  if (p.splits < 1) p.splits = 1;
  p.m_per_split = (int)(up(up(M, p.splits), 64) * 64);
  p.splits = up(M, p.m_per_split);
  return p;
}
// first pixel behind the split that starts at mbeg < M (the splits overshoot M by up to 64 pixels each: mbeg + m_per_split need
// not fit 32 bits)
constexpr int generic_split_end(int M, int mbeg, int m_per_split) {
  return M - mbeg > m_per_split ? mbeg + m_per_split : M;
}

}  // namespace cd
