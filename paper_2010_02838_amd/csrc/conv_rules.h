// Host rules of the convolution and dense-layer launches, in plain integers: no HIP header is needed, so that they can be compiled and
// checked on a machine without a GPU.  (constexpr functions are callable from device code.)
#pragma once
#include <stddef.h>
#include <stdint.h>
#include <algorithm>

namespace cd {

// ---- division by a number that is the same for a whole launch -----------------------------------------------------------------
// n / d for n < 2^31, d >= 1 as (2 n mul / 2^32) >> shift: with 2^shift >= d > 2^(shift - 1) and mul = ceil(2^(31 + shift) / d) < 2^32 the
// excess mul d - 2^(31 + shift) is less than d <= 2^shift, so n times it stays below 2^(31 + shift).
struct FastDiv { uint32_t mul, shift; };
inline FastDiv fast_div(uint32_t d) {
  FastDiv f = {0, 0};
  while ((1ull << f.shift) < d) f.shift++;
  f.mul = (uint32_t)(((1ull << (31 + f.shift)) + d - 1) / d);
  return f;
}

// ---- output tile of the matrix-core convolutions (conv_mfma.hip) ------------------------------------------------------------
// Tiles, measured with random operands that come from memory (constant ones leave the matrix cores a higher clock), on the
// layer shapes of ResNet-50 at batch 256 and 50, Wide-ResNet at 96 and the Transformer (us):
//  - more than 256 tiles of 128x128: 128x256 up to K = 1024 (a short contraction leaves a tile little more than its
//    prologue and epilogue; 200704 x 512 x 128 93 -> 81, 50176 x 256 x 1024 50 -> 46, 8192 x 1536 x 512 28 -> 25; 12544 x 512 x
//    2048 42 either way), 256x128 where its rounds of 512 workgroups are no emptier (50176 x 256 x 2304 80 -> 76: the clock
//    follows the power, and a larger tile moves fewer bytes per product);
//  - of those, launches that also take a BatchNorm's column sums choose by rows first: a tile is one fp32 partial sum, and where
//    256 rows went into one in place of 128 (or the other way) the batch statistics and all roundings behind them moved.  They
//    keep 256x128 for K <= 128 onto N >= 512 and where its last round is 1.2 times fuller, otherwise 128 rows.  (With 256
//    tiles or fewer they choose like the others: a 64-row tile halves the rows of a partial sum, so the statistics of small
//    batches did move when these tiles came.)
//  - where 128x128 tiles do not fill the 256 compute units, or fill them unevenly, 128x64 and 64x64 tiles do: the cost of
//    a tile shape is the number of workgroups on the busiest unit times what one costs there (128x64 0.7 of a 128x128
//    one, 64x64 half), but no less than what one takes alone (1.4, 1.08 and 0.75): 2450 x 512 x 4608 (80 tiles of 128x128)
//    49 -> 26 on 312 of 64x64, 24576 x 320 x 2880 74 -> 66 on 128x64 (five columns of 64 instead of three of 128).
enum { TILE_SQUARE = 0, TILE_TALL = 1, TILE_WIDE = 2, TILE_NARROW = 3, TILE_SMALL = 4, TILE_160 = 5, TILE_256 = 6, TILE_WIDE8 = 7 };   // 128x128 256x128 128x256 128x64 64x64 128x160 256x256 128x256
// M rows, N > 64 columns, contraction K; small_tiles: the 64-wide steps that the last two need fit; sums: takes column sums
inline int conv_tile_rule(int64_t M, int N, int K, bool small_tiles, bool sums) {
  auto cdiv = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
  const int64_t t128 = cdiv(M, 128) * cdiv(N, 128), t256 = cdiv(M, 256) * cdiv(N, 128);
  if (sums && t128 > 256) {
    if (K <= 128 && N >= 512) return TILE_TALL;
    if (N % 256 == 0 && K <= 1024) return TILE_WIDE;
    const double e128 = (double)t128 / (double)(cdiv(t128, 768) * 768), e256 = (double)t256 / (double)(cdiv(t256, 512) * 512);
    if (e256 > 1.2 * e128) return TILE_TALL;
  }
  if (t128 > 256 && N % 256 == 0 && K <= 1024) return TILE_WIDE;
  const double square = std::max(1.4, (double)cdiv(t128, 256));
  double narrow = 1e30, small = 1e30;
  if (small_tiles) {   // (their kernels take 64-wide steps)
    narrow = std::max(1.08, (K <= 1024 ? 0.68 : 0.72) * (double)cdiv(cdiv(M, 128) * cdiv(N, 64), 256));
    small = std::max(0.75, 0.5 * (double)cdiv(cdiv(M, 64) * cdiv(N, 64), 256));
  }
  if (t128 > 256) {
    if (narrow < 0.97 * square) return TILE_NARROW;
    if (sums) return TILE_SQUARE;
    const double e128 = (double)t128 / (double)(cdiv(t128, 512) * 512), e256 = (double)t256 / (double)(cdiv(t256, 512) * 512);
    return t128 > 512 && e256 >= e128 ? TILE_TALL : TILE_SQUARE;
  }
  return small < narrow && small < square ? TILE_SMALL : narrow < square ? TILE_NARROW : TILE_SQUARE;
}

// Tiles of eight waves on a compute unit of their own, 64-wide steps: 128x256 in three stages or 256x256 in two (0: neither; asked first).
// A 32-wide step reads rows in 64-byte segments, 31 B a cycle and compute unit against 52 in 128-byte ones, which two workgroups of 128x256
// tiles wait for (8192 x 2048 x 512: 25000 cycles of loads, 16000 of matrix instructions; 256x256 tiles 10000).  They pay where they fill most
// of a round of 256 compute units: 144 tiles and more of one, or seven eighths of two.  us, without and with, 128x256: 10240 x 512 x 2048 (160) 39
// -> 31, 12544 x 512 x 2048 (196) 41 -> 33, 9408 x 512 x 4608 (148) 54 -> 49, 7168 x 1024 x 1024 (224) 20.1 -> 17.5, 2560 x 2048 x 512
// (160) 12.8 -> 11.5, outside 4096 x 1024 x 1024 (128) 13.4 and 15.7, 5120 x 2048 x 512 (320) 19.5 and 20.2; 256x256: 3840 x 4096 x
// 1024 (240) 38 -> 30, 50176 x 256 x 2304 (196) 75 -> 62, 8192 x 2048 x 512 (256) 27 -> 23.5, 6144 x 1536 x 512 (144) 19.3 -> 16.8, 16384
// x 2048 x 512 (512) 48 -> 41, outside 4096 x 2048 x 512 (128) 14.6 and 17.0, 12288 x 2048 x 512 (384) 37 and 39, 75264 x 256 x 512
// (294) 40 and 46.  Contractions below 256 live on the overlap of several workgroups (802816 x 256 x 64 101 and 122).
inline int conv_eight_waves_rule(int64_t M, int N, int K, bool wide_steps) {   // wide_steps: 64-wide steps fit
  if (N % 256 || K < 256 || !wide_steps) return 0;
  const int64_t half = (M + 127) / 128 * (N / 256), full = (M + 255) / 256 * (N / 256);
  if (half >= 144 && half <= 256) return TILE_WIDE8;
  return (full >= 144 && full <= 256) || (full >= 448 && full <= 512) ? TILE_256 : 0;
}

// Whether a width that 160 divides takes 128x160 tiles instead (asked before conv_tile_rule).  160 columns are two of 128, 37 % of them
// padding, and 320 two and a half; a 128x160 tile also moves a tenth fewer bytes per product than a 128x128 one and two fifths fewer than a
// 128x64 one.  In units of a 128x128 tile a pair of them on a compute unit costs 2.6 and one 1.9; of the narrow ones a
// last round on a fifth of the units does not count.  us, without and with: 98304 x 160 x 1440 74 -> 62, 131072 x 160 x 1440 94 -> 69, 32768 x 160 x 1440 26.7 -> 23, 24576 x 320 x 2880
// 55 -> 48, 32768 x 320 x 2880 64 -> 51, 65536 x 480 x 480 64 -> 56; on the other side of the line 16384 x 160 x 1440 16.1 and 20.8, 12288 x
// 320 x 2880 27.9 and 32, 20480 x 320 x 2880 (narrow tiles, 3.1 a unit) 38 and 46, 6144 x 640 x 5760 43 and 61.  (256x160 tiles of eight
// waves 47 for 24576 x 320 x 2880, 61 for 98304 x 160 x 1440, and behind on fewer rows; a partial sum keeps its 128 rows so.)
inline bool conv_cols160_rule(int64_t M, int N, int K, bool wide_steps) {   // wide_steps: the 64-wide steps that the tile needs fit
  auto cdiv = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
  if (N % 160 || !wide_steps) return false;
  const int64_t per = cdiv(cdiv(M, 128) * (N / 160), 256);   // on the busiest compute unit
  const double each = 2.6 * (double)(per / 2) + 1.9 * (double)(per % 2);
  const double square = std::max(1.4, (double)cdiv(cdiv(M, 128) * cdiv(N, 128), 256));
  const double narrow = std::max(1.08, (K <= 1024 ? 0.68 : 0.72) * (double)cdiv(cdiv(M, 128) * cdiv(N, 64) - 51, 256));
  return each < 0.98 * std::min(square, narrow);
}

// Rows of a tile where there are at most 64 columns (one column tile): 256, but 128 or 64 (64 only from 33 columns on) while those leave
// compute units without a tile.  A launch with column sums takes as many row tiles as the BatchNorm behind it adds up by itself
// (kSumBytes below: 64 KB, 8 bytes a column and tile).  ResNet-20 at batch 128, 256 rows before and now: 8192 x 64 x 576 (32 tiles) 10.1 ->
// 6.3 us, its data gradient with sums 13.7 -> 8.5, 32768 x 32 x 288 (128 tiles) 7.9 -> 6.1 and 10.2 -> 8.3.  A contraction of four 32-wide
// steps or fewer is all prologue and epilogue: 5.6 us either way (8192 x 16 x 32, 2048 x 64 x 32).
inline int conv_rows_rule(int64_t M, int N, int K, bool sums) {
  if (K <= 128) return 256;
  const int64_t most = sums ? (64 << 10) / (8 * (N <= 32 ? 32 : 64)) : 256;
  if (N > 32 && (M + 63) / 64 <= most) return 64;
  return (M + 127) / 128 <= most ? 128 : 256;
}

// Row tiles, i.e. partial sums, of a launch over M rows that takes column sums, at the most: 64-row tiles are chosen only where
// there are at most 256 tiles of 128x128.
inline int64_t conv_stat_chunks_max(int64_t M) { return M <= 256 * 128 ? (M + 63) / 64 : (M + 127) / 128; }
// room for them and for the 32 rows they are folded into, each of `pitch` floats (stat_pitch)
inline bool conv_sums_fit(int64_t M, int64_t pitch, size_t bytes) {
  return (size_t)(conv_stat_chunks_max(M) + 32) * pitch * sizeof(float) <= bytes;
}

// ---- weight gradients of the matrix-core path (conv_mfma.hip) -----------------------------------------------------------------
constexpr int kWgradJobs = 16;     // layers in a launch: their table travels in the kernel arguments
constexpr int kWgradStages = 3;
constexpr int kWgradBlocks = 512;  // workgroups a launch of several layers aims for: two a compute unit
struct WgradShape {
  int64_t M = 0;        // pixels (rows)
  int N = 0, K = 0;     // dw [N][K], per slice
  int taps = 0, slices = 0;
  bool pointwise = false, bias = false;   // bias: the bias gradient comes with it
  int bn() const { return N > 64 ? 128 : 64; }
  int bk() const { return K > 64 ? 128 : 64; }
  int tile_class() const { return (bn() == 128 ? 4 : 0) + (bk() == 128 ? 2 : 0) + (pointwise ? 1 : 0); }
  int64_t tiles() const { return (int64_t)((N + bn() - 1) / bn()) * ((K + bk() - 1) / bk()) * slices; }
  int64_t steps() const { return (M + 31) / 32; }
  int64_t weights() const { return (int64_t)N * K * slices; }
  // bytes of partial sums, each part on a 256-byte boundary
  int64_t partials(int64_t splits) const {
    return splits < 2 ? 0 : (weights() * splits * 4 + 255) / 256 * 256 + (bias ? (N * splits * 8 + 255) / 256 * 256 : 0);
  }
};
struct WgradSplit { int64_t splits, m_per_split; };   // m_per_split: a multiple of the 32 pixels of a step

// How many splits the pixels of n layers (one tile class) in one launch are cut into.  tune > 0: workgroups to aim for instead.
inline void wgrad_plan(const WgradShape* s, int n, size_t partials_bytes, int tune, WgradSplit* out) {
  auto up = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
  auto cut = [&](const WgradShape& h, int64_t splits) {
    WgradSplit r;
    splits = std::max<int64_t>(1, std::min(splits, up(h.M, 4 * 32)));
    r.m_per_split = up(up(h.M, splits), 32) * 32;
    r.splits = up(h.M, r.m_per_split);
    return r;
  };
  if (n == 1) {
    // A layer by itself (measured on the layer shapes of ResNet-50 at batch 256).  Every split writes
    // an fp32 copy of dw, so 1x1 filters with small N*K/(N+K) (few flops per byte of dy and x: the launch
    // is bound by memory traffic whatever the split) run one long workgroup per compute unit; the other
    // 1x1 launches take two, gathers over several taps four.
    const WgradShape& h = s[0];
    int64_t target = 1024;
    if (h.taps == 1) target = (double)h.N * h.K / ((double)h.N + h.K) < 150.0 ? 256 : 512;
    if (tune > 0) target = tune;
    int64_t splits = up(target, h.tiles());
    out[0] = cut(h, splits);
    while (out[0].splits > 1 && h.partials(out[0].splits) > (int64_t)partials_bytes) out[0] = cut(h, out[0].splits - 1);
    return;
  }
  // Several layers: as many steps to a workgroup as give the launch kWgradBlocks of them, the same for every layer, so that they end
  // together; one split each where the tiles alone are that many.
  int64_t work = 0;
  for (int k = 0; k < n; k++) work += s[k].tiles() * s[k].steps();
  const int64_t target = tune > 0 ? tune : kWgradBlocks;
  for (int64_t per = std::max<int64_t>(4, up(work, target));; per += std::max<int64_t>(1, per / 16)) {
    int64_t blocks = 0, bytes = 0;
    bool whole = true;
    for (int k = 0; k < n; k++) {
      out[k] = cut(s[k], up(s[k].steps(), per));
      blocks += s[k].tiles() * out[k].splits;
      bytes += s[k].partials(out[k].splits);
      whole = whole && out[k].splits == 1;
    }
    if (whole || (blocks <= target && bytes <= (int64_t)partials_bytes)) return;
  }
}
// Rows (whole steps) of a split of this layer by itself, whatever launch it is in.
inline int64_t wgrad_own_rows(const WgradShape& h, size_t partials_bytes) {
  WgradSplit r;
  wgrad_plan(&h, 1, partials_bytes, 0, &r);
  return r.m_per_split;
}
// Whether a layer by itself loses little: its splits' partial sums, written and read again, are a small part of what its operands move.
inline bool wgrad_alone(const WgradShape& h, int64_t operand_bytes) {
  WgradSplit r;
  wgrad_plan(&h, 1, ~(size_t)0 >> 1, 0, &r);
  return r.splits == 1 || 4 * (2 * h.partials(r.splits)) <= operand_bytes;
}
// Whether a layer by itself would be over before it has begun: 16 steps a workgroup or fewer, so that most of its time goes into the first
// loads, the stores and the splits' sums.  (ResNet-20's step at batch 128, whose 16-channel layers are 8 steps by themselves: 177 launches and
// ten forks -> 161 and four, 976 -> 905 us replayed from a graph.)
inline bool wgrad_short(const WgradShape& h) {
  WgradSplit r;
  wgrad_plan(&h, 1, ~(size_t)0 >> 1, 0, &r);
  return r.m_per_split <= 16 * 32;
}
// Whether a pass's layers, those that go by themselves included, are so little work altogether (their tiles' steps: 128 in each of 512
// workgroups, some 30 us) that none of them forks: those that wait go at its end, all of them on the caller's stream.  Beside the rest of a small pass they take the compute units that its short launches wait for, and an
// event and a wait are 15 us of the host's time and a gap on the device.  us a pass, with forks and without, by work (512 tile steps): two basic
// blocks of 16 and 32 channels on 80 images of 28x35 (26) 307 and 286, two bottleneck blocks on 30 images of 112x113 (25) 618 and 608, ResNeXt's
// on 19 of 160x161 (42) 905 and 882 and on 45 of 160x160 (96) 1448 and 1422, two Wide-ResNet blocks on 28 images (90) 782 and 744,
// bottleneck blocks on 70 of 96x96 (115) 1036 and 1020; above the line ResNet-20's step at batch 128 (146) 873 and 926, bottleneck blocks on 34
// images of 192x192 (205) 1564 and 1612.  Layers of at most 64 output channels count 1.4: the other launches of their pass leave part of the chip
// idle; basic blocks of 16 and 32 channels on 226 images of 32x32 (98, almost all narrow) 525 and 554, of 64 and 128 on 36 images of 224x225 (96, of
// which 70) 778 and 744.  Where only the waiting layers counted, large batches came back below the line with forks and a late launch: bottleneck blocks
// on 50 images of 192x192 1254, now 1206, ResNeXt's on 90 of 160x160 2341 and 2315, basic ones on 800 of 32x32 795 and 778.  (Behind one fork, when all or half of them have come: slower than either.)
inline bool wgrad_together(int64_t work, int64_t narrow) { return work + narrow * 2 / 5 < (int64_t)kWgradBlocks * 128; }
// Whether the layers collected so far are a launch: tiles enough without a split, or enough work for every compute unit to be busy
// some 20 us (96 steps in each of 512 workgroups), or as much as the pass still has to collect and worth a launch, or all of them:
// launches run beside the data gradients of the layers in front, and what is launched at the end of the pass runs beside nothing (two
// bottleneck blocks on 43 images of 64x96: 774 us a pass with the last launches at its end, 721 with each as soon as its class is
// complete, 743 with a launch per layer; basic blocks at 160x161 698, 664 and 713).
inline bool wgrad_batch_full(int64_t tiles, int64_t work, int jobs, int64_t work_left) {
  return jobs >= kWgradJobs || tiles >= kWgradBlocks || work >= (int64_t)kWgradBlocks * 96 || work_left == 0 ||
         (work >= work_left && work >= (int64_t)kWgradBlocks * 16);
}

// ---- what conv_generic.hip takes ----------------------------------------------------------------------------------------
// 32-bit element offsets, and launches within the runtime's limits: fewer than 2^32 threads along x (256 for each 64 pixels,
// input or output, and for each tile of a weight gradient, at the least 16 x 32 elements), 65535 blocks along y (64 channels
// each).  (The runtime refused a launch of 2^32 threads, but took one of 2^33 - 2^15, whose count does not fit 32 bits, without
// an error.)  Beyond that the plain kernels run, one thread per element with 64-bit offsets.
inline bool generic_conv_fits(int64_t B, int64_t H, int64_t W, int64_t Cin, int64_t Ho, int64_t Wo, int64_t Cout, int64_t kh,
                              int64_t kw, int64_t stride, int64_t pad) {
  const int64_t lim = 1LL << 31, blocks = (1LL << 24) - 1, rows = 64 * blocks, channels = 64 * 65535LL;
  const int64_t in = B * H * W, out = B * Ho * Wo;
  return in <= rows && out <= rows && Cin <= channels && Cout <= channels && in * Cin < lim && out * Cout < lim &&
         Cout * kh * kw * Cin < lim && ((Cout + 15) / 16) * ((kh * kw * Cin + 31) / 32) + 768 <= blocks &&
         H < (1 << 24) && W < (1 << 24) && pad >= 0 && stride >= 1;
}

// Forward and data gradient there: 16-column tiles side by side in a block, and whether its rows are 128 instead of 64: once
// 128-row tiles give every compute unit two workgroups (below that twice as many of 64 rows), with four channels per load.
inline int generic_column_tiles(int N) { return N <= 16 ? 1 : N <= 32 ? 2 : 4; }
inline bool generic_tall_tiles(int64_t M, int N, bool v4) {
  const int64_t bn = 16 * generic_column_tiles(N);
  return v4 && (M + 127) / 128 * ((N + bn - 1) / bn) >= 512;
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
// bytes of the partial sums of dw and of the bias gradient, on 256-byte boundaries (none without a split)
struct GenericWgradRoom { size_t dw, bias; };
inline GenericWgradRoom generic_wgrad_room(const GenericWgradPlan& p, int64_t weights, int N, bool bias) {
  if (p.splits < 2) return {0, 0};
  return {(size_t)((weights * p.splits * 4 + 255) / 256 * 256), bias ? (size_t)((N * p.splits * 8 + 255) / 256 * 256) : 0};
}
// first pixel behind the split that starts at mbeg < M (the splits overshoot M by up to 64 pixels each: mbeg + m_per_split need
// not fit 32 bits)
constexpr int generic_split_end(int M, int mbeg, int m_per_split) {
  return M - mbeg > m_per_split ? mbeg + m_per_split : M;
}

// ---- elementwise passes of the BatchNorms (norm.hip) --------------------------------------------------------------------------
// Channels are cut into groups of at most 64, a block takes one of them for all of its rows.
constexpr int kFoldChunks = 32;   // chunks that long lists of partial sums are folded into
// Lists that col_finalize_k adds up (in fp64) without a fold in front.  In the backward pass the fold, 5 us and a gap in front of a finalize
// of 5, pays from about 1600 chunks on: 72, 136 and 256 channels, from the first launch to the end of the last, with it and without:
// 1024 chunks 10 us and 5.8 to 7.4, 1536 chunks 10 and 8.5 to 10, 2048 chunks 10 and 11.3 to 12.7, 4096 chunks 10 and 21 to 23.
constexpr int kFinalizeChunks = 1600;
// Small tensors' blocks add up the partial sums of their channels themselves, 64 KB at the most, 16 loads a thread.  ResNet-20 at
// batch 128 (0.5 to 4 MB): 240 -> 178 launches, 1330 -> 1192 us a step (1214 with up to 32 KB); a two-block fp32 network (2 MB) 318 -> 309.
// Larger ones lose: 2048 blocks of several trips in ResNet-50 at batch 256, the sums folded to 16 KB for each: forward passes 41 -> 53 us,
// backward 58 -> 74, against 10 us of separate kernels; Wide-ResNet's 16 to 31 MB 9 -> 15, against 5.
constexpr int kSumBytes = 64 << 10;
struct BnGroups { int gc, groups; };
inline BnGroups bn_groups(int C, int vec) {
  BnGroups g;
  const int n = (C + 63) / 64, each = (C + n - 1) / n;
  g.gc = (each + vec - 1) / vec * vec;
  g.groups = (C + g.gc - 1) / g.gc;
  return g;
}
constexpr int64_t kSumTensor = 8 << 20;
inline bool bn_own_sums(int64_t M, int C, int esize, BnGroups g, int chunks) {
  return (int64_t)chunks * g.gc * 8 <= kSumBytes && M * C * esize <= kSumTensor;
}
// Whether a generic convolution leaves that many partial sums for the BatchNorm behind it.  More than a finalize takes need a fold, and where the
// elementwise pass adds up a reduction's sums by itself (kSumTensor) that is a launch more than the reduction: one layer of 16 channels on 128 images
// of 32x32 (2048 chunks, 8 MB).  Larger tensors have a finalize either way, and the fold is shorter than reading them: two-block fp32 network on
// 400 images, three such layers, 909 us with the reduction, 904 with the fold.
inline bool generic_sums_pay(int64_t M, int C, int esize, int64_t chunks) { return chunks <= kFinalizeChunks || M * C * esize > kSumTensor; }
// blocks over M rows: a trip of `unroll` rows a thread
inline int64_t bn_blocks(int64_t M, BnGroups g, int vec, int unroll) {
  const int64_t rows = (int64_t)(256 / (g.gc / vec)) * unroll;
  return (M + rows - 1) / rows * g.groups;
}

// ---- weight gradient of a dense layer (kernels_simple.hip) -----------------------------------------------------------------
// A block per 64 of the F + 1 columns and 4 classes, the column tiles of 4 classes side by side (they read the same part of dy:
// 20000 classes of 512 columns over 256 rows 922 us so, 1388 with the classes side by side), as many classes along x as a
// launch of fewer than 2^32 threads has room for, the rest along y.
struct LinearDwGrid { int64_t x, y; };
inline LinearDwGrid linear_dw_grid(int F, int C) {
  const int64_t tiles = ((int64_t)F + 64) / 64, groups = ((int64_t)C + 3) / 4, most = std::max<int64_t>(1, (1 << 22) / tiles);
  const int64_t per = std::min(groups, most);
  return {tiles * per, (groups + per - 1) / per};
}

}  // namespace cd
