// bf16 implicit-GEMM convolution on the gfx950 matrix cores (v_mfma_f32_32x32x16_bf16), fp32
// accumulation.  These are the contractions of the forward and backward passes of the paper's
// networks (Section 3: ResNet50): fprop, dgrad and wgrad of every convolution.
//
//   fprop  y[m][n]  = sum_k im2col(x)[m][k] * w[n][k]          m = (b,ho,wo), k = (r,s,c)
//   dgrad  dx[m][c] = sum_k gather(dy)[m][k] * wt[c][k]        m = (b,h,w),   k = (r,s,n)
//   wgrad  dw[n][k] = sum_m dy[m][n] * im2col(x)[m][k]
//
// fprop and dgrad share one kernel: both operands are contiguous along the contraction index, so
// a lane's 8-element MFMA operand is one 16-byte load.  Block = 4 waves; buffer loads write global
// memory straight into LDS (two to four stages of unpadded, XOR-swizzled 64- or 128-byte rows:
// conflict-free 16-byte reads) -> MFMA; the fp32 tile is rounded to bf16, transposed through LDS and written as
// full 16-byte vectors along the channels.  The MFMA "A" operand is the filter tile and "B" the
// activation tile, so that a lane's 16 accumulators run along the output channels of one pixel.
#include "kernels.h"
#include "conv_rules.h"
#include <algorithm>

namespace cd {

#define CD_LDS __attribute__((address_space(3)))
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int BK = 32;  // contraction elements per main-loop step of the kernels for short contractions or few channels

struct IgemmArgs {
  const bf16_t* src;  // gathered tensor [B][Hs][Ws][Cs]
  const bf16_t* wt;   // [N][K], K = kh*kw*Cs, laid out (r, s, c)
  bf16_t* dst;        // [M][N]
  int64_t M;
  int N, K;
  int Hs, Ws, Cs, Hd, Wd, kh, kw, stride, pad, pad_w;
  // output row m = (b, hd, wd) is written to row (b*Ho + hd*omul + ooff_h)*Wo + wd*omul + ooff_w of dst
  int omul, ooff_h, ooff_w, Ho, Wo;
  int accumulate;     // the result is added to what dst holds, or to `addend` when that is set
  // accumulate only (nullable): a second tensor [M][N] added instead of the old contents of dst, and
  // (nullable) its gate, one bit per element (bit k of byte i gates element 8i + k): a cleared bit
  // drops the addend's element.  Lets a data gradient pick up the gated gradient of a residual branch
  // without that branch's gradient ever being written out.
  const bf16_t* addend = nullptr;
  const uint8_t* addend_gate = nullptr;
  // (nullable) a tensor [M][N] of which the output is the gradient behind a ReLU: output elements whose element
  // of relu_out is not positive are written as zero (the ReLU's backward pass, without a pass of its own)
  const bf16_t* relu_out = nullptr;
  // Grouped convolutions (sliced launches): the gathered tensor has src_pitch channels per pixel, of which column tile
  // tn reads the Cs = BN channels [tn * BN, (tn + 1) * BN): the slice of channels whose groups the tile's output
  // channels belong to.  The filter rows then hold kh * kw * Cs elements, zero outside a row's own group.
  int src_pitch = 0;   // 0: Cs (an ordinary convolution)
  int sliced = 0;
  int pointwise;  // kh = kw = 1, stride 1, no padding (set by the launcher)
  FastDiv div_w = {0, 0}, div_h = {0, 0};   // by Wd and Hd (set by the launcher)
  int group_m;    // GROUP kernels: tile order in groups of this many row tiles
  int ntiles;
  uint32_t src_bytes, wt_bytes;
  const bf16_t* bias;  // per-column bias added to the output (kernels with EPI >= 1)
  float* stat_partials;  // STATS kernels: [m-tiles][stat_pitch(N)] per-tile column sums and sums of squares
  int sum_parts = 1;     // 256x256 tiles: one partial sum for the 256 rows, or one for every 128 (2)
  // STATS == 2 (a data gradient that completes the gradient of a BatchNorm's output): the sums that BatchNorm's
  // backward pass reduces over the rows, taken from the values as they are stored: dz = the output, gated by the
  // BatchNorm's ReLU bit mask (bn_mask, nullable: no ReLU), and dz * xhat with xhat = (bn_x - mean) * invstd,
  // bn_x [M][N] the BatchNorm's input, bn_stats = [mean[N] | invstd[N]].  Written to stat_partials like the forward sums.
  const bf16_t* bn_x = nullptr;
  const uint8_t* bn_mask = nullptr;
  const float* bn_stats = nullptr;
  // EPI 3: the evaluation-mode BatchNorm behind the convolution (EvalNorm)
  const float* norm_run = nullptr;
  const bf16_t* norm_gamma = nullptr;
  const bf16_t* norm_beta = nullptr;
  const bf16_t* norm_res = nullptr;   // nullable
  int norm_relu = 0;
};

int g_tune_tile = 0, g_tune_co = -1;  // tuning knobs of the microbenchmark

// Blocks are handed to the 8 XCDs round-robin; renumber so that consecutive logical tiles (which
// share activation rows and halos) run on the same XCD and meet in its L2.
__device__ inline unsigned xcd_remap(unsigned bid, unsigned nblocks) {
  const unsigned xcd = bid & 7u, idx = bid >> 3;
  const unsigned per = nblocks >> 3, rem = nblocks & 7u;
  return xcd * per + (xcd < rem ? xcd : rem) + idx;
}

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
// two floats -> two bf16 (round to nearest even) in one instruction
__device__ inline uint32_t pack_bf16x2(float a, float b) {
  const f32x2_t v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));

// Element (c, c) of a 32x32 accumulator tile held in the MFMA output layout (the lane owns column
// lane % 32; register v holds row 8 (v / 4) + 4 (lane / 32) + v % 4), for c = lane % 32: register
// 4 (c / 8) + c % 4, picked by a select tree.  Only the half-wave with lane / 32 == (c / 4) % 2 holds it.
__device__ inline float tile_diagonal(f32x16_t d, int c) {
  const bool b0 = (c & 1) != 0, b1 = (c & 2) != 0, b3 = (c & 8) != 0, b4 = (c & 16) != 0;
  const float u0 = b0 ? d[1] : d[0], u1 = b0 ? d[3] : d[2], u2 = b0 ? d[5] : d[4], u3 = b0 ? d[7] : d[6];
  const float u4 = b0 ? d[9] : d[8], u5 = b0 ? d[11] : d[10], u6 = b0 ? d[13] : d[12], u7 = b0 ? d[15] : d[14];
  const float w0 = b1 ? u1 : u0, w1 = b1 ? u3 : u2, w2 = b1 ? u5 : u4, w3 = b1 ? u7 : u6;
  const float x0 = b3 ? w1 : w0, x1 = b3 ? w3 : w2;
  return b4 ? x1 : x0;
}

// 16 bytes per lane from a buffer straight into LDS: lane l of the wave writes its vector at
// lds_addr + 16*l (lds_addr is uniform over the wave and travels in M0); an offset at or beyond the buffer's size
// writes zeros, so that a masked-out vector costs one select instead of a branch around the load.  The compiler does
// not see these loads: the kernel waits for them itself (wait_vmem) before a barrier publishes the tile.
typedef int rsrc_words_t __attribute__((ext_vector_type(4)));
// the four descriptor words of a raw buffer (stride 0): base address, size in bytes, data format
__device__ inline rsrc_words_t make_rsrc_words(const void* p, uint32_t bytes) {
  const uint64_t b = reinterpret_cast<uint64_t>(p);
  rsrc_words_t w;
  w.x = (int)(uint32_t)b;
  w.y = (int)((uint32_t)(b >> 32) & 0xffffu);
  w.z = (int)bytes;
  w.w = 0x00020000;
  return w;
}
__device__ inline void load_lds16(rsrc_words_t w, uint32_t lds_addr, uint32_t byte_off) {
  asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
               :
               : "s"(lds_addr), "v"(byte_off), "s"(w)
               : "memory");  // M0 cannot be named as a clobber: the compiler treats it as a reserved register (it rejects
                             // "m0" in a clobber list as such), i.e. it never keeps a value in M0 from one statement to
                             // the next and writes M0 itself right before each of its own uses
}
// wait until at most N of this wave's vector memory loads are outstanding
template <int N>
__device__ inline void wait_vmem() {
  static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
  asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}

// the same, and until this wave's LDS reads are done; then the workgroup's barrier.  (Builtins, so that the compiler's own
// count of outstanding LDS reads starts from zero behind it; the empty statements keep memory accesses on their side.)
template <int N>
__device__ inline void wait_step() {
  static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
  asm volatile("" : : : "memory");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));   // vmcnt(N) lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" : : : "memory");
}

// LDS tiles are [row][BKT elements], rows of 64 (BKT = 32) or 128 bytes without padding; the 16-byte column cv of a row
// is stored at column cv ^ swz(row) (element row * BKT + 8 (cv ^ swz(row))), which makes both the 16-byte stores (in lane
// order) and the MFMA fragment reads (16 consecutive rows, one column) bank-conflict free.  A thread's rows are a multiple of 32
// apart and share their swz.
template <int BKT> __device__ inline int lds_swz(int row) { return BKT == 32 ? (row >> 2) & 3 : (row >> 1) & 7; }

// Waves per SIMD that a kernel's registers must leave room for: as many workgroups per compute unit as the LDS allows, up to three
// (128x128 tiles in three 32-wide stages) or two.
constexpr int igemm_waves(int BM, int BN, int WAVES_M, int WAVES_N, int BKT, int NS, int WK) {
  const int tiles = (BM / WAVES_M / 32) * (BN / WAVES_N / 32), stages = NS * (BM + BN) * BKT * 2, waves = WAVES_M * WAVES_N * WK;
  if (waves == 8) return 2;
  if (stages > 80 * 1024) return 1;
  return tiles >= 8 ? 2 : BM == 128 && BN == 128 && NS == 3 ? 3 : 1;
}

// MODE 0: fprop gather, hs = hd*stride - pad + r.
// MODE 1: dgrad gather for stride 1, hs = hd + pad - r.
// (The dgrad of a stride-2 convolution is run as four MODE 0 problems, one per parity of the output
// pixel; see conv_dgrad_mfma.)
//
// Main loop: one barrier per step of BKT contraction elements, NS stages in LDS, the loads NS - 1 steps ahead of their use, the
// fragments of the next sub-step read while the matrix cores work on the current one; what a step waits for stands at the loop.
// The loads are inline assembly: the compiler does not track them, so it cannot serialise them against the LDS reads.
// F32OUT: the output is fp32 [M][N] (dense layers that produce logits); like the bf16 output it is
// transposed through LDS so that a store instruction writes whole 256-byte row segments.
// STATS 1: the epilogue also emits, per m-tile, the column sums and sums of squares of the bf16 values
// it writes (taken from the staged rows with transposing LDS reads and two MFMAs per fragment): the
// BatchNorm that follows a convolution gets its batch statistics without re-reading the tensor.
// STATS 2 (data gradients): per m-tile, the column sums of dz and dz * xhat that the backward pass of the BatchNorm
// whose output gradient this launch completes would otherwise reduce from memory (see IgemmArgs::bn_x).
// NWRAP: 1 when the gathered tensor has at least 32 channels (a 32-element step crosses at most one
// tap boundary), 4 for 8..31 channels.
// REMAP: output rows are placed with the strided row map of IgemmArgs (parity class of a stride-2 dgrad).
// EPI: 0 plain output, 1 per-column bias added, 2 bias and ReLU, 3 the evaluation-mode BatchNorm that follows (its pass over the
// tensor, a read and a write of it, was a third of an evaluation: ResNet-50 at batch 50 1719 us with it, 1353 without).  GROUP: grouped tile order (wide outputs).
// Both are compile-time: the plain kernels pay nothing for them.
// WK: groups of waves that share a tile's places and take equal parts of every step's contraction (1 or 2).
template <int MODE, int BM, int BN, int WAVES_M, int WAVES_N, bool F32OUT = false, int STATS = 0, int NWRAP = 1,
          bool REMAP = false, int EPI = 0, bool GROUP = false, int BKT = 32, int NS = 3, int WK = 1>
__global__ void __launch_bounds__(64 * WAVES_M * WAVES_N * WK, igemm_waves(BM, BN, WAVES_M, WAVES_N, BKT, NS, WK)) igemm_kernel(IgemmArgs a) {
  // (as many waves per SIMD, i.e. workgroups per compute unit, as the LDS allows: two for the tiles whose accumulators take 128
  // registers, three for 128x128 tiles in three 32-wide stages; the bound keeps the other registers within what that leaves)
  constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
  constexpr int TM = WM / 32, TN = WN / 32;
  constexpr int WAVES = WAVES_M * WAVES_N * WK, NT = 64 * WAVES;
  constexpr int EM = WM / WK, TE = TM / WK;    // rows and 32-row tiles of a wave in the epilogue
  static_assert(TM % WK == 0 && (BKT / 16) % WK == 0, "the groups share the sub-steps of a step and the row tiles of the epilogue");
  constexpr int SL = BKT / 8, RPP_L = NT / SL;  // 16-byte slots per LDS row, rows per load pass of the block
  constexpr int AV = BM / RPP_L;                // activation vectors per thread per step
  constexpr int BN_PAD = (BN + RPP_L - 1) / RPP_L * RPP_L;   // filter rows in LDS (whole load passes)
  constexpr int BV = BN_PAD / RPP_L;            // filter vectors per thread per step
  constexpr int STAGE = (BM + BN_PAD) * BKT;    // elements per stage: activation rows, then filter rows
  static_assert(BKT == 32 || (BKT == 64 && NWRAP == 1), "64-wide steps need at least 64 channels per tap");
  constexpr int MAIN_BYTES = NS * STAGE * 2;
  constexpr int EROWS = EM < 64 ? EM : 64;     // rows staged per epilogue pass
  constexpr int EPITCH = WN + 8;
  constexpr int EPI_BYTES = WAVES * EROWS * EPITCH * 2;
  constexpr int RED_BYTES = STATS ? WAVES_M * WK * 2 * BN * 4 : 0;   // column sums behind the staging rows
  constexpr int SMEM = MAIN_BYTES > EPI_BYTES + RED_BYTES ? MAIN_BYTES : EPI_BYTES + RED_BYTES;
  __shared__ __attribute__((aligned(16))) char smem[SMEM];
  // smem: [NS stages][BM + BN_PAD rows][BKT elements], later the epilogue's staging rows

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wmn = wave % (WAVES_M * WAVES_N), kg = wave / (WAVES_M * WAVES_N);   // place in the tile, group along the contraction
  const int wm0 = (wmn % WAVES_M) * WM, wn0 = (wmn / WAVES_M) * WN;
  const int em0 = wm0 + kg * EM;   // first row of this wave in the epilogue
  const unsigned tile = xcd_remap(blockIdx.x, gridDim.x);
  // row and element indices fit 32 bits: every operand is smaller than 2 GiB (conv_mfma_supported)
  unsigned tm = tile / (unsigned)a.ntiles, tn = tile % (unsigned)a.ntiles;
  if (GROUP) {
    // Wide outputs (a filter matrix that does not fit an L2): tiles run down groups of group_m row
    // tiles before moving to the next column tile, so that the workgroups resident at one time share
    // a few filter tiles and a few activation tiles instead of sweeping the whole filter matrix.
    const unsigned per = (unsigned)a.group_m * (unsigned)a.ntiles;
    const unsigned grp = tile / per, loc = tile - grp * per;
    const unsigned mt = (unsigned)((a.M + BM - 1) / BM);
    const unsigned gm = mt - grp * a.group_m < (unsigned)a.group_m ? mt - grp * a.group_m : (unsigned)a.group_m;
    tm = grp * a.group_m + loc % gm;
    tn = loc / gm;
  }
  const int m0 = (int)tm * BM;
  const int n0 = (int)tn * BN;
  const int M = (int)a.M;
  const rsrc_words_t rsrc = make_rsrc_words(a.src, a.src_bytes);
  const rsrc_words_t rwt = make_rsrc_words(a.wt, a.wt_bytes);

  // ---- per-thread gather state ---------------------------------------------------------------------
  // A wave's load instruction fills 64 / SL consecutive tile rows (64 lanes x 16 bytes, in lane order), so thread tid owns
  // LDS slot tid % SL of rows tid / SL + RPP_L j; the slot holds the 16-byte column slot ^ swz(row) of the tile (see
  // lds_swz), the same for all of the thread's rows.
  const int lrow = tid / SL;
  const int kvec = (tid % SL) ^ lds_swz<BKT>(lrow);
  const int P = a.src_pitch ? a.src_pitch : a.Cs;   // channels per pixel of the gathered tensor
  const int cs0 = a.sliced ? n0 : 0;                // first channel this tile gathers (sliced launches)
  int rowoff[AV];                 // element offset of (image, h0, w0, first gathered channel); may be negative
  uint32_t hmask[AV], wmask[AV];  // bit r / s set: tap row r / column s reads inside the image
#pragma unroll
  for (int j = 0; j < AV; j++) {
    const int m = m0 + lrow + RPP_L * j;
    const bool rowok = m < M;
    if (a.pointwise) {  // 1x1 filter, stride 1, no padding: row m of the gathered tensor, every tap inside
      hmask[j] = rowok ? 1u : 0u;
      wmask[j] = 1u;
      rowoff[j] = m * P + cs0;
      continue;
    }
    const unsigned mm = rowok ? (unsigned)m : 0u;
    const unsigned q = div_by(mm, a.div_w);
    const int wd = (int)(mm - q * (unsigned)a.Wd);
    const int b = (int)div_by(q, a.div_h);
    const int hd = (int)(q - (unsigned)b * (unsigned)a.Hd);
    const int hh = MODE == 0 ? hd * a.stride - a.pad : hd + a.pad;
    const int ww = MODE == 0 ? wd * a.stride - a.pad_w : wd + a.pad_w;
    // taps that read inside: bits lo .. hi - 1 (0 <= h + r < n forwards, 0 <= h - r < n backwards; at most 7 taps)
    auto taps = [](int h, int n, int k) {
      const int lo = min(max(MODE == 0 ? -h : h - n + 1, 0), 31), hi = min(max(MODE == 0 ? n - h : h + 1, 0), k);
      return ((1u << hi) - 1u) & ~((1u << lo) - 1u);
    };
    hmask[j] = rowok ? taps(hh, a.Hs, a.kh) : 0u;
    wmask[j] = taps(ww, a.Ws, a.kw);
    rowoff[j] = ((b * a.Hs + hh) * a.Ws + ww) * P + cs0;
  }
  // byte offset of this thread's filter row (+ its 16-byte column); rows past N start beyond every buffer's end (operands
  // are smaller than 2 GiB), so their loads give zeros at every step
  uint32_t woff[BV];
#pragma unroll
  for (int j = 0; j < BV; j++) {
    const int n = n0 + lrow + RPP_L * j;
    woff[j] = ((lrow + RPP_L * j) < BN && n < a.N) ? (uint32_t)(n * a.K + kvec * 8) * 2u : 0x80000000u;
  }
  // position of this thread's vector in the contraction: tap (kr, ks) and channel kc
  int kc = kvec * 8, kr = 0, ks = 0;
  {
    const int tap = kc / a.Cs;
    kc -= tap * a.Cs;
    kr = tap / a.kw;
    ks = tap - kr * a.kw;
  }
  const int KT = (a.K + BKT - 1) / BKT;
  const int tapdir = MODE == 0 ? 1 : -1;

  // LDS byte address of this wave's first rows (1024 bytes a load) of the stage-0 activation tile
  const uint32_t lds_wave = (uint32_t)(uintptr_t)(CD_LDS char*)smem + (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6) * 1024u;
  // The byte offsets of one step's vectors (masked ones beyond the buffer), then the state of the step after it.  A step at
  // or beyond the end of the contraction has every vector masked: its loads cost no memory traffic and write zeros, so the
  // number of loads in flight is the same at every step.
  uint32_t offa[AV], offb[BV];
  constexpr int NPIECE = AV + BV + 1;
  // piece p of the preparation of step kt: one vector's offset, or (last) the step to the next position.  Straight-line code
  // (it sits between the MFMAs): koff, the element offset of the thread's tap and channel, is carried along, masks are or-ed in.
  int koff = tapdir * (kr * a.Ws + ks) * P + kc;
  const int koff_tap = tapdir * P - a.Cs, koff_row = tapdir * (a.Ws - a.kw) * P;
  uint32_t kend = kr < a.kh ? 0u : 0xffffffffu;   // all ones beyond the end of the contraction
  auto prep_piece = [&](int kt, int p) {
    if (p < AV) {
      const uint32_t okb = (hmask[p] >> ((uint32_t)kr & 31u)) & (wmask[p] >> ((uint32_t)ks & 31u)) & 1u;
      offa[p] = ((uint32_t)(rowoff[p] + koff) * 2u) | (okb - 1u) | kend;
    } else if (p < AV + BV) {
      offb[p - AV] = (woff[p - AV] + (uint32_t)kt * (BKT * 2u)) | kend;
    } else {   // NWRAP sub-steps, each crossing at most one tap boundary
#pragma unroll
      for (int u = 0; u < NWRAP; u++) {
        kc += BKT / NWRAP;
        koff += BKT / NWRAP;
        const bool wrap = kc >= a.Cs;
        kc -= wrap ? a.Cs : 0;
        koff += wrap ? koff_tap : 0;
        ks += wrap ? 1 : 0;
        const bool wrap2 = ks == a.kw;
        ks = wrap2 ? 0 : ks;
        koff += wrap2 ? koff_row : 0;
        kr += wrap2 ? 1 : 0;
      }
      kend = kr < a.kh ? 0u : 0xffffffffu;
    }
  };
  // issues prepared load v (activation vectors, then filter vectors) into the stage at byte offset stage_b
  auto issue = [&](uint32_t stage_b, int v) {
    if (v < AV) load_lds16(rsrc, lds_wave + stage_b + (uint32_t)v * (RPP_L * BKT * 2u), offa[v]);
    else load_lds16(rwt, lds_wave + stage_b + (uint32_t)(BM + (v - AV) * RPP_L) * (BKT * 2u), offb[v - AV]);
  };

  // STATS 2: what the epilogue reads besides the tile itself.  The BatchNorm's input at this lane's output vectors is requested
  // now and arrives during the main loop (vector memory operations retire in order: the main loop's first wait also waits for
  // these, and the compiler's own waits for them can only be too strict); its ReLU bits, a byte per vector, follow behind the
  // loop: sixteen registers through the loop would spill (128x256) or cost the third workgroup per compute unit (128x128).
  // (The input's vectors leave the two 128-accumulator tiles of four waves short of 2 registers each: those are stored to scratch memory in
  // front of the loop and loaded behind it.  It takes a request to a call and the row's check for ragged vectors alone, below: with a loop
  // inside the request and the check everywhere they were 13 (256x128) and 9 (128x256), 248 and 239 us a launch of a ResNet-50 step at batch 256
  // where they are 238 and 226 now.)
  constexpr int BS_LPR = WN / 8, BS_RPP = 64 / BS_LPR, BS_EROWS = EM < 64 ? EM : 64;
  // (256x256 tiles, whose vectors are 64 registers, request them pass by pass in the epilogue)
  constexpr bool BS_LATE = BM == 256 && BN == 256;
  constexpr int BS_PP = (BS_EROWS + BS_RPP - 1) / BS_RPP, BS_NV = STATS == 2 ? (BS_LATE ? 1 : EM / BS_EROWS) * BS_PP : 1;
  uint4 bs_x[BS_NV];
  uint32_t bs_bits[BS_NV];
  auto bs_index = [&](int v, bool& ok) {   // element index of vector v in an [M][N] tensor
    const int pass = v / BS_PP, pp = v % BS_PP;
    const int m = m0 + em0 + pass * BS_EROWS + pp * BS_RPP + lane / BS_LPR, n = n0 + wn0 + (lane % BS_LPR) * 8;
    ok = m < M && n < a.N;
    if constexpr (64 % BS_LPR != 0) ok = ok && pp * BS_RPP + lane / BS_LPR < BS_EROWS && lane < BS_RPP * BS_LPR;
    return (unsigned)m * (unsigned)a.N + (unsigned)n;
  };
  auto bs_request_x = [&](int v, int at) {   // vector `at` into place v
    bool ok;
    const unsigned idx = bs_index(at, ok);
    bs_x[v] = make_uint4(0, 0, 0, 0);
    if (ok) bs_x[v] = *reinterpret_cast<const uint4*>(a.bn_x + idx);
  };
  auto bs_request_bits = [&](int v, int at) {
    bool ok;
    const unsigned idx = bs_index(at, ok);
    bs_bits[v] = 0u;
    if (ok) bs_bits[v] = a.bn_mask ? a.bn_mask[idx >> 3] : 0xffu;
  };
  if (STATS == 2 && !BS_LATE) {
#pragma unroll
    for (int v = 0; v < BS_NV; v++) bs_request_x(v, v);
  }
  // EPI: the bias of this lane's channels, requested here so that its latency passes under the main loop (read behind it, element
  // by element, it cost 3 us a tile: 8192 x 2048 x 512 26 us, now 23).  Register v of tile i belongs to channel
  // n0 + wn0 + 32 i + 8 (v / 4) + 4 (lane / 32) + v % 4: four consecutive channels at a time, on 8-byte boundaries.
  constexpr bool BIAS = EPI == 1 || EPI == 2;
  uint2 bias4[BIAS ? TN : 1][4];
  if (BIAS) {
#pragma unroll
    for (int i = 0; i < TN; i++)
#pragma unroll
      for (int g = 0; g < 4; g++) {
        const int n = n0 + wn0 + i * 32 + 8 * g + 4 * (lane >> 5);
        bias4[i][g] = make_uint2(0u, 0u);
        if (n + 3 < a.N) {
          bias4[i][g] = *reinterpret_cast<const uint2*>(a.bias + n);
        } else {   // the last columns of an output whose width is no multiple of four
          uint32_t e[4] = {0u, 0u, 0u, 0u};
#pragma unroll
          for (int q = 0; q < 4; q++)
            if (n + q < a.N) e[q] = a.bias[n + q];
          bias4[i][g] = make_uint2(e[0] | (e[1] << 16), e[2] | (e[3] << 16));
        }
      }
  }
  // EPI 3: the averages and parameters of the eight channels that this lane stores, likewise (the averages start at any element)
  typedef float f32x4_el __attribute__((ext_vector_type(4), aligned(4)));
  f32x4_el nmean[2], nvar[2];
  uint4 ngamma, nbeta;
  if (EPI == 3) {
    const int n = n0 + wn0 + (lane % (WN / 8)) * 8;
    if (n < a.N) {
#pragma unroll
      for (int h = 0; h < 2; h++) {
        nmean[h] = *reinterpret_cast<const f32x4_el*>(a.norm_run + n + 4 * h);
        nvar[h] = *reinterpret_cast<const f32x4_el*>(a.norm_run + a.N + n + 4 * h);
      }
      ngamma = *reinterpret_cast<const uint4*>(a.norm_gamma + n);
      nbeta = *reinterpret_cast<const uint4*>(a.norm_beta + n);
    }
  }
  f32x16_t acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; i++)
#pragma unroll
    for (int j = 0; j < TM; j++)
#pragma unroll
      for (int v = 0; v < 16; v++) acc[i][j][v] = 0.f;

  const int frow = lane & 31, fcv = lane >> 5;
  // Main loop: NS stages rotate, tile kt lies in stage kt % NS.  A step is KK sub-steps of 16; the fragments of the next
  // sub-step are read from LDS while the matrix cores work on the current one, across the step boundary too: before the
  // last sub-step of tile kt the waves wait for their own loads of tile kt+1 (all but the newest NS - 2 tiles') and for
  // their LDS reads of tile kt, and meet at the step's only barrier, which publishes tile kt+1 and frees the stage of tile
  // kt; the loads of tile kt+NS go there.  Their offsets were computed in the shadow of the earlier sub-steps' MFMAs.
  // (Not for the 128-accumulator tiles that also hold the backward sums' operands through the loop: no registers are left for
  // a second fragment buffer, they read a sub-step's fragments and use them.)
  constexpr bool AHEAD = !(STATS == 2 && TN * TM >= 8 && !BS_LATE);
  constexpr int KK = BKT / 16 / WK, TT = TN * TM, FB = AHEAD ? 2 : 1;   // (sub-steps of this wave's group)
  static_assert(KK >= 2 && KK % 2 == 0, "a step ends on the fragment buffer that the next one begins with, and has a sub-step in front of its loads");
  bf16x8_t wf[FB][TN], xf[FB][TM];  // [buffer][tile]
  // byte offset of this lane's fragment of sub-step kk inside a tile row block (swz depends on the lane's row only: tile
  // rows are multiples of 32 apart)
  uint32_t fcol[KK];
#pragma unroll
  for (int kk = 0; kk < KK; kk++)
    fcol[kk] = (uint32_t)(frow * BKT + ((((kg * KK + kk) * 2 + fcv) ^ lds_swz<BKT>(frow)) << 3)) * 2u;
  const uint32_t xbase = (uint32_t)(wm0 * BKT) * 2u, wbase = (uint32_t)((BM + wn0) * BKT) * 2u;
  auto read_frags = [&](int buf, uint32_t stage_b, int kk) {
    const char* xp = smem + (stage_b + xbase + fcol[kk]);
    const char* wp = smem + (stage_b + wbase + fcol[kk]);
#pragma unroll
    for (int i = 0; i < TN; i++) wf[buf][i] = *reinterpret_cast<const bf16x8_t*>(wp + i * 32 * BKT * 2);
#pragma unroll
    for (int j = 0; j < TM; j++) xf[buf][j] = *reinterpret_cast<const bf16x8_t*>(xp + j * 32 * BKT * 2);
  };
  uint32_t cur = 0, nxt = STAGE * 2u;  // byte offsets
#pragma unroll
  for (int t = 0; t < NS; t++) {
#pragma unroll
    for (int p = 0; p < NPIECE; p++) prep_piece(t, p);
#pragma unroll
    for (int v = 0; v < AV + BV; v++) issue(t * STAGE * 2u, v);
  }
  wait_step<(NS - 1) * (AV + BV)>();
  if (AHEAD) read_frags(0, cur, 0);
  __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4));   // lgkmcnt(0): with the scalar loads, so that none is waited for inside
  for (int kt = 0; kt < KT; kt++) {
#pragma unroll
    for (int kk = 0; kk < KK; kk++) {
      if (!AHEAD) read_frags(0, cur, kk);
      if (kk == KK - 1) wait_step<(NS - 2) * (AV + BV)>();
      if (AHEAD) read_frags((kk + 1) & (FB - 1), kk == KK - 1 ? nxt : cur, (kk + 1) % KK);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < TT; i++) {
        acc[i / TM][i % TM] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[kk & (FB - 1)][i / TM], xf[kk & (FB - 1)][i % TM],
                                                                      acc[i / TM][i % TM], 0, 0, 0);
        // in the MFMA's shadow: a share of the next offsets, in the last sub-step of the loads
        if (kk < KK - 1) {
          constexpr int SLOTS = (KK - 1) * TT;
          const int slot = kk * TT + i;
#pragma unroll
          for (int p = 0; p < NPIECE; p++)
            if (p * SLOTS / NPIECE == slot) prep_piece(kt + NS, p);
        } else {
#pragma unroll
          for (int v = 0; v < AV + BV; v++)
            if (v * TT / (AV + BV) == i) issue(cur, v);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    cur = nxt;
    nxt = nxt + STAGE * 2u == NS * STAGE * 2u ? 0 : nxt + STAGE * 2u;
  }
  if (STATS == 2 && !BS_LATE) {
#pragma unroll
    for (int v = 0; v < BS_NV; v++) bs_request_bits(v, v);
  }
  wait_vmem<0>();  // the masked loads past the end still write (zeros) into the stages the epilogue reuses

  // accumulator layout: lane holds pixel column (lane % 32); register v holds channel
  // 8*(v/4) + 4*(lane/32) + v%4 of the 32x32 tile
  if constexpr (WK == 2) {
    // Each of the two waves of a place hands the other one half of its row tiles and adds what it gets (the first group's sum
    // plus the second's, whichever wave adds): 16-byte vectors in lane order.
    constexpr int HALF = TN * TE * 16 * 64;   // floats a wave hands over
    static_assert(WAVES * HALF * 4 <= SMEM, "room for the sums that change hands");
    float* mine = reinterpret_cast<float*>(smem) + wave * HALF + lane * 4;
    const float* theirs = reinterpret_cast<const float*>(smem) + (kg ? wave - WAVES / 2 : wave + WAVES / 2) * HALF + lane * 4;
    __syncthreads();   // the main loop's tiles are no longer read
#pragma unroll
    for (int i = 0; i < TN; i++)
#pragma unroll
      for (int j = 0; j < TE; j++)
#pragma unroll
        for (int g = 0; g < 4; g++) {
          float4 v;
          v.x = kg ? acc[i][j][4 * g] : acc[i][TE + j][4 * g];
          v.y = kg ? acc[i][j][4 * g + 1] : acc[i][TE + j][4 * g + 1];
          v.z = kg ? acc[i][j][4 * g + 2] : acc[i][TE + j][4 * g + 2];
          v.w = kg ? acc[i][j][4 * g + 3] : acc[i][TE + j][4 * g + 3];
          *reinterpret_cast<float4*>(mine + ((i * TE + j) * 4 + g) * 256) = v;
        }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < TN; i++)
#pragma unroll
      for (int j = 0; j < TE; j++)
#pragma unroll
        for (int g = 0; g < 4; g++) {
          const float4 v = *reinterpret_cast<const float4*>(theirs + ((i * TE + j) * 4 + g) * 256);
          acc[i][j][4 * g] = (kg ? acc[i][TE + j][4 * g] : acc[i][j][4 * g]) + v.x;
          acc[i][j][4 * g + 1] = (kg ? acc[i][TE + j][4 * g + 1] : acc[i][j][4 * g + 1]) + v.y;
          acc[i][j][4 * g + 2] = (kg ? acc[i][TE + j][4 * g + 2] : acc[i][j][4 * g + 2]) + v.z;
          acc[i][j][4 * g + 3] = (kg ? acc[i][TE + j][4 * g + 3] : acc[i][j][4 * g + 3]) + v.w;
        }
  }
  if (BIAS) {
#pragma unroll
    for (int i = 0; i < TN; i++)
#pragma unroll
      for (int g = 0; g < 4; g++) {
        const float bv[4] = {__uint_as_float(bias4[i][g].x << 16), __uint_as_float(bias4[i][g].x & 0xffff0000u),
                             __uint_as_float(bias4[i][g].y << 16), __uint_as_float(bias4[i][g].y & 0xffff0000u)};
#pragma unroll
        for (int j = 0; j < TE; j++)
#pragma unroll
          for (int q = 0; q < 4; q++) acc[i][j][4 * g + q] += bv[q];
      }
  }
  if (F32OUT) {
    // one 32-row tile row of the wave at a time: [32][WN] floats (+4 of padding) per wave
    constexpr int FP = WN + 4;
    static_assert(!F32OUT || WAVES * 32 * FP * 4 <= SMEM, "fp32 staging fits the tile memory");
    float* fst = reinterpret_cast<float*>(smem) + wave * 32 * FP;
    float* dst = reinterpret_cast<float*>(a.dst);
    constexpr int FLPR = WN / 4;       // lanes per output row (16-byte vectors)
    constexpr int FRPP = 64 / FLPR;    // rows per store instruction
    const int fr = lane / FLPR, fc = (lane % FLPR) * 4;
    __syncthreads();  // the main loop's tiles are no longer read
#pragma unroll
    for (int j = 0; j < TE; j++) {
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int i = 0; i < TN; i++)
#pragma unroll
        for (int g = 0; g < 4; g++)
          *reinterpret_cast<float4*>(fst + frow * FP + i * 32 + 8 * g + 4 * (lane >> 5)) =
              make_float4(acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]);
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int p = 0; p < 32 / FRPP; p++) {
        const int row = p * FRPP + fr;
        const int m = m0 + em0 + j * 32 + row;
        const int n = n0 + wn0 + fc;
        if (m < M && n < a.N) {
          const float4 v = *reinterpret_cast<const float4*>(fst + row * FP + fc);
          float* dp = dst + ((int64_t)m * a.N + n);
          if (n + 3 < a.N && (a.N & 3) == 0) {
            *reinterpret_cast<float4*>(dp) = v;
          } else {  // ragged or unaligned row ends
            const float e[4] = {v.x, v.y, v.z, v.w};
            for (int q = 0; q < 4 && n + q < a.N; q++) dp[q] = e[q];
          }
        }
      }
    }
    return;
  }
  if (EPI == 2) {
#pragma unroll
    for (int i = 0; i < TN; i++)
#pragma unroll
      for (int j = 0; j < TE; j++)
#pragma unroll
        for (int v = 0; v < 16; v++) acc[i][j][v] = fmaxf(acc[i][j][v], 0.f);
  }
  // ---- epilogue: fp32 -> bf16, transpose through LDS, 16-byte stores along the channels -------------
  bf16_t* stage = reinterpret_cast<bf16_t*>(smem) + wave * EROWS * EPITCH;
  constexpr int LPR = WN / 8;        // lanes per output row
  constexpr int RPP = 64 / LPR;      // rows per pass
  constexpr int PASSES = (EROWS + RPP - 1) / RPP;
  constexpr int TPG = EROWS / 32;    // 32-row tiles per staging pass
  const bool lane_ok = lane < RPP * LPR;   // (all of them where a row's vectors divide 64)
  const int er = lane / LPR, ec = (lane % LPR) * 8;
  // STATS: per-wave column sums [WAVES_M * WK][2][BN], behind the staging rows
  static_assert(STATS != 2 || !REMAP, "the backward sums are taken where the rows are stored in order");
  // STATS 2: running sums of dz and of dz * x over this lane's 8 channels (the same in every pass); the mean and the
  // scale of xhat = (x - mean) * invstd are applied to the tile's sums at the end (the sums are linear in x)
  float bs0[8], bs1[8];
  if (STATS == 2) {
#pragma unroll
    for (int k = 0; k < 8; k++) { bs0[k] = 0.f; bs1[k] = 0.f; }
  }
  // EPI 3: scale and shift of this lane's channels, as running_scale_shift has them
  float nsc[8], nsh[8];
  if (EPI == 3) {
    const uint32_t gg[4] = {ngamma.x, ngamma.y, ngamma.z, ngamma.w}, bb[4] = {nbeta.x, nbeta.y, nbeta.z, nbeta.w};
#pragma unroll
    for (int k = 0; k < 8; k++) {
      const float istd = 1.f / sqrtf(nvar[k >> 2][k & 3] + kBnEps);
      nsc[k] = __uint_as_float(k & 1 ? gg[k >> 1] & 0xffff0000u : gg[k >> 1] << 16) * istd;
      nsh[k] = fmaf(-nmean[k >> 2][k & 3], nsc[k], __uint_as_float(k & 1 ? bb[k >> 1] & 0xffff0000u : bb[k >> 1] << 16));
    }
  }
  float* red = reinterpret_cast<float*>(smem + EPI_BYTES);
  __syncthreads();  // the main loop's tiles are no longer read: the staging rows alias them
#pragma unroll
  for (int g0 = 0; g0 < TE; g0 += TPG) {
    // The staging rows belong to this wave alone, and a wave's LDS accesses execute in program order:
    // no block barrier between its writes, its reads and the next pass's writes.
    uint4 nres[EPI == 3 ? PASSES : 1];   // EPI 3: the residual rows of this pass, requested in front of the staging
    if (EPI == 3 && a.norm_res) {
#pragma unroll
      for (int p = 0; p < PASSES; p++) {
        const int m = m0 + em0 + g0 * 32 + p * RPP + er, n = n0 + wn0 + ec;
        if (m < M && n < a.N && lane_ok && p * RPP + er < EROWS) nres[p] = *reinterpret_cast<const uint4*>(a.norm_res + ((unsigned)m * (unsigned)a.N + (unsigned)n));
      }
    }
    if (STATS == 2 && BS_LATE) {
#pragma unroll
      for (int v = 0; v < BS_NV; v++) bs_request_x(v, g0 / TPG * BS_PP + v);
#pragma unroll
      for (int v = 0; v < BS_NV; v++) bs_request_bits(v, g0 / TPG * BS_PP + v);
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < TN; i++)
#pragma unroll
      for (int j = 0; j < TPG; j++)
#pragma unroll
        for (int g = 0; g < 4; g++) {
          uint2 p;
          p.x = pack_bf16x2(acc[i][g0 + j][4 * g + 0], acc[i][g0 + j][4 * g + 1]);
          p.y = pack_bf16x2(acc[i][g0 + j][4 * g + 2], acc[i][g0 + j][4 * g + 3]);
          *reinterpret_cast<uint2*>(stage + (j * 32 + frow) * EPITCH + i * 32 + 8 * g + 4 * (lane >> 5)) = p;
        }
    __builtin_amdgcn_wave_barrier();
    if (STATS == 1) {
      // Column sums and sums of squares of the staged (rounded) rows on the matrix cores, which idle in
      // the epilogue: the transposing LDS read hands a lane 8 pixels of its column (16 pixels x 32
      // columns per fragment, the operand layout of wgrad_kernel); ones^T Y gives the sums in every row
      // of one accumulator tile, Y^T Y the sums of squares on the diagonal of another.  Rows past M and
      // columns past N were computed from zero-filled operands and add nothing.
      const int grp = lane >> 4, li = lane & 15;
      const int tr_m = 8 * (grp >> 1) + (li >> 2), tr_c = 16 * (grp & 1) + 4 * (li & 3);
      const __bf16 one = (__bf16)1.0f;
      const bf16x8_t ones = {one, one, one, one, one, one, one, one};
      const int wmi = (wmn % WAVES_M) * WK + kg, c = lane & 31;
#pragma unroll 1
      for (int i = 0; i < TN; i++) {   // one 32-column block at a time: two accumulator tiles live
        f32x16_t ds, dq;
#pragma unroll
        for (int v = 0; v < 16; v++) { ds[v] = 0.f; dq[v] = 0.f; }
#pragma unroll
        for (int pc = 0; pc < EROWS / 16; pc++) {
          const bf16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
              (CD_LDS bf16x4_t*)(stage + (pc * 16 + tr_m) * EPITCH + i * 32 + tr_c));
          const bf16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
              (CD_LDS bf16x4_t*)(stage + (pc * 16 + tr_m + 4) * EPITCH + i * 32 + tr_c));
          const bf16x8_t f = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
          ds = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, f, ds, 0, 0, 0);
          dq = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, f, dq, 0, 0, 0);
        }
        // every lane holds the sum of its column, one half-wave per column the sum of squares; a later
        // pass over further rows of the tile adds to what this lane wrote
        float* r0 = red + (wmi * 2 + 0) * BN + wn0 + i * 32 + c;
        float* r1 = red + (wmi * 2 + 1) * BN + wn0 + i * 32 + c;
        const float sq = tile_diagonal(dq, c);
        if (lane < 32) *r0 = g0 == 0 ? ds[0] : *r0 + ds[0];
        if (((c >> 2) & 1) == (lane >> 5)) *r1 = g0 == 0 ? sq : *r1 + sq;
      }
    }
#pragma unroll
    for (int p = 0; p < PASSES; p++) {
      const int row = p * RPP + er;
      int m = m0 + em0 + g0 * 32 + row;
      const int n = n0 + wn0 + ec;
      if (m < M && n < a.N && lane_ok && row < EROWS) {
        uint4 v = *reinterpret_cast<const uint4*>(stage + row * EPITCH + ec);
        if (REMAP) {  // strided placement of the rows (parity class of a stride-2 dgrad)
          const unsigned q = div_by((unsigned)m, a.div_w);
          const int wd = m - (int)(q * (unsigned)a.Wd);
          const int b = (int)div_by(q, a.div_h);
          const int hd = (int)q - b * a.Hd;
          m = (b * a.Ho + hd * a.omul + a.ooff_h) * a.Wo + wd * a.omul + a.ooff_w;
        }
        const unsigned idx = (unsigned)m * (unsigned)a.N + (unsigned)n;
        bf16_t* dp = a.dst + idx;
        if (a.accumulate) {
          const uint4 o = *reinterpret_cast<const uint4*>(a.addend ? a.addend + idx : dp);
          const uint32_t vv[4] = {v.x, v.y, v.z, v.w};
          uint32_t oo[4] = {o.x, o.y, o.z, o.w};
          if (a.addend_gate) {
            const uint32_t bits = a.addend_gate[idx >> 3];
#pragma unroll
            for (int q = 0; q < 4; q++)
              oo[q] &= ((bits >> (2 * q)) & 1u ? 0x0000ffffu : 0u) | ((bits >> (2 * q + 1)) & 1u ? 0xffff0000u : 0u);
          }
          uint32_t r[4];
#pragma unroll
          for (int q = 0; q < 4; q++)
            r[q] = pack_bf16x2(__uint_as_float(vv[q] << 16) + __uint_as_float(oo[q] << 16),
                               __uint_as_float(vv[q] & 0xffff0000u) + __uint_as_float(oo[q] & 0xffff0000u));
          v = make_uint4(r[0], r[1], r[2], r[3]);
        }
        if (a.relu_out) {
          const uint4 y = *reinterpret_cast<const uint4*>(a.relu_out + idx);
          const uint32_t yy[4] = {y.x, y.y, y.z, y.w};
          uint32_t vv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
          for (int q = 0; q < 4; q++)   // a bf16 is positive iff its bits, read as int16, are
            vv[q] &= ((int16_t)(yy[q] & 0xffffu) > 0 ? 0x0000ffffu : 0u) | ((int16_t)(yy[q] >> 16) > 0 ? 0xffff0000u : 0u);
          v = make_uint4(vv[0], vv[1], vv[2], vv[3]);
        }
        if (EPI == 3) {
          const uint32_t vv[4] = {v.x, v.y, v.z, v.w}, rr[4] = {nres[p].x, nres[p].y, nres[p].z, nres[p].w};
          uint32_t o[4];
#pragma unroll
          for (int q = 0; q < 4; q++) {
            float e0 = fmaf(__uint_as_float(vv[q] << 16), nsc[2 * q], nsh[2 * q]);
            float e1 = fmaf(__uint_as_float(vv[q] & 0xffff0000u), nsc[2 * q + 1], nsh[2 * q + 1]);
            if (a.norm_res) { e0 += __uint_as_float(rr[q] << 16); e1 += __uint_as_float(rr[q] & 0xffff0000u); }
            if (a.norm_relu) { e0 = fmaxf(e0, 0.f); e1 = fmaxf(e1, 0.f); }
            o[q] = pack_bf16x2(e0, e1);
          }
          v = make_uint4(o[0], o[1], o[2], o[3]);
        }
        if (STATS == 2) {   // the stored values feed the sums of the BatchNorm's backward pass
          const uint4 xr = bs_x[(BS_LATE ? 0 : g0 / TPG) * PASSES + p];
          const uint32_t bits = bs_bits[(BS_LATE ? 0 : g0 / TPG) * PASSES + p];
          const uint32_t gv[4] = {v.x, v.y, v.z, v.w}, xv[4] = {xr.x, xr.y, xr.z, xr.w};
#pragma unroll
          for (int q = 0; q < 4; q++) {
            const float d0 = (bits >> (2 * q)) & 1u ? __uint_as_float(gv[q] << 16) : 0.f;
            const float d1 = (bits >> (2 * q + 1)) & 1u ? __uint_as_float(gv[q] & 0xffff0000u) : 0.f;
            bs0[2 * q] += d0;
            bs0[2 * q + 1] += d1;
            bs1[2 * q] += d0 * __uint_as_float(xv[q] << 16);
            bs1[2 * q + 1] += d1 * __uint_as_float(xv[q] & 0xffff0000u);
          }
        }
        *reinterpret_cast<uint4*>(dp) = v;
      }
    }
  }
  if (STATS == 2) {
    // lanes that share their 8 channels (one per row of a pass) add up, the first of them hands the wave's sums over
#pragma unroll
    for (int k = 0; k < 8; k++) {
      if constexpr (64 % LPR == 0) {
#pragma unroll
        for (int off = LPR; off < 64; off <<= 1) {
          bs0[k] += __shfl_xor(bs0[k], off, 64);
          bs1[k] += __shfl_xor(bs1[k], off, 64);
        }
      } else {   // (the first LPR lanes hold the sums)
        float t0 = bs0[k], t1 = bs1[k];
#pragma unroll
        for (int r = 1; r < RPP; r++) {
          t0 += __shfl(bs0[k], (lane + r * LPR) & 63, 64);
          t1 += __shfl(bs1[k], (lane + r * LPR) & 63, 64);
        }
        bs0[k] = t0;
        bs1[k] = t1;
      }
    }
    if (lane < LPR) {
      const int wmi = (wmn % WAVES_M) * WK + kg;
#pragma unroll
      for (int k = 0; k < 8; k++) {
        red[(wmi * 2 + 0) * BN + wn0 + ec + k] = bs0[k];
        red[(wmi * 2 + 1) * BN + wn0 + ec + k] = bs1[k];
      }
    }
  }
  if (STATS) {
    // fold the waves of a column
    __syncthreads();
    constexpr int PARTS = BM == 256 && BN == 256 ? 2 : 1, WPP = WAVES_M * WK / PARTS;   // partial sums of the tile at the most, waves to each
    const int parts = PARTS == 1 ? 1 : a.sum_parts, part = PARTS == 1 ? 0 : tid / BN, col = PARTS == 1 ? tid : tid % BN;
    static_assert(PARTS * BN <= NT, "a thread for each of them");
    if (part < parts && tid < PARTS * BN && n0 + col < a.N && m0 + part * (BM / PARTS) < M) {
      float s0 = 0.f, s1 = 0.f;
#pragma unroll
      for (int w = 0; w < WPP; w++) {
        s0 += red[((part * WPP + w) * 2 + 0) * BN + col];
        s1 += red[((part * WPP + w) * 2 + 1) * BN + col];
      }
      if (parts < PARTS) {
#pragma unroll
        for (int w = WPP; w < WPP * PARTS; w++) { s0 += red[(w * 2 + 0) * BN + col]; s1 += red[(w * 2 + 1) * BN + col]; }
      }
      if (STATS == 2) s1 = (s1 - a.bn_stats[n0 + col] * s0) * a.bn_stats[a.N + n0 + col];   // sum dz x -> sum dz xhat
      const int64_t mt = (int64_t)tm * parts + part;
      a.stat_partials[mt * stat_pitch(a.N) + n0 + col] = s0;
      a.stat_partials[mt * stat_pitch(a.N) + a.N + n0 + col] = s1;
    }
  }
}

// Output tile of the wide-output kernels (N > 64), and how their main loop is fed.
//
// What a workgroup's step costs (128x128 tile, 64 contraction elements, cycles at 2.4 GHz; 16 MFMAs a wave take 620 alone): the loads
// from L2 into LDS move 31 B per cycle and compute unit in 64-byte row segments and 52 in 128-byte ones (a line at a time is
// looked up), so 64-wide steps feed the matrix cores where 32-wide ones cannot: 530 against 315 cycles per 16 KB.  A
// workgroup alone on its compute unit takes 1200 cycles a step, two together 860 each.
//  - one workgroup per compute unit or less (at most 256): four stages of 64-wide steps (128 KB), loads three steps ahead, and eight
//    waves, four for the first and four for the second half of every step's contraction (WK): a SIMD's two waves read fragments and
//    multiply in turns, the halves are added in front of the epilogue.  With four waves 6144 x 640 x 5760 49 to 58 us (two cards), now 41 to
//    51, 9800 x 256 x 2304 21.6 -> 18.1, 8192 x 320 x 2880 26.6 -> 22.1, 4096 x 640 x 5760 44.5 -> 35.9; 3840 x 1024 x 4096 and 8192 x 512 x
//    2048, whose rows come from memory once, 42 -> 40.5 and 25.2 -> 24.6 (loads alone: 23.4);
//  - otherwise two stages (64 KB, two workgroups per unit);
//  - many tiles of a short contraction (more than 1024, K <= 512) live on their prologues and epilogues overlapping: three
//    workgroups per unit with 32-wide steps (200704 x 128 x 512: 45 us, 51 with two).
// Before (32-wide steps in three stages for all, fragments read and used in the same step; random operands): 12544 x 512 x
// 4608 76 -> 67 us, 6144 x 640 x 5760 63 -> 52, 8192 x 512 x 2048 28 -> 23, 200704 x 128 x 1152 83 -> 76; the large layers of
// ResNet-50 at batch 256 are bound by memory and by the clock under full matrix load and gain 1 to 3 %.
// (Which tile: conv_tile_rule in conv_rules.h.)
// eight: the eight-wave tiles may be chosen (launches that store their rows in order)
static int igemm_tile(int64_t M, int N, int K, bool small_tiles, bool sums, bool eight) {
  if (N <= 64) return TILE_SQUARE;
  if (g_tune_tile == 2) return TILE_SQUARE;
  if (g_tune_tile == 3) return TILE_TALL;
  if (g_tune_tile == 4) return N % 256 == 0 ? TILE_WIDE : TILE_SQUARE;
  if (g_tune_tile == 5) return TILE_NARROW;
  if (g_tune_tile == 6) return TILE_SMALL;
  if (g_tune_tile == 7 && small_tiles) return TILE_160;
  if (g_tune_tile == 8) eight = false;
  if (eight)
    if (const int t = conv_eight_waves_rule(M, N, K, small_tiles)) return t;
  if (conv_cols160_rule(M, N, K, small_tiles)) return TILE_160;
  return conv_tile_rule(M, N, K, small_tiles, sums);
}
int conv_fprop_tile_class(const ConvGeom& g, bool bias, bool sums) {
  if (g.Cout <= 64) return 2;
  if (g.Cin < BK) return 0;
  const int t = igemm_tile(g.M(), g.Cout, (int)g.K(), g.Cin >= 64, sums, true);
  return t == TILE_SQUARE || (t == TILE_TALL && bias) ? 0 : (t == TILE_WIDE ? 1 : 2);   // (no 256x128 kernel with a bias)
}

template <int MODE, int BM, int BN, int WM, int WN, int STATS, int NWRAP, bool REMAP, int EPI, int BKT, int NS, int WK = 1>
static int launch_tile(IgemmArgs& a, hipStream_t s) {
  a.ntiles = (int)cdiv(a.N, BN);
  const int mt = (int)cdiv(a.M, BM);
  hipLaunchKernelGGL((igemm_kernel<MODE, BM, BN, WM, WN, false, STATS, NWRAP, REMAP, EPI, false, BKT, NS, WK>),
                     dim3((unsigned)((int64_t)mt * a.ntiles)), dim3(64 * WM * WN * WK), 0, s, a);
  return BM == 256 && BN == 256 && a.sum_parts == 2 ? (int)cdiv(a.M, 128) : mt;
}

// returns the number of m-tiles (= statistics chunks when STATS; conv_stat_chunks_max bounds it)
template <int MODE, int STATS, int NWRAP, bool REMAP, int EPI>
static int launch_igemm_w(IgemmArgs a, hipStream_t s) {
  a.pointwise = (a.kh == 1 && a.kw == 1 && a.stride == 1 && a.pad == 0 && a.pad_w == 0 && a.Hs == a.Hd &&
                 a.Ws == a.Wd) ? 1 : 0;
  a.group_m = 1;
  a.div_w = fast_div((uint32_t)a.Wd);
  a.div_h = fast_div((uint32_t)a.Hd);
  if (a.sliced) {   // grouped convolution: one column tile per slice of Cs = 32 or 64 channels
    if (a.Cs == 64) return launch_tile<MODE, 256, 64, 4, 1, STATS, NWRAP, REMAP, EPI, 32, 3>(a, s);
    return launch_tile<MODE, 256, 32, 4, 1, STATS, NWRAP, REMAP, EPI, 32, 3>(a, s);
  }
  if (a.N <= 64) {
    // N <= 64 over few rows (conv_rows_rule): 128x32, and 128x64 or 64x64
    const int rows = conv_rows_rule(a.M, a.N, a.K, STATS != 0);
    if (rows < 256 && a.N <= 32) return launch_tile<MODE, 128, 32, 4, 1, STATS, NWRAP, REMAP, EPI, 32, 3>(a, s);
    if constexpr (NWRAP == 1) {
      if (rows == 64 && a.Cs >= 64) return launch_tile<MODE, 64, 64, 2, 2, STATS, 1, REMAP, EPI, 64, 4>(a, s);
      if (rows == 128 && a.Cs >= 64) return launch_tile<MODE, 128, 64, 2, 2, STATS, 1, REMAP, EPI, 64, 3>(a, s);
    }
    if (rows == 64) return launch_tile<MODE, 64, 64, 2, 2, STATS, NWRAP, REMAP, EPI, 32, 4>(a, s);
    if (rows == 128) return launch_tile<MODE, 128, 64, 2, 2, STATS, NWRAP, REMAP, EPI, 32, 3>(a, s);
  }
  if (a.N <= 32) {
    // few channels, few steps (3 to 9): with more workgroups than two per compute unit, two stages (40 KB, three workgroups per
    // unit, one tile of loads less in front of the first step) against three stages: evaluation of ResNet-20 at
    // batch 8000 (8192000 x 16 x 144 and smaller) 5024 -> 4154 us a pass (4880 before fragments were read ahead), training step at batch 2048
    // 5195 -> 4639; with two workgroups or fewer the third stage hides latency (ResNet-20 step at batch 128 1147 against 1161)
    if (cdiv(a.M, 256) > 512) return launch_tile<MODE, 256, 32, 4, 1, STATS, NWRAP, REMAP, EPI, 32, 2>(a, s);
    return launch_tile<MODE, 256, 32, 4, 1, STATS, NWRAP, REMAP, EPI, 32, 3>(a, s);
  }
  if (a.N <= 64 || g_tune_tile == 1) return launch_tile<MODE, 256, 64, 4, 1, STATS, NWRAP, REMAP, EPI, 32, 3>(a, s);
  if constexpr (NWRAP == 1) {
    const bool w64 = a.Cs >= 64;
    const int tile = igemm_tile(a.M, a.N, a.K, w64, STATS != 0, !REMAP);
    if constexpr (!REMAP) {
      if ((EPI == 0 || EPI == 3) && tile == TILE_TALL) return launch_tile<MODE, 256, 128, 2, 2, STATS, 1, false, EPI, 32, 3>(a, s);
      if (tile == TILE_WIDE) return launch_tile<MODE, 128, 256, 2, 2, STATS, 1, false, EPI, 32, 3>(a, s);
      if (tile == TILE_256) {   // (a partial sum keeps the rows it had in the tiles that these take the place of)
        a.sum_parts = conv_tile_rule(a.M, a.N, a.K, true, true) == TILE_TALL ? 1 : 2;
        return launch_tile<MODE, 256, 256, 2, 4, STATS, 1, false, EPI, 64, 2>(a, s);
      }
      if (tile == TILE_WIDE8) return launch_tile<MODE, 128, 256, 2, 4, STATS, 1, false, EPI, 64, 3>(a, s);
    }
    if (w64) {
      if (tile == TILE_160) return launch_tile<MODE, 128, 160, 4, 1, STATS, 1, REMAP, EPI, 64, 2>(a, s);
      if (tile == TILE_SMALL) return launch_tile<MODE, 64, 64, 2, 2, STATS, 1, REMAP, EPI, 64, 4>(a, s);
      if (tile == TILE_NARROW) return launch_tile<MODE, 128, 64, 2, 2, STATS, 1, REMAP, EPI, 64, 3>(a, s);
      const int64_t wgs = cdiv(a.M, 128) * cdiv(a.N, 128);
      if (wgs <= 256) return launch_tile<MODE, 128, 128, 2, 2, STATS, 1, REMAP, EPI, 64, 4, 2>(a, s);
      if (wgs <= 1024 || a.K > 512) return launch_tile<MODE, 128, 128, 2, 2, STATS, 1, REMAP, EPI, 64, 2>(a, s);
    }
  }
  return launch_tile<MODE, 128, 128, 2, 2, STATS, NWRAP, REMAP, EPI, 32, 3>(a, s);
}
template <int MODE, int STATS, bool REMAP = false, int EPI = 0>
static int launch_igemm(IgemmArgs a, hipStream_t s) {
  return a.Cs >= BK ? launch_igemm_w<MODE, STATS, 1, REMAP, EPI>(a, s) : launch_igemm_w<MODE, STATS, 4, REMAP, EPI>(a, s);
}

bool conv_mfma_supported(const ConvGeom& g) {
  // 32-bit byte offsets into every operand, tap masks of at most 32 bits
  const int64_t lim = 1LL << 31;
  return g.Cin % 8 == 0 && g.Cout % 8 == 0 && (g.stride == 1 || g.stride == 2) && g.kh == g.kw && g.kh <= 7 &&
         g.B * g.H * g.W * (int64_t)g.Cin * 2 < lim && g.M() * (int64_t)g.Cout * 2 < lim &&
         (int64_t)g.Cout * g.K() * 2 < lim;
}

template <int BM, int BN, int EPI, bool GROUP, int BKT, int NS>
static void launch_linear(IgemmArgs a, hipStream_t s) {
  a.ntiles = (int)cdiv(a.N, BN);
  hipLaunchKernelGGL((igemm_kernel<0, BM, BN, 2, 2, true, 0, 1, false, EPI, GROUP, BKT, NS>),
                     dim3((unsigned)(cdiv(a.M, BM) * a.ntiles)), dim3(256), 0, s, a);
}

void linear_fwd_mfma(const bf16_t* x, const bf16_t* w, const bf16_t* bias, float* y, int64_t B, int F, int C,
                     hipStream_t s) {
  IgemmArgs a;
  a.src = x; a.wt = w; a.dst = reinterpret_cast<bf16_t*>(y); a.bias = bias; a.stat_partials = nullptr;
  a.M = B; a.N = C; a.K = F;
  a.Hs = 1; a.Ws = 1; a.Cs = F; a.Hd = 1; a.Wd = 1; a.kh = 1; a.kw = 1; a.stride = 1; a.pad = 0; a.pad_w = 0;
  a.omul = 0; a.ooff_h = a.ooff_w = 0; a.Ho = a.Wo = 1;
  a.accumulate = 0;
  a.pointwise = 1;
  a.group_m = 8;
  a.src_bytes = (uint32_t)(B * (int64_t)F * 2);
  a.wt_bytes = (uint32_t)((int64_t)C * F * 2);
  // a filter matrix beyond an L2's 4 MiB under a wide output: grouped tile order, with a short contraction on 256x128 tiles
  // (8192 x 32768 x 512 inside a training step: 471 us on 128x128 tiles, 459 so; non-temporal stores of the logits, faster when
  // the launch is repeated alone, 368 us, cost it 70 us there; 256x256 tiles of eight waves: the step 0.7 % faster, where the launch runs beside a
  // peer's, but passes of one model 1 to 3 % slower)
  const bool group = (int64_t)C * F * 2 > (4 << 20) && C >= 2048;
  // otherwise 64x64 tiles for few rows as igemm_tile says (256 x 1000 x 2048 18 -> 11 us), and for at most 64 classes up to 16384 rows, a
  // tile for every compute unit: the busiest unit has the same number of tiles of either shape there and a 64x64 one is the shorter
  // chain.  128x128 and 64x64 tiles, 10 classes: 128 rows of 64 8.0 and 3.8 us, of 2048 25.9 and 10.0; 16384 rows of 64 9.2 and 4.5, of 2048
  // 26.1 and 12.9; 64 classes 16384 x 512 9.6 and 5.7.  (Beyond the line 64x64 tiles win less, and lose in places: 32768 rows of 2048
  // onto 64 classes 43 and 34, 65536 of 64 7.9 and 8.2.)
  const bool narrow = C <= 64 && F >= 64 && B <= 64 * 256;
  const int tile = igemm_tile(B, C, F, F >= 64, false, false);
  if (group && F <= 512 && cdiv(B, 256) * cdiv(C, 128) >= 512) {
    a.group_m = 4;
    if (bias) launch_linear<256, 128, 1, true, 32, 3>(a, s); else launch_linear<256, 128, 0, true, 32, 3>(a, s);
  } else if (group && F >= 64) {
    if (bias) launch_linear<128, 128, 1, true, 64, 2>(a, s); else launch_linear<128, 128, 0, true, 64, 2>(a, s);
  } else if (tile == TILE_SMALL || narrow) {
    if (bias) launch_linear<64, 64, 1, false, 64, 4>(a, s); else launch_linear<64, 64, 0, false, 64, 4>(a, s);
  } else if (F >= 64) {
    if (bias) launch_linear<128, 128, 1, false, 64, 2>(a, s); else launch_linear<128, 128, 0, false, 64, 2>(a, s);
  } else {
    if (bias) launch_linear<128, 128, 1, false, 32, 3>(a, s); else launch_linear<128, 128, 0, false, 32, 3>(a, s);
  }
}

static void set_norm(IgemmArgs& a, const EvalNorm& n) {
  a.norm_run = n.running;
  a.norm_gamma = static_cast<const bf16_t*>(n.gamma);
  a.norm_beta = static_cast<const bf16_t*>(n.beta);
  a.norm_res = static_cast<const bf16_t*>(n.res);
  a.norm_relu = n.relu ? 1 : 0;
}

int conv_fprop_mfma(const bf16_t* x, const bf16_t* w, const bf16_t* bias, bool relu, bf16_t* y, const ConvGeom& g,
                    float* stat_partials, hipStream_t s, const EvalNorm* norm) {
  IgemmArgs a;
  a.bias = bias;
  a.stat_partials = stat_partials;
  a.src = x; a.wt = w; a.dst = y;
  a.M = g.M(); a.N = g.Cout; a.K = g.K();
  a.Hs = g.H; a.Ws = g.W; a.Cs = g.Cin; a.Hd = g.Ho; a.Wd = g.Wo;
  a.kh = g.kh; a.kw = g.kw; a.stride = g.stride; a.pad = g.pad; a.pad_w = g.pad;
  a.omul = 0; a.ooff_h = a.ooff_w = 0; a.Ho = g.Ho; a.Wo = g.Wo;
  a.accumulate = 0; a.ntiles = 1;
  a.src_bytes = (uint32_t)(g.B * g.H * g.W * (int64_t)g.Cin * 2);
  a.wt_bytes = (uint32_t)((int64_t)g.Cout * g.K() * 2);
  if (bias) {  // bias (+ ReLU) in the epilogue; no statistics variant (a BatchNorm follows bias-free convolutions)
    if (stat_partials || norm) return -1;
    return relu ? launch_igemm<0, false, false, 2>(a, s) : launch_igemm<0, false, false, 1>(a, s);
  }
  if (relu) return -1;  // ReLU without bias does not occur in the supported graphs
  if (norm) {
    if (stat_partials) return -1;
    set_norm(a, *norm);
    return launch_igemm<0, false, false, 3>(a, s);
  }
  return stat_partials ? launch_igemm<0, true>(a, s) : launch_igemm<0, false>(a, s);
}

__global__ void __launch_bounds__(256) fill_zero16_k(uint4* p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = make_uint4(0, 0, 0, 0);
}

// ---- filter re-layouts of many data gradients in one launch ------------------------------------------------------
constexpr int kLayoutJobs = 48;   // jobs per launch: the table travels in the kernel arguments
struct LayoutBatch { WeightLayoutJob j[kLayoutJobs]; int n; int64_t total; };
static_assert(sizeof(LayoutBatch) <= 4096, "the table travels in the kernel arguments");
// A workgroup transposes one 64x64 tile (output x input channels) of one tap through LDS: 128-byte row segments are read and
// written, where one thread per element read with a stride of the whole filter row (44 M filter elements of the Transformer:
// 537 us, now 56; ResNet-50 256 -> 37).  Channel counts are multiples of 8 and every filter starts on a 16-byte boundary.
constexpr int kLayoutTile = 64, kLayoutPitch = 66;   // 33 words a row: the columns read back fall into different banks
__global__ void __launch_bounds__(256) relayout_weights_k(LayoutBatch b) {
  __shared__ uint32_t sm[kLayoutTile * kLayoutPitch / 2];
  const int64_t i = blockIdx.x;
  int k = 0;
  while (k + 1 < b.n && b.j[k + 1].first <= i) k++;
  const WeightLayoutJob& q = b.j[k];
  const int nc = (q.cin + kLayoutTile - 1) / kLayoutTile, nn = (q.cout + kLayoutTile - 1) / kLayoutTile;
  int t = (int)(i - q.first);
  const int c0 = t % nc * kLayoutTile; t /= nc;
  const int n0 = t % nn * kLayoutTile; t /= nn;
  const int jw = t % q.tw, jh = t / q.tw;
  const int64_t tap = (int64_t)(q.r0 + q.rstep * jh) * q.kw + (q.s0 + q.rstep * jw);
#pragma unroll
  for (int u = 0; u < 2; u++) {
    const int e = threadIdx.x + 256 * u, n = e >> 3, c = (e & 7) * 8;
    if (n0 + n < q.cout && c0 + c < q.cin) {
      const uint4 v = *reinterpret_cast<const uint4*>(q.w + ((int64_t)(n0 + n) * q.kh * q.kw + tap) * q.cin + c0 + c);
      uint32_t* o = sm + (n * kLayoutPitch + c) / 2;
      o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
    }
  }
  __syncthreads();
  const bf16_t* tile = reinterpret_cast<const bf16_t*>(sm);
#pragma unroll
  for (int u = 0; u < 2; u++) {
    const int e = threadIdx.x + 256 * u, c = e >> 3, n = (e & 7) * 8;
    if (c0 + c < q.cin && n0 + n < q.cout) {
      uint32_t o[4];
#pragma unroll
      for (int p = 0; p < 4; p++)
        o[p] = (uint32_t)tile[(n + 2 * p) * kLayoutPitch + c] | ((uint32_t)tile[(n + 2 * p + 1) * kLayoutPitch + c] << 16);
      *reinterpret_cast<uint4*>(q.wt + (((int64_t)(c0 + c) * q.th + jh) * q.tw + jw) * q.cout + n0 + n) =
          make_uint4(o[0], o[1], o[2], o[3]);
    }
  }
}
void relayout_weights_batch(std::vector<WeightLayoutJob>& jobs, hipStream_t s) {
  for (size_t j0 = 0; j0 < jobs.size(); j0 += kLayoutJobs) {
    LayoutBatch b;
    b.n = (int)std::min<size_t>(kLayoutJobs, jobs.size() - j0);
    b.total = 0;
    for (int k = 0; k < b.n; k++) {
      WeightLayoutJob& q = jobs[j0 + k];
      q.first = b.total;
      b.j[k] = q;
      b.total += (int64_t)q.th * q.tw * cdiv(q.cin, kLayoutTile) * cdiv(q.cout, kLayoutTile);
    }
    if (b.total > 0) hipLaunchKernelGGL(relayout_weights_k, dim3((unsigned)b.total), dim3(256), 0, s, b);
  }
}
// The parity classes of a stride-2 data gradient (see conv_dgrad_mfma): calls f(ph, pw, th, tw, tminh, tminw) for every
// class that has taps and pixels.
template <typename F>
static void for_each_parity_class(const ConvGeom& g, F f) {
  for (int ph = 0; ph < 2; ph++)
    for (int pw = 0; pw < 2; pw++) {
      const int loh = ph + g.pad - g.kh + 1, low = pw + g.pad - g.kw + 1;
      const int tminh = loh <= 0 ? -((-loh) >> 1) : (loh + 1) >> 1, tmaxh = (ph + g.pad) >> 1;
      const int tminw = low <= 0 ? -((-low) >> 1) : (low + 1) >> 1, tmaxw = (pw + g.pad) >> 1;
      const int th = tmaxh - tminh + 1, tw = tmaxw - tminw + 1;
      const int hd = (g.H - ph + 1) / 2, wd = (g.W - pw + 1) / 2;
      if (th <= 0 || tw <= 0 || hd <= 0 || wd <= 0) continue;
      f(ph, pw, th, tw, tminh, tminw);
    }
}
int64_t conv_dgrad_layout_elems(const ConvGeom& g) {
  if (g.stride == 1) return (int64_t)g.Cout * g.K();
  int64_t n = 0;
  for_each_parity_class(g, [&](int, int, int th, int tw, int, int) { n += ((int64_t)g.Cin * th * tw * g.Cout + 7) / 8 * 8; });
  return n;
}
void conv_dgrad_layout_jobs(const bf16_t* w, bf16_t* wt, const ConvGeom& g, std::vector<WeightLayoutJob>& jobs) {
  if (g.stride == 1) {   // wt[Cin][kh][kw][Cout] = w[Cout][kh][kw][Cin]
    jobs.push_back(WeightLayoutJob{w, wt, g.Cout, g.kh, g.kw, g.Cin, g.kh, g.kw, 0, 0, 1, 0});
    return;
  }
  int64_t woff = 0;
  for_each_parity_class(g, [&](int ph, int pw, int th, int tw, int tminh, int tminw) {
    jobs.push_back(WeightLayoutJob{w, wt + woff, g.Cout, g.kh, g.kw, g.Cin, th, tw, ph + g.pad - 2 * tminh, pw + g.pad - 2 * tminw,
                                   -2, 0});
    woff += ((int64_t)g.Cin * th * tw * g.Cout + 7) / 8 * 8;
  });
}

int conv_dgrad_mfma(const bf16_t* dy, const bf16_t* w, bf16_t* wt, bf16_t* dx, const ConvGeom& g, bool accumulate,
                    hipStream_t s, const bf16_t* addend, const uint8_t* addend_gate, const bf16_t* relu_out,
                    const BnBackwardSums* bn, bool wt_ready) {
  IgemmArgs a;
  a.bias = nullptr;
  a.stat_partials = nullptr;
  a.src = dy; a.dst = dx;
  a.N = g.Cin;
  a.Hs = g.Ho; a.Ws = g.Wo; a.Cs = g.Cout;
  a.ntiles = 1;
  a.src_bytes = (uint32_t)(g.M() * (int64_t)g.Cout * 2);
  a.Ho = g.H; a.Wo = g.W;
  if (!wt_ready) {
    std::vector<WeightLayoutJob> jobs;
    conv_dgrad_layout_jobs(w, wt, g, jobs);
    relayout_weights_batch(jobs, s);
  }
  if (g.stride == 1) {
    a.wt = wt;
    a.M = g.B * g.H * g.W; a.K = g.kh * g.kw * g.Cout;
    a.Hd = g.H; a.Wd = g.W;
    a.kh = g.kh; a.kw = g.kw; a.stride = 1; a.pad = g.pad; a.pad_w = g.pad;
    a.omul = 0; a.ooff_h = a.ooff_w = 0;
    a.accumulate = (accumulate || addend) ? 1 : 0;
    a.addend = addend;          // stride 1 only (see the declaration); never together with accumulate
    a.addend_gate = addend_gate;
    a.relu_out = relu_out;      // stride 1 only, like the addend
    a.wt_bytes = (uint32_t)((int64_t)g.Cout * g.K() * 2);
    if (bn) {
      a.bn_x = bn->x; a.bn_mask = bn->mask; a.bn_stats = bn->stats; a.stat_partials = bn->partials;
      return launch_igemm<1, 2>(a, s);
    }
    launch_igemm<1, 0>(a, s);
    return 0;
  }
  // Stride 2: input pixel (h, w) receives dy[(h + pad - r)/2, (w + pad - s)/2] * w[., r, s, .] for the taps
  // of matching parity only.  Per parity class (h%2, w%2) that is a stride-1 gather over the half
  // resolution grid h = 2h' + ph with window rows t in [tmin, tmax], ho = h' + t, r = ph + pad - 2t: a
  // MODE 0 problem with its own filter layout, writing every second row / column of dx.
  bool covered_all = true;
  for (int ph = 0; ph < 2; ph++) {
    const int tmax = (ph + g.pad) >> 1, lo = ph + g.pad - g.kh + 1;
    if (tmax < (lo <= 0 ? -((-lo) >> 1) : (lo + 1) >> 1)) covered_all = false;
  }
  if (!accumulate && !covered_all) {
    const int64_t n16 = g.B * g.H * g.W * (int64_t)g.Cin / 8;
    hipLaunchKernelGGL(fill_zero16_k, dim3((unsigned)cdiv(n16, 256)), dim3(256), 0, s, reinterpret_cast<uint4*>(dx), n16);
    accumulate = true;
  }
  int64_t woff = 0;
  for (int ph = 0; ph < 2; ph++)
    for (int pw = 0; pw < 2; pw++) {
      const int loh = ph + g.pad - g.kh + 1, low = pw + g.pad - g.kw + 1;
      const int tminh = loh <= 0 ? -((-loh) >> 1) : (loh + 1) >> 1, tmaxh = (ph + g.pad) >> 1;
      const int tminw = low <= 0 ? -((-low) >> 1) : (low + 1) >> 1, tmaxw = (pw + g.pad) >> 1;
      const int th = tmaxh - tminh + 1, tw = tmaxw - tminw + 1;
      const int hd = (g.H - ph + 1) / 2, wd = (g.W - pw + 1) / 2;
      if (th <= 0 || tw <= 0 || hd <= 0 || wd <= 0) continue;
      bf16_t* wc = wt + woff;
      const int64_t wn = (int64_t)g.Cin * th * tw * g.Cout;
      woff += (wn + 7) / 8 * 8;
      a.wt = wc;
      a.M = g.B * hd * wd; a.K = th * tw * g.Cout;
      a.Hd = hd; a.Wd = wd;
      a.kh = th; a.kw = tw; a.stride = 1; a.pad = -tminh; a.pad_w = -tminw;
      a.omul = 2; a.ooff_h = ph; a.ooff_w = pw;
      a.accumulate = accumulate ? 1 : 0;
      a.wt_bytes = (uint32_t)(wn * 2);
      launch_igemm<0, 0, true>(a, s);
    }
  return 0;
}

// ---- grouped convolutions (Cin = Cout = C, groups of cg = C / groups channels) as sliced launches ----------------
// The channels are cut into slices of SW = 32 or 64 (whole groups).  Column tile s of a launch computes the SW output
// channels of slice s from the SW input channels of the same slice, read in place from the row-major tensor (pitch C),
// with a filter whose rows hold kh * kw * SW elements, zero outside the row's own group: for cg = SW the contraction
// runs over the group's channels only, for smaller groups it spends SW / cg times the grouped arithmetic on zeros.
int grouped_mfma_slice(int C, int groups) {
  if (groups < 1 || C % groups) return 0;
  const int cg = C / groups;
  const int sw = cg > 32 ? 64 : 32;
  return (C % sw == 0 && sw % cg == 0) ? sw : 0;
}

// w [C][taps][cg] -> wd [C][th * tw][SW]: row o, tap (jh, jw), column i holds w[o][r][t][i - its group's first channel
// in the slice] if input channel i of o's slice belongs to o's group, else 0; r = r0 + rstep * jh, t = s0 + rstep * jw.
// TRANSPOSED: wd [C][th * tw][SW] indexed [input channel c][tap][output channel of c's slice] (data gradients).
template <bool TRANSPOSED>
__global__ void __launch_bounds__(256) expand_sliced_weights_k(const bf16_t* __restrict__ w, bf16_t* __restrict__ wd, int C,
                                                               int kh, int kw, int cg, int SW, int th, int tw, int r0, int s0,
                                                               int rstep) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (int64_t)C * th * tw * SW) return;
  const int col = (int)(idx % SW);
  const int t = (int)((idx / SW) % (th * tw));
  const int row = (int)(idx / ((int64_t)SW * th * tw));
  const int slice0 = row / SW * SW;
  const int o = TRANSPOSED ? slice0 + col : row;      // output channel
  const int ci = TRANSPOSED ? row : slice0 + col;     // input channel
  const int r = r0 + rstep * (t / tw), q = s0 + rstep * (t % tw);
  const bool ok = o / cg == ci / cg && r >= 0 && r < kh && q >= 0 && q < kw;
  wd[idx] = ok ? w[(((int64_t)o * kh + r) * kw + q) * cg + ci % cg] : (bf16_t)0;
}

static void fill_sliced(IgemmArgs& a, int C, int SW) {
  a.N = C; a.Cs = SW; a.src_pitch = C; a.sliced = 1;
  a.bias = nullptr; a.addend = nullptr; a.addend_gate = nullptr; a.relu_out = nullptr;
  a.omul = 0; a.ooff_h = a.ooff_w = 0;
  a.accumulate = 0; a.ntiles = 1;
}

int conv_grouped_fprop_mfma(const bf16_t* x, const bf16_t* w, bf16_t* wd, bf16_t* y, const ConvGeom& g, int groups,
                            float* stat_partials, hipStream_t s, const EvalNorm* norm) {
  const int C = g.Cin, cg = C / groups, SW = grouped_mfma_slice(C, groups), taps = g.kh * g.kw;
  const int64_t nw = (int64_t)C * taps * SW;
  hipLaunchKernelGGL(expand_sliced_weights_k<false>, dim3((unsigned)cdiv(nw, 256)), dim3(256), 0, s, w, wd, C, g.kh, g.kw, cg, SW,
                     g.kh, g.kw, 0, 0, 1);
  IgemmArgs a;
  fill_sliced(a, C, SW);
  a.stat_partials = stat_partials;
  a.src = x; a.wt = wd; a.dst = y;
  a.M = g.M(); a.K = taps * SW;
  a.Hs = g.H; a.Ws = g.W; a.Hd = g.Ho; a.Wd = g.Wo;
  a.kh = g.kh; a.kw = g.kw; a.stride = g.stride; a.pad = g.pad; a.pad_w = g.pad;
  a.Ho = g.Ho; a.Wo = g.Wo;
  a.src_bytes = (uint32_t)(g.B * g.H * g.W * (int64_t)C * 2);
  a.wt_bytes = (uint32_t)(nw * 2);
  if (norm) {
    if (stat_partials) return -1;
    set_norm(a, *norm);
    return launch_igemm_w<0, false, 1, false, 3>(a, s);
  }
  return stat_partials ? launch_igemm_w<0, true, 1, false, 0>(a, s) : launch_igemm_w<0, false, 1, false, 0>(a, s);
}

void conv_grouped_dgrad_mfma(const bf16_t* dy, const bf16_t* w, bf16_t* wd, bf16_t* dx, const ConvGeom& g, int groups,
                             bool accumulate, hipStream_t s) {
  const int C = g.Cin, cg = C / groups, SW = grouped_mfma_slice(C, groups);
  IgemmArgs a;
  fill_sliced(a, C, SW);
  a.stat_partials = nullptr;
  a.src = dy; a.dst = dx;
  a.Hs = g.Ho; a.Ws = g.Wo;
  a.src_bytes = (uint32_t)(g.M() * (int64_t)C * 2);
  a.Ho = g.H; a.Wo = g.W;
  if (g.stride == 1) {
    const int64_t nw = (int64_t)C * g.kh * g.kw * SW;
    hipLaunchKernelGGL(expand_sliced_weights_k<true>, dim3((unsigned)cdiv(nw, 256)), dim3(256), 0, s, w, wd, C, g.kh, g.kw, cg,
                       SW, g.kh, g.kw, 0, 0, 1);
    a.wt = wd;
    a.M = g.B * g.H * g.W; a.K = g.kh * g.kw * SW;
    a.Hd = g.H; a.Wd = g.W;
    a.kh = g.kh; a.kw = g.kw; a.stride = 1; a.pad = g.pad; a.pad_w = g.pad;
    a.accumulate = accumulate ? 1 : 0;
    a.wt_bytes = (uint32_t)(nw * 2);
    launch_igemm_w<1, false, 1, false, 0>(a, s);
    return;
  }
  // stride 2: one stride-1 problem per parity class of the input pixel, as in conv_dgrad_mfma
  bool covered_all = true;
  for (int ph = 0; ph < 2; ph++) {
    const int tmax = (ph + g.pad) >> 1, lo = ph + g.pad - g.kh + 1;
    if (tmax < (lo <= 0 ? -((-lo) >> 1) : (lo + 1) >> 1)) covered_all = false;
  }
  if (!accumulate && !covered_all) {
    const int64_t n16 = g.B * g.H * g.W * (int64_t)C / 8;
    hipLaunchKernelGGL(fill_zero16_k, dim3((unsigned)cdiv(n16, 256)), dim3(256), 0, s, reinterpret_cast<uint4*>(dx), n16);
    accumulate = true;
  }
  int64_t woff = 0;
  for (int ph = 0; ph < 2; ph++)
    for (int pw = 0; pw < 2; pw++) {
      const int loh = ph + g.pad - g.kh + 1, low = pw + g.pad - g.kw + 1;
      const int tminh = loh <= 0 ? -((-loh) >> 1) : (loh + 1) >> 1, tmaxh = (ph + g.pad) >> 1;
      const int tminw = low <= 0 ? -((-low) >> 1) : (low + 1) >> 1, tmaxw = (pw + g.pad) >> 1;
      const int th = tmaxh - tminh + 1, tw = tmaxw - tminw + 1;
      const int hd = (g.H - ph + 1) / 2, wdd = (g.W - pw + 1) / 2;
      if (th <= 0 || tw <= 0 || hd <= 0 || wdd <= 0) continue;
      bf16_t* wc = wd + woff;
      const int64_t wn = (int64_t)C * th * tw * SW;
      hipLaunchKernelGGL(expand_sliced_weights_k<true>, dim3((unsigned)cdiv(wn, 256)), dim3(256), 0, s, w, wc, C, g.kh, g.kw, cg,
                         SW, th, tw, ph + g.pad - 2 * tminh, pw + g.pad - 2 * tminw, -2);
      woff += (wn + 7) / 8 * 8;
      a.wt = wc;
      a.M = g.B * hd * wdd; a.K = th * tw * SW;
      a.Hd = hd; a.Wd = wdd;
      a.kh = th; a.kw = tw; a.stride = 1; a.pad = -tminh; a.pad_w = -tminw;
      a.omul = 2; a.ooff_h = ph; a.ooff_w = pw;
      a.accumulate = accumulate ? 1 : 0;
      a.wt_bytes = (uint32_t)(wn * 2);
      launch_igemm_w<0, false, 1, true, 0>(a, s);
    }
}

// ---- wgrad ------------------------------------------------------------------------------------------
// dw[n][k] = sum_m dy[m][n] * im2col(x)[m][k].  The contraction runs over pixels, which is the slow
// axis of both operands in memory.  Tiles are staged in LDS as they lie in memory ([pixel][channel],
// 16-byte vectors along the channels) and read back with the gfx950 LDS transpose load
// (ds_read_b64_tr_b16): in every group of 16 lanes, lane i receives element (i & 3) of the four
// 8-byte chunks addressed by lanes (i >> 2), 4 + (i >> 2), 8 + (i >> 2), 12 + (i >> 2).  Pointing
// chunk 4e+q at pixel e, channels 4q..4q+3 therefore hands lane i four consecutive pixels of channel
// i, which is the MFMA operand layout.
//
// A launch takes the weight gradients of several layers: a tile of any of them is a workgroup.  One layer of a Transformer or of
// a late ResNet stage has 16 to 144 tiles, which fill the chip only if its pixels are cut into many splits, and each split is
// an fp32 copy of dw to be written and added up again; side by side the layers fill it with few splits or none.  (The rule: wgrad_plan in
// conv_rules.h.)  Splits are added by a second kernel in a fixed order.
// One encoder layer (8192 tokens, 512 columns, 2048 inside), sums of the splits included: its four layers one after the other 138 us with
// registers in front of the LDS and two stages, 190 with the bias gradients; one launch 84 and 88, with the folds below 90 and 95; 32768 x 512 over 8192 rows
// 363 -> 308, 256 x 2304 over 50176 99 -> 90.  More stages or 64-pixel steps cost workgroups per compute unit and were no faster.
//
// Main loop: as igemm_kernel's, steps of 32 pixels, NS stages in LDS filled by direct loads NS - 1 steps ahead, one barrier a
// step, the fragments of the next 16 pixels read while the matrix cores work.
struct WgradJob {
  const bf16_t* x;    // [B][H][W][Cin]
  const bf16_t* dy;   // [M][N]
  float* out;         // [splits][slices][N][K]
  double* bias_part;  // column sums of dy, the bias gradient: [splits][N] (more than one split) or null
  float* bias_out;    // [N] (one split) or null
  int M, m_per_split;
  int fold;           // (launches of several layers) steps that one chain of additions covers at the most
  int N, K;
  int H, W, Cin, Ho, Wo, kw, stride, pad;
  int ktiles, tiles_per_slice, tiles;   // tiles along K; of a slice of dw; of dw in all
  // Grouped convolutions (sliced launches): independent problems, slice s taking channels [s * N, (s + 1) * N) of
  // dy and [s * Cin, (s + 1) * Cin) of x, both row-major with `pitch` channels per pixel (N = Cin = the slice width).
  // An ordinary convolution: one slice, x_pitch = Cin, dy_pitch = N.
  int slices, x_pitch, dy_pitch;
  FastDiv div_wo, div_ho, div_cin, div_kw;
  uint32_t x_bytes, dy_bytes;
  uint32_t first;     // workgroups of the jobs in front of this one
};
template <int NJ> struct WgradBatch { WgradJob j[NJ]; int n; };
static_assert(sizeof(WgradBatch<kWgradJobs>) <= 4096, "the table travels in the kernel arguments");

constexpr int WG_MS = 32;   // pixels per main-loop step

// PW: 1x1 filters, stride 1, no padding: row m of x belongs to row m of dy
template <int BN, int BKK, bool PW, int NJ>
__global__ void __launch_bounds__(256, NJ > 1 ? 2 : 1) wgrad_kernel(WgradBatch<NJ> batch) {
  constexpr int NS = kWgradStages;
  constexpr int NVR = BN / 8, KVR = BKK / 8;   // 16-byte vectors per tile row
  constexpr int DV = WG_MS * NVR / 256, XV = WG_MS * KVR / 256;  // vectors per thread per step
  constexpr int DROWS = 256 / NVR, XROWS = 256 / KVR;
  constexpr int WNT = BN / 2, WKT = BKK / 2;   // wave tile (2 x 2 waves)
  constexpr int TN = WNT / 32, TK = WKT / 32, TT = TN * TK, KK = WG_MS / 16;
  constexpr uint32_t DY_BYTES = WG_MS * BN * 2, STAGE_BYTES = DY_BYTES + WG_MS * BKK * 2;
  static_assert(NS * STAGE_BYTES >= 2 * BN * 8, "the bias sums of two waves fit");
  __shared__ __attribute__((aligned(16))) char smem[NS * STAGE_BYTES];   // stage: [32 pixels][BN] of dy, [32 pixels][BKK] of x

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wn0 = (wave & 1) * WNT, wk0 = (wave >> 1) * WKT;
  // One-dimensional grid of jobs x splits x tiles, renumbered per XCD: the tiles of one pixel range (they
  // read the same rows of dy, and the same rows of x up to the filter's reach) run side by side on
  // one XCD and share those rows in its L2 instead of each fetching them from memory.
  const unsigned bid = xcd_remap(blockIdx.x, gridDim.x);
  int jn = 0;
  if (NJ > 1)
    while (jn + 1 < batch.n && batch.j[jn + 1].first <= bid) jn++;
  const WgradJob& a = batch.j[jn];
  const unsigned wg = bid - a.first;
  const unsigned split = wg / (unsigned)a.tiles, tile_all = wg - split * (unsigned)a.tiles;
  const unsigned sl = tile_all / (unsigned)a.tiles_per_slice, tile = tile_all - sl * (unsigned)a.tiles_per_slice;
  const int n0 = (int)(tile / (unsigned)a.ktiles) * BN, k0 = (int)(tile % (unsigned)a.ktiles) * BKK;
  const int dyc0 = (int)sl * a.N, xc0 = (int)sl * a.Cin;   // first channel of this slice in dy and in x
  // pixel and element indices fit 32 bits: every operand is smaller than 2 GiB (conv_mfma_supported)
  const int M = a.M;
  const int mbeg = (int)split * a.m_per_split;
  const int mend = M - mbeg > a.m_per_split ? mbeg + a.m_per_split : M;
  const rsrc_words_t rx = make_rsrc_words(a.x, a.x_bytes), rdy = make_rsrc_words(a.dy, a.dy_bytes);

  // ---- loads: thread tid owns LDS slot tid % NVR (16 bytes) of the tile rows tid / NVR + DROWS j.  The 16-byte column cv of a
  // row lies in slot cv ^ swz(row): a transpose load's four rows of 32 bytes, and the neighbouring 32 bytes that the next
  // sixteen lanes read, then fall into different banks.  A thread's rows are a multiple of 16 apart and share their swz.
  auto swz = [](int row, int vr) { return vr == 16 ? 4 * (row & 3) : 4 * ((row >> 1) & 1); };
  const int drow = tid / NVR, dcv = (tid % NVR) ^ swz(drow, NVR);
  const uint32_t dnot = n0 + dcv * 8 < a.N ? 0u : 0xffffffffu;   // or-ed into an offset: beyond every buffer, reads zeros
  int dm = mbeg + drow;                                          // row of vector 0 in the step at hand
  uint32_t doff = ((uint32_t)dm * (uint32_t)a.dy_pitch + (uint32_t)(dyc0 + n0 + dcv * 8)) * 2u;
  const uint32_t dstep = (uint32_t)WG_MS * (uint32_t)a.dy_pitch * 2u, drstep = (uint32_t)DROWS * (uint32_t)a.dy_pitch * 2u;
  const int xrow = tid / KVR, xcv = (tid % KVR) ^ swz(xrow, KVR);
  const int k = k0 + xcv * 8;
  const uint32_t xnot = k < a.K ? 0u : 0xffffffffu;
  int xm = mbeg + xrow;
  // PW: byte offset of vector 0.  Otherwise: the tap and channel of this thread's column, and each row's pixel
  uint32_t xoff = ((uint32_t)xm * (uint32_t)a.x_pitch + (uint32_t)(xc0 + k)) * 2u;
  const uint32_t xstep = (uint32_t)WG_MS * (uint32_t)a.x_pitch * 2u, xrstep = (uint32_t)XROWS * (uint32_t)a.x_pitch * 2u;
  const int tap = PW || xnot ? 0 : (int)div_by((unsigned)k, a.div_cin);
  const int kc = k - tap * a.Cin, kr = PW ? 0 : (int)div_by((unsigned)tap, a.div_kw), ks = tap - kr * (PW ? 0 : a.kw);
  int pb[PW ? 1 : XV], ph[PW ? 1 : XV], pw[PW ? 1 : XV];
  int adv_b = 0, adv_h = 0, adv_w = 0;
  if (!PW) {
#pragma unroll
    for (int j = 0; j < XV; j++) {
      const unsigned m = (unsigned)(xm + XROWS * j);
      const unsigned q = div_by(m, a.div_wo);
      pw[j] = (int)(m - q * (unsigned)a.Wo);
      pb[j] = (int)div_by(q, a.div_ho);
      ph[j] = (int)(q - (unsigned)pb[j] * (unsigned)a.Ho);
    }
    // one step moves every row WG_MS pixels on: whole images, then whole rows, then columns
    adv_b = WG_MS / (a.Ho * a.Wo);
    const int adv_r = WG_MS % (a.Ho * a.Wo);
    adv_h = adv_r / a.Wo;
    adv_w = adv_r % a.Wo;
  }
  uint32_t offd[DV], offx[XV];
  constexpr int NPIECE = DV + XV + 1;
  // piece p of the preparation of the step at hand: one vector's offset (rows past the split's end are masked in both operands),
  // or (last) the move to the next step; straight-line code between the MFMAs
  auto prep_piece = [&](int p) {
    if (p < DV) {
      offd[p] = (doff + (uint32_t)p * drstep) | dnot | (dm + DROWS * p < mend ? 0u : 0xffffffffu);
    } else if (p < DV + XV) {
      const int j = p - DV;
      const uint32_t out = xnot | (xm + XROWS * j < mend ? 0u : 0xffffffffu);
      if (PW) {
        offx[j] = (xoff + (uint32_t)j * xrstep) | out;
      } else {
        const int hi = ph[j] * a.stride - a.pad + kr, wi = pw[j] * a.stride - a.pad + ks;
        const bool ok = (unsigned)hi < (unsigned)a.H && (unsigned)wi < (unsigned)a.W;
        offx[j] = ((uint32_t)(((pb[j] * a.H + hi) * a.W + wi) * a.x_pitch + xc0 + kc) * 2u) | out | (ok ? 0u : 0xffffffffu);
        pw[j] += adv_w;
        const int cw = pw[j] >= a.Wo ? 1 : 0;
        pw[j] -= cw ? a.Wo : 0;
        ph[j] += adv_h + cw;
        const int ch = ph[j] >= a.Ho ? 1 : 0;
        ph[j] -= ch ? a.Ho : 0;
        pb[j] += adv_b + ch;
      }
    } else {
      dm += WG_MS;
      doff += dstep;
      xm += WG_MS;
      xoff += xstep;
    }
  };
  const uint32_t lds_wave = (uint32_t)(uintptr_t)(CD_LDS char*)smem + (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6) * 1024u;
  auto issue = [&](uint32_t stage_b, int v) {
    if (v < DV) load_lds16(rdy, lds_wave + stage_b + (uint32_t)v * 4096u, offd[v]);
    else load_lds16(rx, lds_wave + stage_b + DY_BYTES + (uint32_t)(v - DV) * 4096u, offx[v - DV]);
  };

  f32x16_t acc[TN][TK];
#pragma unroll
  for (int i = 0; i < TN; i++)
#pragma unroll
    for (int j = 0; j < TK; j++)
#pragma unroll
      for (int v = 0; v < 16; v++) acc[i][j][v] = 0.f;

  // transpose-load addressing of this lane inside a 16-pixel x 32-channel fragment (the second load: four pixels on, same swz)
  const int grp = lane >> 4, li = lane & 15;
  const int tr_m = 8 * (grp >> 1) + (li >> 2);      // pixel row
  const int tr_c = 16 * (grp & 1) + 4 * (li & 3);   // first of the 4 channels this lane points at
  // byte offset of channel c of row m in a tile of vr vectors a row
  auto at = [&](int m, int c, int vr) { return (uint32_t)((m * vr + ((c >> 3) ^ swz(m, vr))) * 16 + (c & 7) * 2); };
  uint32_t fd[TN], fx[TK];
#pragma unroll
  for (int i = 0; i < TN; i++) fd[i] = at(tr_m, wn0 + i * 32 + tr_c, NVR);
#pragma unroll
  for (int j = 0; j < TK; j++) fx[j] = DY_BYTES + at(tr_m, wk0 + j * 32 + tr_c, KVR);
  bf16x8_t df[2][TN], xf[2][TK];  // [buffer][tile]
  auto read_tr = [&](uint32_t b, int pitch) {
    const bf16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((CD_LDS bf16x4_t*)(smem + b));
    const bf16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((CD_LDS bf16x4_t*)(smem + b + 4 * pitch));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  };
  auto read_frags = [&](int buf, uint32_t stage_b, int kk) {
#pragma unroll
    for (int i = 0; i < TN; i++) df[buf][i] = read_tr(stage_b + fd[i] + (uint32_t)(kk * 16 * BN * 2), BN * 2);
#pragma unroll
    for (int j = 0; j < TK; j++) xf[buf][j] = read_tr(stage_b + fx[j] + (uint32_t)(kk * 16 * BKK * 2), BKK * 2);
  };
  // The bias gradient: the workgroups of the first tile column add up the dy fragments that pass through their registers, the
  // two waves of a channel block alternate sub-steps.  A lane holds eight pixels of one channel: their sum is fp32, the sums'
  // sum fp64.
  const bool bias = k0 == 0 && (a.bias_part || a.bias_out);
  const int uwave = __builtin_amdgcn_readfirstlane(tid >> 6);
  double bsum[TN];
#pragma unroll
  for (int i = 0; i < TN; i++) bsum[i] = 0.0;
  float bhalf = 0.f;
  auto add_bias = [&](const bf16x8_t& f, int half, double& s) {   // four pixels at a time: the shadow of one MFMA
    const uint4 u = __builtin_bit_cast(uint4, f);
    const uint32_t w0 = half ? u.z : u.x, w1 = half ? u.w : u.y;
    const float t = (__uint_as_float(w0 << 16) + __uint_as_float(w0 & 0xffff0000u)) +
                    (__uint_as_float(w1 << 16) + __uint_as_float(w1 & 0xffff0000u));
    if (half) s += (double)(bhalf + t); else bhalf = t;
  };

  // FOLD: every a.fold steps the accumulators are added to a second set of fp32 sums, and what that addition rounds away stays behind
  // in the accumulator (compensated summation).  A launch of several layers cuts the rows into few splits or none, and one chain of
  // fp32 additions over all of them was further from the float64 result than the splits it took the place of: a chain now covers the rows
  // of one of those (wgrad_own_rows).  2-norm of the error over that of dw, a layer by itself in splits / one chain / folded:
  // 512 x 512 over 8192 rows 6.7e-8 / 2.8e-7 / 5.7e-8, 640 x 320 over 6144 2.8e-7 / 8.6e-7 / 2.5e-7, 64 x 576 over 8192 2.3e-7 / 4.1e-7 /
  // 2.0e-7.  One encoder layer's four layers alone 83 -> 90 us, steps and passes within 0.2 % of the time with one chain (with a fold every 256
  // rows whatever the layer 95 us, and the one-layer Transformer pass 1581 us where it is 1566).
  // (The bound of two waves per SIMD in the kernel's attributes keeps the accumulators in ordinary registers: moved in and out of the
  // others for each fold, the one-layer Transformer pass took 1707 us.)
  constexpr bool FOLD = NJ > 1;
  f32x16_t sum[FOLD ? TN : 1][FOLD ? TK : 1];
  if constexpr (FOLD) {
#pragma unroll
    for (int i = 0; i < TN; i++)
#pragma unroll
      for (int j = 0; j < TK; j++)
#pragma unroll
        for (int v = 0; v < 16; v++) sum[i][j][v] = 0.f;
  }
  int until_fold = FOLD ? a.fold : 0;
  const int steps = (mend - mbeg + WG_MS - 1) / WG_MS;
  uint32_t cur = 0, nxt = STAGE_BYTES;
#pragma unroll
  for (int t = 0; t < NS; t++) {
#pragma unroll
    for (int p = 0; p < NPIECE; p++) prep_piece(p);
#pragma unroll
    for (int v = 0; v < DV + XV; v++) issue((uint32_t)t * STAGE_BYTES, v);
  }
  wait_step<(NS - 1) * (DV + XV)>();
  read_frags(0, cur, 0);
  __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4));   // lgkmcnt(0): with the scalar loads, so that none is waited for inside
  for (int st = 0; st < steps; st++) {
#pragma unroll
    for (int kk = 0; kk < KK; kk++) {
      if (kk == KK - 1) wait_step<(NS - 2) * (DV + XV)>();
      read_frags((kk + 1) & 1, kk == KK - 1 ? nxt : cur, (kk + 1) % KK);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < TT; i++) {
        acc[i / TK][i % TK] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(df[kk & 1][i / TK], xf[kk & 1][i % TK], acc[i / TK][i % TK],
                                                                      0, 0, 0);
        if (kk < KK - 1) {
          constexpr int SLOTS = (KK - 1) * TT;
          const int slot = kk * TT + i;
#pragma unroll
          for (int p = 0; p < NPIECE; p++)
            if (p * SLOTS / NPIECE == slot) prep_piece(p);
        } else {
#pragma unroll
          for (int v = 0; v < DV + XV; v++)
            if (v * TT / (DV + XV) == i) issue(cur, v);
        }
        if (bias && (uwave >> 1) == (kk & 1)) {
#pragma unroll
          for (int h = 0; h < 2 * TN; h++)
            if (h * TT / (2 * TN) == i) add_bias(df[kk & 1][h >> 1], h & 1, bsum[h >> 1]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    cur = nxt;
    nxt = nxt + STAGE_BYTES == NS * STAGE_BYTES ? 0u : nxt + STAGE_BYTES;
    if constexpr (FOLD) {
      if (--until_fold == 0) {
        until_fold = a.fold;
#pragma unroll
        for (int i = 0; i < TN; i++)
#pragma unroll
          for (int j = 0; j < TK; j++)
#pragma unroll
            for (int v = 0; v < 16; v++) {
              const float b = acc[i][j][v], t = sum[i][j][v] + b;
              // (of an infinite sum the difference is NaN or infinite: a finite remainder leaves the sum as it is.  A real one is at most
              // half a last place, 2^103)
              acc[i][j][v] = __builtin_amdgcn_fmed3f(b - (t - sum[i][j][v]), -0x1p104f, 0x1p104f);
              sum[i][j][v] = t;
            }
      }
    }
  }
  if constexpr (FOLD) {
#pragma unroll
    for (int i = 0; i < TN; i++)
#pragma unroll
      for (int j = 0; j < TK; j++)
#pragma unroll
        for (int v = 0; v < 16; v++) acc[i][j][v] += sum[i][j][v];
  }

  float* out = a.out + ((int64_t)split * a.slices + sl) * a.N * a.K;   // N*K*4 bytes < 2^33: 32-bit element offsets inside
#pragma unroll
  for (int i = 0; i < TN; i++)
#pragma unroll
    for (int j = 0; j < TK; j++) {
      const int kk = k0 + wk0 + j * 32 + (lane & 31);
#pragma unroll
      for (int v = 0; v < 16; v++) {
        const int n = n0 + wn0 + i * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
        if (n < a.N && kk < a.K) out[(uint32_t)n * (uint32_t)a.K + (uint32_t)kk] = acc[i][j][v];
      }
    }
  wait_vmem<0>();   // the masked loads past the end still write (zeros) into the stages
  if (bias) {       // uniform over the workgroup
    __syncthreads();
    double* red = reinterpret_cast<double*>(smem);   // [wave >> 1][BN]
#pragma unroll
    for (int i = 0; i < TN; i++) {
      const double s = bsum[i] + __shfl_xor(bsum[i], 32, 64);
      if (lane < 32) red[(wave >> 1) * BN + wn0 + i * 32 + lane] = s;
    }
    __syncthreads();
    if (tid < BN && n0 + tid < a.N) {
      const double s = red[tid] + red[BN + tid];
      if (a.bias_part) a.bias_part[(int64_t)split * a.N + n0 + tid] = s;
      else a.bias_out[n0 + tid] = (float)s;
    }
  }
}

// The splits of a batch: 256 outputs (four a thread) x 4 split lanes per block, every lane adds every 4th split; of more than 64
// splits (few weights, that is few blocks, and 16 loads and more in a lane's chain) 64 outputs x 16 split lanes: 2304 weights in 512 splits
// 13.0 -> 4.1 us.  Behind a job's outputs a block per 16 channels adds the bias sums, every 16th split to a lane: a layer with a bias and
// few weights has hundreds of splits, and a thread a channel walked them alone (32 channels of 30784 pixels, 240 splits: the launch
// 55.8 -> 5.4 us; step of a two-layer network on 26 images of 37x32 264 -> 219).
struct WgradSum { const float* part; float* out; const double* bias_part; float* bias_out; uint32_t n4; int splits, N; uint32_t first, bias_first; };
constexpr int kBiasCols = 16;
__host__ __device__ inline unsigned wgrad_sum_lanes(int splits) { return splits > 64 ? 16u : 4u; }
template <int NJ> struct WgradSums { WgradSum j[NJ]; int n; };
static_assert(sizeof(WgradSums<kWgradJobs>) <= 4096, "the table travels in the kernel arguments");
template <int NJ>
__global__ void __launch_bounds__(256) wgrad_sum_kernel(WgradSums<NJ> b) {
  __shared__ float4 sm[256];
  int k = 0;
  if (NJ > 1)
    while (k + 1 < b.n && b.j[k + 1].first <= blockIdx.x) k++;
  const WgradSum& q = b.j[k];
  if (blockIdx.x >= q.bias_first) {
    double* bs = reinterpret_cast<double*>(sm);   // [16 lanes][16 channels]
    const int c = (int)(blockIdx.x - q.bias_first) * kBiasCols + (int)threadIdx.x % kBiasCols, lane = (int)threadIdx.x / kBiasCols;
    double s = 0.0;
    if (c < q.N) {
#pragma unroll 8
      for (int j = lane; j < q.splits; j += 256 / kBiasCols) s += q.bias_part[(int64_t)j * q.N + c];
    }
    bs[threadIdx.x] = s;
    __syncthreads();
    if (lane == 0 && c < q.N) {
      for (int l = 1; l < 256 / kBiasCols; l++) s += bs[l * kBiasCols + (int)threadIdx.x];
      q.bias_out[c] = (float)s;
    }
    return;
  }
  const unsigned lanes = wgrad_sum_lanes(q.splits), outs = 256u / lanes;
  const unsigned ol = threadIdx.x & (outs - 1u), lane = threadIdx.x / outs;
  const uint32_t i = (blockIdx.x - q.first) * outs + ol;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  if (i < q.n4) {
    const float4* p = reinterpret_cast<const float4*>(q.part) + i;
#pragma unroll 8
    for (int j = (int)lane; j < q.splits; j += (int)lanes) {
      const float4 v = p[(int64_t)j * q.n4];
      s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
  }
  sm[threadIdx.x] = s;
  __syncthreads();
  if (lane == 0 && i < q.n4) {
    float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
    for (unsigned l = 0; l < lanes; l += 4) {
      const float4 t0 = sm[l * outs + ol], t1 = sm[(l + 1) * outs + ol], t2 = sm[(l + 2) * outs + ol], t3 = sm[(l + 3) * outs + ol];
      t.x += (t0.x + t1.x) + (t2.x + t3.x); t.y += (t0.y + t1.y) + (t2.y + t3.y);
      t.z += (t0.z + t1.z) + (t2.z + t3.z); t.w += (t0.w + t1.w) + (t2.w + t3.w);
    }
    reinterpret_cast<float4*>(q.out)[i] = t;
  }
}

template <int BN, int BKK, bool PW>
static void launch_wgrad(const WgradJob* jobs, int n, unsigned blocks, hipStream_t s) {
  if (n == 1) {
    WgradBatch<1> b;
    b.j[0] = jobs[0]; b.n = 1;
    hipLaunchKernelGGL((wgrad_kernel<BN, BKK, PW, 1>), dim3(blocks), dim3(256), 0, s, b);
  } else {
    WgradBatch<kWgradJobs> b;
    for (int k = 0; k < n; k++) b.j[k] = jobs[k];
    b.n = n;
    hipLaunchKernelGGL((wgrad_kernel<BN, BKK, PW, kWgradJobs>), dim3(blocks), dim3(256), 0, s, b);
  }
}

WgradShape conv_wgrad_shape(const ConvGeom& g, int slices, bool bias) {
  WgradShape h;
  h.bias = bias;
  h.M = g.M(); h.N = g.Cout; h.K = g.K(); h.slices = slices;
  h.taps = g.kh * g.kw;
  h.pointwise = g.kh == 1 && g.kw == 1 && g.stride == 1 && g.pad == 0;
  return h;
}

// p[0 .. n): problems of one tile class (WgradShape::tile_class), at most kWgradJobs
static void wgrad_run(const WgradProblem* p, int n, int pitch, float* partials, size_t partials_bytes, hipStream_t s) {
  WgradJob jobs[kWgradJobs];
  WgradShape shapes[kWgradJobs];
  WgradSplit plan[kWgradJobs];
  for (int k = 0; k < n; k++) {
    shapes[k] = conv_wgrad_shape(p[k].g, p[k].slices, p[k].db != nullptr);
  }
  wgrad_plan(shapes, n, partials_bytes, g_tune_co, plan);
  WgradSums<kWgradJobs> sums;
  sums.n = 0;
  unsigned blocks = 0, sum_blocks = 0;
  char* room = reinterpret_cast<char*>(partials);
  for (int k = 0; k < n; k++) {
    const ConvGeom& g = p[k].g;
    const WgradShape& h = shapes[k];
    WgradJob& a = jobs[k];
    a.x = p[k].x; a.dy = p[k].dy;
    a.M = (int)h.M; a.N = h.N; a.K = h.K;
    a.H = g.H; a.W = g.W; a.Cin = g.Cin; a.Ho = g.Ho; a.Wo = g.Wo; a.kw = g.kw; a.stride = g.stride; a.pad = g.pad;
    a.div_wo = fast_div((uint32_t)g.Wo); a.div_ho = fast_div((uint32_t)g.Ho);
    a.div_cin = fast_div((uint32_t)g.Cin); a.div_kw = fast_div((uint32_t)g.kw);
    a.slices = h.slices;
    a.x_pitch = h.slices > 1 ? pitch : g.Cin;
    a.dy_pitch = h.slices > 1 ? pitch : g.Cout;
    a.x_bytes = (uint32_t)(g.B * g.H * g.W * (int64_t)a.x_pitch * 2);
    a.dy_bytes = (uint32_t)(h.M * (int64_t)a.dy_pitch * 2);
    a.ktiles = (int)cdiv(h.K, h.bk());
    a.tiles_per_slice = (int)(h.tiles() / h.slices);
    a.tiles = (int)h.tiles();
    a.m_per_split = (int)plan[k].m_per_split;
    a.fold = (int)(wgrad_own_rows(h, partials_bytes) / 32);
    a.first = blocks;
    a.out = p[k].dw;
    a.bias_part = nullptr;
    a.bias_out = p[k].db;
    const int splits = (int)plan[k].splits;
    blocks += (unsigned)(h.tiles() * splits);
    if (splits > 1) {
      a.out = reinterpret_cast<float*>(room);
      room += align_up((size_t)(h.weights() * splits) * sizeof(float), 256);
      WgradSum& q = sums.j[sums.n++];
      q.part = a.out; q.out = p[k].dw; q.n4 = (uint32_t)(h.weights() / 4); q.splits = splits; q.N = h.N;
      q.first = sum_blocks;
      sum_blocks += (unsigned)cdiv(q.n4, 256 / wgrad_sum_lanes(splits));
      q.bias_first = sum_blocks;
      q.bias_part = nullptr; q.bias_out = p[k].db;
      if (p[k].db) {
        a.bias_part = reinterpret_cast<double*>(room);
        room += align_up((size_t)h.N * splits * sizeof(double), 256);
        a.bias_out = nullptr;
        q.bias_part = a.bias_part;
        sum_blocks += (unsigned)cdiv(h.N, kBiasCols);
      } else {
        q.bias_first = 0xffffffffu;
      }
    }
  }
  switch (shapes[0].tile_class()) {
    case 0: launch_wgrad<64, 64, false>(jobs, n, blocks, s); break;
    case 1: launch_wgrad<64, 64, true>(jobs, n, blocks, s); break;
    case 2: launch_wgrad<64, 128, false>(jobs, n, blocks, s); break;
    case 3: launch_wgrad<64, 128, true>(jobs, n, blocks, s); break;
    case 4: launch_wgrad<128, 64, false>(jobs, n, blocks, s); break;
    case 5: launch_wgrad<128, 64, true>(jobs, n, blocks, s); break;
    case 6: launch_wgrad<128, 128, false>(jobs, n, blocks, s); break;
    default: launch_wgrad<128, 128, true>(jobs, n, blocks, s); break;
  }
  if (sums.n == 1) {
    WgradSums<1> one;
    one.j[0] = sums.j[0]; one.n = 1;
    hipLaunchKernelGGL(wgrad_sum_kernel<1>, dim3(sum_blocks), dim3(256), 0, s, one);
  } else if (sums.n > 1) {
    hipLaunchKernelGGL(wgrad_sum_kernel<kWgradJobs>, dim3(sum_blocks), dim3(256), 0, s, sums);
  }
}

void conv_wgrad_batch(const WgradProblem* p, int n, float* partials, size_t partials_bytes, hipStream_t s) {
  for (int k = 0; k < n; k += kWgradJobs) wgrad_run(p + k, std::min(n - k, kWgradJobs), 0, partials, partials_bytes, s);
}

void conv_wgrad_mfma(const bf16_t* x, const bf16_t* dy, float* dw, const ConvGeom& g, float* partials,
                     size_t partials_bytes, hipStream_t s) {
  const WgradProblem p = {x, dy, dw, nullptr, g, 1};
  wgrad_run(&p, 1, 0, partials, partials_bytes, s);
}

// dw [C][taps][cg] fp32 of a grouped convolution: dense per-slice gradients dwd [C / SW][SW][taps][SW] (scratch) by the
// sliced launch, then the diagonal blocks.
__global__ void __launch_bounds__(256) extract_sliced_dw_k(const float* __restrict__ dwd, float* __restrict__ dw, int C,
                                                           int taps, int cg, int SW) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (int64_t)C * taps * cg) return;
  const int j = (int)(idx % cg);
  const int t = (int)((idx / cg) % taps);
  const int o = (int)(idx / ((int64_t)cg * taps));
  dw[idx] = dwd[((int64_t)o * taps + t) * SW + (o % SW) / cg * cg + j];
}

void conv_grouped_wgrad_mfma(const bf16_t* x, const bf16_t* dy, float* dwd, float* dw, const ConvGeom& g, int groups,
                             float* partials, size_t partials_bytes, hipStream_t s) {
  const int C = g.Cin, cg = C / groups, SW = grouped_mfma_slice(C, groups), taps = g.kh * g.kw;
  ConvGeom gs = g;
  gs.Cin = gs.Cout = SW;
  const WgradProblem p = {x, dy, dwd, nullptr, gs, C / SW};   // C / SW independent problems on slices of the row-major tensors
  wgrad_run(&p, 1, C, partials, partials_bytes, s);
  const int64_t n = (int64_t)C * taps * cg;
  hipLaunchKernelGGL(extract_sliced_dw_k, dim3((unsigned)cdiv(n, 256)), dim3(256), 0, s, dwd, dw, C, taps, cg, SW);
}

// eight elements per thread (two 16-byte loads, one 16-byte store); the ragged tail element by element
__global__ void __launch_bounds__(256) cast_f32_bf16_k(const float* __restrict__ in, bf16_t* __restrict__ out, int64_t n) {
  const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 8;
  if (i + 8 <= n) {
    const float4 a = *reinterpret_cast<const float4*>(in + i), b = *reinterpret_cast<const float4*>(in + i + 4);
    *reinterpret_cast<uint4*>(out + i) =
        make_uint4(pack_bf16x2(a.x, a.y), pack_bf16x2(a.z, a.w), pack_bf16x2(b.x, b.y), pack_bf16x2(b.z, b.w));
  } else {
    for (int64_t j = i; j < n; j++) out[j] = f32_to_bf16(in[j]);
  }
}
void cast_f32_bf16(const float* in, bf16_t* out, int64_t n, hipStream_t s) {   // in, out 16-byte aligned
  hipLaunchKernelGGL(cast_f32_bf16_k, dim3((unsigned)cdiv(cdiv(n, 8), 256)), dim3(256), 0, s, in, out, n);
}

// ---- layout helpers ---------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) pad_c3_to_c8_k(const bf16_t* __restrict__ in, bf16_t* __restrict__ out,
                                                      int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const uint32_t a = in[3 * i], b = in[3 * i + 1], c = in[3 * i + 2];
  reinterpret_cast<uint4*>(out)[i] = make_uint4(a | (b << 16), c, 0u, 0u);
}
void pad_c3_to_c8(const bf16_t* in, bf16_t* out, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(pad_c3_to_c8_k, dim3((unsigned)cdiv(n, 256)), dim3(256), 0, s, in, out, n);
}
// ---- space-to-depth form of a stride-2 convolution on 3-channel images ------------------------------
// x[b][2I+p][2J+q][c] -> xs[b][I][J][(2p+q)*3 + c] (16 channels, the last four zero): a k x k stride-2
// filter with padding pad becomes a ks x ks stride-1 filter on xs with padding P = ceil(pad / 2),
// ks = ceil((k + 2P - pad) / 2), whose tap (R, S), channel (2p+q)*3 + c is the original tap
// r = 2R + p - (2P - pad), s = 2S + q - (2P - pad) (zero where that falls outside the filter).  The
// contraction shrinks from k*k*8 (channels padded to a 16-byte vector) to ks*ks*16.
__global__ void __launch_bounds__(256) s2d_pack_x_k(const bf16_t* __restrict__ x, bf16_t* __restrict__ xs, int64_t n,
                                                    int Hs, int Ws) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;  // (b, I, J)
  if (i >= n) return;
  const int J = (int)(i % Ws);
  const int64_t q = i / Ws;
  const int I = (int)(q % Hs);
  const int64_t b = q / Hs;
  const int W = 2 * Ws;
  const bf16_t* r0 = x + ((b * 2 * Hs + 2 * I) * W + 2 * J) * 3;  // six contiguous elements per image row
  const bf16_t* r1 = r0 + (int64_t)W * 3;
  uint32_t u[8];
  u[0] = r0[0] | ((uint32_t)r0[1] << 16); u[1] = r0[2] | ((uint32_t)r0[3] << 16); u[2] = r0[4] | ((uint32_t)r0[5] << 16);
  u[3] = r1[0] | ((uint32_t)r1[1] << 16); u[4] = r1[2] | ((uint32_t)r1[3] << 16); u[5] = r1[4] | ((uint32_t)r1[5] << 16);
  u[6] = 0; u[7] = 0;
  uint4* o = reinterpret_cast<uint4*>(xs + i * 16);
  o[0] = make_uint4(u[0], u[1], u[2], u[3]);
  o[1] = make_uint4(u[4], u[5], u[6], u[7]);
}
void s2d_pack_x(const bf16_t* x, bf16_t* xs, int64_t B, int H, int W, hipStream_t s) {
  const int64_t n = B * (H / 2) * (W / 2);
  hipLaunchKernelGGL(s2d_pack_x_k, dim3((unsigned)cdiv(n, 256)), dim3(256), 0, s, x, xs, n, H / 2, W / 2);
}
// w[n][k][k][3] -> ws[n][ks][ks][16]
__global__ void __launch_bounds__(256) s2d_pack_w_k(const bf16_t* __restrict__ w, bf16_t* __restrict__ ws, int cout,
                                                    int k, int ks, int shift) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= cout * ks * ks * 16) return;
  const int ch = i & 15, S = (i >> 4) % ks, R = (i >> 4) / ks % ks, n = (i >> 4) / (ks * ks);
  bf16_t v = 0;
  if (ch < 12) {
    const int pq = ch / 3, c = ch - pq * 3;
    const int r = 2 * R + (pq >> 1) - shift, t = 2 * S + (pq & 1) - shift;
    if (r >= 0 && r < k && t >= 0 && t < k) v = w[((n * k + r) * k + t) * 3 + c];
  }
  ws[i] = v;
}
void s2d_pack_w(const bf16_t* w, bf16_t* ws, int cout, int k, int ks, int shift, hipStream_t s) {
  hipLaunchKernelGGL(s2d_pack_w_k, dim3((unsigned)cdiv(cout * ks * ks * 16, 256)), dim3(256), 0, s, w, ws, cout, k, ks,
                     shift);
}
// fp32 dws[n][ks][ks][16] -> dw[n][k][k][3]
__global__ void __launch_bounds__(256) s2d_unpack_dw_k(const float* __restrict__ dws, float* __restrict__ dw, int cout,
                                                       int k, int ks, int shift) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= cout * k * k * 3) return;
  const int c = i % 3, t = i / 3 % k, r = i / 3 / k % k, n = i / 3 / (k * k);
  const int rr = r + shift, tt = t + shift;
  dw[i] = dws[((n * ks + (rr >> 1)) * ks + (tt >> 1)) * 16 + ((rr & 1) * 2 + (tt & 1)) * 3 + c];
}
void s2d_unpack_dw(const float* dws, float* dw, int cout, int k, int ks, int shift, hipStream_t s) {
  hipLaunchKernelGGL(s2d_unpack_dw_k, dim3((unsigned)cdiv(cout * k * k * 3, 256)), dim3(256), 0, s, dws, dw, cout, k, ks,
                     shift);
}

__global__ void __launch_bounds__(256) unpad_c8_to_c3_k(const float* __restrict__ in, float* __restrict__ out,
                                                        int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= 3 * n) return;
  out[i] = in[(i / 3) * 8 + i % 3];
}
void unpad_c8_to_c3(const float* in, float* out, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(unpad_c8_to_c3_k, dim3((unsigned)cdiv(3 * n, 256)), dim3(256), 0, s, in, out, n);
}
}  // namespace cd
