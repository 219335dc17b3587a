// fp32 contractions on the bf16 matrix cores: Eq. 4 (forward, mode 0) and the second half of Eq. 5 (gradient
// to the conv input, mode 1) of 'same' stride-1 3x3 and 1x1 layers.
//
// An fp32 value is the exact sum of three bf16 values (8 + 8 + 8 significant bits: x = h + m + l, each the
// rounded remainder of the ones before), so a product of two is nine bf16 products, each exact in fp32.  Six
// of them are taken - hh, hm, mh, mm, hl, lh; the dropped ones (ml, lm, ll) are 2^-28 of the product on average and
// below 2^-24, an fp32 rounding, at worst (above 2^-26 for 3 pairs of significands in 100).  A loop of
// v_mfma_f32_16x16x32_bf16 on random registers does 2050 TFLOP/s, one of v_mfma_f32_16x16x4_f32 154: six of the former take
// 0.45 of the time of the fp32 product; and the sum is rounded once per 32 terms and product instead of once per 4 terms.  The five small
// products have an accumulator of their own: added to the large one they would each round at its magnitude
// (relative error of a 2304-term contraction against 64 bits: fp32 matrix cores 8.6e-7, one accumulator
// 7.4e-7, two 2.9e-7).  The parts are taken of 2^23 x: those of the smallest fp32 values (multiples of 2^-149) are normal
// bf16 values then, and every other result is the same bit for bit.  What the split cannot carry - infinities, values
// from 2^105 on, sums from 2^82 on - gives an infinity or a NaN; an output that is not finite is computed again from the
// fp32 operands by exact_output().
//
// One block = a run of up to 112 consecutive pixels (of one image, or across images where that makes fewer
// tiles) x 16 NT WN output channels.  Its input patch (the rows of those pixels and the filter's border) is
// split once, on the way into LDS, CHUNKS 32-channel chunks at a time.  3x3: every eight channels of a part are a
// plane of 16 bytes per position, planes multiples of 256 bytes apart: the 16-byte reads of a fragment - 16
// positions, four planes - then touch every bank once, whichever lanes the LDS serves together (with a position's
// channels side by side they took twice the cycles; 64 -> 64 @56x56 95 -> 87 us).  1x1: a position's channels side
// by side, which loads whole lines of the input (1024 -> 256 @14x14 45 us, in planes 48).  Weights go from the L2 straight
// into registers, one k-step (32 contraction channels of one tap) ahead; every wave has output channels of its own, so
// a block reads nothing twice.  PRE: they come as the parts that SplitWeights describes, split once per call, in six whole
// kilobytes a k-step instead of 16 gathers and 88 vector instructions.  (Where no workspace is at hand the kernel splits them.)
// A wave computes 112 pixels x 16 NT channels: 7 NT tiles, 21 reads and 42 NT MFMAs per k-step.
// What the k-loop needs to stay at the matrix cores' rate (us before / with all of it, in a stack, both traced on one card: 3x3
// 256 -> 256 @14x14 75.7 / 71.9, gradient with sums 80.1 / 75.9; 1x1 1024 -> 256 48.3 / 44.5, its mirror's gradient 49.7 / 46.2;
// 1x1 256 -> 1024 58.0 / 56.4, gradient 58.6 / 56.9; 3x3 64 -> 64 @56x56 106 / 89, gradient 114 / 97; layer call with bf16 operands
// and 8-bit codes 53 / 43 and 76 / 56 (with its weights further ahead 33 and 45, see AHEAD).  In the first four the card's power is the bound: the weight gradients between them, the same
// kernels on both sides, took 58 and 62):
//  - two sets of weight registers in turn.  With one, its copy at every step waits for everything in flight, the next phase's
//    input too.  (An odd number of steps leaves one copy, at the end of a phase, where the input is awaited anyway.)
//  - loads without branches around them, and the next phase's input after the weights of a step, not before.
//  - the wave that is behind first: left to itself a SIMD runs its older wave to the barrier, and the other alone gets
//    80 % of the matrix rate (a phase of nine steps 31.6 thousand cycles, with falling priorities 30.0, both at full rate 24.2).
//  - nothing of the epilogue held in registers through the contraction: it spilled 58 registers of the 1x1 gradient.
//  - few copies of the step's code: with all four variants of a phase written out (56 KB) the 3x3 layer went from 74 to 92 us;
//    the instruction cache is cold when a kernel starts.
// (Splits between the k-steps instead of in front of them gained nothing: vector and matrix instructions of a SIMD's two
// waves overlap little.)
// KS = 2: the chunks of a phase go to two groups of waves whose sums meet in LDS at the end - two waves per
// SIMD also where a layer gives only one block per compute unit - and the patch has two buffers.
// KS = 1: one buffer, two blocks per compute unit cover each other's staging (with fp32 operands one where a 3x3 patch has more
// than 256 positions).
// With bf16 operands (ABL_MATH_BF16) the same kernel runs with one part per operand: rounded once, one product.

#include <type_traits>

#include "abl_internal.h"

namespace abl {
namespace {

constexpr int MT = 7;   // 16-pixel tiles per wave and block
constexpr int WN = 4;   // waves along the output channels

struct Tiling {
  int run;           // pixels per tile
  int unit, ntr;     // a tile never crosses a multiple of `unit` pixels (an image, or the whole batch): ntr tiles each
  int tiles, per;    // tiles in all, tiles per block (consecutive)
  int gm;            // blocks along the pixels
  int npos;          // positions of a patch
  Divisor w, pw, h, ph, hw, per_unit;   // by W, W + 2, H, H + 2, H W, ntr
};

// One output from the operands themselves (products and sums in 64 bits), for values that are not finite.
template <int MODE, int TAPS, int FUSE>
__device__ inline float exact_output(const float* in, const float* wgt, const float* stats, int H, int W, int Cin, int Cout,
                                     int p, int n) {
  const int Cg = MODE == 0 ? Cin : Cout;
  const int HW = H * W;
  const int img = p / HW, h = (p - img * HW) / W, w = p - img * HW - h * W;
  double s = 0.0;
  for (int tap = 0; tap < TAPS; ++tap) {
    const int hi = h + (TAPS == 9 ? tap / 3 - 1 : 0), wi = w + (TAPS == 9 ? tap % 3 - 1 : 0);
    const bool in_image = hi >= 0 && hi < H && wi >= 0 && wi < W;   // (the border's zeros take part)
    const float* a = in + (in_image ? ((size_t)(img * H + hi) * W + wi) * Cg : 0);
    const float* b = MODE == 0 ? wgt + (size_t)tap * Cin * Cout + n : wgt + ((size_t)(TAPS - 1 - tap) * Cin + n) * Cout;
    for (int c = 0; c < Cg; ++c) {
      float x = in_image ? a[c] : 0.0f;
      if (FUSE != 0 && in_image) {   // Eq. 1-3
        const float a1 = (x - stats[P_MEAN * Cin + c]) * stats[P_RSTD * Cin + c];
        const float a2 = stats[P_GAMMA * Cin + c] * a1 + stats[P_BETA * Cin + c];
        x = a2 > 0.0f ? a2 : 0.0f;
      }
      s += (double)x * (double)(MODE == 0 ? b[(size_t)c * Cout] : b[c]);
      if (s != s) return (float)s;
    }
  }
  return (float)s;
}

// EPI: 0 none; 1 = sums of y and y^2 per channel (first pass of the next layer's Eq. 1); 4 / 8 = the Eq. 6-7
// sums from the layer's K-bit codes.  Row blockIdx of sums: [gm][2][Ng] doubles.
// Bytes of LDS of a block besides its sums: the patch (KS of them), later the exchange of the groups' sums and the codes.
__host__ __device__ constexpr int patch_bytes(int taps, int ks, int cpp, int su, int np) {
  const int c8 = 4 * ks * cpp, npos = su * 64 * WN * ks / c8;
  return taps == 9 ? 16 * np * c8 * npos : npos * (16 * np * c8 + 16);
}
__host__ __device__ constexpr int exchange_bytes(int nt, int ks) { return ks == 2 ? 4 * nt * 1024 * WN * ks : 0; }
__host__ __device__ constexpr int area_bytes(int taps, int nt, int ks, int cpp, int su, int np) {
  const int a = ks * patch_bytes(taps, ks, cpp, su, np);
  const int b = exchange_bytes(nt, ks) + 16 * MT * (16 * nt * WN + 16);   // (8-bit codes: a byte per channel)
  return a > b ? a : b;
}

// NP = 3: operands in three parts, as above; NP = 1: rounded to bf16.
// FUSE = K (4 or 8, 3x3 forward): `in` is the layer input x; Eq. 1-3 are applied on the way into LDS and the K-bit codes of
// the block's own pixels written to `packed` (the blocks along the output channels take turns over the phases).
// ONE: the contraction is a single phase (1x1 gradients with 64 channels to contract).  Code for both kinds of phase asks for
// the next phase's input and for the epilogue's codes, and holds registers for both: with 128 channels per block and 8-bit
// codes 14 of them were spilled (1x1 256 <- 64, backward, us, ONE / without: @55x55 N=14, K=8 62.5 / 66.3, N=40, K=8 140 / 151,
// K=4 131 / 135; @56x56 N=64, K=8 231 / 247; with a branch between the two inside one kernel N=40, K=4 161).
template <int MODE, int TAPS, int NT, int KS, int CPP, int SU, int EPI, int NP, bool PRE, int FUSE = 0, bool ONE = false>
__global__ __launch_bounds__(64 * WN * KS, 2) void split_conv_kernel(const float* __restrict__ in,
                                                                          const float* __restrict__ wgt,
                                                                          const uint4* __restrict__ parts,
                                                                          const float* skip, float* out,
                                                                          double* __restrict__ sums,
                                                                          const uint8_t* __restrict__ codes,
                                                                          const float* __restrict__ stats, ConvGeom g,
                                                                          Tiling tl, uint8_t* packed, int pack_pad) {
  constexpr int THREADS = 64 * WN * KS;
  constexpr int CHUNKS = KS * CPP, CH = 32 * CHUNKS;   // per phase
  constexpr int BN = 16 * NT * WN;
  constexpr bool DB = KS > 1;
  constexpr int C8 = CH / 8;                           // staging items per position
  constexpr int STEPS = TAPS * CPP;                    // k-steps of a phase and wave
  // pixel fragments of a k-step (7 tiles, NP parts), and registers for as many as are read ahead.  (A wave that has to wait
  // for each tile's reads leaves its SIMD idle as soon as the other wave waits at a barrier.)
  // (1x1, bf16 operands and weights split here: six reads ahead of a step's fourteen products only put off its weights, which
  // are few.  us, one ahead / six: gradient with sums 512 <- 128 @28x28 N=40, K=8 79.3 / 81.9, N=64, K=4 101.6 / 106.4, 256 <- 64
  // @56x56 N=14, K=8 55.9 / 58.2, forward 64 -> 256 @55x55 N=12 29.1 / 30.5; not so a long forward contraction, which takes 64
  // channels per block, 2048 -> 512 @7x7 N=80 68.4 / 64.4.)
  constexpr bool SHORT = TAPS == 1 && NP == 1 && !PRE;
  constexpr int NF = MT * NP, SLOTS = 7, LOOK = SHORT && (MODE == 1 || NT == 2) ? 1 : SLOTS - 1;
  // the next phase's input asked for in front of a phase's only step (us, in front / behind its weights: gradient 512 <- 2048
  // @7x7 N=26 53.9 / 61.9, 256 <- 1024 @14x14 N=14 38.4 / 42.1, forward 2048 -> 512 @8x8 N=26 43.4 / 48.9)
  constexpr bool INPUT_FIRST = SHORT && KS == 2;
  // 3x3 layers with bf16 operands: weights are asked for AHEAD steps before their use, into the registers of the step that has
  // read them.  A step is 7 or 14 products, 112 or 224 cycles, and with weights one step ahead it waited for the L2; loads come
  // back in order, so weights that are asked for behind the next phase's input wait for that as well, and with all nine taps'
  // in flight the input has the whole phase.  With 128 channels per block three sets fit.  (us, forward / gradient, one step
  // ahead, three, nine: 64 -> 64 @56x56 N=64, 8-bit codes, 43.1 / 56.4, 35.5 / 49.1, 33.4 / 44.5; 256 -> 256 @14x14 N=64 27.4 /
  // 28.6, 24.3 / 25.3.  fp32 operands, 42 products a step: 64 -> 64 84.5 / 92.3, three ahead 84.1 / 91.3, and five times the code.)
  constexpr int AHEAD = PRE && NP == 1 && STEPS == 9 ? (NT == 1 ? 9 : 3) : 0;
  // the lane's offset into the parts, opaque as that of the weights below: 60 registers less with three sets of 128 channels (11
  // spilled without).  Elsewhere the free order of the loads is worth more (us: nine sets 33.4 / 44.5, opaque 36.8 / 50.6; fp32 256
  // -> 256 @14x14 70.2 / 76.3, opaque 73.2 / 79.1; bf16 1x1 1024 -> 256 22.0 / 23.0, opaque 22.6 / 24.0, four waves 33.3 / 32.1)
  constexpr bool OPAQUE = NP == 1 && NT == 2 && (TAPS == 9 || KS == 1);
  // Remainders by dot products (split3): 1x1 layers (1024 -> 256 @14x14 in a layer call 217 -> 211 us, plain forwards 0.99 of the time,
  // 0.95 to 1.04) and 3x3 kernels with the weights in parts and no prologue.  Other 3x3 kernels depend on the grid: 0.92 to 1.05 of the
  // time in stage calls, and with the prologue 512 -> 128 @31x31 N=35 in a layer call 257 us without, 282 with.
  constexpr bool DOT = TAPS != 9 || (PRE && FUSE == 0);
  static_assert(NF % SLOTS == 0, "a k-step starts in the slot of the one before");
  // the patch: bytes from a position, eight channels, a part and a chunk to the next
  constexpr int NPOS = SU * THREADS / C8;
  constexpr int POS_B = TAPS == 9 ? 16 : 64 * NP * CHUNKS + 16, C8_B = TAPS == 9 ? 16 * NPOS : 16;
  constexpr int PART_B = 4 * C8_B, CHUNK_B = 4 * NP * C8_B;
  constexpr int bufsz = patch_bytes(TAPS, KS, CPP, SU, NP);
  static_assert(TAPS == 1 || C8_B % 256 == 0, "planes on the same banks");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  double* const sum_lds = reinterpret_cast<double*>(smem + area_bytes(TAPS, NT, KS, CPP, SU, NP));   // [KS][2][BN]

  const int Cg = MODE == 0 ? g.Cin : g.Cout;
  const int Ng = MODE == 0 ? g.Cout : g.Cin;
  const int H = g.H, W = g.W, PW = W + 2;
  const int Mg = g.N * H * W;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wn = wave % WN, kg = wave / WN;
  const int li = lane & 15, lk = lane >> 4;
  // ids 8 apart share an XCD and its L2: the blocks that read the same pixels for different output channels
  // run there back to back
  const int nblk = Ng / BN;
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int mb = (slot / nblk) * 8 + xcd;
  const int nb = (slot % nblk) * BN, n0 = nb + 16 * NT * wn;
  if (mb >= tl.gm) return;
  const int t_end = min((mb + 1) * tl.per, tl.tiles);
  const int nph = Cg / CH;

  // weights of a k-step: forward: the lane's column in eight rows; gradient: 32 contiguous bytes
  uint32_t w_lane = 4u * (MODE == 0 ? (uint32_t)(8 * lk * g.Cout + li) : (uint32_t)(li * g.Cout + 8 * lk));
  auto load_w = [&](auto& raw, int tap, int c0) __attribute__((always_inline)) {
    // (opaque: the lane's 32-bit offset stays a register beside the scalar base instead of a 64-bit address)
    asm volatile("" : "+v"(w_lane));
    if constexpr (MODE == 0) {
      const char* wb = reinterpret_cast<const char*>(wgt + ((size_t)(tap * g.Cin + c0) * g.Cout + n0));
#pragma unroll
      for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int j = 0; j < NT; ++j)
          raw[j][e] = *reinterpret_cast<const uint32_t*>(wb + (size_t)(4 * e) * g.Cout + 64 * j + w_lane);
    } else {
      const char* wb = reinterpret_cast<const char*>(wgt + ((size_t)((TAPS - 1 - tap) * g.Cin + n0) * g.Cout + c0));
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const floatx4 v = *reinterpret_cast<const floatx4*>(wb + (size_t)(64 * j) * g.Cout + 16 * q + w_lane);
#pragma unroll
          for (int e = 0; e < 4; ++e) raw[j][4 * q + e] = __float_as_uint(v[e]);
        }
    }
  };

  // PRE: the parts of a k-step in fragment order, a kilobyte per output-channel tile and part
  uint32_t p_lane = 16u * lane;
  auto load_parts = [&](auto& raw, int tap, int c0) __attribute__((always_inline)) {
    if constexpr (OPAQUE) asm volatile("" : "+v"(p_lane));   // (as above)
    const char* wb = reinterpret_cast<const char*>(parts + ((size_t)(tap * (Cg / 32) + c0 / 32) * (Ng / 16) + n0 / 16) * (64 * NP));
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        const uint4 v = *reinterpret_cast<const uint4*>(wb + (j * NP + q) * 1024 + p_lane);
        raw[j][4 * q] = v.x, raw[j][4 * q + 1] = v.y, raw[j][4 * q + 2] = v.z, raw[j][4 * q + 3] = v.w;
      }
  };

  if (FUSE != 0 && blockIdx.x == 0 && tid < pack_pad)   // the tail of the store's last 128-byte row
    packed[((int64_t)Mg * Cg * FUSE) / 8 + tid] = 0;
  if (EPI != 0)
    for (int i = tid; i < KS * 2 * BN; i += THREADS) sum_lds[i] = 0.0;

  // ---- staging: per thread SU items of eight channels of a position; the first phase of the next tile is requested
  // before the epilogue of this one
  int s_off[SU];   // element offset of the item's channels (phase 0), -1 = zeros
  uint32_t own = 0;   // (FUSE) items whose position is a pixel of the tile
  float sv[SU][8];
  auto load_item = [&](int ph, int u, int keep) __attribute__((always_inline)) {
    const float* src = in + ph * CH + ((s_off[u] < 0 ? 0 : s_off[u]) & keep);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const floatx4 v = *reinterpret_cast<const floatx4*>(src + 4 * q);
#pragma unroll
      for (int e = 0; e < 4; ++e) sv[u][4 * q + e] = v[e];
    }
  };
  auto stage_load = [&](int ph, bool exists) __attribute__((always_inline)) {
    // (past the last phase every lane reads the first channels again: no branch, behind which the compiler would wait for all
    // that is in flight)
    const bool none = !exists && ph >= nph;
#pragma unroll
    for (int u = 0; u < SU; ++u) load_item(none ? 0 : ph, u, none ? 0 : -1);
  };
  auto store_item = [&](unsigned char* buf, int u) __attribute__((always_inline)) {
    bf16x8_t h, m, l;   // (NP = 1: the first only)
    if (TAPS == 9 || s_off[u] < 0)
#pragma unroll
      for (int e = 0; e < 8; ++e) sv[u][e] = s_off[u] < 0 ? 0.0f : sv[u][e];
    if constexpr (NP == 3) split3<DOT>(sv[u], h, m, l);
    else h = to_bf16x8(sv[u]);
    const int it = tid + THREADS * u;
    const int pos = TAPS == 9 ? (it & 15) + 16 * (it / (16 * C8)) : it / C8;
    const int c8 = TAPS == 9 ? (it >> 4) % C8 : it % C8;
    unsigned char* to = buf + (c8 >> 2) * CHUNK_B + (c8 & 3) * C8_B + pos * POS_B;
    *reinterpret_cast<bf16x8_t*>(to) = h;
    if constexpr (NP == 3) {
      *reinterpret_cast<bf16x8_t*>(to + PART_B) = m;
      *reinterpret_cast<bf16x8_t*>(to + 2 * PART_B) = l;
    }
  };
  // a tile: pixels p0 .. p_end - 1; its patch starts a row above the first of them, in rows of images padded to H + 2
  auto first_pixel = [&](int t) __attribute__((always_inline)) {
    const int q = tl.per_unit.of(t);
    return q * tl.unit + (t - q * tl.ntr) * tl.run;
  };
  auto last_pixel = [&](int t) __attribute__((always_inline)) {
    return min(min(first_pixel(t) + tl.run, (tl.per_unit.of(t) + 1) * tl.unit), Mg);
  };
  auto first_row = [&](int p0) __attribute__((always_inline)) { return tl.w.of(p0) + 2 * tl.hw.of(p0); };
  auto begin_tile = [&](int t) __attribute__((always_inline)) {
    const int p0 = first_pixel(t), p_end = last_pixel(t), row0 = first_row(p0);
    own = 0;
#pragma unroll
    for (int u = 0; u < SU; ++u) {
      const int it = tid + THREADS * u;
      const int pos = TAPS == 9 ? (it & 15) + 16 * (it / (16 * C8)) : it / C8;
      const int c8 = TAPS == 9 ? (it >> 4) % C8 : it % C8;
      if (TAPS == 9) {
        const int prow = tl.pw.of(pos), w = pos - prow * PW - 1;
        const int n = tl.ph.of(row0 + prow), h = row0 + prow - n * (H + 2) - 1;
        s_off[u] = pos < tl.npos && n < g.N && h >= 0 && h < H && w >= 0 && w < W ? ((n * H + h) * W + w) * Cg + 8 * c8 : -1;
        if constexpr (FUSE != 0) {
          const int p = (n * H + h) * W + w;
          own |= s_off[u] >= 0 && p >= p0 && p < p_end ? 1u << u : 0u;
        }
      } else {
        s_off[u] = p0 + pos < p_end ? (p0 + pos) * Cg + 8 * c8 : -1;
      }
    }
    stage_load(0, true);
  };
  begin_tile(mb * tl.per);
  for (int t = mb * tl.per; t < t_end; ++t) {
    const int p0 = first_pixel(t), p_end = last_pixel(t), row0 = first_row(p0);
    auto stage_store = [&](unsigned char* buf, int ph) __attribute__((always_inline)) {
      if constexpr (FUSE != 0) {
        // (a thread's items are the same eight channels of different positions)
        static_assert(THREADS % (16 * C8) == 0, "one channel group per thread");
        const int c = ph * CH + 8 * ((tid >> 4) % C8);
        const bool packs = ph % nblk == slot % nblk;   // block-uniform
        float mean[8], rstd[8], gm[8], bt[8], cq[8];
        int32_t fb[8];
#pragma unroll
        for (int q = 0; q < 8; q += 4) {
          const floatx4 m4 = *reinterpret_cast<const floatx4*>(stats + P_MEAN * Cg + c + q);
          const floatx4 r4 = *reinterpret_cast<const floatx4*>(stats + P_RSTD * Cg + c + q);
          const floatx4 g4 = *reinterpret_cast<const floatx4*>(stats + P_GAMMA * Cg + c + q);
          const floatx4 b4 = *reinterpret_cast<const floatx4*>(stats + P_BETA * Cg + c + q);
          const floatx4 c4 = *reinterpret_cast<const floatx4*>(stats + P_CQ * Cg + c + q);
          const int4 f4 = *reinterpret_cast<const int4*>(stats + P_FB * Cg + c + q);
          const int32_t f[4] = {f4.x, f4.y, f4.z, f4.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            mean[q + e] = m4[e]; rstd[q + e] = r4[e]; gm[q + e] = g4[e]; bt[q + e] = b4[e]; cq[q + e] = c4[e]; fb[q + e] = f[e];
          }
        }
#pragma unroll
        for (int u = 0; u < SU; ++u) {
          float a2[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float d = sv[u][e] - mean[e];
            const float a1 = d * rstd[e];                    // Eq. 1
            const float t2 = gm[e] * a1;
            a2[e] = t2 + bt[e];                              // Eq. 2
            sv[u][e] = a2[e] > 0.0f ? a2[e] : 0.0f;          // Eq. 3 (the border is zeroed below)
          }
          if (packs && ((own >> u) & 1u)) {
            uint32_t word[2] = {0, 0};
#pragma unroll
            for (int e = 0; e < 8; ++e)
              word[e * FUSE / 32] |= quant_code<FUSE>(a2[e], cq[e], fb[e]) << ((e * FUSE) % 32);   // Eq. 9
            uint8_t* to = packed + (size_t)(s_off[u] + ph * CH) * FUSE / 8;
            if (FUSE == 4) *reinterpret_cast<uint32_t*>(to) = word[0];
            else *reinterpret_cast<uint2*>(to) = make_uint2(word[0], word[1]);
          }
        }
      }
#pragma unroll
      for (int u = 0; u < SU; ++u) store_item(buf, u);
    };
    int a_base[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      int m = 16 * i + li;
      if (TAPS == 9) {
        const int p = p0 + m < p_end ? p0 + m : p_end - 1;   // slots past the tile: any position of it, never stored
        const int row = tl.w.of(p);
        m = (row + 2 * tl.h.of(row) - row0) * PW + p - row * W;
      }
      a_base[i] = m * POS_B + kg * CPP * CHUNK_B + lk * C8_B;
    }

    floatx4 hi[NT][MT], lo[NT][MT];
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int i = 0; i < MT; ++i) hi[j][i] = lo[j][i] = floatx4{0.f, 0.f, 0.f, 0.f};

    constexpr int I0 = 4;   // KS = 2: group 0 finishes the first four pixel tiles, group 1 the others
    // Eq. 6-7: the tile's codes go through LDS in whole 16-byte pieces (loaded where they are used, two bytes per
    // lane and channel tile, they took half as long as the contraction: 1x1 256 -> 64 @56x56 122 us, without them 88)
    constexpr int CPR = EPI > 1 ? BN * EPI / 128 : 1;                        // pieces per pixel
    constexpr int CU = (16 * MT * CPR + THREADS - 1) / THREADS;              // ... per thread
    constexpr int CPITCH = 16 * CPR + 16;
    uint4 cq[CU];
    // Weights of two k-steps in turn: the set that a step reads and the one that it asks for.  (One set and a copy of it waits for
    // everything in flight at the copy.)  Where the kernel splits them one set does: a step splits it before it asks for the next.
    constexpr int RW = PRE ? 4 * NP : 8;
    constexpr int ODD = PRE ? 1 : 0;   // set of the steps with odd numbers
    uint32_t wset[AHEAD > 0 ? AHEAD : 1 + ODD][NT][RW];
    auto load_set = [&](uint32_t (&w)[NT][RW], int tap, int c0) __attribute__((always_inline)) {
      if constexpr (PRE) load_parts(w, tap, c0);
      else load_w(w, tap, c0);
    };
#pragma unroll
    for (int d = 0; d < (AHEAD > 0 ? AHEAD : 1); ++d) load_set(wset[d], d, kg * CPP * 32);
    // the epilogue's codes, behind the last k-steps
    auto load_codes = [&]() __attribute__((always_inline)) {
      if constexpr (EPI > 1) {
        const uint8_t* cs = codes + ((size_t)p0 * Ng + nb) * EPI / 8;
#pragma unroll
        for (int u = 0; u < CU; ++u) {
          const int it = min(tid + THREADS * u, (p_end - p0) * CPR - 1);
          cq[u] = *reinterpret_cast<const uint4*>(cs + (uint32_t)(it / CPR * (Ng * EPI / 8) + it % CPR * 16));
        }
      }
    };
    auto step_off = [&](int ks) __attribute__((always_inline)) {
      const int cc = ks / TAPS, tap = ks - cc * TAPS;
      return (TAPS == 9 ? (tap / 3) * PW + tap % 3 : 0) * POS_B + cc * CHUNK_B;
    };
    bf16x8_t a[SLOTS];
    auto read_a = [&](const unsigned char* at, int f) __attribute__((always_inline)) {
      a[f % SLOTS] = *reinterpret_cast<const bf16x8_t*>(at + a_base[f / NP] + (f % NP) * PART_B);
    };
    // k-step ks of phase ph, whose patch is at cur; last: 1 = the phase is the tile's last, 0 = it is not, 2 = either
    auto k_step = [&](uint32_t (&use)[NT][RW], uint32_t (&fill)[NT][RW], int ph, int ks, const unsigned char* cur, bool first,
                      int last) __attribute__((always_inline)) {
      bf16x8_t bh[NT], bm[NT], bl[NT];
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        if constexpr (PRE) {
          bh[j] = __builtin_bit_cast(bf16x8_t, make_uint4(use[j][0], use[j][1], use[j][2], use[j][3]));
          if constexpr (NP == 3) {
            bm[j] = __builtin_bit_cast(bf16x8_t, make_uint4(use[j][4], use[j][5], use[j][6], use[j][7]));
            bl[j] = __builtin_bit_cast(bf16x8_t, make_uint4(use[j][8], use[j][9], use[j][10], use[j][11]));
          }
        } else {
          float x[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) x[e] = __uint_as_float(use[j][e]);
          if constexpr (NP == 3) split3<DOT>(x, bh[j], bm[j], bl[j]);
          else bh[j] = to_bf16x8(x);
        }
      }
      // the next k-step's weights (the very last step asks for its own again: no branch)
      const bool wrap = ks + 1 == STEPS, end = wrap && ph + 1 == nph;
      if constexpr (AHEAD == 0) {
        const int nks = end ? ks : wrap ? 0 : ks + 1;
        const int ncc = nks / TAPS, ntap = nks - ncc * TAPS;
        load_set(fill, ntap, (wrap && !end ? ph + 1 : ph) * CH + (kg * CPP + ncc) * 32);
      }
      // after them the input of the next phase (two steps' weights come back before it has to)
      if (first && !INPUT_FIRST) {
        if (last != 1) stage_load(ph + 1, last == 0);
        if (last == 1 || (last == 2 && ph + 1 == nph)) load_codes();
      }
      const unsigned char *const ab = cur + step_off(ks), *const nab = cur + step_off(wrap ? ks : ks + 1);
      // fragment by fragment, LOOK reads in flight
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        const int i = f / NP, q = f % NP;
        if (f + LOOK < NF) read_a(ab, f + LOOK);
        else if (STEPS > 1) read_a(nab, f + LOOK - NF);   // (past a phase's last step: read, not used)
        __builtin_amdgcn_sched_barrier(0);
        const bf16x8_t& x = a[f % SLOTS];
        if constexpr (NP == 3) {
          if (q == 0)
#pragma unroll
            for (int j = 0; j < NT; ++j) lo[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bl[j], x, lo[j][i], 0, 0, 0);
        }
        if (q == 0)
#pragma unroll
          for (int j = 0; j < NT; ++j) hi[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bh[j], x, hi[j][i], 0, 0, 0);
        if constexpr (NP == 3) {
          if (q < 2)
#pragma unroll
            for (int j = 0; j < NT; ++j) lo[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bm[j], x, lo[j][i], 0, 0, 0);
          if (q > 0)
#pragma unroll
            for (int j = 0; j < NT; ++j) lo[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bh[j], x, lo[j][i], 0, 0, 0);
        }
      }
      if constexpr (AHEAD > 0) {   // into the registers that the step has read
        if (ks + AHEAD < STEPS) load_set(fill, ks + AHEAD, ph * CH + kg * 32);
        else if (last != 1) load_set(fill, ks + AHEAD - STEPS, (last == 2 && ph + 1 == nph ? ph : ph + 1) * CH + kg * 32);
      }
    };
    auto phase = [&](int ph, auto last_c) __attribute__((always_inline)) {
      constexpr int last = decltype(last_c)::value;
      unsigned char* const cur = smem + (DB ? (ph & 1) * bufsz : 0);
      // (two buffers: this one was last read a phase ago, before the barrier that followed)
      if (!DB || ph == 0) __syncthreads();
      stage_store(cur, ph);
      __syncthreads();
      if constexpr (INPUT_FIRST) {
        if constexpr (last == 1) load_codes();
        else stage_load(ph + 1, last == 0);
      }
#pragma unroll
      for (int f = 0; f < LOOK; ++f) read_a(cur + step_off(0), f);
      // each set in its own registers; an odd number of steps leaves the next weights in the wrong one.  (Few copies of the
      // step's code: a kernel starts with a cold instruction cache.)
      if constexpr (STEPS >= 9) __builtin_amdgcn_s_setprio(3);
      if constexpr (AHEAD > 0) {
#pragma unroll
        for (int ks = 0; ks < STEPS; ++ks) {
          if (ks == 3) __builtin_amdgcn_s_setprio(2);
          else if (ks == 5) __builtin_amdgcn_s_setprio(1);
          else if (ks == 7) __builtin_amdgcn_s_setprio(0);
          k_step(wset[ks % AHEAD], wset[ks % AHEAD], ph, ks, cur, ks == 0, last);
        }
        return;
      }
      k_step(wset[0], wset[ODD], ph, 0, cur, true, last);
      if constexpr (STEPS == 2) k_step(wset[ODD], wset[0], ph, 1, cur, false, last);
      if constexpr (STEPS >= 9) {
#pragma unroll 1
        for (int ks = 1; ks < STEPS; ks += 2) {
          // two waves of a SIMD that are to meet at the end of the phase: the one that is behind goes first
          if (ks == 3) __builtin_amdgcn_s_setprio(2);
          else if (ks == 5) __builtin_amdgcn_s_setprio(1);
          else if (ks == 7) __builtin_amdgcn_s_setprio(0);
          k_step(wset[ODD], wset[0], ph, ks, cur, false, last);
          k_step(wset[0], wset[ODD], ph, ks + 1, cur, false, last);
        }
      }
      if constexpr (PRE && STEPS % 2 == 1) {
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
          for (int e = 0; e < RW; ++e) wset[0][j][e] = wset[1][j][e];
      }
    };
    if constexpr (ONE) {
      phase(0, std::integral_constant<int, 1>{});
    } else if constexpr (NP == 1) {   // (short code: a tile's last phase apart)
      for (int ph = 0; ph + 1 < nph; ++ph) phase(ph, std::integral_constant<int, 0>{});
      phase(nph - 1, std::integral_constant<int, 1>{});
    } else {
      for (int ph = 0; ph < nph; ++ph) phase(ph, std::integral_constant<int, 2>{});
    }

    if (t + 1 < t_end) begin_tile(t + 1);
    // ---- the lane holds channels n0 + 16 j + 4 lk .. +3 of pixel slot 16 i + li
    // (opaque: addresses and constants of the epilogue, formed ahead of the contraction, had no registers to wait in)
    int tid_e = tid;
    asm volatile("" : "+v"(tid_e));
    const int lane_e = tid_e & 63, li_e = lane_e & 15, lk_e = lane_e >> 4;
    floatx4 v[NT][MT];
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int i = 0; i < MT; ++i) v[j][i] = NP == 3 ? kDown * (hi[j][i] + lo[j][i]) : hi[j][i];
    unsigned char* const cbuf = smem + exchange_bytes(NT, KS);
    if (KS == 2 || EPI > 1) __syncthreads();      // every wave has finished reading the patch
    if constexpr (EPI > 1) {
#pragma unroll
      for (int u = 0; u < CU; ++u) {
        const int it = tid_e + THREADS * u;
        if (it < 16 * MT * CPR) *reinterpret_cast<uint4*>(cbuf + it / CPR * CPITCH + it % CPR * 16) = cq[u];
      }
      if (KS == 1) __syncthreads();
    }
    if constexpr (KS == 2) {
      unsigned char* dst = smem + (size_t)((wave ^ WN) * I0 * NT) * 1024 + lane_e * 16;
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int i = 0; i < MT; ++i)
          if ((i < I0) == (kg == 1)) *reinterpret_cast<floatx4*>(dst + (j * I0 + (i < I0 ? i : i - I0)) * 1024) = v[j][i];
      __syncthreads();
      const unsigned char* srcp = smem + (size_t)(wave * I0 * NT) * 1024 + lane_e * 16;
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int i = 0; i < MT; ++i)
          if ((i < I0) == (kg == 0)) v[j][i] += *reinterpret_cast<const floatx4*>(srcp + (j * I0 + (i < I0 ? i : i - I0)) * 1024);
    }
    int px[MT];   // the lane's pixels, -1 = none
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      px[i] = p0 + 16 * i + li_e;
      if (px[i] >= p_end) px[i] = -1;
    }
    // outputs that are not finite: again from the fp32 operands, one after the other
    if constexpr (NP == 3) {
      float bad = 0.0f;
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) bad = fmaf(v[j][i][r], 0.0f, bad);
      if (__builtin_expect(bad != 0.0f, 0)) {   // (a NaN)
        for (int e = 0; e < NT * MT * 4; ++e) {
          float x = 0.0f;
          int p = -1;
#pragma unroll
          for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
              for (int r = 0; r < 4; ++r)
                if (e == (j * MT + i) * 4 + r && (KS == 1 || (i < I0) == (kg == 0))) x = v[j][i][r], p = px[i];
          if (fabsf(x) < INFINITY || p < 0) continue;
          x = exact_output<MODE, TAPS, FUSE>(in, wgt, stats, H, W, g.Cin, g.Cout, p, n0 + 16 * (e / (4 * MT)) + 4 * lk_e + (e & 3));
#pragma unroll
          for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
              for (int r = 0; r < 4; ++r) v[j][i][r] = e == (j * MT + i) * 4 + r ? x : v[j][i][r];
        }
      }
    }
    // a pixel's channels one after the other: the two halves of a 128-byte line leave together (64 -> 256
    // channels at 56x56: 60 us, channel tile by channel tile 89 us)
    if (MODE == 0 && skip != nullptr) {
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        if (KS == 2 && (i < I0) != (kg == 0)) continue;
#pragma unroll
        for (int j = 0; j < NT; ++j)
          v[j][i] += *reinterpret_cast<const floatx4*>(skip + (size_t)(px[i] < 0 ? 0 : px[i]) * Ng + n0 + 16 * j + 4 * lk_e);
      }
    }
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      if (KS == 2 && (i < I0) != (kg == 0)) continue;
      if (px[i] < 0) continue;
#pragma unroll
      for (int j = 0; j < NT; ++j)
        *reinterpret_cast<floatx4*>(out + (size_t)px[i] * Ng + n0 + 16 * j + 4 * lk_e) = v[j][i];
    }
    // the sums, a channel tile at a time: one tile's sums and constants only are live
    if constexpr (EPI != 0)
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int nch = n0 + 16 * j + 4 * lk_e;
      double s1[4] = {0.0, 0.0, 0.0, 0.0}, s2[4] = {0.0, 0.0, 0.0, 0.0};
      floatx4 st4;
      float offh[4];   // code + offh = Eq. 10 over its step (exact below 2^23; from there on the half is rounded away)
      if constexpr (EPI > 1) {
        st4 = *reinterpret_cast<const floatx4*>(stats + P_STEP * Ng + nch);
        const int4 fb4 = *reinterpret_cast<const int4*>(stats + P_FB * Ng + nch);
        const int32_t fbv[4] = {fb4.x, fb4.y, fb4.z, fb4.w};
#pragma unroll
        for (int r = 0; r < 4; ++r) offh[r] = (float)(fbv[r] - (1 << (EPI - 1))) + 0.5f;
      }
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        if (KS == 2 && (i < I0) != (kg == 0)) continue;
        const bool ok = px[i] >= 0;
        uint32_t cw = 0;
        if constexpr (EPI > 1) {
          const unsigned char* ca = cbuf + (16 * i + li_e) * CPITCH + (16 * (NT * wn + j) + 4 * lk_e) * EPI / 8;
          cw = EPI == 4 ? (uint32_t) * reinterpret_cast<const uint16_t*>(ca) : *reinterpret_cast<const uint32_t*>(ca);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if constexpr (EPI == 1) {
            const double y = ok ? v[j][i][r] : 0.0f;
            s1[r] += y;
            s2[r] = __builtin_fma(y, y, s2[r]);
          } else if constexpr (EPI > 1) {
            const float q = (float)((cw >> (EPI * r)) & ((1u << EPI) - 1u)) + offh[r];
            const float da2 = ok && st4[r] * q > 0.0f ? v[j][i][r] : 0.0f;   // Eq. 10, Eq. 6
            s1[r] += (double)da2;
            s2[r] = __builtin_fma((double)q, (double)da2, s2[r]);
          }
        }
      }
      if constexpr (EPI != 0) {
        // over the 16 pixel lanes, then onto the wave's own row of sums
        double* row = sum_lds + (size_t)kg * 2 * BN + 16 * NT * wn;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const double t1 = row16_sum(s1[r]), t2 = row16_sum(s2[r]);
          if (li_e == 0) {
            row[16 * j + 4 * lk_e + r] += t1;
            row[BN + 16 * j + 4 * lk_e + r] += t2;
          }
        }
      }
    }
    if (DB) __syncthreads();   // the exchange area is the next tile's patch
  }
  if constexpr (EPI != 0) {
    __syncthreads();
    for (int c = tid; c < BN; c += THREADS) {
      double t1 = 0.0, t2 = 0.0;
#pragma unroll
      for (int k = 0; k < KS; ++k) {
        t1 += sum_lds[(size_t)k * 2 * BN + c];
        t2 += sum_lds[(size_t)k * 2 * BN + BN + c];
      }
      // Eq. 7 by linearity: with A~2 = step q, sum A~1 dA2 = (step sum q dA2 - beta sum dA2) / gamma
      if (EPI > 1)
        t2 = ((double)stats[P_STEP * Ng + nb + c] * t2 - (double)stats[P_BETA * Ng + nb + c] * t1) /
             (double)stats[P_GAMMA * Ng + nb + c];
      sums[((size_t)mb * 2) * Ng + nb + c] = t1;
      sums[((size_t)mb * 2 + 1) * Ng + nb + c] = t2;
    }
  }
}

// ---- which configuration a layer takes ---------------------------------------------------------------
struct Plan {
  int nt, ks, cpp, su;   // the kernel's parameters
  Tiling tl;
  size_t lds;
  int bn;
};

bool supported(const ConvGeom& g, int mode) {
  const int Cg = mode == 0 ? g.Cin : g.Cout, Ng = mode == 0 ? g.Cout : g.Cin;
  const bool k3 = g.R == 3 && g.S == 3 && g.pad == 1, k1 = g.R == 1 && g.S == 1 && g.pad == 0;
  const int64_t M = (int64_t)g.N * g.H * g.W;
  return g.stride == 1 && (k3 || k1) && Cg % 32 == 0 && Ng % 64 == 0 && M * g.Cin < ((int64_t)1 << 31) &&
         M * g.Cout < ((int64_t)1 << 31);
}

// Positions of a 3x3 patch up to which four-wave blocks share a compute unit in pairs (fp32: its LDS; four staging items a thread).
constexpr int kPairPositions = 256;

// What `tiles` tiles in four-wave blocks take, nblk blocks along the output channels: rounds of one block per unit, or
// of two (34 of 50 where the last round has one only).
int64_t rounds_cost(int64_t tiles, int64_t nblk, bool pairs) {
  const int64_t per = (tiles + kMaxPartialBlocks - 1) / kMaxPartialBlocks, n = (tiles + per - 1) / per * nblk;
  if (!pairs) return per * 40 * ((n + 255) / 256);
  const int64_t last = n % 512;
  return per * (50 * (n / 512) + (last == 0 ? 0 : last <= 256 ? 34 : 50));
}

// The configuration with nt, ks for this layer; false where its sizes do not fit.
bool fit_plan(const ConvGeom& g, int mode, int np, int nt, int ks, Plan& p) {
  const int Cg = mode == 0 ? g.Cin : g.Cout, Ng = mode == 0 ? g.Cout : g.Cin;
  const bool k3 = g.R == 3;
  p.nt = nt;
  p.ks = ks;
  p.cpp = !k3 && ks == 1 ? 2 : 1;                                // 1x1: two k-steps between barriers
  p.su = k3 ? (ks == 2 ? 3 : nt == 2 ? 4 : 7) : ks == 2 ? 2 : 4;   // staging items per thread, at most
  p.bn = 16 * nt * WN;
  if (Ng % p.bn != 0 || Cg % (32 * ks * p.cpp) != 0) return false;
  const int threads = 64 * WN * ks, c8 = 4 * ks * p.cpp, bm = 16 * MT;
  const int M = g.N * g.H * g.W, HW = g.H * g.W, W = g.W;
  Tiling& t = p.tl;
  if (!k3) {
    t.run = bm;
    t.unit = M;
    t.ntr = t.tiles = (M + bm - 1) / bm;
    t.npos = bm;
  } else {
    // image by image, the tiles of an image of equal lengths
    t.unit = HW;
    t.ntr = (HW + bm - 1) / bm;
    t.run = (HW + t.ntr - 1) / t.ntr;
    t.tiles = g.N * t.ntr;
    int rows = t.run % W == 0 ? t.run / W : (t.run + W - 2) / W + 1;   // that a run touches
    if (rows > g.H) rows = g.H;
    t.npos = (rows + 2) * (W + 2);
    // across images, where the patch has room for the two rows of border that each of them brings: runs of
    // any pixels, or of whole images
    const int room = p.su * threads / c8, xtiles = (M + bm - 1) / bm;
    int xrows = bm % W == 0 ? bm / W : (bm + W - 2) / W + 1;
    xrows += 2 + 2 * ((xrows + g.H - 2) / g.H);
    int imgs = bm / HW;
    if (imgs > room / ((g.H + 2) * (W + 2))) imgs = room / ((g.H + 2) * (W + 2));
    const bool run = xtiles < t.tiles && xrows * (W + 2) <= room;
    Tiling x = t;
    if (run) {
      x.run = bm;
      x.npos = xrows * (W + 2);
    } else if (imgs > 1) {
      x.run = imgs * HW;
      x.npos = imgs * (g.H + 2) * (W + 2);
    }
    x.unit = M;
    x.ntr = x.tiles = (M + x.run - 1) / x.run;
    // (A few tiles less do not make up for the unit's second block.  us, forward of the layer, runs across images / image by
    // image: 128 -> 128 @27x27 N=64 137 / 87, N=80 162 / 137, @29x29 N=56 137 / 87, 64 -> 64 @33x33 N=64 64 / 53, @40x40 N=64
    // 83 / 60, 256 -> 256 @22x22 N=20 128 / 78; but one round of single blocks beats a few pairs: 64 -> 64 @32x32 N=28, 256
    // blocks / 280, 29.5 / 31.4, 128 -> 128 @26x26 N=20, 242 / 280, 42.6 / 45.4.)
    const bool loses_pairs = x.npos > kPairPositions && t.npos <= kPairPositions &&
                             rounds_cost(x.tiles, Ng / p.bn, false) >= rounds_cost(t.tiles, Ng / p.bn, true);
    if ((run || imgs > 1) && !loses_pairs) t = x;
  }
  if (t.npos * c8 > p.su * threads) return false;
  if (p.su == 7 && t.npos * c8 <= 4 * threads) p.su = 4;
  t.per = (t.tiles + kMaxPartialBlocks - 1) / kMaxPartialBlocks;   // one row of sums per block
  t.gm = (t.tiles + t.per - 1) / t.per;
  p.lds = (size_t)area_bytes(k3 ? 9 : 1, nt, ks, p.cpp, p.su, np) + (size_t)ks * 2 * p.bn * sizeof(double);
  return p.lds <= (size_t)160 * 1024;
}

// How many consecutive tiles a block of an accepted plan takes: fewer rounds of the chip's places (two four-wave blocks per compute
// unit; with fp32 operands one where a patch has more than kPairPositions) that stay filled.  (1x1 gradient 256 <- 64 @56x56, two blocks along the
// channels: 896 blocks of four tiles, 1.75 rounds, 125 us; 512 of seven 116; 256 of fourteen, one per unit, 147.  Grids of one tile
// per block stay: 896 blocks of one or 448 of two, 1x1 256 -> 1024 @14x14 52 us both.  One block per unit: 64 -> 64 @55x55 N=64,
// forward, 448 blocks of four 150, 256 of seven 135, @57x57 N=40 387 of three 119, 233 of five 102; but a last round that is
// nearly empty costs less than it counts here: runs across images of 128 -> 128 @27x27 N=80, 522 blocks of two 142, 210 of five 162.
// With bf16 operands such patches leave room for two: gradient 64 <- 64 @55x55 N=64 448 blocks of four 114, 256 of seven 131, N=28
// 392 of two 68.5, 196 of four 81.)
void balance(const ConvGeom& g, int mode, int np, Plan& p) {
  if (p.tl.per == 1) return;
  const bool alone = np == 3 && p.su > 4;
  const int64_t nblk = (mode == 0 ? g.Cout : g.Cin) / p.bn, places = alone ? 256 : 512, least = alone ? 160 : 448;
  auto blocks = [&](int per) { return (p.tl.tiles + per - 1) / per * nblk; };
  auto cost = [&](int per) { return (blocks(per) + places - 1) / places * (2 * per + 1); };   // in half tiles: a start costs about one
  int best = p.tl.per;
  for (int per = p.tl.per + 1; per <= 16 * p.tl.per && blocks(per) >= least; ++per)
    if (cost(per) < cost(best)) best = per;
  p.tl.per = best;
  p.tl.gm = (p.tl.tiles + best - 1) / best;
}

// Whether the halo kernel is the faster one on a 3x3 layer's four-wave grid (fp32).  Its tiles of 64 pixels, all in one
// round of the compute units, take less than a 112-pixel tile here (us, layer, halo kernel / here: 64 -> 64 @32x32 N=12 25.5 /
// 27.1, backward 45.8 / 51.3; with more of them it is two rounds, N=24 29.3 here).  A patch of more than 256 positions
// (a round of runs across 32-pixel-wide images, rows of 45 and more) leaves LDS for one block per unit only; a tile then takes 15.5
// us per 64 input channels, the halo kernel 11.1 per round of 64 pixels, 20 of 128, 35.5 of 224 (layer, halo kernel / here: 64 -> 64
// @55x55 N=24 78.1 / 64.5, N=20 58.7 / 63.1).  Where both take about the same this kernel stays: its sums are the closer ones.
bool halo_is_faster(const ConvGeom& g, int mode, const Plan& p) {
  const int Ng = mode == 0 ? g.Cout : g.Cin;
  const bool alone = p.su > 4;
  // (256 blocks of 64 pixels and 64 channels at most: no need to ask for a plan beyond)
  if (!alone && (int64_t)g.N * g.H * g.W * Ng > 256 * 64 * 64) return false;
  int pixels;
  int64_t blocks;
  if (!halo_grid(g, mode, &pixels, &blocks)) return false;
  if (pixels == 64 && blocks <= 256) return true;
  if (!alone) return false;
  const int64_t rounds = (blocks + 255) / 256;
  Plan q = p;
  balance(g, mode, 3, q);
  const double here = 1.5 + 15.5 * (double)(q.tl.per * (((int64_t)q.tl.gm * (Ng / q.bn) + 255) / 256));
  const double there = pixels == 64 ? 3.7 + 11.1 * rounds : pixels == 128 ? 3.0 + 20.0 * rounds : 2.5 + 35.5 * rounds;
  return 1.1 * there < here;
}

// Tiles of 128 pixels x 64 channels that the other kernels have, each XCD's share rounded up.
int64_t other_tiles(const ConvGeom& g, int Ng) { return ((int64_t)g.N * g.H * g.W + 1023) / 1024 * 8 * (Ng / 64); }

// Whether a grid of four-wave blocks - two to a compute unit, 512 at a time - is faster than the kernel that would
// run otherwise.  A grid a little over one block per unit, or a little over 512, takes as long as a much larger one (the
// units with one block more decide), while the other kernels' tiles may just fit.  (us, here / the other kernel, n blocks.
// fp32 1x1, where the pointwise kernel's tiles fit one round of the units (two for blocks of 128 channels): 256 -> 128
// @27x27 N=20, n = 262, 16.1 / 13.5, 512 -> 64 @28x28 N=39, n = 274, 29.7 / 23.5, 64 -> 512 @16x16 N=32, n = 296 of 128
// channels, 11.8 / 10.6, gradient 256 <- 128 @20x20 N=81, n = 290 of 128, 24.9 / 22.4; just beyond: 256 -> 256 @14x14 N=44,
// n = 308, 16.6 / 22.7, 192 -> 256 @29x29 N=10, n = 304, 13.1 / 16.5, gradient 256 <- 128 @27x27 N=49, n = 319 of 128, 25.2 /
// 29.8.  Longer contractions than 256 share the pointwise kernel's last round out: gradient 384 <- 64 @29x29 N=41, n = 308,
// 23.6 / 20.4.  256 -> 64 @56x56 of two tiles per block N=20, n = 280, 30.9 / 23.6, N=28, n = 392, 33.0 / 32.1; 64 -> 256
// @56x56 N=8, n = 448, 12.3 / 14.8, N=20, n = 560, 28.9 / 27.4, but 128 -> 512 @28x28 N=20, also 560, 23.8 / 26.7.  bf16
// 1x1: 128 -> 512 @28x28 N=10, n = 280, 10.4 / 9.0, N=12, n = 336, 10.7 / 11.5, N=20, n = 560, 14.5 / 13.2, N=24, n = 672,
// 14.7 / 17.2; 256 -> 512 @15x15 N=77, n = 620, 19.2 / 24.6; 64 -> 256 @56x56 N=14, n = 784, 15.3 / 13.4; 512 -> 128 @28x28
// N=40, n = 280, 23.8 / 18.9, N=56, n = 392, 24.9 / 23.7; 512 -> 256 @15x15 N=77, n = 310, 21.0 / 23.4; 64 -> 128 @57x57 N=20
// of two tiles, n = 291, 16.0 / 11.5; gradient 256 <- 1024 @14x14 N=40, n = 280, 30.3 / 24.5.  bf16 3x3: 64 -> 64 @56x56 of two tiles per block
// N=20, n = 280, 24.5 / 21.1; 64 -> 64 @57x57 of two tiles, patches of more than 256 positions, N=27, step 53.5 / 46.9;
// 128 -> 128 @60x60 N=10, n = 644, 47.4 / 42.8, N=14, n = 900, 54.8 / 60.2, its gradient 62.8 / 53.4; gradient 128 <- 128
// @28x28 N=40, n = 280 of 128 channels, 43.6 / 36.7, N=67, n = 469, 44.2 / 51.9, @30x30 N=58 of two tiles 83.4 / 55.6, 256 <-
// 256 @15x15 N=73, n = 294, 78.6 / 68.6, @17x17 N=100, n = 518, 120.7 / 89.6.)
bool four_waves_pay(const ConvGeom& g, int mode, int np, bool sums, const Plan& p) {
  const int Cg = mode == 0 ? g.Cin : g.Cout, Ng = mode == 0 ? g.Cout : g.Cin;
  const int64_t n = (int64_t)p.tl.gm * (Ng / p.bn);
  const bool over_one = n > 256 && n < 320, over_two = n > 512 && n < 660;
  // whole rounds of one block per unit that this grid is larger than, and whether the other kernels fit them
  const int64_t rounds = (n - 1) / 256, others = other_tiles(g, Ng);
  const bool fit = rounds > 0 && others <= 256 * rounds * p.nt;
  if (g.R == 3) {
    if (np == 3) return p.nt == 2 || !halo_is_faster(g, mode, p);
    if (sums) return true;
    if (mode == 1 && p.nt == 2) return n <= 256 || (n >= 400 && n <= 512 && p.tl.per == 1);
    return !(p.nt == 1 && p.tl.per > 1 && over_one) && !(p.su > 4 && (p.tl.per > 1 || over_two || (mode == 1 && n > 512)));
  }
  // with the Eq. 6-7 sums the other kernels need a pass of their own or lose their weight gradient's launch: fp32 is faster
  // here throughout, bf16 with 64 channels per block and less than 1024 to contract only (1024 <- 256 @14x14 N=40,
  // n = 560 of 128 channels each, backward 65.6 / 57.9; 256 <- 1024 N=40 59.4 / 55.3)
  if (np == 3) {
    if (sums) return true;
    // (512 -> 128 @28x28 N=40, n = 280: 42.6 / 59.1; 128 -> 512 @20x20 N=18, n = 260: 14.1 / 16.3)
    if (p.nt == 2 && (Cg >= 512 || Cg == 128)) return true;
    if (fit && (rounds == 1 || (rounds == 2 && Cg < 128))) return false;
    if (over_one && p.nt == 1 && Cg > 256 && (Ng == 64 || Ng % 128 == 0)) return false;
    return !(n > 256 && n < 400 && p.tl.per > 1);
  }
  // (bf16, layer, us, other kernel / here.  Gradient, blocks of 128 channels: 1024 <- 256 @14x14 N=64, n = 896, 80.0 / 75.5, N=40,
  // n = 560, 58.0 / 60.6; 2048 <- 512 @7x7 N=64, n = 448, 65.8 / 60.6, N=40, n = 288, 51.6 / 54.3; 256 <- 64 @56x56 N=40, n = 748,
  // 119 / 112, N=20, n = 560, 68.4 / 72.0; 512 <- 128 @28x28 N=64 112 / 106.  Forward: 1024 -> 256 @14x14 N=40 53.8 / 47.2; 2048 ->
  // 512 @8x8 N=64 77.2 / 62.3; 256 -> 1024 @15x15 N=64, n = 1032, 48.7 / 42.0; 128 -> 512 @28x28 N=52, n = 1456, 46.6 / 42.4, N=20,
  // n = 560, 29.1 / 29.6.
  // Blocks of several tiles with 128 and more channels to contract, K = 8 / 4: 512 <- 128 @30x30 N=80 149 / 145 against 162 / 146,
  // @28x28 N=80 135 / 133 against 138 / 132; with 64 here, 256 <- 64 @56x56 N=80 273 / 262 against 264 / 244.  Forward with 64
  // channels to contract: 64 -> 256 @56x56 N=14, n = 784, 31.3 / 32.1, @55x55 N=16, n = 866, 31.6 / 32.4.)
  if (mode == 1) return sums && (p.nt == 1 ? Cg < 1024 : (n >= 440 && n <= 512) || (n >= 720 && (p.tl.per == 1 || Cg < 128)));
  return Cg >= 1024 || n >= (Cg < 128 ? 1024 : 720) || (!fit && !(over_one && p.tl.per > 1));
}

// 128 output channels per block where that fills the chip, else 64.  About one block per compute unit: the
// contraction in two groups of waves; more: four-wave blocks, two per unit.  (us, blocks of 8 / 4 waves: 3x3
// 256 -> 256 @14x14, 256 blocks 79 / 89; 1x1 1024 -> 256 @14x14, 224 blocks 45 / 55; 3x3 128 -> 128 @28x28,
// 448 blocks 79 / 74; 1x1 256 -> 1024 @14x14, 896 blocks 54 / 45; with 64 channels per block 3x3 512 -> 512 @7x7
// 88 / 105 instead of 125 / 160 with 128 channels on 112 blocks.)  Grids of fewer than 96 blocks stay on the other
// kernels, and four-wave blocks where they do not pay.  sums: with the Eq. 6-7 sums in the epilogue.
bool make_plan(const ConvGeom& g, int mode, int np, bool sums, Plan& p) {
  if (!supported(g, mode)) return false;
  const int Cg = mode == 0 ? g.Cin : g.Cout, Ng = mode == 0 ? g.Cout : g.Cin;
  const bool k3 = g.R == 3;
  for (int nt = 2; nt >= 1; --nt)
    for (int ks = 2; ks >= 1; --ks) {
      if (!fit_plan(g, mode, np, nt, ks, p)) continue;
      const int64_t blocks = (int64_t)p.tl.gm * (Ng / p.bn);
      if (blocks < (nt == 2 ? 200 : 96) || (ks == 2 && blocks > 256)) continue;
      // (the gradient of 1x1 layers with 64 channels to contract and more to write: two groups of waves have nothing to share;
      // exact storage 256 <- 64 @16x16 N=12, backward 32.4 us against the pointwise kernel's 30.1)
      if (ks == 2) return k3 || np != 3 || sums || mode == 0 || Cg >= 128 || Ng < 128;
      if (four_waves_pay(g, mode, np, sums, p)) return true;
      // (long 1x1 contractions on 257 to 319 four-wave blocks: half as many of eight waves with 128 channels, which take what
      // the pointwise kernel takes or less, and their sums are the closer ones.  us, here / pointwise kernel: 1024 -> 512
      // @14x14 N=20 43.1 / 42.5, 384 -> 512 @15x15 N=18 19.3 / 18.8, 1024 -> 384 @20x20 N=14 43.7 / 60.7; gradient 512 <- 256
      // @29x29 N=10 23.2 / 25.2, but 5 to 12 % slower where its tiles fit one round)
      return !k3 && np == 3 && nt == 1 && blocks < 320 && Cg >= 384 && (mode == 0 || other_tiles(g, Ng) > 256) &&
             fit_plan(g, mode, np, 2, 2, p);
    }
  return false;
}

Tiling with_divisors(const ConvGeom& g, Tiling t) {
  t.w = Divisor(g.W);
  t.pw = Divisor(g.W + 2);
  t.h = Divisor(g.H);
  t.ph = Divisor(g.H + 2);
  t.hw = Divisor(g.H * g.W);
  t.per_unit = Divisor(t.ntr);
  return t;
}

template <int MODE, int NP, bool PRE, int TAPS, int NT, int KS, int CPP, int SU>
int launch_cfg(hipStream_t st, const ConvGeom& g, const Plan& p, const float* in, const float* w, const void* parts,
               const float* skip, float* out, double* sums, const uint8_t* codes, const float* stats, int epi) {
  const int Ng = MODE == 0 ? g.Cout : g.Cin;
  const unsigned grid = (unsigned)((p.tl.gm + 7) / 8 * 8 * (Ng / p.bn));
  // (weights are split once for gradients with sums only)
  auto kern = split_conv_kernel<MODE, TAPS, NT, KS, CPP, SU, MODE == 1 && PRE ? 4 : 0, NP, PRE>;
  if constexpr (MODE == 0) {
    if (epi == 1) kern = split_conv_kernel<MODE, TAPS, NT, KS, CPP, SU, 1, NP, PRE>;
  } else {
    if (PRE && epi == 0) return ABL_ERR_ARG;
    if (epi == 4) kern = split_conv_kernel<MODE, TAPS, NT, KS, CPP, SU, 4, NP, PRE>;
    if (epi == 8) kern = split_conv_kernel<MODE, TAPS, NT, KS, CPP, SU, 8, NP, PRE>;
    if constexpr (TAPS == 1 && KS == 1 && NP == 3 && !PRE)
      if (epi != 0 && g.Cout == 32 * KS * CPP)
        kern = epi == 4 ? split_conv_kernel<MODE, TAPS, NT, KS, CPP, SU, 4, NP, PRE, 0, true>
                        : split_conv_kernel<MODE, TAPS, NT, KS, CPP, SU, 8, NP, PRE, 0, true>;
  }
  if (int e = allow_full_lds(reinterpret_cast<const void*>(kern))) return e;
  kern<<<grid, 64 * WN * KS, p.lds, st>>>(in, w, static_cast<const uint4*>(parts), skip, out, sums, codes, stats, g,
                                          with_divisors(g, p.tl), nullptr, 0);
  return hip_status();
}

template <int MODE, int NP, bool PRE>
int launch_as(hipStream_t st, const ConvGeom& g, const Plan& p, const float* in, const float* w, const void* parts,
              const float* skip, float* out, double* sums, const uint8_t* codes, const float* stats, int epi) {
  auto run = [&](auto f) { return f(st, g, p, in, w, parts, skip, out, sums, codes, stats, epi); };
  if (g.R == 3) {
    if (p.ks == 2) return run(p.nt == 2 ? launch_cfg<MODE, NP, PRE, 9, 2, 2, 1, 3> : launch_cfg<MODE, NP, PRE, 9, 1, 2, 1, 3>);
    if (p.nt == 2) return run(launch_cfg<MODE, NP, PRE, 9, 2, 1, 1, 4>);
    return run(p.su == 4 ? launch_cfg<MODE, NP, PRE, 9, 1, 1, 1, 4> : launch_cfg<MODE, NP, PRE, 9, 1, 1, 1, 7>);
  }
  if (p.ks == 2) return run(p.nt == 2 ? launch_cfg<MODE, NP, PRE, 1, 2, 2, 1, 2> : launch_cfg<MODE, NP, PRE, 1, 1, 2, 1, 2>);
  return run(p.nt == 2 ? launch_cfg<MODE, NP, PRE, 1, 2, 1, 2, 4> : launch_cfg<MODE, NP, PRE, 1, 1, 1, 2, 4>);
}

template <int MODE, int NP>
int launch(hipStream_t st, const ConvGeom& g, const Plan& p, const float* in, const float* w, const void* parts,
           const float* skip, float* out, double* sums, const uint8_t* codes, const float* stats, int epi) {
  return parts != nullptr ? launch_as<MODE, NP, true>(st, g, p, in, w, parts, skip, out, sums, codes, stats, epi)
                          : launch_as<MODE, NP, false>(st, g, p, in, w, parts, skip, out, sums, codes, stats, epi);
}

template <int FUSE, int KS, int SU, bool PRE>
int launch_fused(hipStream_t st, const ConvGeom& g, const Plan& p, const float* x, const float* stats, const float* w,
                 const void* parts, const float* skip, float* y, uint8_t* packed, double* sums) {
  const unsigned grid = (unsigned)((p.tl.gm + 7) / 8 * 8 * (g.Cout / p.bn));
  const int64_t raw = (int64_t)g.N * g.H * g.W * g.Cin * FUSE / 8;
  auto kern = sums != nullptr ? split_conv_kernel<0, 9, 1, KS, 1, SU, 1, 3, PRE, FUSE>
                              : split_conv_kernel<0, 9, 1, KS, 1, SU, 0, 3, PRE, FUSE>;
  if (int e = allow_full_lds(reinterpret_cast<const void*>(kern))) return e;
  kern<<<grid, 64 * WN * KS, p.lds, st>>>(x, w, static_cast<const uint4*>(parts), skip, y, sums, nullptr, stats, g,
                                          with_divisors(g, p.tl), packed, (int)((raw + 127) / 128 * 128 - raw));
  return hip_status();
}

// The fused forward: 64 output channels per block (the constants of Eq. 1-3 take the registers of the second tile) in
// four waves.
bool fit_fused_plan(const ConvGeom& g, Plan& p) {
  return g.R == 3 && supported(g, 0) && fit_plan(g, 0, 3, 1, 1, p);
}

}  // namespace

int split_conv_blocks(const ConvGeom& g, int mode, bool bf16, bool sums) {
  Plan p;
  if (!make_plan(g, mode, bf16 ? 1 : 3, sums, p)) return 0;
  balance(g, mode, bf16 ? 1 : 3, p);
  return p.tl.gm;
}

// On a launch that is there anyway: 3x3 layers, and 1x1 layers of 4096 pixels and more whose gradient contracts 256 channels and
// more; a forward of two k-steps from three times as many pixels on.  (Layer, us, split by the blocks / once: gradient 2048 <- 512 @7x7 N=14 48.2 / 52.3, 512 <- 128 @28x28 N=26 73.8 / 78.5,
// 256 <- 64 @56x56 N=26 94.0 / 96.8; forward 512 -> 2048 @7x7 N=14 30.3 / 32.3, 256 -> 1024 @15x15 N=14 29.7 / 31.2, but 1024
// -> 256 @14x14 N=40 72 / 64; bf16 64 -> 256 @55x55 N=12 29.1 / 30.2, @56x56 N=20 36.9 / 36.5.)
// A launch of its own costs 4 us: those whose waves take enough k-steps, counted over all of a grid's rounds; bf16 1x1 layers
// split little at a step, and only more channels per block make it count.  (Backward, us, split by the blocks / once.  3x3: 64
// <- 64 @8x8 N=128, 9 steps, 39.3 / 40.5, @28x28 N=24, 9, 46.0 / 47.3, N=40, 18, 60.3 / 60.7, bf16 46.8 / 45.0, N=128, 31, 98.3 /
// 95.8; 128 <- 128 @14x14 N=64, 18, 63.4 / 63.3, bf16 50.0 / 49.8; 512 <- 512 @7x7 N=40, 72, 124 / 122, bf16 83 / 74.  1x1: 64
// <- 256 @55x55 N=14, 8, 46.4 / 47.4, N=40, 16.9, 94.6 / 91.7; 128 <- 512 @28x28 N=14, 8, 45.5 / 46.8, N=26, 16, 63.3 / 61.9; 1024
// <- 256 @14x14 N=40, 8.8, 84.9 / 87.7; 256 <- 1024 N=40, 32, 87.3 / 81.2.  bf16, steps times channel tiles: 64 <- 256 @56x56
// N=34, 15, 65.4 / 68.3, N=64, 28, 130 / 127; 128 <- 512 @28x28 N=28, 16, 43.7 / 44.5; 256 <- 1024 @14x14 N=34, 16, 45.3 / 46.3,
// N=64, 32, 58.8 / 56.8; 1024 <- 256 N=52, 23, 68.5 / 69.1, @15x15 N=52, 26, 79.6 / 77.5.)
bool parts_pay(const ConvGeom& g, int mode, bool bf16, bool own_launch) {
  const int64_t pixels = (int64_t)g.N * g.H * g.W;
  if (g.R != 3 && (pixels < 4096 || (mode == 1 && g.Cout < 256) || (mode == 0 && g.Cin < 128 && pixels < 3 << 14))) return false;
  if (!own_launch) return true;
  Plan p;
  if (!make_plan(g, mode, bf16 ? 1 : 3, mode == 1, p)) return false;
  const int Cg = mode == 0 ? g.Cin : g.Cout, Ng = mode == 0 ? g.Cout : g.Cin;
  const int64_t steps = (int64_t)g.R * g.S * (Cg / 32) / p.ks, n = (int64_t)p.tl.tiles * (Ng / p.bn);
  const int64_t all = steps * (n > 512 ? n : 512) * (bf16 && g.R == 1 ? p.nt : 1);   // (places for 512 blocks)
  return all >= 512 * (g.R == 3 ? 18 : bf16 ? 24 : 16);
}

// (us, layer forward / backward, image kernel against here: 512 -> 512 @7x7 N=40, two rounds of images, 72 / 113 against 46 /
// 74, N=120 125 / 224 against 57 / 116; 256 -> 256 @14x14 N=20 35.2 / 58.1 against 32.9 / 53.0, N=64 40.5 / 79.9 against 40.6 /
// 78.1, N=120 65.4 / 134 against 59.1 / 119; 128 -> 128 @14x14 N=28 26.5 / 50.0 against 22.7 / 45.1, N=64 29.4 / 55.3 against
// 26.6 / 49.6.  Four-wave blocks of 64 channels a little over one per unit lose: 256 -> 256 @14x14 N=40, n = 280, 37.1 / 68.1
// against 46.3 / 72.9, 128 -> 128 N=80 30.9 / 56.1 against 33.2 / 56.3, n = 420 wins again, 33.9 / 63.0 against 32.9 / 60.2; so
// do a few blocks with a long contraction beside one round of images: 512 -> 512 @7x7 N=28, n = 112, 43.4 / 70.4 against 45.5 /
// 69.5.  Nor does an image that is no more than a tile here, while one round of the units takes them all - forward: 256 -> 256 @7x7
// N=64 27.9 against 30.4, @8x8 N=40 25.7 / 29.1, @10x10 N=52 31.4 / 32.8, 128 -> 128 @8x8 N=64 19.3 / 20.5, but @12x12 N=64 27.3 /
// 23.8; gradients, with the sums, below 64 pixels: @7x7 N=64 49.0 / 50.5, @8x8 N=40 48.1 / 47.8, @10x10 N=64 71.4 / 69.5.)
bool split_beats_image(const ConvGeom& g, int mode) {
  Plan p;
  if (!make_plan(g, mode, 1, false, p)) return false;
  const int Cg = mode == 0 ? g.Cin : g.Cout, Ng = mode == 0 ? g.Cout : g.Cin;
  const int64_t n = (int64_t)p.tl.gm * (Ng / p.bn);
  if ((int64_t)g.N * (Ng / 64) <= 256 && g.H * g.W <= (mode == 0 ? 16 * MT : 63)) return false;
  if (p.nt == 1 && p.ks == 1) return n >= 384;
  return n >= 128 || Cg < 512 || (int64_t)g.N * (Ng / 64) > 256;
}

// ... and where the weights come in parts, which the image kernel does not read: with 512 channels and more to contract (us, layer,
// image kernel / here: 512 -> 512 @8x8 N=40 192 / 117, N=14 112 / 93, @7x7 N=28 115 / 100; 256 -> 256 about the same on both, @14x14
// N=40 105.7 / 106.4, @10x10 N=52 91.0 / 87.8).  Not on images of a tile or two where that kernel's grid is one round of the compute
// units (forward of 512 -> 64 @3x3 N=108 28.9 / 34.6, 512 -> 128 @4x5 N=74 33.8 / 36.6; both equal below 60 blocks, and 512 -> 512
// @3x5 N=58, two rounds, 44.1 / 37.8; gradients, with their sums, 0.81 to 1 of the time there too).
bool split_parts_beat_image(const ConvGeom& g, int mode) {
  if (split_beats_image(g, mode)) return true;
  const int Cg = mode == 0 ? g.Cin : g.Cout, Ng = mode == 0 ? g.Cout : g.Cin;
  const int64_t blocks = (int64_t)g.N * (Ng / 64);
  if (Cg < 512 || (mode == 0 && g.H * g.W <= 20 && blocks > 60 && blocks <= 256)) return false;
  Plan p;
  return make_plan(g, mode, 1, mode == 1, p);
}

// Four-wave grids that fill less than three quarters of their 512 places are not (512 -> 128 @28x28, step, us, with the
// pass / with the prologue: N=16, eight-wave blocks, 40.0 / 41.6; N=24, n = 336, 56.7 / 53.0; N=28, n = 392, 59.9 / 64.9),
// nor are shorter contractions, but for 256 -> 256 and where the pointwise kernel's tiles are more than a round of the units
// and the ones here no more than their 512 places (128 -> 256 @28x28 N=5 18.4 / 15.8, N=24 34.5 / 30.8; 256 -> 128 @14x14
// N=40 26.6 / 21.9, @27x27 N=36, n = 470, 40.3 / 44.1, @28x28 N=40, n = 560, 49.5 / 45.6; 320 -> 192 @13x13 N=56 40.8 / 31.7;
// but 384 -> 192 @28x28 N=20 45.1 / 53.1, 256 -> 256 @14x14 N=56 34.3 / 37.2; @28x28 N=40, n = 560, 62.7 / 59.7).
bool split_beats_prologue(const ConvGeom& g) {
  Plan p;
  if (g.R != 1 || g.Cin < 256 || !make_plan(g, 0, 3, false, p)) return false;
  const int64_t n = (int64_t)p.tl.gm * (g.Cout / p.bn);
  if (g.Cin < 384 && g.Cout < 256)
    return g.Cout >= 128 && other_tiles(g, g.Cout) > 256 && (int64_t)p.tl.tiles * (g.Cout / 64) <= 512;
  if (p.ks == 2) return p.nt == 1 || n >= 200 || g.Cin >= 1024;
  if (p.nt == 2 && n > 256 && n < 320 && g.Cin < 512) return false;   // (384 -> 128 @29x29 N=41 70.5 / 62.2)
  return p.nt == 2 ? g.Cin >= 384 || n <= 512 || n >= 660 : n >= 350;
}

int launch_split_conv(hipStream_t st, const ConvGeom& g, int mode, bool bf16, const float* in, const float* w,
                      const float* skip, float* out, double* sums, const void* parts) {
  Plan p;
  if (!make_plan(g, mode, bf16 ? 1 : 3, false, p)) return ABL_ERR_SHAPE;
  balance(g, mode, bf16 ? 1 : 3, p);
  const int epi = sums != nullptr ? 1 : 0;
  if (mode == 0)
    return bf16 ? launch<0, 1>(st, g, p, in, w, parts, skip, out, sums, nullptr, nullptr, epi)
                : launch<0, 3>(st, g, p, in, w, parts, skip, out, sums, nullptr, nullptr, epi);
  return bf16 ? launch<1, 1>(st, g, p, in, w, nullptr, nullptr, out, nullptr, nullptr, nullptr, 0)
              : launch<1, 3>(st, g, p, in, w, nullptr, nullptr, out, nullptr, nullptr, nullptr, 0);
}

int split_forward3(const ConvGeom& g, int* rows) {
  Plan p;
  if (g.R != 3 || !make_plan(g, 0, 3, false, p)) return 0;
  const bool weighed = p.nt == 1 && p.ks == 1;   // (make_plan has compared this one with the halo kernel)
  if (!fit_fused_plan(g, p) || (!weighed && halo_is_faster(g, 0, p))) return -1;
  balance(g, 0, 3, p);
  *rows = p.tl.gm;
  return 1;
}

int launch_split_fwd_fused(hipStream_t st, const ConvGeom& g, int K, const float* x, const void* stats, const float* w,
                           const float* skip, float* y, void* packed, double* sums, const void* parts) {
  Plan p;
  if (!fit_fused_plan(g, p) || (K != 4 && K != 8)) return ABL_ERR_SHAPE;
  balance(g, 0, 3, p);
  const float* sp = static_cast<const float*>(stats);
  uint8_t* pk = static_cast<uint8_t*>(packed);
  auto run = [&](auto f) { return f(st, g, p, x, sp, w, parts, skip, y, pk, sums); };
  if (parts != nullptr) {
    if (p.su == 4) return run(K == 4 ? launch_fused<4, 1, 4, true> : launch_fused<8, 1, 4, true>);
    return run(K == 4 ? launch_fused<4, 1, 7, true> : launch_fused<8, 1, 7, true>);
  }
  if (p.su == 4) return run(K == 4 ? launch_fused<4, 1, 4, false> : launch_fused<8, 1, 4, false>);
  return run(K == 4 ? launch_fused<4, 1, 7, false> : launch_fused<8, 1, 7, false>);
}

int launch_split_dgrad_reduce(hipStream_t st, const ConvGeom& g, int K, bool bf16, const float* dy, const float* w,
                              const void* packed, const void* stats, float* da3, double* partial, const void* parts) {
  Plan p;
  if (!make_plan(g, 1, bf16 ? 1 : 3, true, p) || (K != 4 && K != 8)) return ABL_ERR_SHAPE;
  balance(g, 1, bf16 ? 1 : 3, p);
  const uint8_t* codes = static_cast<const uint8_t*>(packed);
  const float* sp = static_cast<const float*>(stats);
  return bf16 ? launch<1, 1>(st, g, p, dy, w, parts, nullptr, da3, partial, codes, sp, K)
              : launch<1, 3>(st, g, p, dy, w, parts, nullptr, da3, partial, codes, sp, K);
}

}  // namespace abl
