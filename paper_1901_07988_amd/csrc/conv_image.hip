// 3x3 'same' stride-1 convolutions on small images (up to 208 pixels: the 14x14 and 7x7 stages of
// an ImageNet network) in fp32: Eq. 4 (forward, mode 0) and the second half of Eq. 5 (gradient to
// the conv input, mode 1), the latter optionally with the Eq. 6-7 sums of the BN backward in its
// epilogue.
//
// One block = one image x 64 output channels, and the image stays in LDS, 64 contraction channels
// (one phase) at a time: (H+2)(W+2) positions of 64 floats with their zero border, 68 KB for 14x14,
// in two buffers that take turns - the next phase's channels are requested during this phase's
// MFMAs and written to the other buffer after them, so that only the first phase's loads are
// waited for.  That is what the 160 KB of LDS per compute unit are for: every input element is
// fetched once per block instead of once per tile of a pixel grid.  The four waves split the
// CONTRACTION: of the 9 taps x 4 sixteen-channel chunks of a phase each wave takes 9, and each
// keeps the block's whole output tile (up to 13 x 4 MFMA tiles = 208 accumulator registers) to
// itself.  So an activation fragment is read from LDS once per block and k-step (one 16-byte
// read feeds four MFMAs of each of the four channel tiles), no weights are shared (each wave
// streams its own k-steps' weights from the L2 straight into registers) and the main loop has no
// barrier and next to no vector-ALU work: per k-step 208 MFMAs against 13 LDS reads, 16 loads and
// some thirty other instructions.  The four partial tiles are added through the same LDS at the
// end in a fixed wave order; the wave that owns an output-channel tile adds the shortcut, stores,
// and takes the per-channel sums (of y for the next layer's Eq. 1, or Eq. 6-7 from the layer's
// codes).
//
// The file also holds another kernel built for one block per compute unit with its results in accumulator
// registers: the weight gradient of 1x1 layers from the packed codes with bf16 operands (rows_wgrad_bf16_kernel).
//
// The MFMAs are written as inline assembly with the accumulator tied to the result: left to the
// register allocator, some tiles get a result register of their own and are copied back every
// k-step.  The compiler does not know these are matrix-core results, so the wait states they need
// before another kind of instruction reads them are inserted by hand after the loop.

#include <type_traits>

#include "abl_internal.h"

namespace abl {
namespace {

constexpr int kThreads = 256;
constexpr int IMG_NB = 64;    // output channels per block
constexpr int IMG_PC = 64;    // contraction channels per phase; two phases' patches are resident

template <int MODE, int MT, int EPI>
__global__ __launch_bounds__(kThreads, 1) void image_f32_kernel(const float* __restrict__ in,
                                                                const float* __restrict__ wgt, const float* skip,
                                                                float* out, double* __restrict__ sums,
                                                                const uint8_t* __restrict__ codes,
                                                                const float* __restrict__ stats, ConvGeom g) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int H = g.H, W = g.W, HW = H * W, PW = W + 2;
  const int Cg = MODE == 0 ? g.Cin : g.Cout;   // contraction channels: 16, 32, or a multiple of 64
  const int Ng = MODE == 0 ? g.Cout : g.Cin;   // output channels: a multiple of 64
  const int PC = Cg < IMG_PC ? Cg : IMG_PC;    // channels per phase (a power of two)
  const int pitch = 4 * PC + 16;               // bytes per patch position: the 16-byte fragments of 16
                                               // consecutive positions fall into different banks
  const int bufsz = (H + 2) * PW * pitch;      // one phase's patch; two of them take turns
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lk = lane >> 4;
  // ids 8 apart share an XCD and its L2: the blocks of one image (same input) run there
  const int nblk = Ng / IMG_NB;
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int img = (slot / nblk) * 8 + xcd;
  const int n0 = (slot % nblk) * IMG_NB;
  if (img >= g.N) return;

  // ---- the zero border of both patch buffers, once (the phases rewrite the interior only)
  {
    const int per = pitch >> 4;   // 16-byte pieces per position
    const int nz = (2 * PW + 2 * H) * per;
    for (int i0 = 0; i0 < nz; i0 += kThreads) {
      const int it = i0 + tid < nz ? i0 + tid : nz - 1;   // (a lane past the end repeats the last piece)
      const int bp = it / per, piece = it - bp * per;
      int pos;
      if (bp < PW) pos = bp;
      else if (bp < 2 * PW) pos = (H + 1) * PW + (bp - PW);
      else pos = (((bp - 2 * PW) >> 1) + 1) * PW + (((bp - 2 * PW) & 1) ? PW - 1 : 0);
      *reinterpret_cast<uint4*>(smem + pos * pitch + piece * 16) = make_uint4(0u, 0u, 0u, 0u);
      *reinterpret_cast<uint4*>(smem + bufsz + pos * pitch + piece * 16) = make_uint4(0u, 0u, 0u, 0u);
    }
  }

  // ---- fragment addresses.  acc[jj] is the output-channel tile (wave + jj) % 4, so that a wave's
  // own tile (the one it finishes) is acc[0] whatever the wave.
  int a_base[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    int m = 16 * i + li;
    m = m < HW ? m : HW - 1;   // rows past the image: any valid address, never stored
    const int h = m / W, w = m - h * W;
    a_base[i] = (h * PW + w) * pitch + lk * 16;
    asm volatile("" : "+v"(a_base[i]));   // kept in its register, not recomputed in the loop
  }
  const int cch_sh = __builtin_ctz((unsigned)PC) - 4;   // log2 of 16-channel chunks per phase
  const int T = 9 << cch_sh;
  const int ks_begin = wave * T / 4, ks_end = (wave + 1) * T / 4;
  auto a_offset = [&](int ks) __attribute__((always_inline)) {
    const int tap = ks >> cch_sh, cc = ks - (tap << cch_sh);
    const int r = tap / 3, s = tap - 3 * r;
    return (r * PW + s) * pitch + cc * 64;
  };
  // weights of one k-step: MFMA t of a chunk contracts channels 4 lk + t, so the lane's four
  // registers are four consecutive channels of its column (forward: four rows of W; gradient: 16
  // contiguous bytes).  Uniform part of the address in scalar registers, the lane's part a 32-bit
  // byte offset.
  uint32_t w_lane[4];
#pragma unroll
  for (int t = 0; t < 4; ++t)
    w_lane[t] = 4u * (MODE == 0 ? (uint32_t)((4 * lk + t) * g.Cout + li) : (uint32_t)(li * g.Cout + 4 * lk));
  int ph = 0;
  // part p of 8 (forward: two rows of one channel tile; gradient: parts 0, 2, 4, 6 a whole tile) or,
  // p < 0, everything
  auto load_w = [&](floatx4 (&dst)[4], int ks, int p) __attribute__((always_inline)) {
    const int tap = ks >> cch_sh, c0 = ph * PC + (ks - (tap << cch_sh)) * 16;
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      if (p >= 0 && (p >> 1) != jj) continue;
      const int nt = n0 + 16 * ((wave + jj) & 3);
      if (MODE == 0) {
        const char* wb = reinterpret_cast<const char*>(wgt + ((size_t)(tap * g.Cin + c0) * g.Cout + nt));
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          if (p >= 0 && (t >> 1) != (p & 1)) continue;
          // (opaque to the optimizer: the 32-bit offset stays a register operand of the load beside
          // the scalar base instead of being widened to a 64-bit address outside the loop)
          asm volatile("" : "+v"(w_lane[t]));
          dst[jj][t] = *reinterpret_cast<const float*>(wb + w_lane[t]);
        }
      } else {
        // gradient to the input: tap (r', s') of the patch pairs with W[2 - r'][2 - s'][n][c]
        if (p >= 0 && (p & 1) != 0) continue;
        const char* wb = reinterpret_cast<const char*>(wgt + ((size_t)((8 - tap) * g.Cin + nt) * g.Cout + c0));
        asm volatile("" : "+v"(w_lane[0]));
        dst[jj] = *reinterpret_cast<const floatx4*>(wb + w_lane[0]);
      }
    }
  };

  floatx4 acc[4][MT];
#pragma unroll
  for (int jj = 0; jj < 4; ++jj)
#pragma unroll
    for (int i = 0; i < MT; ++i) acc[jj][i] = floatx4{0.f, 0.f, 0.f, 0.f};

  const int c4sh = __builtin_ctz((unsigned)PC) - 2;    // log2 of float4 per pixel and phase
  const int total = HW << c4sh;
  const uint32_t wmagic = 65536u / (unsigned)W + 1u;   // pix / W for pix * W < 65536
  const int nph = Cg / PC;
  // Staging of one phase, in two halves so that the next phase's loads can be in flight during
  // this phase's MFMAs: SU float4 per lane (13 for 14x14x64).  No branch anywhere (a guarded load
  // or store makes the compiler wait for everything in flight): a lane past the end repeats the
  // last item, which rewrites the same value.
  constexpr int SU = (16 * MT * (IMG_PC / 4) + kThreads - 1) / kThreads;
  floatx4 sv[SU];
  auto stage_load = [&](int p) __attribute__((always_inline)) {
    const float* src = in + (size_t)img * HW * Cg + p * PC;
#pragma unroll
    for (int u = 0; u < SU; ++u) {
      const int f = tid + kThreads * u;
      const int fi = f < total ? f : total - 1;
      const int pix = fi >> c4sh, c4 = fi - (pix << c4sh);
      sv[u] = *reinterpret_cast<const floatx4*>(src + (size_t)pix * Cg + 4 * c4);
    }
  };
  auto stage_store = [&](unsigned char* buf) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < SU; ++u) {
      const int f = tid + kThreads * u;
      const int fi = f < total ? f : total - 1;
      const int pix = fi >> c4sh, c4 = fi - (pix << c4sh);
      const int h = (int)(((unsigned)pix * wmagic) >> 16), w = pix - h * W;
      *reinterpret_cast<floatx4*>(buf + ((h + 1) * PW + w + 1) * pitch + c4 * 16) = sv[u];
    }
  };
  stage_load(0);
  stage_store(smem);
  for (ph = 0; ph < nph; ++ph) {
    const unsigned char* cur = smem + (ph & 1) * bufsz;
    unsigned char* nxt = smem + ((ph + 1) & 1) * bufsz;
    const bool more_ph = ph + 1 < nph;
    // two sets of weight registers take turns by k-step; the next k-step's weights are requested in
    // eight parts behind the first eight tiles' MFMAs (every vector instruction between two MFMAs
    // costs the matrix pipe some cycles; a burst of them empties it)
    floatx4 w0[4], w1[4];
    load_w(w0, ks_begin, -1);
    __syncthreads();   // this phase's patch is complete; every wave is done with the other buffer
    // One set of activation fragments, refreshed in place: a tile's fragment of the next k-step
    // is requested as soon as its MFMAs of this k-step have been issued, a whole k-step ahead.
    floatx4 a[MT];
    {
      const int off = a_offset(ks_begin);
#pragma unroll
      for (int i = 0; i < MT; ++i) a[i] = *reinterpret_cast<const floatx4*>(cur + a_base[i] + off);
    }
    auto kstep = [&](const floatx4 (&wc)[4], floatx4 (&wn)[4], int ks) __attribute__((always_inline)) {
      const int kn = ks + 1 < ks_end ? ks + 1 : ks;   // the last k-step asks for its own operands again: no branch
      const int offn = a_offset(kn);
      __builtin_amdgcn_sched_barrier(0);
      // the order below is the schedule
#pragma unroll
      for (int i = 0; i < MT; ++i) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
          for (int jj = 0; jj < 4; ++jj)
            asm volatile("v_mfma_f32_16x16x4_f32 %0, %1, %2, %0" : "+a"(acc[jj][i]) : "v"(wc[jj][t]), "v"(a[i][t]));
        a[i] = *reinterpret_cast<const floatx4*>(cur + a_base[i] + offn);
        constexpr int PP = (8 + MT - 1) / MT;   // parts per tile: all eight within the MT tiles
#pragma unroll
        for (int q = 0; q < PP; ++q)
          if (i * PP + q < 8) load_w(wn, kn, i * PP + q);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    // The next phase's channels are requested behind the first k-step's MFMAs and have the rest
    // of the phase to arrive (the load counter retires in order: requested any earlier, the first
    // k-step's wait for its weights would wait for them too); they go to the other buffer after
    // the last k-step.
    for (int ks = ks_begin; ks < ks_end; ks += 2) {
      kstep(w0, w1, ks);
      if (ks == ks_begin && more_ph) stage_load(ph + 1);
      __builtin_amdgcn_sched_barrier(0);
      if (ks + 1 < ks_end) kstep(w1, w0, ks + 1);
    }
    if (more_ph) stage_store(nxt);
  }

  // the last MFMAs' results are read below by instructions the compiler does not know to depend
  // on a matrix-core result: more wait states than the longest such hazard (18)
  asm volatile("s_nop 15\n\ts_nop 15");
  // ---- the four partial tiles -> one: wave w sends acc[jj], jj = 1..3, to the owner (w + jj) % 4,
  // which adds what it receives in the order jj = 1, 2, 3 of the senders
  __syncthreads();   // every wave has finished reading the image
#pragma unroll
  for (int jj = 1; jj < 4; ++jj) {
    const int owner = (wave + jj) & 3;
    unsigned char* dst = smem + (size_t)((owner * 3 + (jj - 1)) * MT) * 1024 + lane * 16;
#pragma unroll
    for (int i = 0; i < MT; ++i) *reinterpret_cast<floatx4*>(dst + i * 1024) = acc[jj][i];
  }
  __syncthreads();
  const int nch = n0 + 16 * wave + 4 * lk;
  floatx4 v[MT];
  size_t o[MT];   // element offset of the lane's four channels; rows past the image: the last pixel's
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    v[i] = acc[0][i];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const floatx4 t = *reinterpret_cast<const floatx4*>(smem + (size_t)((wave * 3 + q) * MT + i) * 1024 + lane * 16);
      v[i][0] += t[0]; v[i][1] += t[1]; v[i][2] += t[2]; v[i][3] += t[3];
    }
    const int m = 16 * i + li;
    o[i] = ((size_t)img * HW + (m < HW ? m : HW - 1)) * Ng + nch;
  }
  double s1[4] = {0.0, 0.0, 0.0, 0.0}, s2[4] = {0.0, 0.0, 0.0, 0.0};
  if (MODE == 0) {
    if (skip != nullptr) {
      // all the shortcut loads together, none of them guarded
      floatx4 sv[MT];
#pragma unroll
      for (int i = 0; i < MT; ++i) sv[i] = *reinterpret_cast<const floatx4*>(skip + o[i]);
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        v[i][0] += sv[i][0]; v[i][1] += sv[i][1]; v[i][2] += sv[i][2]; v[i][3] += sv[i][3];
      }
    }
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      if (16 * i + li < HW) {
        *reinterpret_cast<floatx4*>(out + o[i]) = v[i];
        if (sums != nullptr) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            s1[r] += (double)v[i][r];
            s2[r] += (double)v[i][r] * (double)v[i][r];
          }
        }
      }
    }
  } else {
    if constexpr (EPI != 0) {
      // Eq. 6-7 from the layer's K-bit codes: the codes of the lane's four channels per pixel
      uint32_t cw[MT];
#pragma unroll
      for (int i = 0; i < MT; ++i)
        cw[i] = EPI == 4 ? (uint32_t) * reinterpret_cast<const uint16_t*>(codes + (o[i] >> 1))
                         : *reinterpret_cast<const uint32_t*>(codes + o[i]);
      const floatx4 st4 = *reinterpret_cast<const floatx4*>(stats + P_STEP * Ng + nch);
      const floatx4 bt4 = *reinterpret_cast<const floatx4*>(stats + P_BETA * Ng + nch);
      const floatx4 gm4 = *reinterpret_cast<const floatx4*>(stats + P_GAMMA * Ng + nch);
      const int4 fb4 = *reinterpret_cast<const int4*>(stats + P_FB * Ng + nch);
      const int32_t fbv[4] = {fb4.x, fb4.y, fb4.z, fb4.w};
      float ig[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) ig[r] = 1.0f / gm4[r];
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        if (16 * i + li < HW) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const uint32_t code = (cw[i] >> (EPI * r)) & ((1u << EPI) - 1u);
            const int32_t j = (int32_t)code - (1 << (EPI - 1)) + fbv[r];
            const float a2t = st4[r] * ((float)j + 0.5f);        // Eq. 10
            const float da2 = a2t > 0.0f ? v[i][r] : 0.0f;       // Eq. 6
            const float a1t = (a2t - bt4[r]) * ig[r];            // inverse of Eq. 2
            s1[r] += (double)da2;
            s2[r] += (double)a1t * (double)da2;
          }
        }
      }
    }
#pragma unroll
    for (int i = 0; i < MT; ++i)
      if (16 * i + li < HW) *reinterpret_cast<floatx4*>(out + o[i]) = v[i];
  }
  if (sums != nullptr && (MODE == 0 || EPI != 0)) {
    // row `img` of [N][2][Ng]: the two sums over the image, added over the 16 pixel lanes
#pragma unroll
    for (int r = 0; r < 4; ++r) {
#pragma unroll
      for (int d = 1; d < 16; d <<= 1) {
        s1[r] += __shfl_xor(s1[r], d, 64);
        s2[r] += __shfl_xor(s2[r], d, 64);
      }
    }
    if (li == 0) {
      double* row = sums + (size_t)img * 2 * Ng;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        row[nch + r] = s1[r];
        row[Ng + nch + r] = s2[r];
      }
    }
  }
}


// Copies of dW that a layer's workspace has had room for on 14-pixel-wide images (tiles of 32 x 64 channels).
constexpr int WG_CI = 32, WG_CO = 64;

int image_wgrad_splits(const ConvGeom& g) {
  const int tiles = (g.Cin / WG_CI) * (g.Cout / WG_CO);
  int s = 256 / tiles;
  if (s > g.N) s = g.N;
  if (s > 16) s = 16;
  return s < 1 ? 1 : s;
}

// ---- weight gradient (first half of Eq. 5) of 1x1 stride-1 layers from the packed codes, bf16 operands ----
// dW[ci][co] = sum over the N H W pixels of A3~[pixel][ci] * dy[pixel][co], A3~ = ReLU of Eq. 10: one matrix
// product whose contraction index is the pixel (v_mfma_f32_16x16x32_bf16: 32 pixels per MFMA, a lane supplies eight
// of them per operand register set).  One block owns a 64 (ci) x 256 (co) tile and a share of the pixels; each wave
// keeps 64 x 64 of it (16 accumulator tiles) in registers.  The rows and columns of an MFMA tile need not be
// neighbouring channels: lane li supplies FOUR input channels (4 li .. 4 li + 3) and FOUR output channels (4 li ..
// 4 li + 3 of the wave's 64), and the 4 x 4 register sets are the 16 MFMAs of a chunk.  Only the dequantized
// activation goes through LDS, shared by the four waves.  Each share of the pixels leaves its own copy of dW,
// summed in a fixed order by the caller's launch.  Both operands are rounded to bf16 by the hardware's packed
// convert, which takes its two inputs from any two registers - so the regrouping from "four channels of one pixel"
// (what a 16-byte load delivers) to "eight pixels of one channel" (what the MFMA wants) costs nothing beyond the
// conversion itself: dy goes from eight 16-byte global loads (the lane's eight pixels) through 16 converts into the
// four operand sets; the activation is dequantized (Eq. 10 with its step, ReLU: the rounded value is that of the
// tiled bf16 kernel), converted in pairs of neighbouring pixels and written to LDS as [pixel group][e][li][8
// pixels], from where a lane's operand set e is one 16-byte read.  dy runs four chunks ahead in a ring of 128 registers.
constexpr int PW_CI = 64, PW_CO = 256, PW_PX = 16;
constexpr int PB_PX = 32;

template <int K>
__global__ __launch_bounds__(kThreads, 1) void rows_wgrad_bf16_kernel(const uint8_t* __restrict__ codes,
                                                                      const float* __restrict__ stats,
                                                                      const float* __restrict__ dy,
                                                                      float* __restrict__ dst, ConvGeom g,
                                                                      int splits) {
  __shared__ __attribute__((aligned(16))) uint32_t AL[2][4][4][16][4];   // [buffer][pixel group][e][li][4 pixel pairs]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lk = lane >> 4;
  const int n_ci = g.Cin / PW_CI, n_co = g.Cout / PW_CO;
  int ci_blk, pair;
  if ((n_co * splits) % 8 == 0) {
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    pair = (slot / n_ci) * 8 + xcd;
    ci_blk = slot % n_ci;
  } else {
    pair = blockIdx.x / n_ci;
    ci_blk = blockIdx.x % n_ci;
  }
  const int co_blk = pair % n_co, split = pair / n_co;
  const int ci0 = ci_blk * PW_CI, co0 = co_blk * PW_CO + 64 * wave;
  const int chunks = (int)(((int64_t)g.N * g.H * g.W) / PB_PX);   // N H W is a multiple of 32
  const int c_begin = (int)((int64_t)split * chunks / splits), c_end = (int)((int64_t)(split + 1) * chunks / splits);

  // ---- staging role: channels ci0 + 4 cg .., pixels 2 q and 2 q + 1 of a chunk (q = 4 wave + lk: wave w
  // stages pixel group w).  Eq. 10 as one add and one multiply: step * (code + offh), offh = fb - 2^(K-1) + 0.5.
  const int cg = tid & 15, q = tid >> 4;
  float stp[4], offh[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int c = ci0 + 4 * cg + e;
    stp[e] = stats[P_STEP * g.Cin + c];
    offh[e] = (float)(reinterpret_cast<const int32_t*>(stats)[P_FB * g.Cin + c] - (1 << (K - 1))) + 0.5f;
  }
  uint32_t c_lane = (uint32_t)((2 * q * g.Cin + ci0 + 4 * cg) * K / 8);
  const size_t c_chunk = (size_t)PB_PX * g.Cin * K / 8;          // bytes of codes per chunk
  const size_t c_pixel = (size_t)g.Cin * K / 8;                   // ... per pixel
  // the four codes of a pixel are 16 or 32 bits; kept in a word of their own size until they are
  // taken apart (widened on arrival they would have to be waited for at the top of the loop)
  using code_t = typename std::conditional<K == 4, uint16_t, uint32_t>::type;
  code_t cw[4][2];                                                // ring of four chunks: [slot][pixel]
  // (a chunk index past the tensor's last one asks for the last one again: never used)
  auto load_codes = [&](code_t (&w)[2], int c) __attribute__((always_inline)) {
    const uint8_t* cb = codes + (size_t)(c < chunks ? c : chunks - 1) * c_chunk;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      asm volatile("" : "+v"(c_lane));
      w[p] = *reinterpret_cast<const code_t*>(cb + p * c_pixel + c_lane);
    }
  };
  auto stage = [&](const code_t (&w)[2], int buf) __attribute__((always_inline)) {
    float v[2][4];
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t code = ((uint32_t)w[p] >> (K * e)) & ((1u << K) - 1u);
        v[p][e] = fmaxf(stp[e] * ((float)code + offh[e]), 0.0f);   // Eq. 10, then the ReLU
      }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const __bf16 lo = (__bf16)v[0][e], hi = (__bf16)v[1][e];
      AL[buf][q >> 2][e][cg][q & 3] = (uint32_t)__builtin_bit_cast(uint16_t, lo) | ((uint32_t)__builtin_bit_cast(uint16_t, hi) << 16);
    }
  };

  // ---- operands.  dy: the lane's pixels are 8 lk .. 8 lk + 7 of the chunk, its channels co0 + 4 li ..
  uint32_t d_lane = 4u * (uint32_t)(8 * lk * g.Cout + co0 + 4 * li);
  const size_t d_chunk = (size_t)PB_PX * g.Cout;                 // floats of dy per chunk
  floatx4 dyr[4][8];                                             // ring of four chunks: [slot][pixel]
  auto load_dy = [&](int slot, int c) __attribute__((always_inline)) {
    const float* db = dy + (size_t)(c < chunks ? c : chunks - 1) * d_chunk;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      asm volatile("" : "+v"(d_lane));
      dyr[slot][i] = *reinterpret_cast<const floatx4*>(reinterpret_cast<const char*>(db + (size_t)i * g.Cout) + d_lane);
    }
  };
  // (one set: the next chunk's fragments are read after this chunk's MFMAs have been issued)
  bf16x8_t af[4];                                                // [e]: eight pixels of channel 4 li + e
  auto read_a = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 4; ++e) af[e] = *reinterpret_cast<const bf16x8_t*>(&AL[buf][lk][e][li][0]);
  };

  floatx4 acc[4][4];   // [e][j]: rows = input channels 4 (4 lk + r) + e, column = output channel 4 li + j
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[e][j] = floatx4{0.f, 0.f, 0.f, 0.f};

  // One chunk, ring slot SLOT (= chunk index mod 4 from the block's first): convert its dy, contract,
  // ask for dy of the chunk four ahead into the slot, dequantize the next chunk into the other buffer
  // and ask for the codes of the chunk four after that one.  One barrier per chunk: the buffer written here was
  // last read in the previous chunk, before that chunk's barrier.
  auto chunk = [&](auto slot_c, int c) __attribute__((always_inline)) {
    constexpr int SLOT = decltype(slot_c)::value, PAR = SLOT & 1;
    // (the fences keep the phases in this order: left alone, the scheduler starts on the code words of
    // later chunks at the top of the loop and waits for every load in flight to get at them)
    __builtin_amdgcn_sched_barrier(0);
    bf16x8_t d[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
      d[j] = bf16x8_t{(__bf16)dyr[SLOT][0][j], (__bf16)dyr[SLOT][1][j], (__bf16)dyr[SLOT][2][j], (__bf16)dyr[SLOT][3][j],
                      (__bf16)dyr[SLOT][4][j], (__bf16)dyr[SLOT][5][j], (__bf16)dyr[SLOT][6][j], (__bf16)dyr[SLOT][7][j]};
    // (the converted operands exist before the slot is asked for again: otherwise the conversions sink
    // below the loads and the old contents of the slot are copied out of their way first)
#pragma unroll
    for (int j = 0; j < 4; ++j) asm volatile("" : "+v"(d[j]));
    __builtin_amdgcn_sched_barrier(0);
    load_dy(SLOT, c + 4);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[e][j]) : "v"(af[e]), "v"(d[j]));
    __builtin_amdgcn_sched_barrier(0);
    stage(cw[(SLOT + 1) & 3], PAR ^ 1);
    __builtin_amdgcn_sched_barrier(0);
    load_codes(cw[(SLOT + 1) & 3], c + 5);
    __syncthreads();
    read_a(PAR ^ 1);
    __builtin_amdgcn_sched_barrier(0);
  };

  if (c_begin < c_end) {
#pragma unroll
    for (int t = 0; t < 4; ++t) load_codes(cw[t], c_begin + t);
#pragma unroll
    for (int t = 0; t < 4; ++t) load_dy(t, c_begin + t);
    stage(cw[0], 0);
    load_codes(cw[0], c_begin + 4);
    __syncthreads();
    read_a(0);
    const int n = c_end - c_begin;
    int i = 0;
    for (; i + 3 < n; i += 4) {
      chunk(std::integral_constant<int, 0>{}, c_begin + i);
      chunk(std::integral_constant<int, 1>{}, c_begin + i + 1);
      chunk(std::integral_constant<int, 2>{}, c_begin + i + 2);
      chunk(std::integral_constant<int, 3>{}, c_begin + i + 3);
    }
    if (i < n) chunk(std::integral_constant<int, 0>{}, c_begin + i);
    if (i + 1 < n) chunk(std::integral_constant<int, 1>{}, c_begin + i + 1);
    if (i + 2 < n) chunk(std::integral_constant<int, 2>{}, c_begin + i + 2);
  }
  // the MFMAs' results are read below by instructions the compiler does not know to depend on a
  // matrix-core result: more wait states than the longest such hazard, tied to the accumulator written last
  asm volatile("s_nop 15\n\ts_nop 15" : "+a"(acc[3][3]));
  float* out = dst + (size_t)split * g.Cin * g.Cout;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int ci = ci0 + 4 * (4 * lk + r);
#pragma unroll
    for (int e = 0; e < 4; ++e)
      *reinterpret_cast<floatx4*>(out + (size_t)(ci + e) * g.Cout + co0 + 4 * li) =
          floatx4{acc[e][0][r], acc[e][1][r], acc[e][2][r], acc[e][3][r]};
  }
}

int rows_wgrad_splits(const ConvGeom& g) {
  const int tiles = (g.Cin / PW_CI) * (g.Cout / PW_CO);
  return tiles <= 256 ? 256 / tiles : 0;
}

int image_mt(const ConvGeom& g) {
  const int tiles = (g.H * g.W + 15) / 16;
  return tiles <= 4 ? 4 : tiles <= 8 ? 8 : tiles <= 13 ? 13 : 0;
}

size_t image_lds_bytes(const ConvGeom& g, int mode) {
  const int Cg = mode == 0 ? g.Cin : g.Cout;
  const int PC = Cg < IMG_PC ? Cg : IMG_PC;
  const size_t patch = (size_t)2 * (g.H + 2) * (g.W + 2) * (4 * PC + 16);
  const size_t red = (size_t)12 * image_mt(g) * 1024;
  return patch > red ? patch : red;
}

template <int MODE, int EPI>
int launch_mt(hipStream_t st, const ConvGeom& g, const float* in, const float* w, const float* skip, float* out,
              double* sums, const uint8_t* codes, const float* stats) {
  const int Ng = MODE == 0 ? g.Cout : g.Cin;
  const int mt = image_mt(g);
  const size_t lds = image_lds_bytes(g, MODE);
  const unsigned grid = (unsigned)((g.N + 7) / 8 * 8 * (Ng / IMG_NB));
  auto kern = mt == 4 ? image_f32_kernel<MODE, 4, EPI> : mt == 8 ? image_f32_kernel<MODE, 8, EPI>
                                                                  : image_f32_kernel<MODE, 13, EPI>;
  if (int e = allow_full_lds(reinterpret_cast<const void*>(kern))) return e;
  kern<<<grid, kThreads, lds, st>>>(in, w, skip, out, sums, codes, stats, g);
  return hip_status();
}

}  // namespace

bool image_f32_supported(const ConvGeom& g, int mode) {
  const int Cg = mode == 0 ? g.Cin : g.Cout, Ng = mode == 0 ? g.Cout : g.Cin;
  if (g.R != 3 || g.S != 3 || g.stride != 1 || g.pad != 1) return false;
  if (Cg < 16 || (Cg < IMG_PC ? (Cg & (Cg - 1)) != 0 : Cg % IMG_PC != 0) || Ng % IMG_NB != 0) return false;
  if (image_mt(g) == 0 || g.N > kMaxPartialBlocks) return false;
  // one block per compute unit and round is what the kernel is built for: with fewer blocks than
  // most of a 256-unit round the tiled kernels are faster (measured: 64 images x 128 channels, 128
  // blocks, 64 us against 44)
  if ((int64_t)g.N * (Ng / IMG_NB) < 224) return false;
  if (image_lds_bytes(g, mode) > (size_t)160 * 1024) return false;
  const int64_t e_in = (int64_t)g.N * g.H * g.W * g.Cin, e_out = (int64_t)g.N * g.Ho * g.Wo * g.Cout;
  return e_in < ((int64_t)1 << 31) && e_out < ((int64_t)1 << 31);
}

int launch_image_f32(hipStream_t st, const ConvGeom& g, int mode, const float* in, const float* w,
                     const float* skip, float* out, double* sums) {
  if (!image_f32_supported(g, mode)) return ABL_ERR_SHAPE;
  if (mode == 0) return launch_mt<0, 0>(st, g, in, w, skip, out, sums, nullptr, nullptr);
  return launch_mt<1, 0>(st, g, in, w, nullptr, out, nullptr, nullptr, nullptr);
}

int launch_image_dgrad_reduce(hipStream_t st, const ConvGeom& g, int K, const float* dy, const float* w,
                              const void* packed, const void* stats, float* da3, double* partial) {
  if (!image_f32_supported(g, 1) || (K != 4 && K != 8)) return ABL_ERR_SHAPE;
  const uint8_t* codes = static_cast<const uint8_t*>(packed);
  const float* sp = static_cast<const float*>(stats);
  if (K == 4) return launch_mt<1, 4>(st, g, dy, w, nullptr, da3, partial, codes, sp);
  return launch_mt<1, 8>(st, g, dy, w, nullptr, da3, partial, codes, sp);
}

int image_wgrad_copies(const ConvGeom& g, int K) {
  if (g.R != 3 || g.S != 3 || g.stride != 1 || g.pad != 1 || (K != 4 && K != 8)) return 0;
  if (g.W != 14 || g.H < 2 || g.H > 14 || (g.H * g.W) % 4 != 0) return 0;
  if (g.Cin % WG_CI != 0 || g.Cout % WG_CO != 0) return 0;
  const int s = image_wgrad_splits(g);
  if ((int64_t)s * (g.Cin / WG_CI) * (g.Cout / WG_CO) < 224) return 0;   // built for one block per compute unit
  const int64_t e_in = (int64_t)g.N * g.H * g.W * g.Cin, e_out = (int64_t)g.N * g.Ho * g.Wo * g.Cout;
  if (e_in >= ((int64_t)1 << 31) || e_out >= ((int64_t)1 << 31)) return 0;
  return s;
}

int rows_wgrad_copies(const ConvGeom& g, int K, bool bf16) {
  if (g.R != 1 || g.S != 1 || g.stride != 1 || g.pad != 0 || (K != 4 && K != 8)) return 0;
  if (g.Cin % PW_CI != 0 || g.Cout % PW_CO != 0) return 0;
  const int64_t M = (int64_t)g.N * g.H * g.W;
  if (M % (bf16 ? PB_PX : PW_PX) != 0) return 0;
  const int s = rows_wgrad_splits(g);
  if ((int64_t)s * (g.Cin / PW_CI) * (g.Cout / PW_CO) < 224) return 0;   // built for one block per compute unit
  if (M / PW_PX < (int64_t)16 * s) return 0;                             // ... with a long share of the pixels each
  if (M * g.Cin >= ((int64_t)1 << 30) || M * g.Cout >= ((int64_t)1 << 30)) return 0;   // 32-bit byte offsets
  return s;
}

int launch_rows_wgrad(hipStream_t st, const ConvGeom& g, int K, const void* packed, const float* stats,
                      const float* dy, float* copies) {
  const int s = rows_wgrad_copies(g, K, true);
  if (s == 0) return ABL_ERR_SHAPE;
  const unsigned grid = (unsigned)(s * (g.Cin / PW_CI) * (g.Cout / PW_CO));
  auto kern = K == 4 ? rows_wgrad_bf16_kernel<4> : rows_wgrad_bf16_kernel<8>;
  kern<<<grid, kThreads, 0, st>>>(static_cast<const uint8_t*>(packed), stats, dy, copies, g, s);
  return hip_status();
}

}  // namespace abl
