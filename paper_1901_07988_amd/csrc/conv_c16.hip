// 3x3 'same' stride-1 layers with 16 input and 16 output channels, fp32 operands split into three bf16 parts (as in
// conv_split.hip): the layers of a CIFAR-sized residual network's first stage.
//
//   c16_fwd_kernel   Eq. 1 (second pass), Eq. 1-3 and Eq. 9 while the patch is staged, Eq. 4, shortcut, first pass of Eq. 1 of y
//   c16_bwd_kernel   Eq. 5 (both gradients) and the first pass of Eq. 6-7; with CHAIN its dy is Eq. 8 of the layer above, second
//                    pass of Eq. 7 included
//
// What bounds a layer of this size (2 million elements) is not a rate but a chain: a dependent launch costs some 4 us whatever it
// does, and inside a kernel the first loads, the staging arithmetic, the contraction and the epilogue follow each other, all
// blocks in step.  So the launches between two convolutions go into the convolutions' first loads (each block sums the 256
// rows of 32 doubles itself: 64 KB from the L2 while the patch is on its way), and the contraction is as short as it gets: two
// taps of 16 channels are one 32-deep step, 30 MFMAs of 16 cycles for 16 pixels where the fp32 instruction took 36 of 32.
// A block of eight waves takes up to 512 pixels, whole rows of one image: one block per compute unit at 128 images of 32x32.
// There (8 MB tensors, a stack of 18 layers, us a layer): forward 12.6, of which first loads with the sums 3, constants 0.7, staging
// 1.8, contraction with epilogue 3.6 (vector instructions 4 and MFMAs 1.6 of them all); before, with fp32 MFMAs, 14.0 + 4.4 for the
// second pass.  Backward 17.4 / 20 (without / with the residual stream's update), before 20.2 + 4.8 + 5.5.  The stack 874 -> 569.
//
// LDS: planes of 16-byte pieces, eight channels of one part of one position; pieces of neighbouring positions are adjacent, so
// that the 16 pixels of a fragment fall on all banks.  The weight gradient, whose contraction index is the pixel, reads the
// same planes with ds_read_b64_tr_b16: 16 lanes fetch four positions' 16 channels and receive one channel's four positions each.
//
// Codes are compared bit for bit with an IEEE fp32 evaluation: this file is compiled with floating-point contraction off.

#include <algorithm>
#include <type_traits>

#include "abl_internal.h"

#pragma clang fp contract(off)

namespace abl {
namespace {

constexpr int kC = 16, kT = 512, kWaves = kT / 64;
constexpr int kPos = 640;                      // positions of a patch at most
constexpr int kPlane = kPos * 16;              // bytes of a plane
constexpr int kOperand = 6 * kPlane;           // three parts, two halves of the channels
constexpr int kWtPart = 20 * 16 * 16;          // weights: [part][10 taps x 2 halves][16 rows] pieces (the tenth tap is zero)
constexpr int kSlots = (2 * kPos + kT - 1) / kT;
constexpr int kPixels = 512;                   // of a tile at most: 4 x kT pieces of four channels

struct C16Plan {
  int H, W, TH, tiles_h, tiles, PW, npos;
  Divisor by_pw, by_w, by_tiles;
};

// Six of the nine products of two split operands (the others are below 2^-24 of it): the large one, the rest.  (Two sums of the
// rest in turn: an MFMA waits for the one before it on the same registers.)
__device__ inline void six(const bf16x8_t (&a)[3], const bf16x8_t (&b)[3], floatx4& big, floatx4& r0, floatx4& r1) {
  r0 = mfma32(a[2], b[0], r0);
  r1 = mfma32(a[0], b[2], r1);
  big = mfma32(a[0], b[0], big);
  r0 = mfma32(a[1], b[1], r0);
  r1 = mfma32(a[1], b[0], r1);
  r0 = mfma32(a[0], b[1], r0);
}

// Totals of `nb` rows of 32 doubles, in a fixed order; `part` is this thread's share, to be asked for early.
struct RowSums {
  double a = 0.0, b = 0.0;
  template <int ROWS>
  __device__ inline void take(const double* __restrict__ rows, int nb) {
    typedef double double2_t __attribute__((ext_vector_type(2)));
    const int first = threadIdx.x >> 4;
    double2_t r[ROWS];
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
      const int i = first + 32 * k;
      r[k] = *reinterpret_cast<const double2_t*>(rows + (i < nb ? i : 0) * 32 + 2 * (threadIdx.x & 15));
    }
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
      a += first + 32 * k < nb ? r[k][0] : 0.0;
      b += first + 32 * k < nb ? r[k][1] : 0.0;
    }
  }
  __device__ inline void load(const double* __restrict__ rows, int nb) {
    if (nb <= 64) take<2>(rows, nb);
    else if (nb <= 128) take<4>(rows, nb);
    else if (nb <= 256) take<8>(rows, nb);
    else take<16>(rows, nb);
  }
  // one row of sums per wave, [wave][32]; total() after a barrier
  __device__ inline void leave(double* sm) {
    a += __shfl_xor(a, 16);
    b += __shfl_xor(b, 16);
    a += __shfl_xor(a, 32);
    b += __shfl_xor(b, 32);
    if ((threadIdx.x & 63) < 16) {
      sm[(threadIdx.x >> 6) * 32 + 2 * (threadIdx.x & 15)] = a;
      sm[(threadIdx.x >> 6) * 32 + 2 * (threadIdx.x & 15) + 1] = b;
    }
  }
  static __device__ inline double total(const double* sm, int v) {
    double t = sm[v];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) t += sm[w * 32 + v];
    return t;
  }
};

// ---- forward --------------------------------------------------------------------------------------------------
struct C16Fwd {
  const float *x, *w, *skip;
  const double* partial;    // nb rows of the statistics' sums, taken around `shift` (nullable); nb = 0: `stats` is there already
  int nb;
  const float *shift, *gamma, *beta;
  float *stats, *y;
  uint8_t* packed;
  int pack_pad;
  double* out_partial;      // nullable: sums of y and y^2, a row per block
  int64_t M;
};

constexpr int kFwdSm = kOperand + 3 * kWtPart, kFwdCst = kFwdSm + kWaves * 32 * 8, kFwdLds = kFwdCst + 8 * kC * 4;

template <int K>
__global__ __launch_bounds__(kT) void c16_fwd_kernel(C16Fwd a, C16Plan p) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  char* const wt = lds + kOperand;
  double* const sm = reinterpret_cast<double*>(lds + kFwdSm);
  float* const cst = reinterpret_cast<float*>(lds + kFwdCst);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, lk = lane >> 4;
  const int img = p.by_tiles.of(blockIdx.x), h0 = ((int)blockIdx.x - img * p.tiles_h) * p.TH;
  const int rows = p.H - h0 < p.TH ? p.H - h0 : p.TH, npix = rows * p.W;
  const int base = (img * p.H + h0) * p.W * kC;   // of the tile's first pixel; its pixels are contiguous

  // the patch: eight channels of a position each
  float4 rx[kSlots][2];
  int at[kSlots];      // element offset, -1 outside the image
  const int half = tid & 1;
#pragma unroll
  for (int j = 0; j < kSlots; ++j) {
    const int pos = (tid + kT * j) >> 1, r = p.by_pw.of(pos), c = pos - r * p.PW;
    const bool ok = pos < p.npos && (unsigned)(h0 + r - 1) < (unsigned)p.H && (unsigned)(c - 1) < (unsigned)p.W;
    at[j] = ok ? base + ((r - 1) * p.W + c - 1) * kC + 8 * half : -1;
    const float4* src = reinterpret_cast<const float4*>(a.x + (ok ? at[j] : 0));
    rx[j][0] = src[0];
    rx[j][1] = src[1];
  }
  // a piece of the weights: output channel row, eight input channels
  float wv[8];
  const int wtap = tid >> 5, wrow = tid & 15, whalf = (tid >> 4) & 1;
#pragma unroll
  for (int e = 0; e < 8; ++e) wv[e] = wtap < 9 ? a.w[(wtap * kC + 8 * whalf + e) * kC + wrow] : 0.0f;
  float gm = 0.f, bt = 0.f, sh = 0.f;
  if (tid < kC && a.nb > 0) {
    gm = a.gamma[tid];
    bt = a.beta[tid];
    sh = a.shift != nullptr ? a.shift[tid] : 0.0f;
  }
  if (a.nb > 0) {
    RowSums s;
    s.load(a.partial, a.nb);
    s.leave(sm);
  } else if (tid < 8 * kC) {
    cst[tid] = a.stats[tid];
  }
  if (tid < 320) {
    bf16x8_t h, m, l;
    split3(wv, h, m, l);
    put(wt + tid * 16, h);
    put(wt + kWtPart + tid * 16, m);
    put(wt + 2 * kWtPart + tid * 16, l);
  }
  __syncthreads();
  if (a.nb > 0) {
    if (tid < kC) {
      float v[8];
      channel_constants(RowSums::total(sm, tid), RowSums::total(sm, kC + tid), sh, a.M, gm, bt, K, v);
#pragma unroll
      for (int i = 0; i < 8; ++i) cst[i * kC + tid] = v[i];
      if (blockIdx.x == 0)
#pragma unroll
        for (int i = 0; i < 8; ++i) a.stats[i * kC + tid] = v[i];
    }
    __syncthreads();
  }
  if (blockIdx.x == 0 && tid < a.pack_pad) a.packed[a.M * kC * K / 8 + tid] = 0;   // the tail of the store

  // Eq. 1-3, Eq. 9
  {
    float mean[8], rstd[8], g8[8], b8[8], cq[8];
    int32_t fb[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int c = 8 * half + e;
      mean[e] = cst[P_MEAN * kC + c];
      rstd[e] = cst[P_RSTD * kC + c];
      g8[e] = cst[P_GAMMA * kC + c];
      b8[e] = cst[P_BETA * kC + c];
      cq[e] = cst[P_CQ * kC + c];
      fb[e] = __float_as_int(cst[P_FB * kC + c]);
    }
#pragma unroll
    for (int j = 0; j < kSlots; ++j) {
      const int idx = tid + kT * j, pos = idx >> 1;
      if (pos >= p.npos) continue;
      const float xs[8] = {rx[j][0].x, rx[j][0].y, rx[j][0].z, rx[j][0].w, rx[j][1].x, rx[j][1].y, rx[j][1].z, rx[j][1].w};
      float v[8];
      uint32_t code[8];
      const bool ok = at[j] >= 0;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float d = xs[e] - mean[e];
        const float a1 = d * rstd[e];           // Eq. 1
        const float t = g8[e] * a1;
        const float a2 = t + b8[e];             // Eq. 2
        v[e] = ok && a2 > 0.0f ? a2 : 0.0f;     // Eq. 3
        code[e] = quant_code<K>(a2, cq[e], fb[e]);
      }
      bf16x8_t h, m, l;
      split3(v, h, m, l);
      char* const to = lds + half * kPlane + pos * 16;
      put(to, h);
      put(to + 2 * kPlane, m);
      put(to + 4 * kPlane, l);
      // the codes of the tile's own pixels
      if (ok && at[j] >= base && at[j] < base + npix * kC) {
        if constexpr (K == 4) {
          uint32_t word = 0;
#pragma unroll
          for (int e = 0; e < 8; ++e) word |= code[e] << (4 * e);
          *reinterpret_cast<uint32_t*>(a.packed + (at[j] >> 1)) = word;
        } else {
          uint2 word = make_uint2(0u, 0u);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            word.x |= code[e] << (8 * e);
            word.y |= code[4 + e] << (8 * e);
          }
          *reinterpret_cast<uint2*>(a.packed + at[j]) = word;
        }
      }
    }
  }
  __syncthreads();

  // ---- Eq. 4: 16 pixels at a time, D[output channel][pixel]; a lane holds four channels of one pixel ----
  bf16x8_t wf[5][3];
  int off[5];           // of the lane's operand of a step from its pixel's first tap
#pragma unroll
  for (int s = 0; s < 5; ++s) {
#pragma unroll
    for (int q = 0; q < 3; ++q) wf[s][q] = piece(wt + q * kWtPart + (s * 64 + lane) * 16);
    const int tap = 2 * s + (lk >> 1) < 9 ? 2 * s + (lk >> 1) : 8;   // (the tenth tap's weights are zero)
    off[s] = ((tap / 3) * p.PW + tap % 3) * 16 + (lk & 1) * kPlane;
  }
  double s1[4] = {0.0, 0.0, 0.0, 0.0}, s2[4] = {0.0, 0.0, 0.0, 0.0};
  const int ntile = (npix + 15) / 16;
  struct Tile {
    bf16x8_t f[5][3];
    float4 sk;
  };
  auto fetch = [&](int i, Tile& t) __attribute__((always_inline)) {
    const int m = 16 * i + li, mc = m < npix ? m : 0;
    const int h = p.by_w.of(mc);
    const char* const src = lds + (h * p.PW + mc - h * p.W) * 16;
    t.sk = make_float4(0.f, 0.f, 0.f, 0.f);
    if (a.skip != nullptr) t.sk = *reinterpret_cast<const float4*>(a.skip + base + mc * kC + 4 * lk);
#pragma unroll
    for (int s = 0; s < 5; ++s)
#pragma unroll
      for (int q = 0; q < 3; ++q) t.f[s][q] = piece(src + off[s] + 2 * q * kPlane);
  };
  auto store = [&](int m, const float (&o)[4], const float4& sk) __attribute__((always_inline)) {
    const float v[4] = {o[0] + sk.x, o[1] + sk.y, o[2] + sk.z, o[3] + sk.w};
    *reinterpret_cast<float4*>(a.y + base + m * kC + 4 * lk) = make_float4(v[0], v[1], v[2], v[3]);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      s1[r] += (double)v[r];
      s2[r] += (double)v[r] * (double)v[r];
    }
  };
  uint32_t again = 0;   // tiles with values beyond what the parts carry
  auto finish = [&](int i, const Tile& t) __attribute__((always_inline)) {
    const int m = 16 * i + li;
    floatx4 big = {0.f, 0.f, 0.f, 0.f}, rest = big, more = big;
#pragma unroll
    for (int s = 0; s < 5; ++s) six(wf[s], t.f[s], big, s % 2 == 0 ? rest : more, s % 2 == 0 ? more : rest);
    float o[4];
    bool fine = true;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      o[r] = (big[r] + (rest[r] + more[r])) * kDown;
      fine = fine && finite(o[r]);
    }
    if (__any(!fine)) again |= 1u << (i / kWaves);
    else if (m < npix) store(m, o, t.sk);
  };
  {
    // (the next tile's operands are read in front of this one's MFMAs)
    Tile one, two;
    fetch(wave, one);
#pragma unroll 1
    for (int i = wave; i < ntile; i += 2 * kWaves) {
      fetch(i + kWaves, two);
      finish(i, one);
      if (i + kWaves >= ntile) break;
      fetch(i + 2 * kWaves, one);
      finish(i + kWaves, two);
    }
  }
#pragma unroll 1
  for (int i = wave; again != 0; i += kWaves, again >>= 1) {   // from the fp32 operands
    const int m = 16 * i + li;
    if ((again & 1u) == 0 || m >= npix) continue;
    const int h = p.by_w.of(m), wq = m - h * p.W;
    float o[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int tap = 0; tap < 9; ++tap) {
      const int ih = h0 + h + tap / 3 - 1, iw = wq + tap % 3 - 1;
      const bool in = (unsigned)ih < (unsigned)p.H && (unsigned)iw < (unsigned)p.W;   // (zeros outside take part, as in the patch)
#pragma unroll 1
      for (int c = 0; c < kC; ++c) {
        const float d = (in ? a.x[((img * p.H + ih) * p.W + iw) * kC + c] : 0.0f) - cst[P_MEAN * kC + c];
        const float a1 = d * cst[P_RSTD * kC + c];
        const float u = cst[P_GAMMA * kC + c] * a1;
        const float a2 = u + cst[P_BETA * kC + c];
#pragma unroll
        for (int r = 0; r < 4; ++r) o[r] = __builtin_fmaf(in && a2 > 0.0f ? a2 : 0.0f, a.w[(tap * kC + c) * kC + 4 * lk + r], o[r]);
      }
    }
    float4 sk = make_float4(0.f, 0.f, 0.f, 0.f);
    if (a.skip != nullptr) sk = *reinterpret_cast<const float4*>(a.skip + base + m * kC + 4 * lk);
    store(m, o, sk);
  }
  if (a.out_partial == nullptr) return;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const double u1 = row16_sum(s1[r]), u2 = row16_sum(s2[r]);
    if (li == 0) {
      sm[wave * 32 + 4 * lk + r] = u1;
      sm[wave * 32 + kC + 4 * lk + r] = u2;
    }
  }
  __syncthreads();
  if (tid < 32) a.out_partial[(int64_t)blockIdx.x * 32 + tid] = RowSums::total(sm, tid);
}

// ---- backward -------------------------------------------------------------------------------------------------
// Eq. 8 of a layer, from its dA3, codes, statistics and the means of Eq. 8.
struct C16Apply {
  const float* da3;
  const uint8_t* packed;
  const float *stats, *means;
};
struct C16Bwd {
  const float *dy, *w;          // CHAIN: dy = nullptr
  const uint8_t* packed;
  const float* stats;
  float* da3;
  double* partial;              // a row of the Eq. 6-7 sums per block
  float* wpartial;              // a copy of dW per block
  // CHAIN: dy = Eq. 8 of the layer above (+ add), whose second pass of Eq. 7 and whose sum of dW's copies are done here
  C16Apply up;                  // (up.means is written)
  float* up_means;
  const double* up_partial;
  int up_nb;
  float *up_dgamma, *up_dbeta;
  const float* add;             // nullable
  const float* up_wpartial;
  int up_copies;
  float* up_dw;
  // s += Eq. 8 of the first layer of the group above, on the block's own pixels (nullable)
  C16Apply res;
  float* s;
  int64_t M;
};

constexpr int kBwdWt = 2 * kOperand, kBwdSm = kBwdWt + 3 * kWtPart, kBwdTot = kBwdSm + kWaves * 32 * 8, kBwdCst = kBwdTot + 32 * 8,
              kBwdWs = kBwdCst + 24 * kC * 4, kBwdLds = kBwdWs + kWaves * 16 * 4;
static_assert(kWaves * 9 * 256 * 4 <= 2 * kOperand, "the waves' sums of dW take the patches' place");
static_assert(kBwdLds <= 160 * 1024, "LDS of a compute unit");

template <int K>
__device__ inline float eq8(float g, uint32_t q, float step, int32_t fb, float bt, float gm, float ig, float rstd, float m1, float m2) {
  const float a2t = dequant<K>(q, step, fb);
  const float da2 = a2t > 0.0f ? g : 0.0f;                 // Eq. 6
  const float a1t = (a2t - bt) * ig;
  const float da1 = gm * da2;                              // Eq. 7
  const float t = (da1 - m1) - a1t * m2;
  return rstd * t;                                         // Eq. 8
}
// codes of channels c0 .. c0 + 7 or + 3 of the element with offset e (a multiple of 8, of 4)
template <int K>
__device__ inline uint2 codes8(const uint8_t* p, int e) {
  if constexpr (K == 4) return make_uint2(*reinterpret_cast<const uint32_t*>(p + (e >> 1)), 0u);
  else return *reinterpret_cast<const uint2*>(p + e);
}
template <int K>
__device__ inline uint32_t code_of(const uint2& w, int e) {
  if constexpr (K == 4) return (w.x >> (4 * e)) & 15u;
  else return ((e < 4 ? w.x : w.y) >> (8 * (e & 3))) & 255u;
}
template <int K>
__device__ inline uint32_t code_at(const uint8_t* p, int e) {
  if constexpr (K == 4) return (p[e >> 1] >> (4 * (e & 1))) & 15u;
  else return p[e];
}

// Constants in LDS, [row][16]: of the layer above (rows 0-7), of the layer itself (8-13), of Eq. 8 for s (16-23).
enum CstRow { U_STEP = 0, U_FB, U_BETA, U_GAMMA, U_IG, U_RSTD, U_M1, U_M2, L_STEP, L_FB, L_BETA, L_IG, R_FIRST = 16 };

template <int K, bool CHAIN>
__global__ __launch_bounds__(kT) void c16_bwd_kernel(C16Bwd a, C16Plan p) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  char* const act = lds + kOperand;
  char* const wt = lds + kBwdWt;
  double* const sm = reinterpret_cast<double*>(lds + kBwdSm);
  float* const cst = reinterpret_cast<float*>(lds + kBwdCst);
  float* const ws = reinterpret_cast<float*>(lds + kBwdWs);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, lk = lane >> 4;
  const int img = p.by_tiles.of(blockIdx.x), h0 = ((int)blockIdx.x - img * p.tiles_h) * p.TH;
  const int rows = p.H - h0 < p.TH ? p.H - h0 : p.TH, npix = rows * p.W;
  const int base = (img * p.H + h0) * p.W * kC;
  const float* const grad = CHAIN ? a.up.da3 : a.dy;

  float4 rg[kSlots][2], ra[CHAIN ? kSlots : 1][2];
  uint2 rc[kSlots], ru[CHAIN ? kSlots : 1];
  int at[kSlots];
  const int half = tid & 1;
#pragma unroll
  for (int j = 0; j < kSlots; ++j) {
    const int pos = (tid + kT * j) >> 1, r = p.by_pw.of(pos), c = pos - r * p.PW;
    const bool ok = pos < p.npos && (unsigned)(h0 + r - 1) < (unsigned)p.H && (unsigned)(c - 1) < (unsigned)p.W;
    at[j] = ok ? base + ((r - 1) * p.W + c - 1) * kC + 8 * half : -1;
    const int e = ok ? at[j] : 0;
    const float4* src = reinterpret_cast<const float4*>(grad + e);
    rg[j][0] = src[0];
    rg[j][1] = src[1];
    rc[j] = codes8<K>(a.packed, e);
    if constexpr (CHAIN) {
      ru[j] = codes8<K>(a.up.packed, e);
      if (a.add != nullptr) {
        const float4* sa = reinterpret_cast<const float4*>(a.add + e);
        ra[j][0] = sa[0];
        ra[j][1] = sa[1];
      }
    }
  }
  // the residual stream's own pixels (C16Bwd::s)
  float4 xg[CHAIN ? 4 : 1], xs[CHAIN ? 4 : 1];
  uint32_t xc[CHAIN ? 4 : 1];
  if constexpr (CHAIN)
    if (a.s != nullptr)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int i = tid + kT * j, e = base + (i < npix * 4 ? 4 * i : 0);
        xg[j] = *reinterpret_cast<const float4*>(a.res.da3 + e);
        xs[j] = *reinterpret_cast<const float4*>(a.s + e);
        if constexpr (K == 4) xc[j] = *reinterpret_cast<const uint16_t*>(a.res.packed + (e >> 1));
        else xc[j] = *reinterpret_cast<const uint32_t*>(a.res.packed + e);
      }
  // a piece of the weights: input channel row, eight output channels
  float wv[8];
  const int wtap = tid >> 5, wrow = tid & 15, whalf = (tid >> 4) & 1;
  {
    const float4* src = reinterpret_cast<const float4*>(a.w + ((wtap < 9 ? wtap : 0) * kC + wrow) * kC + 8 * whalf);
    const float4 u = src[0], v = src[1];
    const float z[8] = {u.x, u.y, u.z, u.w, v.x, v.y, v.z, v.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) wv[e] = wtap < 9 ? z[e] : 0.0f;
  }
  // constants: thread = (row of 16 threads, channel)
  if (tid < kC) {
    cst[L_STEP * kC + tid] = a.stats[P_STEP * kC + tid];
    cst[L_FB * kC + tid] = a.stats[P_FB * kC + tid];
    cst[L_BETA * kC + tid] = a.stats[P_BETA * kC + tid];
    cst[L_IG * kC + tid] = 1.0f / a.stats[P_GAMMA * kC + tid];
  }
  if constexpr (CHAIN) {
    auto consts = [&](const float* st, int row, int c) __attribute__((always_inline)) {
      cst[(row + U_STEP) * kC + c] = st[P_STEP * kC + c];
      cst[(row + U_FB) * kC + c] = st[P_FB * kC + c];
      cst[(row + U_BETA) * kC + c] = st[P_BETA * kC + c];
      const float g = st[P_GAMMA * kC + c];
      cst[(row + U_GAMMA) * kC + c] = g;
      cst[(row + U_IG) * kC + c] = 1.0f / g;
      cst[(row + U_RSTD) * kC + c] = st[P_RSTD * kC + c];
    };
    if (tid >= 64 && tid < 64 + kC) consts(a.up.stats, 0, tid - 64);
    if (a.s != nullptr && tid >= 128 && tid < 128 + kC) {
      const int c = tid - 128;
      consts(a.res.stats, R_FIRST, c);
      cst[(R_FIRST + U_M1) * kC + c] = a.res.means[c];
      cst[(R_FIRST + U_M2) * kC + c] = a.res.means[kC + c];
    }
    RowSums s;
    s.load(a.up_partial, a.up_nb);
    s.leave(sm);
    // copies of the layer above's dW: 16 of its elements a block
    for (int o = blockIdx.x; o < 144; o += gridDim.x) {
      const float4* src = reinterpret_cast<const float4*>(a.up_wpartial + 16 * o) + (tid & 3);
      float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
      for (int k = tid >> 2; k < a.up_copies; k += kT / 4) {
        const float4 v = src[(int64_t)k * (2304 / 4)];
        t.x += v.x; t.y += v.y; t.z += v.z; t.w += v.w;
      }
#pragma unroll
      for (int d = 4; d < 64; d <<= 1) {
        t.x += __shfl_xor(t.x, d); t.y += __shfl_xor(t.y, d); t.z += __shfl_xor(t.z, d); t.w += __shfl_xor(t.w, d);
      }
      if (lane < 4) *reinterpret_cast<float4*>(ws + wave * 16 + 4 * lane) = t;
      __syncthreads();
      if (tid < 16) {
        float u = ws[tid];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) u += ws[w * 16 + tid];
        a.up_dw[16 * o + tid] = u;
      }
      __syncthreads();
    }
  }
  if (tid < 320) {
    bf16x8_t h, m, l;
    split3(wv, h, m, l);
    put(wt + tid * 16, h);
    put(wt + kWtPart + tid * 16, m);
    put(wt + 2 * kWtPart + tid * 16, l);
  }
  __syncthreads();
  if constexpr (CHAIN) {
    if (tid < kC) {
      const double t0 = RowSums::total(sm, tid), t1 = RowSums::total(sm, kC + tid);
      const double g = (double)cst[U_GAMMA * kC + tid];
      const float m1 = (float)(g * t0 / (double)a.M), m2 = (float)(g * t1 / (double)a.M);
      cst[U_M1 * kC + tid] = m1;
      cst[U_M2 * kC + tid] = m2;
      if (blockIdx.x == 0) {
        a.up_dbeta[tid] = (float)t0;
        a.up_dgamma[tid] = (float)t1;
        a.up_means[tid] = m1;
        a.up_means[kC + tid] = m2;
      }
    }
    __syncthreads();
    // the residual stream's gradient, of the block's own pixels (before their dA3 is overwritten)
    if (a.s != nullptr) {
      const int c0 = 4 * (tid & 3);
      const float* const rc0 = cst + R_FIRST * kC + c0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int i = tid + kT * j, e = base + 4 * i;
        if (i >= npix * 4) continue;
        const float4 g = xg[j], s0 = xs[j];
        const uint32_t w = xc[j];
        const float gv[4] = {g.x, g.y, g.z, g.w}, sv[4] = {s0.x, s0.y, s0.z, s0.w};
        float o[4];
#pragma unroll
        for (int v = 0; v < 4; ++v)
          o[v] = sv[v] + eq8<K>(gv[v], (w >> (K * v)) & ((1u << K) - 1u), rc0[U_STEP * kC + v], __float_as_int(rc0[U_FB * kC + v]),
                                rc0[U_BETA * kC + v], rc0[U_GAMMA * kC + v], rc0[U_IG * kC + v], rc0[U_RSTD * kC + v],
                                rc0[U_M1 * kC + v], rc0[U_M2 * kC + v]);
        *reinterpret_cast<float4*>(a.s + e) = make_float4(o[0], o[1], o[2], o[3]);
      }
    }
  }

  // Whether the whole numbers 2 t (Eq. 10 is step t) of all positive activations are exact in one bf16.
  bool narrow;
  {
    const int32_t fb = __float_as_int(cst[L_FB * kC + li]);
    const int32_t top = (1 << K) - 1 + 2 * (cst[L_STEP * kC + li] > 0.0f ? fb : -fb);
    narrow = __all(top <= 256) != 0;
  }

  // ---- staging: dy in three parts, 2 t of the positive activations in one or three ----
  {
    float st8[8];
    int32_t fb8[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      st8[e] = cst[L_STEP * kC + 8 * half + e];
      fb8[e] = __float_as_int(cst[L_FB * kC + 8 * half + e]);
    }
#pragma unroll
    for (int j = 0; j < kSlots; ++j) {
      const int pos = (tid + kT * j) >> 1;
      if (pos >= p.npos) continue;
      const bool ok = at[j] >= 0;
      const float gs[8] = {rg[j][0].x, rg[j][0].y, rg[j][0].z, rg[j][0].w, rg[j][1].x, rg[j][1].y, rg[j][1].z, rg[j][1].w};
      float v[8], t2[8];
      if constexpr (CHAIN) {
        const float* const uc = cst + 8 * half;
#pragma unroll
        for (int e = 0; e < 8; ++e)
          v[e] = eq8<K>(gs[e], code_of<K>(ru[j], e), uc[U_STEP * kC + e], __float_as_int(uc[U_FB * kC + e]), uc[U_BETA * kC + e],
                        uc[U_GAMMA * kC + e], uc[U_IG * kC + e], uc[U_RSTD * kC + e], uc[U_M1 * kC + e], uc[U_M2 * kC + e]);
        if (a.add != nullptr) {
          const float as[8] = {ra[j][0].x, ra[j][0].y, ra[j][0].z, ra[j][0].w, ra[j][1].x, ra[j][1].y, ra[j][1].z, ra[j][1].w};
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] = as[e] + v[e];
        }
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = gs[e];
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        v[e] = ok ? v[e] : 0.0f;
        const int32_t q = (int32_t)code_of<K>(rc[j], e) - (1 << (K - 1)) + fb8[e];
        const float t = (float)q + 0.5f;
        t2[e] = ok && st8[e] * t > 0.0f ? t + t : 0.0f;     // Eq. 10, Eq. 3
      }
      bf16x8_t h, m, l;
      split3<false>(v, h, m, l);   // (the channels of a pixel are columns of dW)
      char* const to = lds + half * kPlane + pos * 16;
      put(to, h);
      put(to + 2 * kPlane, m);
      put(to + 4 * kPlane, l);
      if (narrow) {
        put(to + kOperand, to_bf16x8(t2));
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) t2[e] *= kDown * kUp;    // (split3 takes 2^23 times its argument)
        split3<false>(t2, h, m, l);
        put(to + kOperand, h);
        put(to + kOperand + 2 * kPlane, m);
        put(to + kOperand + 4 * kPlane, l);
      }
    }
  }
  __syncthreads();

  // dy of one element from memory, for what the parts do not carry
  auto dy_at = [&](int e, int c) __attribute__((always_inline)) -> float {
    if constexpr (!CHAIN) return a.dy[e + c];
    const float d = eq8<K>(a.up.da3[e + c], code_at<K>(a.up.packed, e + c), cst[U_STEP * kC + c], __float_as_int(cst[U_FB * kC + c]),
                           cst[U_BETA * kC + c], cst[U_GAMMA * kC + c], cst[U_IG * kC + c], cst[U_RSTD * kC + c],
                           cst[U_M1 * kC + c], cst[U_M2 * kC + c]);
    return a.add != nullptr ? a.add[e + c] + d : d;
  };
  // 2 t of four channels 4 lk .. of a position, as staged
  auto act4 = [&](int pos, float (&t2)[4]) __attribute__((always_inline)) {
    const char* const src = act + (lk >> 1) * kPlane + pos * 16 + (lk & 1) * 8;
    auto four = [&](const char* q, int r) { return __uint_as_float((uint32_t)reinterpret_cast<const uint16_t*>(q)[r] << 16); };
#pragma unroll
    for (int r = 0; r < 4; ++r) t2[r] = four(src, r);
    if (!narrow)
#pragma unroll
      for (int r = 0; r < 4; ++r) t2[r] = (t2[r] + four(src + 2 * kPlane, r)) + four(src + 4 * kPlane, r);
  };

  // ---- Eq. 5, gradient to the input: D[input channel][pixel] ----
  {
    bf16x8_t wf[5][3];
    int off[5];
#pragma unroll
    for (int s = 0; s < 5; ++s) {
#pragma unroll
      for (int q = 0; q < 3; ++q) wf[s][q] = piece(wt + q * kWtPart + (s * 64 + lane) * 16);
      const int tap = 2 * s + (lk >> 1) < 9 ? 2 * s + (lk >> 1) : 8;
      off[s] = ((2 - tap / 3) * p.PW + 2 - tap % 3) * 16 + (lk & 1) * kPlane;
    }
    float st4[4], bt4[4], ig4[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      st4[r] = cst[L_STEP * kC + 4 * lk + r];
      bt4[r] = cst[L_BETA * kC + 4 * lk + r];
      ig4[r] = cst[L_IG * kC + 4 * lk + r];
    }
    double s1[4] = {0.0, 0.0, 0.0, 0.0}, s2[4] = {0.0, 0.0, 0.0, 0.0};
    const int ntile = (npix + 15) / 16;
    struct Tile {
      bf16x8_t f[5][3];
      float t2[4];
    };
    auto fetch = [&](int i, Tile& t) __attribute__((always_inline)) {
      const int m = 16 * i + li, mc = m < npix ? m : 0;
      const int h = p.by_w.of(mc), pos = h * p.PW + mc - h * p.W;
      const char* const src = lds + pos * 16;
#pragma unroll
      for (int s = 0; s < 5; ++s)
#pragma unroll
        for (int q = 0; q < 3; ++q) t.f[s][q] = piece(src + off[s] + 2 * q * kPlane);
      act4(pos + p.PW + 1, t.t2);
    };
    auto store = [&](int m, const float (&o)[4], const float (&t2)[4]) __attribute__((always_inline)) {
      *reinterpret_cast<float4*>(a.da3 + base + m * kC + 4 * lk) = make_float4(o[0], o[1], o[2], o[3]);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float a3t = st4[r] * (0.5f * t2[r]);
        const float da2 = a3t > 0.0f ? o[r] : 0.0f;               // Eq. 6
        const float a1t = (a3t - bt4[r]) * ig4[r];                // inverse of Eq. 2
        s1[r] += (double)da2;
        s2[r] += (double)a1t * (double)da2;
      }
    };
    uint32_t again = 0;
    auto finish = [&](int i, const Tile& t) __attribute__((always_inline)) {
      const int m = 16 * i + li;
      floatx4 big = {0.f, 0.f, 0.f, 0.f}, rest = big, more = big;
#pragma unroll
      for (int s = 0; s < 5; ++s) six(wf[s], t.f[s], big, s % 2 == 0 ? rest : more, s % 2 == 0 ? more : rest);
      float o[4];
      bool fine = true;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        o[r] = (big[r] + (rest[r] + more[r])) * kDown;
        fine = fine && finite(o[r]);
      }
      if (__any(!fine)) again |= 1u << (i / kWaves);
      else if (m < npix) store(m, o, t.t2);
    };
    {
      Tile one, two;
      fetch(wave, one);
#pragma unroll 1
      for (int i = wave; i < ntile; i += 2 * kWaves) {
        fetch(i + kWaves, two);
        finish(i, one);
        if (i + kWaves >= ntile) break;
        fetch(i + 2 * kWaves, one);
        finish(i + kWaves, two);
      }
    }
#pragma unroll 1
    for (int i = wave; again != 0; i += kWaves, again >>= 1) {
      const int m = 16 * i + li;
      if ((again & 1u) == 0 || m >= npix) continue;
      const int h = p.by_w.of(m), wq = m - h * p.W;
      float o[4] = {0.f, 0.f, 0.f, 0.f}, t2[4];
#pragma unroll 1
      for (int tap = 0; tap < 9; ++tap) {
        const int ih = h0 + h + 1 - tap / 3, iw = wq + 1 - tap % 3;
        const bool in = (unsigned)ih < (unsigned)p.H && (unsigned)iw < (unsigned)p.W;
#pragma unroll 1
        for (int c = 0; c < kC; ++c) {
          const float d = in ? dy_at(((img * p.H + ih) * p.W + iw) * kC, c) : 0.0f;
#pragma unroll
          for (int r = 0; r < 4; ++r) o[r] = __builtin_fmaf(d, a.w[(tap * kC + 4 * lk + r) * kC + c], o[r]);
        }
      }
      act4(h * p.PW + wq + p.PW + 1, t2);
      store(m, o, t2);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double u1 = row16_sum(s1[r]), u2 = row16_sum(s2[r]);
      if (li == 0) {
        sm[wave * 32 + 4 * lk + r] = u1;
        sm[wave * 32 + kC + 4 * lk + r] = u2;
      }
    }
  }

  // ---- Eq. 5, weight gradient: D[input channel][output channel], 32 pixels a step ----
  floatx4 wb[9], wr[9];
#pragma unroll
  for (int t = 0; t < 9; ++t) wb[t] = wr[t] = floatx4{0.f, 0.f, 0.f, 0.f};
  {
    const int chunk = ((li >> 1) & 1) * kPlane + (li & 1) * 8;   // this lane's eight bytes of a position's 16 channels
    const int nstep = (npix + 31) / 32;
    auto contract = [&](auto wide) __attribute__((always_inline)) {
#pragma unroll 1
      for (int s = wave; s < nstep; s += kWaves) {
        int from[2], apart[2];
        const char* z[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int m = 32 * s + 8 * lk + 4 * j + (li >> 2), mc = m < npix ? m : 0;
          const int h = p.by_w.of(mc), pos = h * p.PW + mc - h * p.W;
          from[j] = chunk + pos * 16;
          // (pixels past the tile's end: the weights' tenth tap, zeros)
          z[j] = m < npix ? lds + from[j] + (p.PW + 1) * 16 : wt + 288 * 16;
          apart[j] = m < npix ? 2 * kPlane : 0;
        }
        bf16x8_t g[3], x[9];
#pragma unroll
        for (int q = 0; q < 3; ++q) g[q] = transposed(z[0] + q * apart[0], z[1] + q * apart[1]);
        auto taps = [&](int part) __attribute__((always_inline)) {
#pragma unroll
          for (int t = 0; t < 9; ++t) {
            const int o = ((t / 3) * p.PW + t % 3) * 16 + 2 * part * kPlane;
            x[t] = transposed(act + from[0] + o, act + from[1] + o);
          }
        };
        taps(0);
#pragma unroll
        for (int t = 0; t < 9; ++t) wb[t] = mfma32(x[t], g[0], wb[t]);
#pragma unroll
        for (int q = 2; q > 0; --q)
#pragma unroll
          for (int t = 0; t < 9; ++t) wr[t] = mfma32(x[t], g[q], wr[t]);
        if constexpr (decltype(wide)::value) {
          taps(1);
#pragma unroll
          for (int q = 1; q >= 0; --q)
#pragma unroll
            for (int t = 0; t < 9; ++t) wr[t] = mfma32(x[t], g[q], wr[t]);
          taps(2);
#pragma unroll
          for (int t = 0; t < 9; ++t) wr[t] = mfma32(x[t], g[0], wr[t]);
        }
      }
    };
    if (narrow) contract(std::false_type{});
    else contract(std::true_type{});
  }
  __syncthreads();   // every wave is done with the patches
  float* const wred = reinterpret_cast<float*>(lds);
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) wred[(wave * 9 + t) * 256 + (4 * lk + r) * kC + li] = wb[t][r] + wr[t][r];
  if (tid < 32) a.partial[(int64_t)blockIdx.x * 32 + tid] = RowSums::total(sm, tid);
  __syncthreads();
  float* const dst = a.wpartial + (int64_t)blockIdx.x * 2304;
  for (int i = tid; i < 2304; i += kT) {
    float t = wred[i];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) t += wred[w * 2304 + i];
    const int c = (i >> 4) & 15;
    t = (t * 0x1p-24f) * cst[L_STEP * kC + c];   // 2^23 dy, 2 t
    if (!finite(t)) {
      const int tap = i >> 8, co = i & 15;
      t = 0.f;
#pragma unroll 1
      for (int m = 0; m < npix; ++m) {
        const int h = p.by_w.of(m), ih = h0 + h + tap / 3 - 1, iw = m - h * p.W + tap % 3 - 1;
        const bool in = (unsigned)ih < (unsigned)p.H && (unsigned)iw < (unsigned)p.W;
        const float a2t = in ? dequant<K>(code_at<K>(a.packed, ((img * p.H + ih) * p.W + iw) * kC + c), cst[L_STEP * kC + c],
                                          __float_as_int(cst[L_FB * kC + c]))
                             : 0.0f;
        t = __builtin_fmaf(a2t > 0.0f ? a2t : 0.0f, dy_at(base + m * kC, co), t);
      }
    }
    dst[i] = t;
  }
}

// Tiles of whole rows.  The chip takes 256 blocks at a time, and what a block does besides its rows is worth about ten of them; a
// row of sums each, at most `limit` blocks.  (Narrow tiles of very wide images would be mostly border.)
bool make_plan(const ConvGeom& g, int64_t limit, C16Plan& p) {
  if (g.R != 3 || g.S != 3 || g.stride != 1 || g.pad != 1 || g.Cin != kC || g.Cout != kC) return false;
  const int most = std::min(kPixels / g.W, kPos / (g.W + 2) - 2);
  if (most < 1 || (most < 6 && most < g.H)) return false;
  int64_t best = -1;
  for (int t = (g.H + most - 1) / most; t <= g.H; ++t) {
    const int64_t blocks = (int64_t)g.N * t;
    if (blocks > limit) break;
    const int th = (g.H + t - 1) / t;
    if ((g.H + th - 1) / th != t) continue;
    const int64_t cost = (blocks + 255) / 256 * (10 + th);
    if (best >= 0 && cost >= best) continue;
    best = cost;
    p.TH = th;
    p.tiles_h = t;
  }
  if (best < 0) return false;
  p.H = g.H;
  p.W = g.W;
  p.tiles = g.N * p.tiles_h;
  p.PW = g.W + 2;
  p.npos = (p.TH + 2) * p.PW;
  p.by_pw = Divisor(p.PW);
  p.by_w = Divisor(g.W);
  p.by_tiles = Divisor(p.tiles_h);
  return true;
}

// (the copies of dW have room for so many blocks)
bool make_plan(const ConvGeom& g, C16Plan& p) {
  const size_t room = halo_wgrad_partial_bytes(g) / (2304 * sizeof(float));
  return make_plan(g, (int64_t)std::min(room, (size_t)kMaxPartialBlocks), p);
}

}  // namespace

int c16_tiles(const ConvGeom& g, int mode) {
  C16Plan p;
  if (g.Cin != kC) return 0;
  return (mode == 0 ? make_plan(g, kMaxPartialBlocks, p) : make_plan(g, p)) ? p.tiles : 0;
}

int launch_c16_fwd(hipStream_t st, const ConvGeom& g, int K, const float* x, const float* w, const double* partial, int nb,
                   const float* shift, const float* gamma, const float* beta, void* stats, const float* skip, float* y, void* packed,
                   double* out_partial) {
  C16Plan p;
  if (!make_plan(g, kMaxPartialBlocks, p)) return ABL_ERR_SHAPE;
  if (nb > 0 && partial == out_partial) return ABL_ERR_ARG;   // (a block reads all rows and leaves its own before others begin)
  const int64_t M = (int64_t)g.N * g.H * g.W, raw = M * kC * K / 8;
  const C16Fwd a{x, w, skip, partial, nb, shift, gamma, beta, static_cast<float*>(stats), y, static_cast<uint8_t*>(packed),
                 (int)((raw + 127) / 128 * 128 - raw), out_partial, M};
  auto kern = K == 4 ? c16_fwd_kernel<4> : c16_fwd_kernel<8>;
  if (int e = allow_full_lds(reinterpret_cast<const void*>(kern))) return e;
  kern<<<p.tiles, kT, kFwdLds, st>>>(a, p);
  return hip_status();
}

int launch_c16_bwd(hipStream_t st, const ConvGeom& g, int K, const float* dy, const float* w, const void* packed, const void* stats,
                   float* da3, double* partial, float* copies) {
  C16Plan p;
  if (!make_plan(g, p)) return ABL_ERR_SHAPE;
  C16Bwd a{};
  a.dy = dy;
  a.w = w;
  a.packed = static_cast<const uint8_t*>(packed);
  a.stats = static_cast<const float*>(stats);
  a.da3 = da3;
  a.partial = partial;
  a.wpartial = copies;
  a.M = (int64_t)g.N * g.H * g.W;
  auto kern = K == 4 ? c16_bwd_kernel<4, false> : c16_bwd_kernel<8, false>;
  if (int e = allow_full_lds(reinterpret_cast<const void*>(kern))) return e;
  kern<<<p.tiles, kT, kBwdLds, st>>>(a, p);
  return hip_status();
}

int c16_stack_tiles(const abl_layer* layers, int L, int K, int skip_every, size_t room) {
  if (skip_every != 2 || L < 2 || L % 2 != 0 || K == 32) return 0;
  const ConvGeom g = geom_of(layers[0].shape);
  const int tiles = c16_tiles(g, 1);
  if (tiles == 0 || (size_t)2 * tiles * 2304 * sizeof(float) > room) return 0;
  for (int i = 1; i < L; ++i) {
    const abl_shape &a = layers[0].shape, &b = layers[i].shape;
    if (a.N != b.N || a.H != b.H || a.W != b.W || a.Cin != b.Cin || a.Cout != b.Cout || a.R != b.R || a.S != b.S ||
        a.stride != b.stride || a.pad != b.pad)
      return 0;
  }
  return tiles;
}

// The gradients of a group go S -> T -> S: its last layer takes S + Eq. 8 of the group above as its dy and leaves its dA3 in T, its
// first layer takes Eq. 8 of that and leaves its dA3 in da3; S itself moves on to the group's own output there, when no block
// reads its neighbours' pixels of it.
int launch_c16_stack_bwd(hipStream_t st, const abl_layer* layers, int L, int K, float* s, float* t, float* da3, double* const (&rows)[2],
                         float* copies, float* means, float* const* trace) {
  const ConvGeom g = geom_of(layers[0].shape);
  C16Plan p;
  if (!make_plan(g, p)) return ABL_ERR_SHAPE;
  const size_t copy = (size_t)p.tiles * 2304;
  const int64_t M = (int64_t)g.N * g.H * g.W;
  if (int e = trace_copy(st, trace, L - 1, s, (size_t)M * kC)) return e;
  auto apply_of = [&](int i) {
    return C16Apply{i % 2 == 0 ? da3 : t, static_cast<const uint8_t*>(layers[i].packed), static_cast<const float*>(layers[i].stats),
                    means + 2 * kC * (i & 1)};
  };
  for (int i = L - 1; i >= 0; --i) {
    const abl_layer& l = layers[i];
    C16Bwd a{};
    a.dy = s;
    a.w = l.W;
    a.packed = static_cast<const uint8_t*>(l.packed);
    a.stats = static_cast<const float*>(l.stats);
    a.da3 = i % 2 == 0 ? da3 : t;
    a.partial = rows[i & 1];
    a.wpartial = copies + copy * (i & 1);
    a.M = M;
    const bool chain = i < L - 1;
    if (chain) {
      const abl_layer& u = layers[i + 1];
      a.up = apply_of(i + 1);
      a.up_means = means + 2 * kC * ((i + 1) & 1);
      a.up_partial = rows[(i + 1) & 1];
      a.up_nb = p.tiles;
      a.up_dgamma = u.dgamma;
      a.up_dbeta = u.dbeta;
      a.up_wpartial = copies + copy * ((i + 1) & 1);
      a.up_copies = p.tiles;
      a.up_dw = u.dW;
      if (i % 2 == 1) {
        a.add = s;
      } else if (i + 2 < L) {
        a.res = apply_of(i + 2);
        a.s = s;
      }
    }
    auto kern = K == 4 ? (chain ? c16_bwd_kernel<4, true> : c16_bwd_kernel<4, false>)
                       : (chain ? c16_bwd_kernel<8, true> : c16_bwd_kernel<8, false>);
    if (int e = allow_full_lds(reinterpret_cast<const void*>(kern))) return e;
    kern<<<p.tiles, kT, kBwdLds, st>>>(a, p);
    if (int e = hip_status()) return e;
    // its dy, which the kernel had in registers: what that was made of is still there
    if (chain && trace != nullptr && trace[i] != nullptr) {
      if (a.add != nullptr)
        if (int e = trace_copy(st, trace, i, a.add, (size_t)M * kC)) return e;
      if (int e = launch_bn_bwd_apply(st, a.up.packed, a.up.stats, a.up.da3, M, kC, K, a.add != nullptr, a.up_means, trace[i])) return e;
    }
  }
  return ABL_OK;
}

}  // namespace abl
