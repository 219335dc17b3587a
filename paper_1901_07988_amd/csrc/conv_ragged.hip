// Convolutions whose channel counts are not multiples of 16 (narrowed layers, image inputs): Eq. 4, both
// halves of Eq. 5, any filter, stride and padding, fp32.
//
// The matrix instructions want operands in tiles of 16, and a row of 20 channels cannot be read 16 bytes at
// a time by every lane.  So the contraction is flattened - (tap, channel) is one index - and both operands
// are gathered element by element into LDS tiles whose ends are filled with zeros; from there on it is a
// plain GEMM on the fp32 matrix cores.  A block is 64 rows x up to 64 columns with the four waves on 16
// rows each, and a 32-deep chunk of the contraction per barrier, the next chunk's elements in flight in
// registers meanwhile.  What bounds it is the gather (one address and one 4-byte load per element of the
// unfolded operand), which the small tiles keep on many blocks: 50 x 27 x 21, 3x3, 20 -> 36 channels takes
// 18 us forward, 24 us for the input's gradient and 36 us for the weights', where one thread per output
// element took 75, 246 and 456 us.

#include "abl_internal.h"

namespace abl {
namespace {

constexpr int kThreads = 256;
constexpr int RB_M = 64;    // rows of the output tile per block (16 per wave)
constexpr int RB_K = 32;    // contraction elements per chunk
constexpr int RB_LD = 36;   // floats per LDS row of a chunk: 16-byte fragments of 16 rows on different banks

// One output from the positions inside the image alone, for values that are not finite: in the tiles a position outside
// is a zero, which an infinite weight would turn into a NaN.
template <int MODE>
__device__ inline float output_inside(const float* in, const float* wgt, const ConvGeom& g, int p, int n) {
  const int Hi = MODE == 0 ? g.H : g.Ho, Wi = MODE == 0 ? g.W : g.Wo;
  const int Hq = MODE == 0 ? g.Ho : g.H, Wq = MODE == 0 ? g.Wo : g.W;
  const int Cg = MODE == 0 ? g.Cin : g.Cout;
  const int t = p / Wq, img = t / Hq, wq = p - t * Wq, hq = t - img * Hq;
  double sum = 0.0;
  for (int r = 0; r < g.R; ++r)
    for (int s = 0; s < g.S; ++s) {
      int hi, wi;
      if (MODE == 0) {
        hi = hq * g.stride + r - g.pad;
        wi = wq * g.stride + s - g.pad;
      } else {
        const int hh = hq + g.pad - r, ww = wq + g.pad - s;
        if (hh < 0 || ww < 0 || hh % g.stride != 0 || ww % g.stride != 0) continue;
        hi = hh / g.stride;
        wi = ww / g.stride;
      }
      if (hi < 0 || hi >= Hi || wi < 0 || wi >= Wi) continue;
      const float* a = in + (int64_t)((img * Hi + hi) * Wi + wi) * Cg;
      const float* b = wgt + (int64_t)(r * g.S + s) * g.Cin * g.Cout + (MODE == 0 ? n : (int64_t)n * g.Cout);
      for (int c = 0; c < Cg; ++c) {
        sum += (double)a[c] * (double)b[MODE == 0 ? (int64_t)c * g.Cout : c];
        if (sum != sum) return (float)sum;
      }
    }
  return (float)sum;
}

// Contractions of a few elements: one thread per output, the sum in order.  The tiles below spend a chunk of 32 on them.
template <int MODE>
__global__ __launch_bounds__(kThreads) void direct_conv_kernel(const float* __restrict__ in, const float* __restrict__ wgt,
                                                               const float* skip, float* out, ConvGeom g) {
  const int Hi = MODE == 0 ? g.H : g.Ho, Wi = MODE == 0 ? g.W : g.Wo;
  const int Hq = MODE == 0 ? g.Ho : g.H, Wq = MODE == 0 ? g.Wo : g.W;
  const int Cg = MODE == 0 ? g.Cin : g.Cout, Ng = MODE == 0 ? g.Cout : g.Cin;
  const uint32_t o = blockIdx.x * kThreads + threadIdx.x;
  if (o >= (uint32_t)(g.N * Hq * Wq) * Ng) return;
  const int p = (int)(o / Ng), n = (int)(o - (uint32_t)p * Ng);
  const int t = p / Wq, img = t / Hq, wq = p - t * Wq, hq = t - img * Hq;
  float sum = 0.0f;
  for (int r = 0; r < g.R; ++r) {
    const int hh = MODE == 0 ? hq * g.stride + r - g.pad : hq + g.pad - r;
    const int hi = MODE == 0 ? hh : hh / g.stride;
    if (hh < 0 || hi >= Hi || (MODE == 1 && hi * g.stride != hh)) continue;
    for (int s = 0; s < g.S; ++s) {
      const int ww = MODE == 0 ? wq * g.stride + s - g.pad : wq + g.pad - s;
      const int wi = MODE == 0 ? ww : ww / g.stride;
      if (ww < 0 || wi >= Wi || (MODE == 1 && wi * g.stride != ww)) continue;
      const float* a = in + (size_t)((img * Hi + hi) * Wi + wi) * Cg;
      const float* b = wgt + (size_t)(r * g.S + s) * g.Cin * g.Cout + (MODE == 0 ? n : (size_t)n * g.Cout);
      for (int c = 0; c < Cg; ++c) sum = fmaf(a[c], b[MODE == 0 ? (size_t)c * g.Cout : c], sum);
    }
  }
  out[o] = skip != nullptr ? sum + skip[o] : sum;
}

// MODE 0: out[p][co] = sum_{tap, ci} a3[p at tap][ci] W[tap][ci][co] (+ skip)
// MODE 1: out[p][ci] = sum_{tap, co} dy[p at tap][co] W[tap][ci][co]
// STRIDED: stride other than 1 (in mode 1 a tap then reaches only every stride-th pixel).
template <int MODE, int NT, bool STRIDED>
__global__ __launch_bounds__(kThreads, NT == 4 || (NT == 3 && MODE == 0) ? 4 : 1) void ragged_conv_kernel(const float* __restrict__ in,
                                                               const float* __restrict__ wgt, const float* skip,
                                                               float* out, ConvGeom g) {
  constexpr int BN = 16 * NT;
  constexpr int A_N = RB_M * RB_K / kThreads;   // elements of the A chunk per thread: 8
  constexpr int B_N = BN * RB_K / kThreads;     // ... of the B chunk: 2 NT
  __shared__ __attribute__((aligned(16))) float As[2][RB_M * RB_LD];
  __shared__ __attribute__((aligned(16))) float Bs[2][BN * RB_LD];
  const int Hi = MODE == 0 ? g.H : g.Ho, Wi = MODE == 0 ? g.W : g.Wo;
  const int Hq = MODE == 0 ? g.Ho : g.H, Wq = MODE == 0 ? g.Wo : g.W;
  const int Cg = MODE == 0 ? g.Cin : g.Cout;
  const int Ng = MODE == 0 ? g.Cout : g.Cin;
  const uint32_t Mg = (uint32_t)(g.N * Hq * Wq);
  const uint32_t KK = (uint32_t)(g.R * g.S * Cg);   // (at most 2^31 - 1: indexes past it stay unsigned)
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int ncol = (Ng + BN - 1) / BN;
  const uint32_t blk = block_of_grid();
  const uint32_t m0 = blk / ncol * RB_M;
  const int n0 = (int)(blk % ncol) * BN;
  if (m0 >= Mg) return;

  // A: the thread's column of the chunk is fixed (tid % 32), its rows are tid / 32 + 8 i
  const int a_k = tid & (RB_K - 1), a_row = tid >> 5;
  int a_base[A_N], a_h[A_N], a_w[A_N];   // offset of the row's image, position of tap (0, 0); a_h: far outside = no row
#pragma unroll
  for (int i = 0; i < A_N; ++i) {
    const uint32_t p = m0 + a_row + 8 * i;
    const bool ok = p < Mg;
    const int pp = ok ? (int)p : 0;
    const int t = pp / Wq, n = t / Hq;
    const int wq = pp - t * Wq, hq = t - n * Hq;
    a_base[i] = n * Hi * Wi;
    a_h[i] = ok ? (MODE == 0 ? hq * g.stride - g.pad : hq + g.pad) : -(1 << 28);
    a_w[i] = MODE == 0 ? wq * g.stride - g.pad : wq + g.pad;
  }
  float ra[A_N], rb[B_N];
  auto fetch = [&](uint32_t k0) __attribute__((always_inline)) {
    const uint32_t kk = k0 + a_k;
    const int tap = (int)kk / Cg, c = (int)kk - tap * Cg;   // (not used where kk >= KK)
    const int r = tap / g.S, s = tap - r * g.S;
#pragma unroll
    for (int i = 0; i < A_N; ++i) {
      int hi, wi;
      bool ok = kk < KK;
      if (MODE == 0) {
        hi = a_h[i] + r;
        wi = a_w[i] + s;
      } else {
        const int hh = a_h[i] - r, ww = a_w[i] - s;
        hi = STRIDED ? hh / g.stride : hh;
        wi = STRIDED ? ww / g.stride : ww;
        if (STRIDED) ok = ok && hh >= 0 && ww >= 0 && hi * g.stride == hh && wi * g.stride == ww;
      }
      ok = ok && hi >= 0 && hi < Hi && wi >= 0 && wi < Wi;
      const uint32_t o = ((uint32_t)a_base[i] + (uint32_t)hi * Wi + wi) * Cg + c;   // (tensors have fewer than 2^31 elements)
      const float v = in[ok ? o : 0u];
      ra[i] = ok ? v : 0.f;
    }
#pragma unroll
    for (int j = 0; j < B_N; ++j) {
      // forward: lanes along the output channel (contiguous in W); gradient: along the contraction
      const int idx = tid + kThreads * j;
      const int n = MODE == 0 ? idx % BN : idx / RB_K;
      const uint32_t kb = MODE == 0 ? k0 + idx / BN : kk;   // (idx % RB_K is the thread's own column)
      const bool ok = kb < KK && n0 + n < Ng;
      const uint32_t o = MODE == 0 ? kb * g.Cout + n0 + n : ((uint32_t)tap * g.Cin + n0 + n) * g.Cout + c;
      const float v = wgt[ok ? o : 0u];
      rb[j] = ok ? v : 0.f;
    }
  };
  auto stage = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < A_N; ++i) As[buf][(a_row + 8 * i) * RB_LD + a_k] = ra[i];
#pragma unroll
    for (int j = 0; j < B_N; ++j) {
      const int idx = tid + kThreads * j;
      const int n = MODE == 0 ? idx % BN : idx / RB_K;
      const int kb = MODE == 0 ? idx / BN : idx % RB_K;
      Bs[buf][n * RB_LD + kb] = rb[j];
    }
  };
  // transposed product (first operand = weights): a lane ends up with four consecutive channels of a pixel.
  // Two sums per output, of the two halves of every chunk: chains half as long round half as often.
  floatx4 acc[2][NT][1];
#pragma unroll
  for (int j = 0; j < NT; ++j) acc[0][j][0] = acc[1][j][0] = floatx4{0.f, 0.f, 0.f, 0.f};
  const uint32_t chunks = (KK + RB_K - 1) / RB_K;
  fetch(0);
  stage(0);
  __syncthreads();
  for (uint32_t it = 0; it < chunks; ++it) {
    const int cur = it & 1;
    if (it + 1 < chunks) fetch((it + 1) * RB_K);
#pragma unroll
    for (int h = 0; h < RB_K; h += 16) {
      float4 bf[NT], af[1];
#pragma unroll
      for (int j = 0; j < NT; ++j) bf[j] = *reinterpret_cast<const float4*>(&Bs[cur][(16 * j + li) * RB_LD + h + 4 * lk]);
      af[0] = *reinterpret_cast<const float4*>(&As[cur][(16 * wave + li) * RB_LD + h + 4 * lk]);
      mma_k4<false, NT, 1>(bf, af, acc[h / 16]);
    }
    if (it + 1 < chunks) stage(cur ^ 1);   // (the other buffer: its readers passed the barrier of the last chunk)
    __syncthreads();
  }
  const uint32_t p = m0 + 16 * wave + li;
  if (p >= Mg) return;
  uint32_t odd = 0;   // outputs that are not finite
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int n = n0 + 16 * j + 4 * lk + r;
      if (n >= Ng) continue;
      const size_t o = (size_t)p * Ng + n;
      const float v = acc[0][j][0][r] + acc[1][j][0][r];
      const bool fin = fabsf(v) < INFINITY;
      odd |= fin ? 0u : 1u << (4 * j + r);
      if (fin) out[o] = skip != nullptr ? v + skip[o] : v;
    }
  for (; __builtin_expect(odd != 0, 0); odd &= odd - 1) {
    const int e = __builtin_ctz(odd), n = n0 + 16 * (e >> 2) + 4 * lk + (e & 3);
    const size_t o = (size_t)p * Ng + n;
    const float v = output_inside<MODE>(in, wgt, g, (int)p, n);
    out[o] = skip != nullptr ? v + skip[o] : v;
  }
}

// p / d for p < 2^31 with m = floor(2^32 / d) + 1 (d > 1): the high product is the quotient or one more.
__device__ inline int div_magic(int p, int d, uint32_t m) {
  if (d == 1) return p;
  const int q = (int)__umulhi((uint32_t)p, m);
  return (int64_t)q * d > p ? q - 1 : q;
}
inline uint32_t magic_of(int d) { return d > 1 ? (uint32_t)((1ull << 32) / (uint32_t)d + 1) : 0u; }

// One sum of the weight gradient over the pixels p_begin .. p_end - 1 that the tap reaches inside the image with an
// activation that is not zero, for values that are not finite (an infinite dy times a zero of the tile is a NaN).
template <int K>
__device__ inline float sum_inside(const uint8_t* packed, const float* stats, const float* dy, const ConvGeom& g,
                                   int relu32, int tap, int ci, int co, int64_t p_begin, int64_t p_end) {
  const float step = K == 32 ? 0.f : stats[P_STEP * g.Cin + ci];
  const int32_t fb = K == 32 ? 0 : reinterpret_cast<const int32_t*>(stats)[P_FB * g.Cin + ci];
  const int tr = tap / g.S, ts = tap - tr * g.S;
  double sum = 0.0;
  for (int64_t p = p_begin; p < p_end; ++p) {
    const int t = (int)p / g.Wo, n = t / g.Ho;
    const int wi = ((int)p - t * g.Wo) * g.stride - g.pad + ts, hi = (t - n * g.Ho) * g.stride - g.pad + tr;
    if (hi < 0 || hi >= g.H || wi < 0 || wi >= g.W) continue;
    const int64_t e = (int64_t)((n * g.H + hi) * g.W + wi) * g.Cin + ci;
    float v;
    if constexpr (K == 32) {
      v = reinterpret_cast<const float*>(packed)[e];
      if (relu32 != 0 && v < 0.f) continue;
    } else {
      v = dequant<K>(K == 4 ? (packed[e >> 1] >> ((e & 1) * 4)) & 15u : packed[e], step, fb);
      if (!(v > 0.f)) continue;
    }
    sum += (double)v * (double)dy[p * g.Cout + co];
    if (sum != sum) return (float)sum;
  }
  return (float)sum;
}

// dW[(tap, ci)][co] = sum over output pixels of A3~[p at tap][ci] dy[p][co].  Rows of the tile = flattened
// (tap, ci), contraction = the pixels of this block's share, 32 per chunk; the shares' copies of dW are
// summed by the caller.  Both tiles lie in LDS with the pixel outermost, which is how they are read from
// memory and how the 4-deep fp32 MFMA wants its operands (one 4-byte read per lane, the four pixels of a
// step on different quarters of the banks).
template <int K, int NT>
__global__ __launch_bounds__(kThreads) void ragged_wgrad_kernel(const uint8_t* __restrict__ packed,
                                                                const float* __restrict__ stats,
                                                                const float* __restrict__ dy,
                                                                float* __restrict__ dst, ConvGeom g, int relu32,
                                                                int chunks, int split, uint32_t wo_magic,
                                                                uint32_t ho_magic) {
  constexpr int BN = 16 * NT;
  constexpr int LDA = RB_M + 16, LDB = (BN % 64 == 16 || BN % 64 == 48) ? BN : BN + 16;   // 16 or 48 words past a multiple of 64
  constexpr int A_N = RB_M * RB_K / kThreads, B_N = BN * RB_K / kThreads;
  __shared__ float As[2][RB_K * LDA];
  __shared__ float Bs[2][RB_K * LDB];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lk = lane >> 4;
  const int MR = g.R * g.S * g.Cin;
  const int ncol = (g.Cout + BN - 1) / BN, nrow = (int)(((uint32_t)MR + RB_M - 1) / RB_M);
  const uint32_t blk = block_of_grid();
  const int part = (int)(blk / (uint32_t)(ncol * nrow)), tile = (int)(blk - (uint32_t)part * (ncol * nrow));
  if (part >= split) return;
  const uint32_t m0 = (uint32_t)(tile / ncol) * RB_M;
  const int n0 = (tile % ncol) * BN;
  const int c_begin = (int)((int64_t)part * chunks / split), c_end = (int)((int64_t)(part + 1) * chunks / split);
  const int Mg = g.N * g.Ho * g.Wo;   // at most 2^31 - 1; pixel numbers past it wrap to negative ones

  // the thread's row (tap, ci) is fixed: lane of the block's 64 rows; its pixels are wave + 4 i
  const uint32_t row = m0 + lane;
  const bool row_ok = row < (uint32_t)MR;
  const int rr = row_ok ? (int)row : 0;
  const int tap = rr / g.Cin, ci = rr - tap * g.Cin;
  const int tr = tap / g.S, ts = tap - tr * g.S;
  const float step = K == 32 ? 0.f : stats[P_STEP * g.Cin + ci];
  const int32_t fb = K == 32 ? 0 : reinterpret_cast<const int32_t*>(stats)[P_FB * g.Cin + ci];

  float ra[A_N], rb[B_N];
  auto fetch = [&](int chunk) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < A_N; ++i) {
      const int p = (int)((unsigned)chunk * RB_K + wave + 4 * i);   // the same for the whole wave
      const bool in_p = (unsigned)p < (unsigned)Mg;
      const int pc = in_p ? p : 0;
      const int t = div_magic(pc, g.Wo, wo_magic), n = div_magic(t, g.Ho, ho_magic);
      const int wi = (pc - t * g.Wo) * g.stride - g.pad + ts, hi = (t - n * g.Ho) * g.stride - g.pad + tr;
      const bool ok = row_ok && in_p && hi >= 0 && hi < g.H && wi >= 0 && wi < g.W;
      const uint32_t e = ok ? (uint32_t)(((n * g.H + hi) * g.W + wi) * g.Cin + ci) : 0u;
      float v;
      if constexpr (K == 32) {
        v = reinterpret_cast<const float*>(packed)[e];
        ra[i] = ok && !(relu32 != 0 && v < 0.f) ? v : 0.f;
      } else {
        const uint32_t code = K == 4 ? (packed[e >> 1] >> ((e & 1) * 4)) & 15u : packed[e];
        v = dequant<K>(code, step, fb);                  // Eq. 10
        ra[i] = ok && v > 0.f ? v : 0.f;                 // Eq. 3
      }
    }
#pragma unroll
    for (int j = 0; j < B_N; ++j) {
      const int idx = tid + kThreads * j;
      const int p = (int)((unsigned)chunk * RB_K + idx / BN), n = n0 + idx % BN;
      const bool ok = (unsigned)p < (unsigned)Mg && n < g.Cout;
      const float v = dy[ok ? (uint32_t)p * (uint32_t)g.Cout + n : 0u];
      rb[j] = ok ? v : 0.f;
    }
  };
  auto stage = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < A_N; ++i) As[buf][(wave + 4 * i) * LDA + lane] = ra[i];
#pragma unroll
    for (int j = 0; j < B_N; ++j) {
      const int idx = tid + kThreads * j;
      Bs[buf][(idx / BN) * LDB + idx % BN] = rb[j];
    }
  };
  floatx4 acc[2][NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) acc[0][j] = acc[1][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  if (c_begin < c_end) {
    fetch(c_begin);
    stage(0);
  }
  __syncthreads();
  for (int it = c_begin; it < c_end; ++it) {
    const int cur = (it - c_begin) & 1;
    if (it + 1 < c_end) fetch(it + 1);
#pragma unroll
    for (int q = 0; q < RB_K / 4; ++q) {
      const float a = As[cur][(4 * q + lk) * LDA + 16 * wave + li];
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[q & 1][j] = mfma16(a, Bs[cur][(4 * q + lk) * LDB + 16 * j + li], acc[q & 1][j]);
    }
    if (it + 1 < c_end) stage(cur ^ 1);
    __syncthreads();
  }
  float* d = dst + (size_t)part * MR * g.Cout;
  uint32_t odd = 0;   // sums that are not finite
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const uint32_t m = m0 + 16 * wave + 4 * lk + r;
      const int n = n0 + 16 * j + li;
      const float v = acc[0][j][r] + acc[1][j][r];
      if (m < (uint32_t)MR && n < g.Cout) {
        odd |= fabsf(v) < INFINITY ? 0u : 1u << (4 * j + r);
        d[(size_t)m * g.Cout + n] = v;
      }
    }
  for (; __builtin_expect(odd != 0, 0); odd &= odd - 1) {
    const int e = __builtin_ctz(odd), n = n0 + 16 * (e >> 2) + li;
    const uint32_t m = m0 + 16 * wave + 4 * lk + (e & 3);
    const int64_t p_end = (int64_t)c_end * RB_K;
    d[(size_t)m * g.Cout + n] = sum_inside<K>(packed, stats, dy, g, relu32, (int)(m / (uint32_t)g.Cin),
                                              (int)(m % (uint32_t)g.Cin), n, (int64_t)c_begin * RB_K, p_end < Mg ? p_end : Mg);
  }
}

// column tiles per block: no more than the channels fill
inline int ragged_nt(int channels) { return channels > 32 ? (channels > 48 ? 4 : 3) : (channels > 16 ? 2 : 1); }

template <int MODE>
int launch_ragged(hipStream_t st, const ConvGeom& g, const float* in, const float* w, const float* skip, float* out) {
  const int Ng = MODE == 0 ? g.Cout : g.Cin;
  const int64_t Mg = MODE == 0 ? (int64_t)g.N * g.Ho * g.Wo : (int64_t)g.N * g.H * g.W;
  // (1x1, us, a thread per output / tiles: 3 -> 16 @112x112 N=8, 1.6 10^6 outputs, 7.7 / 11.4; 7 -> 9 8.1 / 10.3; gradient
  // 16 <- 5 9.7 / 11.8; but 16 -> 5 12.6 / 10.1, 10 -> 64 30.7 / 22.5, gradient 64 <- 3, 6.4 10^6 outputs, 29.2 / 24.0.  Up to
  // 16 elements on few outputs: a chunk's round trip is all there is; backward of 512 -> 10 on 128 pixels 22.5 / 25.9)
  const int kk = g.R * g.S * (MODE == 0 ? g.Cin : g.Cout);
  if ((kk <= 9 && Mg * Ng < 3000000) || (kk <= 16 && Mg * Ng < 100000)) {
    direct_conv_kernel<MODE><<<(unsigned)((Mg * Ng + kThreads - 1) / kThreads), kThreads, 0, st>>>(in, w, skip, out, g);
    return hip_status();
  }
  const int nt = ragged_nt(Ng);
  const dim3 grid = grid_of(((Mg + RB_M - 1) / RB_M) * ((Ng + 16 * nt - 1) / (16 * nt)));
  constexpr bool ST = MODE == 1;   // (the forward only multiplies by the stride)
  const bool st1 = !ST || g.stride == 1;
  auto kern = nt == 1 ? (st1 ? ragged_conv_kernel<MODE, 1, false> : ragged_conv_kernel<MODE, 1, ST>)
            : nt == 2 ? (st1 ? ragged_conv_kernel<MODE, 2, false> : ragged_conv_kernel<MODE, 2, ST>)
            : nt == 3 ? (st1 ? ragged_conv_kernel<MODE, 3, false> : ragged_conv_kernel<MODE, 3, ST>)
                      : (st1 ? ragged_conv_kernel<MODE, 4, false> : ragged_conv_kernel<MODE, 4, ST>);
  kern<<<grid, kThreads, 0, st>>>(in, w, skip, out, g);
  return hip_status();
}

template <int K>
void run_ragged_wgrad(hipStream_t st, const ConvGeom& g, const void* packed, const float* stats, const float* dy,
                      float* dst, int relu32, int chunks, int split, int64_t tiles, int nt) {
  auto kern = nt == 1 ? ragged_wgrad_kernel<K, 1> : nt == 2 ? ragged_wgrad_kernel<K, 2>
            : nt == 3 ? ragged_wgrad_kernel<K, 3> : ragged_wgrad_kernel<K, 4>;
  kern<<<grid_of(tiles * split), kThreads, 0, st>>>(static_cast<const uint8_t*>(packed), stats, dy, dst, g, relu32,
                                                     chunks, split, magic_of(g.Wo), magic_of(g.Ho));
}

}  // namespace

int launch_ragged_conv(hipStream_t st, const ConvGeom& g, int mode, const float* in, const float* w, const float* skip,
                       float* out) {
  return mode == 0 ? launch_ragged<0>(st, g, in, w, skip, out) : launch_ragged<1>(st, g, in, w, skip, out);
}

int ragged_wgrad_copies(const ConvGeom& g, size_t room) {
  const int nt = ragged_nt(g.Cout);
  const int64_t MR = (int64_t)g.R * g.S * g.Cin;
  const int64_t tiles = ((MR + RB_M - 1) / RB_M) * ((g.Cout + 16 * nt - 1) / (16 * nt));
  const int64_t chunks = ((int64_t)g.N * g.Ho * g.Wo + RB_K - 1) / RB_K;
  // A block per element of dW is over sooner than a walk over chunks, and needs no launch to sum copies (backward, us,
  // elements / chunks: 1x1 64 -> 10 @14x14 N=16, 2.0 10^6 products, 26.5 / 30.4; 20 -> 36, 2.3 10^6, 27.0 / 33.2; 512 ->
  // 10 on 128 pixels 23.1 / 28.0; but 33 -> 65 @14x14, 6.7 10^6, 49.5 / 38.7).
  if (MR * g.Cout * (int64_t)g.N * g.Ho * g.Wo < 2500000) return 0;
  // about four blocks per compute unit, at least four chunks each (a chunk is a round trip to memory)
  int64_t split = 1024 / tiles;
  if (split > chunks / 4) split = chunks / 4;
  if (split < 1) split = 1;
  const int64_t fit = (int64_t)(room / ((size_t)MR * g.Cout * sizeof(float)));
  // one copy needs no room: it is dW itself
  if (split > fit) split = fit > 1 ? fit : 1;
  // A block walks its share one chunk after the other, about a microsecond each; with shares of more than
  // 64 chunks the kernel with a block per element of dW is the faster one.
  return chunks / split > 64 ? 0 : (int)split;
}

// (241 layers of 3 to 64 channels, us: 0.72 to 1.2 of it)
double ragged_dgrad_us(const ConvGeom& g) {
  const int nt = ragged_nt(g.Cin), chunks = (g.R * g.S * g.Cout + RB_K - 1) / RB_K;
  const int64_t blocks = (((int64_t)g.N * g.H * g.W + RB_M - 1) / RB_M) * ((g.Cin + 16 * nt - 1) / (16 * nt));
  const double rounds = (double)blocks / 1024 * (nt + 1);
  return 3.5 + chunks * (g.stride > 1 ? 1.44 + 0.19 * nt + rounds : 0.73 + 0.19 * nt + 0.55 * rounds);
}
// (270 layers: 0.77 to 1.2 of it)
double ragged_wgrad_us(const ConvGeom& g, size_t room) {
  const double n = (double)g.R * g.S * g.Cin * g.Cout, pixels = (double)g.N * g.Ho * g.Wo;
  const int copies = ragged_wgrad_copies(g, room);
  if (copies == 0) return 2.6 + 1.6e-3 * pixels + 5.8e-4 * n + 2.1e-6 * n * pixels;
  return 3.8 + 2.3 * pixels / RB_K / copies + 0.02 * copies + 3.5e-6 * n * copies + 2.6e-8 * n * pixels;
}

int launch_ragged_wgrad(hipStream_t st, const ConvGeom& g, int K, const void* packed, const float* stats,
                        const float* dy, int copies, float* dst, bool relu32) {
  const int nt = ragged_nt(g.Cout);
  const int64_t MR = (int64_t)g.R * g.S * g.Cin;
  const int64_t tiles = ((MR + RB_M - 1) / RB_M) * ((g.Cout + 16 * nt - 1) / (16 * nt));
  const int chunks = (int)(((int64_t)g.N * g.Ho * g.Wo + RB_K - 1) / RB_K);
  const int r32 = relu32 ? 1 : 0;
  if (K == 4) run_ragged_wgrad<4>(st, g, packed, stats, dy, dst, r32, chunks, copies, tiles, nt);
  else if (K == 8) run_ragged_wgrad<8>(st, g, packed, stats, dy, dst, r32, chunks, copies, tiles, nt);
  else run_ragged_wgrad<32>(st, g, packed, stats, dy, dst, r32, chunks, copies, tiles, nt);
  return hip_status();
}

}  // namespace abl
