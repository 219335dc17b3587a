// Weight gradient (first half of Eq. 5) of 'same' stride-1 3x3 and 1x1 layers from the K-bit codes (K = 4 / 8), fp32
// results on the bf16 matrix cores.
//
//   dW[tap][ci][co] = |step[ci]| / 2 * sum over pixels of v[pixel + tap][ci] * dy[pixel][co],
//
// where step (n + 1/2) is Eq. 10 and v = |2 n + 1| where that is positive, else 0.  v is a whole number below
// 2^K + 2 |fb|, exact in one bf16 up to 256; 2^23 dy is the exact sum of three bf16 values (as in conv_split.hip).  So
// three bf16 products - each exact - replace one fp32 product, with nothing dropped, in 0.22 of its matrix-core time
// (loops on registers: 2050 TFLOP/s of bf16, 154 of fp32), and the sums are rounded once per 32 pixels and part instead of
// once per 4 pixels (relative error of a sum over 12544 pixels against 64 bits 0.95e-6, fp32 matrix cores 1.4e-6).
// A block whose channels reach beyond 256 (8-bit codes with a positive fb) but not beyond 511 stores v - 1 there - v
// is odd - and the missing ones are made from the stored bits: two more products, with the upper two parts of dy
// (the third is below 2^-17 of dy and the bit 2^-8 of v: below 2^-25 of the sum's terms).  Larger v go in two or three bf16 parts, one pass after the other.
//
// One block = a 32 (ci) x 64 (co) tile of all nine taps and a share of the pixels, chunk by chunk (rows of an image
// or a few whole images, at most 128 positions).  The contraction index of the MFMAs is the pixel, eight
// consecutive ones of a row per lane, so both operands are staged in groups of eight positions of a channel: dy as
// [part][group][co], v as [row][group][ci] with the border rows; rows start at multiples of eight positions and are
// filled up with zeros.  The left and right taps of a row are the middle one's fragment shifted
// by one element (four v_alignbit each, with one neighbouring word on either side), so v is stored once.
// The 16-byte groups of neighbouring channels are neighbours and those of neighbouring groups multiples of 256 bytes
// apart: no bank is touched twice by a read or a write (with a channel's positions side by side a third of the
// kernel's time were bank conflicts).  To that end a thread's channels go to slots a quarter or half of the tile
// apart; the epilogue undoes the permutation.
// Eight waves in two groups that take alternate k-steps (32 positions); a wave keeps one 16-channel tile of ci and
// two of co for all nine taps, 54 MFMAs per k-step from 6 + 9 reads and 24 shifts.  Two buffers; while one group
// stages the next chunk the other contracts this one and then they change places, so that on every SIMD the
// staging arithmetic of a wave runs under the MFMAs of another.  Each share of the pixels leaves its own copy of
// dW, summed in a fixed order by the caller's launch.
#include <type_traits>

#include "abl_internal.h"

namespace abl {
namespace {

constexpr int TCI = 32, TCO = 64, THREADS = 512;
constexpr int POS = 128;                         // positions of dy per chunk
constexpr int DPART = POS / 8 * TCO * 16;        // bytes of one part of dy
constexpr int AGRP = TCI * 16;                   // bytes of a group of v

constexpr float kUp = 0x1p23f, kDown = 0x1p-23f;   // dy is split as 2^23 times its values: the parts of the smallest are normal

// One share's sum of one element from dy and the codes themselves (summed in 64 bits), for sums that are not finite.
template <int K>
__device__ inline float exact_sum(const uint8_t* codes, const float* stats, const float* dy, int H, int W, int Cin,
                                  int Cout, int tap, int ci, int co, int px_begin, int px_end) {
  const float step = stats[P_STEP * Cin + ci];
  const int32_t fb = reinterpret_cast<const int32_t*>(stats)[P_FB * Cin + ci];
  const int dh = tap / 3 - 1, dw = tap % 3 - 1;
  double s = 0.0;
  for (int p = px_begin; p < px_end; ++p) {
    const int row = p / W, w = p - row * W + dw, h = row % H + dh;
    float v = 0.0f;   // (the border's zeros take part: times an infinity they are NaN)
    if (h >= 0 && h < H && w >= 0 && w < W) {
      const size_t e = ((size_t)(row + dh) * W + w) * Cin + ci;
      const uint32_t code = K == 4 ? (codes[e >> 1] >> (4 * (e & 1))) & 15u : codes[e];
      v = fmaxf(dequant<K>(code, step, fb), 0.0f);
    }
    s += (double)v * (double)dy[(size_t)p * Cout + co];
    if (s != s) return (float)s;
  }
  return (float)s;
}

// How a block's codes become v = max(s2 code + off, 0) - the sign of the step folded in - and how far they reach.
template <int K>
__device__ inline float decode_consts(const float* stats, int Cin, int c, float& s2, float& off) {
  const float st = stats[P_STEP * Cin + c];
  const float sg = st > 0.0f ? 1.0f : st < 0.0f ? -1.0f : 0.0f;
  s2 = 2.0f * sg;
  off = sg * (2.0f * (float)(reinterpret_cast<const int32_t*>(stats)[P_FB * Cin + c] - (1 << (K - 1))) + 1.0f);
  return fmaxf(off, off + s2 * (float)((1 << K) - 1));
}
// ... and (bf16 operands) Eq. 10 itself, max(step code + step (fb - 2^(K-1) + 1/2), 0) before it is rounded: a sum of
// code and a constant, exact, times the step
template <int K>
__device__ inline void decode_consts_bf16(const float* stats, int Cin, int c, float& step, float& off) {
  step = stats[P_STEP * Cin + c];
  off = (float)(reinterpret_cast<const int32_t*>(stats)[P_FB * Cin + c] - (1 << (K - 1))) + 0.5f;
}
// 0: exact in one bf16; 1: the ones beyond 256 from the stored bits; 2, 3: that many parts, pass by pass
__device__ inline int decode_mode(float vmax) { return vmax <= 256.0f ? 0 : vmax < 512.0f ? 1 : vmax < 65536.0f ? 2 : 3; }

// the upper halves of two floats (bf16 by truncation: exact for whole numbers up to 256, v - 1 for odd ones up to 511)
__device__ inline uint32_t upper2(float a, float b) {
  return __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);
}
// part `part` of the truncations of a and b
__device__ inline uint32_t part2(float a, float b, int part) {
  uint32_t u = upper2(a, b);
  for (int t = 0; t < part; ++t) {
    a -= __uint_as_float(u << 16);
    b -= __uint_as_float(u & 0xFFFF0000u);
    u = upper2(a, b);
  }
  return u;
}
__device__ inline uint32_t round2(float a, float b) {
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, bf16x2_t{(__bf16)a, (__bf16)b});
}
// 1.0 for every stored value of 256 and more, else 0
__device__ inline uint4 missing_ones(uint4 h) {
  typedef unsigned short ushort2_t __attribute__((ext_vector_type(2)));
  auto f = [](uint32_t w) __attribute__((always_inline)) {
    ushort2_t x = __builtin_bit_cast(ushort2_t, w);
    const ushort2_t lim = {0x437F, 0x437F}, one = {1, 1}, bits = {0x3F80, 0x3F80};
    x = __builtin_elementwise_sub_sat(x, lim);
    x = __builtin_elementwise_min(x, one) * bits;
    return __builtin_bit_cast(uint32_t, x);
  };
  return make_uint4(f(h.x), f(h.y), f(h.z), f(h.w));
}
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
// the NP parts of eight floats of dy, two to a word
template <int NP>
__device__ inline void split_dy(const float (&x)[8], uint4 (&u)[NP]) {
  uint32_t w[NP][4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    float a = NP == 3 ? kUp * x[2 * q] : x[2 * q], b = NP == 3 ? kUp * x[2 * q + 1] : x[2 * q + 1];
#pragma unroll
    for (int t = 0; t < NP; ++t) {
      w[t][q] = __builtin_bit_cast(uint32_t, bf16x2_t{(__bf16)a, (__bf16)b});
      if (t + 1 == NP) break;
      a = less_low(a, w[t][q]);    // (pixels of one channel: the same sums)
      b = less_high(b, w[t][q]);
    }
  }
#pragma unroll
  for (int t = 0; t < NP; ++t) u[t] = make_uint4(w[t][0], w[t][1], w[t][2], w[t][3]);
}
// N codes of K bits in a word -> v, or (bf16 operands) the dequantized activation
template <int K, bool BF16, int N>
__device__ inline void decode(uint32_t w, const float (&s2)[N], const float (&off)[N], float (&v)[N]) {
  uint32_t by[2] = {w, w};
  if (K == 4) {   // one code per byte: a byte converts in one instruction
    by[0] = w & 0x0F0F0F0Fu;
    by[1] = (w >> 4) & 0x0F0F0F0Fu;
  }
#pragma unroll
  for (int e = 0; e < N; ++e) {
    const uint32_t code = K == 4 ? (by[e & 1] >> (8 * (e >> 1))) & 0xFFu : (w >> (8 * e)) & 0xFFu;
    v[e] = BF16 ? fmaxf(s2[e] * ((float)code + off[e]), 0.0f) : fmaxf(fmaf(s2[e], (float)code, off[e]), 0.0f);
  }
}

struct Chunking {
  int TI, R;         // a chunk: R rows of one image, or (R = H) TI images
  int nch, chunks;   // chunks per image (TI = 1), chunks in all
  int dw8, aw8;      // groups of eight positions per row of dy / of v
  int agroups;       // groups of v, with a group of zeros before and after
  int splits;
};

// NP = 3: dy in three parts, as above; NP = 1: both operands rounded to bf16.
template <int K, int NP>
__global__ __launch_bounds__(THREADS, 2) void split_wgrad_kernel(const uint8_t* __restrict__ codes,
                                                                 const float* __restrict__ stats,
                                                                 const float* __restrict__ dy, float* __restrict__ dst,
                                                                 ConvGeom g, Chunking ck) {
  constexpr int DBYTES = NP * DPART;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int abytes = ck.agroups * AGRP;
  unsigned char* const D0 = smem;                  // [2][part][group][co]
  unsigned char* const A0 = smem + 2 * DBYTES;     // [2][zeros, rows of groups, zeros][ci]
  const int H = g.H, W = g.W, Cin = g.Cin, Cout = g.Cout;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lk = lane >> 4;
  const int kg = wave >> 2, wc = wave & 1, wo = (wave >> 1) & 1;
  // ids 8 apart share an XCD and its L2: the blocks that stage the same dy (same co tile and share of the
  // pixels, different ci tiles) run there
  const int n_ci = Cin / TCI, n_co = Cout / TCO;
  int ci_blk, pair;
  if ((n_co * ck.splits) % 8 == 0) {
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    pair = (slot / n_ci) * 8 + xcd;
    ci_blk = slot % n_ci;
  } else {
    pair = blockIdx.x / n_ci;
    ci_blk = blockIdx.x % n_ci;
  }
  const int co_blk = pair % n_co, split = pair / n_co;
  const int ci0 = ci_blk * TCI, co0 = co_blk * TCO;
  const int c_begin = (int)((int64_t)split * ck.chunks / ck.splits), c_end = (int)((int64_t)(split + 1) * ck.chunks / ck.splits);

  // the zeros before and after v: neighbours of its first and last positions
  if (tid < 4 * TCI) {
    const int b = tid & 1;
    *reinterpret_cast<uint4*>(A0 + b * abytes + ((tid & 2) ? abytes - AGRP : 0) + (tid >> 2) * 16) = make_uint4(0u, 0u, 0u, 0u);
  }

  // ---- staging roles.  dy: eight positions of two channels; v: eight positions of four channels, its few items
  // spread over the SIMDs and the two groups of waves
  const int Hc = ck.TI > 1 ? H : ck.R;             // rows of an image in a chunk
  const int drows = ck.TI * Hc, arows = ck.TI * (Hc + 2);
  const int dgr = tid >> 5, dcp = tid & 31;
  const int drow = dgr / ck.dw8, dw0 = 8 * (dgr - drow * ck.dw8);
  const int dti = drow / Hc, dh = drow - dti * Hc;
  const int atid = lane + 64 * (wave ^ ((wave & 1) << 2));
  const int agr = atid >> 3, ac4 = atid & 7;
  const int arow = agr / ck.aw8, aw0 = 8 * (agr - arow * ck.aw8);
  const int ati = arow / (Hc + 2), ah = arow - ati * (Hc + 2) - 1;
  const bool a_role = arow < arows;
  unsigned char* const d_st = D0 + (dgr * TCO + dcp) * 16;               // channel 2 dcp + ch: slot dcp + 32 ch
  unsigned char* const a_st = A0 + (agr + 1) * AGRP + ac4 * 16;          // channel 4 ac4 + e: slot ac4 + 8 e
  float s2[4], off[4];
  float vmax = 0.0f;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if constexpr (NP == 3) vmax = fmaxf(vmax, decode_consts<K>(stats, Cin, ci0 + 4 * ac4 + e, s2[e], off[e]));
    else decode_consts_bf16<K>(stats, Cin, ci0 + 4 * ac4 + e, s2[e], off[e]);
  }
  // (eight neighbouring lanes hold all 32 channels)
#pragma unroll
  for (int d = 1; d < 8; d <<= 1) vmax = fmaxf(vmax, __shfl_xor(vmax, d, 64));
  const int mode = __builtin_amdgcn_readfirstlane(decode_mode(vmax));

  using code_t = typename std::conditional<K == 4, uint16_t, uint32_t>::type;
  // bytes from the chunk's first pixel (v: from the row above it) to the item's columns, the last one again past
  // the row; items outside the image load the chunk's first pixel
  uint32_t d_off[8], a_off[8];
  // (elements first, then bytes: a chunk of many channels has up to 2^31 of them, and their bits do not fit 32)
  const uint32_t a_row = (uint32_t)(W * Cin) / (8 / K);
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    d_off[i] = (uint32_t)(((dti * H + dh) * W + min(dw0 + i, W - 1)) * Cout + 2 * dcp) * 4u;
    a_off[i] = ((uint32_t)((ati * H + ah + 1) * W + min(aw0 + i, W - 1)) * Cin + 4 * ac4) / (8 / K);
  }
  float2 dv[8];
  uint32_t cw[8];
  bool d_ok = false, a_ok = false;
  auto stage_load = [&](int c) __attribute__((always_inline)) {
    const int im = ck.TI > 1 ? c * ck.TI : c / ck.nch;
    const int h0 = ck.TI > 1 ? 0 : (c - im * ck.nch) * ck.R;
    const size_t p0 = (size_t)(im * H + h0) * W;
    {
      d_ok = drow < drows && im + dti < g.N && h0 + dh < H;
      const char* src = reinterpret_cast<const char*>(dy + p0 * Cout + co0);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        uint32_t o = d_ok ? d_off[i] : 0u;
        asm volatile("" : "+v"(o));   // (a select, not a branch around the load: behind one the loads before it are waited for)
        dv[i] = *reinterpret_cast<const float2*>(src + o);
      }
    }
    if (a_role) {
      const int h = h0 + ah;
      a_ok = im + ati < g.N && h >= 0 && h < H;
      const char* src = reinterpret_cast<const char*>(codes) + (p0 * Cin + ci0) * K / 8 - a_row;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        uint32_t o = a_ok ? a_off[i] : a_row;
        asm volatile("" : "+v"(o));
        cw[i] = *reinterpret_cast<const code_t*>(src + o);
      }
    }
  };
  auto stage_store = [&](int buf, int part) __attribute__((always_inline)) {
#pragma unroll
    for (int ch = 0; ch < 2; ++ch) {
      float x[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) x[i] = d_ok && dw0 + i < W ? (ch == 0 ? dv[i].x : dv[i].y) : 0.0f;
      uint4 u[NP];
      split_dy<NP>(x, u);
#pragma unroll
      for (int t = 0; t < NP; ++t) *reinterpret_cast<uint4*>(d_st + buf * DBYTES + ch * 512 + t * DPART) = u[t];
    }
    if (a_role) {
      float v[8][4];
#pragma unroll
      for (int i = 0; i < 8; ++i) decode<K, NP == 1>(cw[i], s2, off, v[i]);
      uint32_t keep[4];
#pragma unroll
      for (int q = 0; q < 4; ++q)
        keep[q] = (a_ok && aw0 + 2 * q < W ? 0xFFFFu : 0u) | (a_ok && aw0 + 2 * q + 1 < W ? 0xFFFF0000u : 0u);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        uint32_t u[4];
        if (NP == 1) {
#pragma unroll
          for (int q = 0; q < 4; ++q) u[q] = round2(v[2 * q][e], v[2 * q + 1][e]) & keep[q];
        } else if (part == 0) {
#pragma unroll
          for (int q = 0; q < 4; ++q) u[q] = upper2(v[2 * q][e], v[2 * q + 1][e]) & keep[q];
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q) u[q] = part2(v[2 * q][e], v[2 * q + 1][e], part) & keep[q];
        }
        *reinterpret_cast<uint4*>(a_st + buf * abytes + e * 128) = make_uint4(u[0], u[1], u[2], u[3]);
      }
    }
  };

  floatx4 acc[9][2];
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int o = 0; o < 2; ++o) acc[t][o] = floatx4{0.f, 0.f, 0.f, 0.f};

  // fragment addresses of the group's two k-steps kg and kg + 2: positions 8 (4 ks + lk) ..
  int a_ad[2], d_ad[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int gr = 4 * (kg + 2 * s) + lk;
    int row = gr / ck.dw8;
    const int w8 = gr - row * ck.dw8;
    row = row < drows ? row + 2 * (row / Hc) : 0;   // (past the rows dy is zero: any finite v)
    a_ad[s] = (row * ck.aw8 + w8 + 1) * AGRP + (16 * wc + li) * 16;
    d_ad[s] = (gr * TCO + 16 * wo + li) * 16;   // the wave's tiles: slots 16 wo .. and 32 + 16 wo ..
  }
  // nks: k-steps of the chunk
  auto contract = [&](int buf, int nks, auto ones) __attribute__((always_inline)) {
    const unsigned char* Ab = A0 + buf * abytes;
    const unsigned char* Db = D0 + buf * DBYTES;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      if (kg + 2 * s >= nks) continue;
      bf16x8_t d[2][NP];
#pragma unroll
      for (int o = 0; o < 2; ++o)
#pragma unroll
        for (int t = 0; t < NP; ++t) d[o][t] = *reinterpret_cast<const bf16x8_t*>(Db + d_ad[s] + o * 512 + t * DPART);
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        const unsigned char* ap = Ab + a_ad[s] + r * ck.aw8 * AGRP;
        const uint4 m = *reinterpret_cast<const uint4*>(ap);
        const uint32_t lw = *reinterpret_cast<const uint32_t*>(ap - AGRP + 12), rw = *reinterpret_cast<const uint32_t*>(ap + AGRP);
        const uint4 l = make_uint4(__builtin_amdgcn_alignbit(m.x, lw, 16), __builtin_amdgcn_alignbit(m.y, m.x, 16),
                                   __builtin_amdgcn_alignbit(m.z, m.y, 16), __builtin_amdgcn_alignbit(m.w, m.z, 16));
        const uint4 h = make_uint4(l.y, l.z, l.w, __builtin_amdgcn_alignbit(rw, m.w, 16));
        const uint4 a[3] = {l, m, h};
        if constexpr (decltype(ones)::value) {
#pragma unroll
          for (int q = 0; q < 3; ++q) {
            const bf16x8_t one = __builtin_bit_cast(bf16x8_t, missing_ones(a[q]));
#pragma unroll
            for (int t = 1; t >= 0; --t)
#pragma unroll
              for (int o = 0; o < 2; ++o)
                acc[3 * r + q][o] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(d[o][t], one, acc[3 * r + q][o], 0, 0, 0);
          }
        }
        // (the small parts first; consecutive MFMAs on different accumulators)
#pragma unroll
        for (int t = NP - 1; t >= 0; --t)
#pragma unroll
          for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int o = 0; o < 2; ++o)
              acc[3 * r + q][o] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(d[o][t], __builtin_bit_cast(bf16x8_t, a[q]),
                                                                          acc[3 * r + q][o], 0, 0, 0);
      }
    }
  };
  auto pass = [&](int part, auto ones) __attribute__((always_inline)) {
    if (c_begin < c_end) stage_load(c_begin);
    __syncthreads();   // (the buffers of the part before have been read)
    stage_store(0, part);
    if (c_begin + 1 < c_end) stage_load(c_begin + 1);
    __syncthreads();
    for (int c = c_begin; c < c_end; ++c) {
      const int buf = (c - c_begin) & 1;
      const bool more = c + 1 < c_end;
      if (kg == 0 && more) {
        stage_store(buf ^ 1, part);
        if (c + 2 < c_end) stage_load(c + 2);
      }
      // (the last chunk of an image has fewer rows)
      const int rows = ck.TI > 1 ? drows : min(ck.R, H - c % ck.nch * ck.R);
      contract(buf, (rows * ck.dw8 + 3) / 4, ones);
      if (kg == 1 && more) {
        stage_store(buf ^ 1, part);
        if (c + 2 < c_end) stage_load(c + 2);
      }
      __syncthreads();
    }
  };
  if constexpr (NP == 1) {
    pass(0, std::false_type{});
  } else if (mode == 1) {
    pass(0, std::true_type{});
  } else {
    const int parts = mode == 0 ? 1 : mode;
#pragma unroll 1
    for (int part = 0; part < parts; ++part) pass(part, std::false_type{});
  }

  // ---- the two groups' sums: group 0 finishes the taps 0 .. 4, group 1 the others
  {
    unsigned char* to = smem + (size_t)((wave ^ 4) * 10) * 1024 + lane * 16;
    const unsigned char* from = smem + (size_t)(wave * 10) * 1024 + lane * 16;
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
      for (int o = 0; o < 2; ++o)
        if ((t < 5) == (kg == 1)) *reinterpret_cast<floatx4*>(to + ((t < 5 ? t : t - 5) * 2 + o) * 1024) = acc[t][o];
    __syncthreads();
    // the lane holds output channels co + 2 r + o of input channel ci (slot 16 wc + li)
    const int ci = ci0 + 4 * (li & 7) + 2 * wc + (li >> 3), co = co0 + 32 * wo + 8 * lk;
    const float half_step = NP == 1 ? 1.0f : 0.5f * fabsf(stats[P_STEP * Cin + ci]);
    float bad = 0.0f;
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
      for (int o = 0; o < 2; ++o)
        if ((t < 5) == (kg == 0)) {
          acc[t][o] = half_step * (acc[t][o] + *reinterpret_cast<const floatx4*>(from + ((t < 5 ? t : t - 5) * 2 + o) * 1024));
          if (NP == 3) acc[t][o] *= kDown;   // (last: the product before it is normal wherever the result is not zero)
#pragma unroll
          for (int r = 0; r < 4; ++r) bad = fmaf(acc[t][o][r], 0.0f, bad);
        }
    // sums that are not finite (an infinity in dy, or a value that rounds to an infinite bf16, splits into NaN):
    // again from the operands, one after the other
    if (NP == 3 && __builtin_expect(bad != 0.0f, 0)) {
      const int rows_all = g.N * H;
      const int r0 = ck.TI > 1 ? c_begin * ck.TI * H : c_begin / ck.nch * H + c_begin % ck.nch * ck.R;
      const int r1 = ck.TI > 1 ? c_end * ck.TI * H : c_end / ck.nch * H + c_end % ck.nch * ck.R;
      for (int e = 0; e < 9 * 2 * 4; ++e) {
        float x = 0.0f;
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
          for (int o = 0; o < 2; ++o)
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (e == (t * 2 + o) * 4 + r && (t < 5) == (kg == 0)) x = acc[t][o][r];
        if (fabsf(x) < INFINITY) continue;
        x = exact_sum<K>(codes, stats, dy, H, W, Cin, Cout, e / 8, ci, co + 2 * (e & 3) + ((e >> 2) & 1), r0 * W,
                         min(r1, rows_all) * W);
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
          for (int o = 0; o < 2; ++o)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[t][o][r] = e == (t * 2 + o) * 4 + r ? x : acc[t][o][r];
      }
    }
    float* out = dst + ((size_t)split * 9 * Cin + ci) * Cout + co;
#pragma unroll
    for (int t = 0; t < 9; ++t)
      if ((t < 5) == (kg == 0)) {
        const floatx4 x = acc[t][0], y = acc[t][1];
        *reinterpret_cast<floatx4*>(out + (size_t)t * Cin * Cout) = floatx4{x[0], y[0], x[1], y[1]};
        *reinterpret_cast<floatx4*>(out + (size_t)t * Cin * Cout + 4) = floatx4{x[2], y[2], x[3], y[3]};
      }
  }
}

// ---- 1x1 stride-1 layers ---------------------------------------------------------------------------------
// The same products with one tap and no border: dW[ci][co] = step / 2 * sum over pixels of v[pixel][ci] * dy[pixel][co],
// a plain matrix product over all N H W pixels.  One block owns a CI x CO tile and a share of the pixels, 64 at a time
// in two buffers; its eight waves are two groups of 2 x 2, a group takes one of the chunk's two k-steps, a wave a
// quarter of the tile.  A 128 x 128 tile has 48 MFMAs per wave and k-step for 16 reads and, per chunk, some 150
// vector instructions of staging (dy is split once per 128 input channels, a code decoded once per 128 output
// channels), which run under the other group's MFMAs.
constexpr int PX1 = 64;                          // pixels per chunk

template <int K, int CI, int CO, int NP>
__global__ __launch_bounds__(THREADS, 2) void split_wgrad1_kernel(const uint8_t* __restrict__ codes,
                                                                  const float* __restrict__ stats,
                                                                  const float* __restrict__ dy, float* __restrict__ dst,
                                                                  int M, int Cin, int Cout, int splits) {
  constexpr int DPART1 = PX1 / 8 * CO * 16, DB = NP * DPART1, AB = PX1 / 8 * CI * 16, IT = CI / 32, OT = CO / 32;   // 16-channel tiles of a wave
  constexpr int DCH = CO / 64, ACH = CI / 64;    // channels per staging item (eight pixels of them)
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  unsigned char* const D0 = smem;                // [2][part][group][co]
  unsigned char* const A0 = smem + 2 * DB;       // [2][group][ci]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lk = lane >> 4;
  const int kg = wave >> 2, wc = wave & 1, wo = (wave >> 1) & 1;
  const int n_ci = Cin / CI, n_co = Cout / CO;
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
  const int ci0 = ci_blk * CI, co0 = co_blk * CO;
  const int chunks = (M + PX1 - 1) / PX1;
  const int c_begin = (int)((int64_t)split * chunks / splits), c_end = (int)((int64_t)(split + 1) * chunks / splits);

  // staging role: pixels 8 sg .. of channels DCH sc .. (dy) and ACH sc .. (v)
  const int sg = wave, sc = lane;
  float s2[ACH], off[ACH];
  float vmax = 0.0f;
#pragma unroll
  for (int e = 0; e < ACH; ++e) {
    if constexpr (NP == 3) vmax = fmaxf(vmax, decode_consts<K>(stats, Cin, ci0 + ACH * sc + e, s2[e], off[e]));
    else decode_consts_bf16<K>(stats, Cin, ci0 + ACH * sc + e, s2[e], off[e]);
  }
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) vmax = fmaxf(vmax, __shfl_xor(vmax, d, 64));   // (a wave holds all CI channels)
  const int mode = __builtin_amdgcn_readfirstlane(decode_mode(vmax));

  using code_t = typename std::conditional<K * ACH == 16, uint16_t, uint8_t>::type;   // ACH codes
  constexpr bool HALF = K * ACH == 4;            // one 4-bit code: half a byte
  const uint32_t d_lane = (uint32_t)(DCH * sc) * 4u, c_lane = (uint32_t)(ACH * sc * K / 8);
  float dv[DCH][8];
  uint32_t cw[8];
  int left = 0;                                  // pixels from the item's first to the tensor's end
  auto stage_load = [&](int c) __attribute__((always_inline)) {
    const int px0 = c * PX1 + 8 * sg;            // (uniform: a wave's item rows)
    left = M - px0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int p = min(px0 + i, M - 1);
      const char* src = reinterpret_cast<const char*>(dy + (size_t)p * Cout + co0);
      if constexpr (DCH == 2) {
        const float2 v = *reinterpret_cast<const float2*>(src + d_lane);
        dv[0][i] = v.x;
        dv[1][i] = v.y;
      } else {
        dv[0][i] = *reinterpret_cast<const float*>(src + d_lane);
      }
      const uint8_t* cs = codes + ((size_t)p * Cin + ci0) * K / 8;
      cw[i] = *reinterpret_cast<const code_t*>(cs + c_lane);
    }
  };
  auto stage_store = [&](int buf, int part) __attribute__((always_inline)) {
    if (left < 8) {
#pragma unroll
      for (int ch = 0; ch < DCH; ++ch)
#pragma unroll
        for (int i = 0; i < 8; ++i) dv[ch][i] = i < left ? dv[ch][i] : 0.0f;
    }
#pragma unroll
    for (int ch = 0; ch < DCH; ++ch) {
      uint4 u[NP];
      split_dy<NP>(dv[ch], u);
#pragma unroll
      for (int t = 0; t < NP; ++t)
        *reinterpret_cast<uint4*>(D0 + buf * DB + t * DPART1 + (sg * CO + 64 * ch + sc) * 16) = u[t];
    }
    float v[8][ACH];
#pragma unroll
    for (int i = 0; i < 8; ++i) decode<K, NP == 1>(cw[i] >> (HALF ? 4 * (sc & 1) : 0), s2, off, v[i]);
#pragma unroll
    for (int e = 0; e < ACH; ++e) {
      uint32_t u[4];
      if (NP == 1) {
#pragma unroll
        for (int q = 0; q < 4; ++q) u[q] = round2(v[2 * q][e], v[2 * q + 1][e]);
      } else if (part == 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q) u[q] = upper2(v[2 * q][e], v[2 * q + 1][e]);
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) u[q] = part2(v[2 * q][e], v[2 * q + 1][e], part);
      }
      *reinterpret_cast<uint4*>(A0 + buf * AB + (sg * CI + 64 * e + sc) * 16) = make_uint4(u[0], u[1], u[2], u[3]);
    }
  };

  floatx4 acc[IT][OT];
#pragma unroll
  for (int i = 0; i < IT; ++i)
#pragma unroll
    for (int o = 0; o < OT; ++o) acc[i][o] = floatx4{0.f, 0.f, 0.f, 0.f};
  // tile i / o of a wave: slots 64 (i / 2) + 32 wc + 16 (i % 2) ..; channel c of two per thread sits in slot c / 2 + 64 (c % 2)
  const int a_ad = ((4 * kg + lk) * CI + 32 * wc + li) * 16;
  const int d_ad = ((4 * kg + lk) * CO + 32 * wo + li) * 16;
  auto contract = [&](int buf, auto ones) __attribute__((always_inline)) {
    bf16x8_t a[IT], one[IT];
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      a[i] = *reinterpret_cast<const bf16x8_t*>(A0 + buf * AB + a_ad + (64 * (i >> 1) + 16 * (i & 1)) * 16);
      if constexpr (decltype(ones)::value) one[i] = __builtin_bit_cast(bf16x8_t, missing_ones(__builtin_bit_cast(uint4, a[i])));
    }
#pragma unroll
    for (int o = 0; o < OT; ++o) {
      bf16x8_t d[NP];
#pragma unroll
      for (int t = 0; t < NP; ++t) d[t] = *reinterpret_cast<const bf16x8_t*>(D0 + buf * DB + d_ad + (64 * (o >> 1) + 16 * (o & 1)) * 16 + t * DPART1);
      if constexpr (decltype(ones)::value) {
#pragma unroll
        for (int t = 1; t >= 0; --t)
#pragma unroll
          for (int i = 0; i < IT; ++i) acc[i][o] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(d[t], one[i], acc[i][o], 0, 0, 0);
      }
#pragma unroll
      for (int t = NP - 1; t >= 0; --t)   // (the small parts first)
#pragma unroll
        for (int i = 0; i < IT; ++i) acc[i][o] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(d[t], a[i], acc[i][o], 0, 0, 0);
    }
  };
  auto pass = [&](int part, auto ones) __attribute__((always_inline)) {
    if (c_begin < c_end) stage_load(c_begin);
    __syncthreads();   // (the buffers of the part before have been read)
    stage_store(0, part);
    if (c_begin + 1 < c_end) stage_load(c_begin + 1);
    __syncthreads();
    for (int c = c_begin; c < c_end; ++c) {
      const int buf = (c - c_begin) & 1;
      const bool more = c + 1 < c_end;
      if (kg == 0 && more) {
        stage_store(buf ^ 1, part);
        if (c + 2 < c_end) stage_load(c + 2);
      }
      contract(buf, ones);
      if (kg == 1 && more) {
        stage_store(buf ^ 1, part);
        if (c + 2 < c_end) stage_load(c + 2);
      }
      __syncthreads();
    }
  };
  if constexpr (NP == 1) {
    pass(0, std::false_type{});
  } else if (mode == 1) {
    pass(0, std::true_type{});
  } else {
    const int parts = mode == 0 ? 1 : mode;
#pragma unroll 1
    for (int part = 0; part < parts; ++part) pass(part, std::false_type{});
  }

  // the two groups' sums: group 0 finishes the lower half of the tiles of ci, group 1 the upper
  constexpr int IH = IT / 2;
  unsigned char* to = smem + (size_t)((wave ^ 4) * IH * OT) * 1024 + lane * 16;
  const unsigned char* from = smem + (size_t)(wave * IH * OT) * 1024 + lane * 16;
#pragma unroll
  for (int i = 0; i < IT; ++i)
#pragma unroll
    for (int o = 0; o < OT; ++o)
      if ((i < IH) == (kg == 1)) *reinterpret_cast<floatx4*>(to + ((i % IH) * OT + o) * 1024) = acc[i][o];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    if ((i < IH) != (kg == 0)) continue;
    const int ci = ci0 + ACH * (32 * wc + 16 * (i & 1) + li) + (i >> 1);
    const float half_step = NP == 1 ? 1.0f : 0.5f * fabsf(stats[P_STEP * Cin + ci]);
#pragma unroll
    for (int o = 0; o < OT; ++o) {
      acc[i][o] = half_step * (acc[i][o] + *reinterpret_cast<const floatx4*>(from + ((i % IH) * OT + o) * 1024));
      if (NP == 3) acc[i][o] *= kDown;   // (last: the product before it is normal wherever the result is not zero)
    }
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      // the lane's output channels co .. in order: element r of tile p (and of tile p + 2)
      const int co = co0 + DCH * (32 * wo + 16 * p + 4 * lk);
      float s[4 * DCH];
      float bad = 0.0f;
#pragma unroll
      for (int e = 0; e < 4 * DCH; ++e) {
        s[e] = DCH == 2 ? acc[i][p + 2 * (e & 1)][e >> 1] : acc[i][p][e];
        bad = fmaf(s[e], 0.0f, bad);
      }
      if (NP == 3 && __builtin_expect(bad != 0.0f, 0))   // (as above)
#pragma unroll 1
        for (int r = 0; r < 4 * DCH; ++r) {
          float was = 0.0f;
#pragma unroll
          for (int q = 0; q < 4 * DCH; ++q) was = q == r ? s[q] : was;
          if (fabsf(was) < INFINITY) continue;
          const float x = exact_sum<K>(codes, stats, dy, 1, 1, Cin, Cout, 4, ci, co + r, c_begin * PX1, min(c_end * PX1, M));
#pragma unroll
          for (int q = 0; q < 4 * DCH; ++q) s[q] = q == r ? x : s[q];
        }
      float* out = dst + ((size_t)split * Cin + ci) * Cout + co;
#pragma unroll
      for (int h = 0; h < DCH; ++h)
        *reinterpret_cast<floatx4*>(out + 4 * h) = floatx4{s[4 * h], s[4 * h + 1], s[4 * h + 2], s[4 * h + 3]};
    }
  }
}

struct Tile1 {
  int ci, co, splits;
};

bool make_tile1(const ConvGeom& g, int K, size_t room, Tile1& t) {
  if (g.R != 1 || g.S != 1 || g.stride != 1 || g.pad != 0 || (K != 4 && K != 8)) return false;
  if (g.Cin % 64 != 0 || g.Cout % 64 != 0) return false;
  const int64_t M = (int64_t)g.N * g.H * g.W;
  if (M * g.Cin >= ((int64_t)1 << 31) || M * g.Cout >= ((int64_t)1 << 31)) return false;
  t.ci = g.Cin % 128 == 0 ? 128 : 64;
  t.co = g.Cout % 128 == 0 ? 128 : 64;
  const int tiles = (g.Cin / t.ci) * (g.Cout / t.co);
  const size_t n = (size_t)g.Cin * g.Cout * sizeof(float);
  int64_t s = 256 / tiles;
  if (s > (int64_t)(room / n)) s = (int64_t)(room / n);
  if (s > M / (4 * PX1)) s = M / (4 * PX1);
  if (s < 1) s = 1;
  t.splits = (int)s;
  return s * tiles >= 96;
}

template <int K, int NP, int CI, int CO>
int launch_tile1(hipStream_t st, const ConvGeom& g, const Tile1& t, const void* packed, const float* stats, const float* dy,
                 float* dst) {
  auto kern = split_wgrad1_kernel<K, CI, CO, NP>;
  if (int e = allow_full_lds(reinterpret_cast<const void*>(kern))) return e;
  constexpr size_t stage = (size_t)2 * (PX1 / 8) * 16 * (NP * CO + CI), xch = (size_t)8 * (CI / 64) * (CO / 32) * 1024;
  const unsigned grid = (unsigned)(t.splits * (g.Cin / CI) * (g.Cout / CO));
  kern<<<grid, THREADS, stage > xch ? stage : xch, st>>>(static_cast<const uint8_t*>(packed), stats, dy, dst, g.N * g.H * g.W,
                                                         g.Cin, g.Cout, t.splits);
  return hip_status();
}

template <int K, int NP>
int launch_1x1(hipStream_t st, const ConvGeom& g, const Tile1& t, const void* packed, const float* stats, const float* dy,
               float* dst) {
  if (t.ci == 128) return t.co == 128 ? launch_tile1<K, NP, 128, 128>(st, g, t, packed, stats, dy, dst)
                                      : launch_tile1<K, NP, 128, 64>(st, g, t, packed, stats, dy, dst);
  return t.co == 128 ? launch_tile1<K, NP, 64, 128>(st, g, t, packed, stats, dy, dst)
                     : launch_tile1<K, NP, 64, 64>(st, g, t, packed, stats, dy, dst);
}

// Whether the shares are long enough for the multiplications they do: a share's launch costs some 5 us more than a tiled
// kernel's and its k-steps about 1.9 us each, a tiled kernel 0.34 us per 10^6 multiplications and tap (bf16 operands a little
// less).  What counts is the longest share, in k-steps of one of the two groups of waves: rows that fill no k-step and
// images that fill no chunk make it long.  (us, here / tiled: 64 -> 64 @10x10 N=64, 5 steps for 26, 22.4 / 17.0; 64 -> 64
// @15x15 N=32, 4 for 29, 21.1 / 17.8; 96 -> 192 @9x9 N=32, 8 for 48, 28.9 / 26.0; 64 -> 64 @16x16 N=32, 2 for 34, 18.1 /
// 20.6; 96 -> 192 @11x11 N=64, 15 for 143, 41.8 / 50.0; bf16 128 -> 128 @9x9 N=32, 6 for 42, 21.8 / 20.3.)
bool shares_pay(const ConvGeom& g, bool bf16, const Chunking& c) {
  const int per = (c.chunks + c.splits - 1) / c.splits;   // chunks of the longest share
  const int rows = c.TI > 1 ? c.TI * c.R : c.R, last = g.H - (c.nch - 1) * c.R;
  const int short_ones = c.nch > 1 ? per / c.nch : 0;
  auto steps = [&](int r) { return ((r * c.dw8 + 3) / 4 + 1) / 2; };
  const double most = (double)(per - short_ones) * steps(rows) + (double)short_ones * steps(last);
  const double work = 1e-6 * g.N * g.H * g.W * g.Cin * g.Cout;
  return bf16 ? 6.5 * most + 20.0 < work : 5.5 * most + 14.0 < work;
}

bool make_chunking(const ConvGeom& g, int K, bool bf16, size_t room, Chunking& c) {
  if (g.R != 3 || g.S != 3 || g.stride != 1 || g.pad != 1 || (K != 4 && K != 8)) return false;
  if (g.Cin % TCI != 0 || g.Cout % TCO != 0) return false;
  const int64_t M = (int64_t)g.N * g.H * g.W;
  if (M * g.Cin >= ((int64_t)1 << 31) || M * g.Cout >= ((int64_t)1 << 31)) return false;
  c.dw8 = (g.W + 7) / 8;
  c.aw8 = (g.W + 8) / 8;   // at least one zero after a row
  int rows = POS / 8 / c.dw8;
  if (rows < 1) return false;
  // (60 groups of v: one item per thread, and both buffers in 160 KB)
  while (rows > 1 && (rows + 2) * c.aw8 > 60) --rows;
  if ((rows + 2) * c.aw8 > 60) return false;
  c.TI = 1;
  c.R = rows;
  if (rows >= g.H) {
    c.R = g.H;
    c.TI = rows / g.H;
    while (c.TI > 1 && c.TI * (g.H + 2) * c.aw8 > 60) --c.TI;
  }
  c.nch = (g.H + c.R - 1) / c.R;
  c.chunks = c.TI > 1 ? (g.N + c.TI - 1) / c.TI : g.N * c.nch;
  c.agroups = c.TI * (c.R + 2) * c.aw8 + 2;
  const int tiles = (g.Cin / TCI) * (g.Cout / TCO);
  const size_t n = (size_t)9 * g.Cin * g.Cout * sizeof(float);
  int64_t s = 256 / tiles;
  if (s > (int64_t)(room / n)) s = (int64_t)(room / n);
  if (s > c.chunks) s = c.chunks;
  if (s < 1) s = 1;
  c.splits = (int)s;
  return s * tiles >= 96 && shares_pay(g, bf16, c);
}

}  // namespace

int split_wgrad_copies(const ConvGeom& g, int K, bool bf16, size_t room) {
  Tile1 t;
  if (make_tile1(g, K, room, t)) return t.splits;
  Chunking c;
  return make_chunking(g, K, bf16, room, c) ? c.splits : 0;
}

int launch_split_wgrad(hipStream_t st, const ConvGeom& g, int K, bool bf16, const void* packed, const float* stats,
                       const float* dy, float* dst, size_t room) {
  Tile1 t;
  if (make_tile1(g, K, room, t)) {
    if (bf16) return K == 4 ? launch_1x1<4, 1>(st, g, t, packed, stats, dy, dst) : launch_1x1<8, 1>(st, g, t, packed, stats, dy, dst);
    return K == 4 ? launch_1x1<4, 3>(st, g, t, packed, stats, dy, dst) : launch_1x1<8, 3>(st, g, t, packed, stats, dy, dst);
  }
  Chunking c;
  if (!make_chunking(g, K, bf16, room, c)) return ABL_ERR_SHAPE;
  size_t lds = 2 * ((size_t)(bf16 ? 1 : 3) * DPART + c.agroups * AGRP);
  if (lds < (size_t)80 * 1024) lds = (size_t)80 * 1024;   // the exchange of the two groups' sums
  const unsigned grid = (unsigned)(c.splits * (g.Cin / TCI) * (g.Cout / TCO));
  auto kern = bf16 ? (K == 4 ? split_wgrad_kernel<4, 1> : split_wgrad_kernel<8, 1>)
                   : (K == 4 ? split_wgrad_kernel<4, 3> : split_wgrad_kernel<8, 3>);
  if (int e = allow_full_lds(reinterpret_cast<const void*>(kern))) return e;
  kern<<<grid, THREADS, lds, st>>>(static_cast<const uint8_t*>(packed), stats, dy, dst, g, c);
  return hip_status();
}

}  // namespace abl
