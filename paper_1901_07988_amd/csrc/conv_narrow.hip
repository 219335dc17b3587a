// Layers of few channels (up to 64 in, 128 out) on small tensors: any filter up to 5x5, stride 1 or 2, any padding, channel counts
// that no tile divides.  fp32 operands split into three bf16 parts (as in conv_split.hip).
//
//   narrow_fwd_kernel   Eq. 1 (second pass), Eq. 1-3 and Eq. 9 while the patch is staged, Eq. 4, shortcut, first pass of Eq. 1 of y;
//                       or Eq. 4 of a given A3
//   narrow_bwd_kernel   Eq. 5 and the first pass of Eq. 6-7: blocks that contract the gradient to the input and blocks that contract
//                       the gradient of the weights side by side in one launch
//
// What bounds such a layer is a chain of dependent launches of 4-5 us each and, within a kernel, the chain of first loads, staging,
// contraction and epilogue; the chip is rarely full.  So there are few launches, and a block stages its patch once, whole rows of
// one image with all channels, and contracts all taps from it.  The contraction index is flattened into (tap, eight channels): a
// table in LDS says where piece k of a pixel lies and which weights belong to it, so that a 32-deep step takes four pieces whatever
// the filter is.  The data gradient of a strided layer takes the pixels class by class of (row, column) modulo the stride, with the
// taps that reach the class.  Weights are split by the waves that use them, a step ahead.
//
// LDS: planes of 16-byte pieces of eight channels; the three parts of a position are adjacent (a pitch of 48 bytes: the 16
// positions of a fragment fall on all banks, and the parts are constant offsets).  The weight gradient reads the planes with
// ds_read_b64_tr_b16, as in conv_c16.hip.
//
// Where the time goes (3x3 64 -> 64 @8x8 N=128, us in a kernel): forward first loads with the sums 2.8, staging 1.5, contraction 7
// (per 32-deep step and wave some 75 vector instructions, 52 of them the split of the weights, and 6 MFMAs a pixel tile), epilogue
// 1; data gradient 2.2, 9, 2; weight gradient beside it 5.3, 3, 3 + 3 for two images, 1.3 for its copy.  The layer 60 -> 48, with
// 3x3 16 -> 32 stride 2 @32x32 N=128 73 -> 53, 20 -> 36 @27x21 N=50 104 -> 62.
//
// Codes are compared bit for bit with an IEEE fp32 evaluation: this file is compiled with floating-point contraction off.

#include <algorithm>
#include <cstring>
#include <type_traits>

#include "abl_internal.h"

#pragma clang fp contract(off)

namespace abl {
namespace {

constexpr int kT = 512, kWaves = kT / 64;
constexpr int kLds = 160 * 1024;
constexpr int kPitch = 48;      // bytes of a position in three parts
constexpr int kUnits = 6;      // (16 x 16 channels, three taps) of dW that a wave keeps at most

// Rows of tiles of one role of one direction.
struct Tiles {
  int TH, per_image, count;    // output rows of a tile
  int PH, PW, npos, plane;     // positions of the input patch at most, bytes of a plane of it
  int DH, DW, dpos, dplane;    // of the patch of dy
  int rows;                    // of the input that a tile owns at most
};
struct NarrowPlan {
  int N, H, W, Ho, Wo, Cin, Cout, R, S, st, pad;
  int ip, op;                  // pieces of eight channels
  Tiles t;                     // of the forward, of the gradient to the input
  int steps, entries;
  bool outside;                // zeros around the image take part next to infinities (channel counts in tiles)
  bool masked;                 // pieces or rows of the weights with fewer channels than they hold
  int kw;                      // waves that share the steps of a unit of work
  int blocks, lds;
  Tiles w;                     // of the weight gradient
  int per_wave, nsub, copies, wlds;   // units of a wave, blocks that share a copy
  float fwd_us, dgrad_us, wgrad_us;   // what the plans expect
  Divisor by_pw, by_wo, by_tiles, by_ip, by_op, by_dw, by_nw0, by_nw1, wby_pw, wby_tiles;
};

// Channels c0 .. c0 + 7 of C as they are in memory (past the last: any; `below` clears them where they are used - a select next to
// the load would wait for it).
template <bool VEC>
__device__ inline void load8(const float* __restrict__ p, int c0, int C, float (&v)[8]) {
  if constexpr (VEC) {
    const float4 a = *reinterpret_cast<const float4*>(p + c0), b = *reinterpret_cast<const float4*>(p + (c0 + 4 < C ? c0 + 4 : c0));
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = p[c0 + e < C ? c0 + e : C - 1];
  }
}
__device__ inline void below(int n, float (&v)[8]) {
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = e < n ? v[e] : 0.0f;
}
// Asks for one value of each line of a part of the weights, another part in the next block of the same XCD: together they bring
// them into its L2 while the patches are staged.
__device__ inline float warm(const float* __restrict__ w, int n, int block) {
  const int parts = (n + 32 * kT - 1) / (32 * kT), k = 32 * ((int)threadIdx.x + (block >> 3) % parts * kT);
  return w[k < n ? k : 0];
}

template <int K>
__device__ inline uint32_t code_at(const uint8_t* p, int64_t e) {
  if constexpr (K == 4) return (p[e >> 1] >> (4 * (e & 1))) & 15u;
  else return p[e];
}
// Codes of four channels c0 .. c0 + 3 (those below C), element e = channel c0.
template <int K, bool VEC>
__device__ inline uint32_t codes4(const uint8_t* p, int64_t e, int c0, int C) {
  if constexpr (VEC && K == 4) return *reinterpret_cast<const uint16_t*>(p + (e >> 1));
  if constexpr (VEC) return *reinterpret_cast<const uint32_t*>(p + e);
  uint32_t w = 0;
#pragma unroll
  for (int r = 0; r < 4; ++r) w |= (c0 + r < C ? code_at<K>(p, e + r) : 0u) << (K * r);
  return w;
}

// A piece of the contraction: where it lies from the pixel's first, where its weights begin, how many of its channels exist.
struct Entry {
  int off, w, n, pad;
};

template <int MT>
struct Acc {
  floatx4 big[2][MT], rest[2][MT];
  __device__ inline void clear() {
#pragma unroll
    for (int t = 0; t < MT; ++t) big[0][t] = big[1][t] = rest[0][t] = rest[1][t] = floatx4{0.f, 0.f, 0.f, 0.f};
  }
  // six of the nine products (the others are below 2^-24 of it); the large ones of even and odd steps apart: half the roundings
  template <int S>
  __device__ inline void step(const bf16x8_t (&a)[3], const bf16x8_t (&b)[MT][3]) {
#pragma unroll
    for (int t = 0; t < MT; ++t) rest[0][t] = mfma32(a[2], b[t][0], rest[0][t]);
#pragma unroll
    for (int t = 0; t < MT; ++t) rest[1][t] = mfma32(a[0], b[t][2], rest[1][t]);
#pragma unroll
    for (int t = 0; t < MT; ++t) big[S][t] = mfma32(a[0], b[t][0], big[S][t]);
#pragma unroll
    for (int t = 0; t < MT; ++t) rest[0][t] = mfma32(a[1], b[t][1], rest[0][t]);
#pragma unroll
    for (int t = 0; t < MT; ++t) rest[1][t] = mfma32(a[1], b[t][0], rest[1][t]);
#pragma unroll
    for (int t = 0; t < MT; ++t) rest[0][t] = mfma32(a[0], b[t][1], rest[0][t]);
  }
  __device__ inline float sum(int t, int r) const { return (big[0][t][r] + big[1][t][r]) + (rest[0][t][r] + rest[1][t][r]); }
};

// The sums of `kw` waves for the same unit, wave = kq * nu + unit: left in LDS by the others (the patch has been read by then) and
// added by the first in order.  Every wave of the block comes here.
template <int MT>
__device__ inline void together(char* lds, int kw, int kq, int unit, int nu, bool work, const Acc<MT>& acc, float (&o)[MT][4]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) o[t][r] = acc.sum(t, r);
  if (kw > 1) {
    __syncthreads();
    if (work && kq > 0)
#pragma unroll
      for (int t = 0; t < MT; ++t)
        reinterpret_cast<float4*>(lds)[(((kq - 1) * nu + unit) * MT + t) * 64 + lane] = make_float4(o[t][0], o[t][1], o[t][2], o[t][3]);
    __syncthreads();
    if (work && kq == 0)
      for (int k = 1; k < kw; ++k)
#pragma unroll
        for (int t = 0; t < MT; ++t) {
          const float4 v = reinterpret_cast<const float4*>(lds)[(((k - 1) * nu + unit) * MT + t) * 64 + lane];
          o[t][0] += v.x; o[t][1] += v.y; o[t][2] += v.z; o[t][3] += v.w;
        }
  }
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) o[t][r] *= kDown;
}

// Steps s0 .. s1 - 1 of the pieces from `tab` for MT pixels of 16; weights(entry, v) asks for a lane's eight; `row`: the lane's row of
// the weights exists.  Weights are asked for two steps ahead, the pixels' pieces one, the table's entries three: what a step waits
// for has come by then (without that a step of 24 MFMAs took twice its instructions' time).
template <int MT, class Weights>
__device__ inline void contract(const char* lds, const Entry* tab, int s0, int s1, const int (&base)[MT], int lk, bool masked, bool row,
                                Acc<MT>& acc, Weights&& weights) {
  if (s0 >= s1) return;
  float w[2][8];
  bf16x8_t b[2][MT][3];
  auto entry = [&](int s) __attribute__((always_inline)) { return tab[4 * (s < s1 ? s : s1 - 1) + lk]; };
  auto fetch = [&](int off, bf16x8_t (&to)[MT][3]) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
      for (int q = 0; q < 3; ++q) to[t][q] = piece(lds + base[t] + off + 16 * q);
  };
  Entry e0 = entry(s0), e1 = entry(s0 + 1), e2 = entry(s0 + 2);
  weights(e0, w[0]);
  weights(e1, w[1]);
  fetch(e0.off, b[0]);
  auto one = [&](auto par, int s) __attribute__((always_inline)) {
    constexpr int P = decltype(par)::value;
    fetch(e1.off, b[1 - P]);
    const Entry e3 = entry(s + 3);
    __builtin_amdgcn_sched_barrier(0);
    bf16x8_t a[3];
    if (masked) below(row ? e0.n : 0, w[P]);
    split3(w[P], a[0], a[1], a[2]);
    __builtin_amdgcn_sched_barrier(0);
    weights(e2, w[P]);
    acc.template step<P>(a, b[P]);
    e0 = e1;
    e1 = e2;
    e2 = e3;
  };
#pragma unroll 1
  for (int s = s0; s + 1 < s1; s += 2) {
    one(std::integral_constant<int, 0>{}, s);
    one(std::integral_constant<int, 1>{}, s + 1);
  }
  if ((s1 - s0) % 2 != 0) one(std::integral_constant<int, 0>{}, s1 - 1);
}

// ---- forward --------------------------------------------------------------------------------------------------
struct NarrowFwd {
  const float *x, *w, *skip;   // x: the layer's input, or A3 (K = 0)
  const double* partial;       // nb rows of the statistics' sums, taken around `shift` (nullable); nb = 0: `stats` is there already
  int nb;
  const float *shift, *gamma, *beta;
  float *stats, *y;
  uint8_t* packed;
  int pack_pad;
  double* out_partial;         // nullable: sums of y and y^2, a row per block
  int64_t M;
};

// K = 0: no prologue, x is A3.  MT: pixels in sixteens of a unit of work (16 output channels).  VEC: channels in fours.
template <int K, int MT, bool VEC>
__global__ __launch_bounds__(kT, 2) void narrow_fwd_kernel(NarrowFwd a, NarrowPlan p) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int ip = p.ip, nj = (p.Cout + 15) / 16, cp = 8 * ip, plane = p.t.plane;
  Entry* const tab = reinterpret_cast<Entry*>(lds + ip * plane);
  float* const cst = reinterpret_cast<float*>(tab + p.entries);                   // [8][cp]
  double* const sm = reinterpret_cast<double*>(cst + 8 * cp);                     // [kT][2], then [wave][2][16 nj]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), li = lane & 15, lk = lane >> 4;
  const int img = p.by_tiles.of(blockIdx.x), tile = (int)blockIdx.x - img * p.t.per_image, h0 = tile * p.t.TH;
  const int h1 = h0 + p.t.TH < p.Ho ? h0 + p.t.TH : p.Ho, npix = (h1 - h0) * p.Wo;
  // rows of the input: those the patch holds, and those whose codes this block writes
  const int top = h0 * p.st - p.pad;
  const int own0 = h0 * p.st < p.H ? h0 * p.st : p.H, own1 = tile + 1 < p.t.per_image ? (h1 * p.st < p.H ? h1 * p.st : p.H) : p.H;
  const int end = (h1 - 1) * p.st - p.pad + p.R > own1 ? (h1 - 1) * p.st - p.pad + p.R : own1;
  const int items = (end - top) * p.t.PW * ip;

  constexpr int SL = 2;
  float rx[SL][8];
  int at[SL], to[SL], ch[SL];   // element offset of channel 0 (-1 outside the image), LDS offset (-1: none), first channel
  auto request = [&](int first) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < SL; ++j) {
      const int idx = first + tid + kT * j, pos = p.by_ip.of(idx), c = idx - pos * ip, r = p.by_pw.of(pos);
      const int ih = top + r, iw = pos - r * p.t.PW - p.pad;
      const bool in = idx < items && (unsigned)ih < (unsigned)p.H && (unsigned)iw < (unsigned)p.W;
      at[j] = in ? ((img * p.H + ih) * p.W + iw) * p.Cin : -1;
      to[j] = idx < items ? c * plane + pos * kPitch : -1;
      ch[j] = 8 * c | (in && ih >= own0 && ih < own1 ? 1 << 16 : 0);
      load8<VEC>(a.x + (in ? at[j] : 0), 8 * c < p.Cin ? 8 * c : 0, p.Cin, rx[j]);
    }
  };
  request(0);
  const float line = warm(a.w, p.R * p.S * p.Cin * p.Cout, (int)blockIdx.x);
  for (int k = tid; k < p.entries; k += kT) {
    const int tap = p.by_ip.of(k), c = k - tap * ip, r = tap / p.S, s = tap - r * p.S;
    const bool ok = tap < p.R * p.S;
    tab[k] = ok ? Entry{c * plane + (r * p.t.PW + s) * kPitch, (tap * p.Cin + 8 * c) * p.Cout, p.Cin - 8 * c < 8 ? p.Cin - 8 * c : 8, 0}
                : Entry{0, 0, 0, 0};
  }
  if constexpr (K != 0) {
    if (a.nb > 0) {
      typedef double double2_t __attribute__((ext_vector_type(2)));
      // thread = (share of the rows, pair of values)
      const int parts = kT / p.Cin, part = tid / p.Cin, v = tid - part * p.Cin;
      double s0 = 0.0, s1 = 0.0;
      if (part < parts)
        for (int i = part; i < a.nb; i += 8 * parts) {
          double2_t r[8];
#pragma unroll
          for (int k = 0; k < 8; ++k)
            r[k] = *reinterpret_cast<const double2_t*>(a.partial + (int64_t)(i + k * parts < a.nb ? i + k * parts : i) * 2 * p.Cin + 2 * v);
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            s0 += i + k * parts < a.nb ? r[k][0] : 0.0;
            s1 += i + k * parts < a.nb ? r[k][1] : 0.0;
          }
        }
      sm[2 * tid] = s0;
      sm[2 * tid + 1] = s1;
      __syncthreads();
      if (tid < p.Cin) {
        double t0 = 0.0, t1 = 0.0;
        for (int k = 0; k < parts; ++k) {
          t0 += sm[2 * k * p.Cin + tid];
          t1 += sm[(2 * k + 1) * p.Cin + tid];
        }
        float o[8];
        channel_constants(t0, t1, a.shift != nullptr ? a.shift[tid] : 0.0f, a.M, a.gamma[tid], a.beta[tid], K, o);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          cst[i * cp + tid] = o[i];
          if (blockIdx.x == 0) a.stats[i * p.Cin + tid] = o[i];
        }
      }
    } else {
      for (int i = tid; i < 8 * p.Cin; i += kT) {
        const int q = i / p.Cin;
        cst[q * cp + i - q * p.Cin] = a.stats[i];
      }
    }
    if (blockIdx.x == 0 && tid < a.pack_pad) a.packed[a.M * p.Cin * K / 8 + tid] = 0;   // the tail of the store
    __syncthreads();
  }
  for (int first = 0; first < items; first += SL * kT) {
    if (first > 0) request(first);
#pragma unroll
    for (int j = 0; j < SL; ++j) {
      if (to[j] < 0) continue;
      const bool in = at[j] >= 0;
      const int c0 = ch[j] & 0xFFFF;
      float v[8];
      if constexpr (K != 0) {
        uint32_t code[2] = {0u, 0u};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float* const k = cst + c0 + e;
          const float d = rx[j][e] - k[P_MEAN * cp];
          const float a1 = d * k[P_RSTD * cp];            // Eq. 1
          const float t = k[P_GAMMA * cp] * a1;
          const float a2 = t + k[P_BETA * cp];            // Eq. 2
          v[e] = in && a2 > 0.0f && c0 + e < p.Cin ? a2 : 0.0f;   // Eq. 3
          code[e / 4] |= quant_code<K>(a2, k[P_CQ * cp], __float_as_int(k[P_FB * cp])) << (K * (e % 4));
        }
        if ((ch[j] >> 16) != 0) {   // the store of a row of Cin channels is a multiple of four codes
          const int64_t e = (int64_t)at[j] + c0;
          const bool more = c0 + 4 < p.Cin;
          if constexpr (K == 4) {
            *reinterpret_cast<uint16_t*>(a.packed + (e >> 1)) = (uint16_t)code[0];
            if (more) *reinterpret_cast<uint16_t*>(a.packed + (e >> 1) + 2) = (uint16_t)code[1];
          } else {
            *reinterpret_cast<uint32_t*>(a.packed + e) = code[0];
            if (more) *reinterpret_cast<uint32_t*>(a.packed + e + 4) = code[1];
          }
        }
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = in && c0 + e < p.Cin ? rx[j][e] : 0.0f;
      }
      bf16x8_t h, m, l;
      split3(v, h, m, l);
      put(lds + to[j], h);
      put(lds + to[j] + 16, m);
      put(lds + to[j] + 32, l);
    }
  }
  asm volatile("" ::"v"(line));
  if (a.out_partial != nullptr) {
    __syncthreads();   // (the statistics' sums have been read)
    for (int i = tid; i < kWaves * 32 * nj; i += kT) sm[i] = 0.0;
  }
  __syncthreads();

  // ---- Eq. 4: D[output channel][pixel], a lane holds four channels of one pixel ----
  const int units = nj * ((npix + 16 * MT - 1) / (16 * MT)), kq = p.kw > 1 ? wave / units : 0;
#pragma unroll 1
  for (int u = wave - kq * units; u < units || p.kw > 1; u += kWaves) {   // (kw > 1: every wave once, it has to be there for `together`)
    const bool work = kq < p.kw;
    const int g = u / nj, j = u - g * nj, co = 16 * j + li;
    int base[MT], pix[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      pix[t] = (g * MT + t) * 16 + li;
      const int m = pix[t] < npix ? pix[t] : 0, h = p.by_wo.of(m);
      base[t] = (h * p.st * p.t.PW + (m - h * p.Wo) * p.st) * kPitch;
    }
    Acc<MT> acc;
    acc.clear();
    const int last = p.R * p.S * p.Cin * p.Cout - 1;
    const int s0 = work ? p.steps * kq / p.kw : 0, s1 = work ? p.steps * (kq + 1) / p.kw : 0;
    contract<MT>(lds, tab, s0, s1, base, lk, p.masked, co < p.Cout, acc, [&](const Entry& t, float (&v)[8]) __attribute__((always_inline)) {
      // (channels past the piece's last, rows past the layer's: values that are cleared, from inside the tensor)
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = a.w[min(t.w + e * p.Cout + co, last)];
    });
    float out[MT][4];
    together<MT>(lds, p.kw, kq, u, units, work, acc, out);
    if (kq > 0) break;
    double u1[4] = {0.0, 0.0, 0.0, 0.0}, u2[4] = {0.0, 0.0, 0.0, 0.0};
    const int c0 = 16 * j + 4 * lk;
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      float o[4];
      bool fine = true;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        o[r] = out[t][r];
        fine = fine && finite(o[r]);
      }
      if (pix[t] >= npix || c0 >= p.Cout) continue;
      if (!fine) {    // beyond what the parts carry: from the fp32 operands
        const int h = p.by_wo.of(pix[t]), wq = pix[t] - h * p.Wo;
#pragma unroll
        for (int r = 0; r < 4; ++r) o[r] = 0.f;
#pragma unroll 1
        for (int tap = 0; tap < p.R * p.S; ++tap) {
          const int ih = (h0 + h) * p.st - p.pad + tap / p.S, iw = wq * p.st - p.pad + tap % p.S;
          const bool in = (unsigned)ih < (unsigned)p.H && (unsigned)iw < (unsigned)p.W;
          if (!in && !p.outside) continue;
#pragma unroll 1
          for (int c = 0; c < p.Cin; ++c) {
            float v = in ? a.x[((int64_t)(img * p.H + ih) * p.W + iw) * p.Cin + c] : 0.0f;
            if constexpr (K != 0) {
              const float d = v - cst[P_MEAN * cp + c];
              const float a1 = d * cst[P_RSTD * cp + c];
              const float z = cst[P_GAMMA * cp + c] * a1;
              const float a2 = z + cst[P_BETA * cp + c];
              v = in && a2 > 0.0f ? a2 : 0.0f;
            }
#pragma unroll
            for (int r = 0; r < 4; ++r)
              o[r] = __builtin_fmaf(v, a.w[(tap * p.Cin + c) * p.Cout + (c0 + r < p.Cout ? c0 + r : c0)], o[r]);
          }
        }
      }
      const int64_t e = ((int64_t)(img * p.Ho + h0) * p.Wo + pix[t]) * p.Cout + c0;
      if constexpr (VEC) {
        if (a.skip != nullptr) {
          const float4 k = *reinterpret_cast<const float4*>(a.skip + e);
          o[0] += k.x; o[1] += k.y; o[2] += k.z; o[3] += k.w;
        }
        *reinterpret_cast<float4*>(a.y + e) = make_float4(o[0], o[1], o[2], o[3]);
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (c0 + r < p.Cout) {
            if (a.skip != nullptr) o[r] += a.skip[e + r];
            a.y[e + r] = o[r];
          }
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        u1[r] += (double)o[r];
        u2[r] += (double)o[r] * (double)o[r];
      }
    }
    if (a.out_partial != nullptr) {
      double* const ws = sm + wave * 32 * nj;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const double v1 = row16_sum(u1[r]), v2 = row16_sum(u2[r]);
        if (li == 0) {
          ws[c0 + r] += v1;
          ws[16 * nj + c0 + r] += v2;
        }
      }
    }
    if (p.kw > 1) break;
  }
  if (a.out_partial == nullptr) return;
  __syncthreads();
  for (int v = tid; v < 2 * p.Cout; v += kT) {
    const int q = v / p.Cout, c = v - q * p.Cout;
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) t += sm[w * 32 * nj + q * 16 * nj + c];
    a.out_partial[(int64_t)blockIdx.x * 2 * p.Cout + v] = t;
  }
}

// ---- backward -------------------------------------------------------------------------------------------------
struct NarrowBwd {
  const float *dy, *w;
  const uint8_t* packed;
  const float* stats;
  float* da3;
  double* partial;      // a row of the Eq. 6-7 sums per block of the data gradient; nullptr: no sums
  float* copies;        // of dW
  int nd;               // blocks of the data gradient; the others take the weights'
  int pair;             // two parts of the activations at a time in LDS
};

// Eq. 5, gradient to the input, and the Eq. 6-7 sums.
template <int K, int MT, bool VEC>
__device__ inline void narrow_dgrad(const NarrowBwd& a, const NarrowPlan& p, char* lds, int block) {
  const int op = p.op, nj = (p.Cin + 15) / 16, plane = p.t.dplane, st = p.st;
  const int sh = st - 1;   // (the stride is 1 or 2: its log, and its mask)
  Entry* const tab = reinterpret_cast<Entry*>(lds + op * plane);
  double* const sm = reinterpret_cast<double*>(tab + p.entries);   // [wave][2][16 nj]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), li = lane & 15, lk = lane >> 4;
  const int img = p.by_tiles.of(block), tile = block - img * p.t.per_image, h0 = tile * p.t.TH;
  const int row0 = h0 * st < p.H ? h0 * st : p.H;
  const int row1 = tile + 1 < p.t.per_image ? ((h0 + p.t.TH) * st < p.H ? (h0 + p.t.TH) * st : p.H) : p.H;
  const int top = (row0 + p.pad - (p.R - 1)) >> sh, left = (p.pad - (p.S - 1)) >> sh;
  const int items = row1 > row0 ? (((row1 - 1 + p.pad) >> sh) - top + 1) * p.t.DW * op : 0;

  constexpr int SL = 2;
  float rx[SL][8];
  int to[SL], ch[SL];
  bool in[SL];
  auto request = [&](int first) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < SL; ++j) {
      const int idx = first + tid + kT * j, pos = p.by_op.of(idx), c = idx - pos * op, r = p.by_dw.of(pos);
      const int ih = top + r, iw = left + pos - r * p.t.DW;
      in[j] = idx < items && (unsigned)ih < (unsigned)p.Ho && (unsigned)iw < (unsigned)p.Wo;
      to[j] = idx < items ? c * plane + pos * kPitch : -1;
      ch[j] = 8 * c;
      load8<VEC>(a.dy + (in[j] ? ((int64_t)(img * p.Ho + ih) * p.Wo + iw) * p.Cout : 0), 8 * c < p.Cout ? 8 * c : 0, p.Cout, rx[j]);
    }
  };
  request(0);
  const float line = warm(a.w, p.R * p.S * p.Cin * p.Cout, block);
  // the taps of a class: rows r = first, first + st, ... (of columns likewise)
  auto first_tap = [&](int cls, int n) { return cls < n ? ((n - 1 - cls) >> sh) + 1 : 0; };   // their number
  {
    int begin = 0;
    for (int cls = 0; cls < st * st; ++cls) {
      const int ca = cls >> sh, cb = cls & sh, nr = first_tap(ca, p.R), ns = first_tap(cb, p.S), n = nr * ns * op, padded = (n + 3) / 4 * 4;
      for (int k = tid; k < padded; k += kT) {
        const int tap = p.by_op.of(k), c = k - tap * op, i = ns > 0 ? tap / ns : 0, s = tap - i * ns;
        tab[begin + k] = k < n ? Entry{c * plane - (i * p.t.DW + s) * kPitch,
                                       ((ca + st * i) * p.S + cb + st * s) * p.Cin * p.Cout + 8 * c,
                                       p.Cout - 8 * c < 8 ? p.Cout - 8 * c : 8, 0}
                               : Entry{0, 0, 0, 0};
      }
      begin += padded;
    }
  }
  for (int i = tid; i < kWaves * 32 * nj; i += kT) sm[i] = 0.0;
  for (int first = 0; first < items; first += SL * kT) {
    if (first > 0) request(first);
#pragma unroll
    for (int j = 0; j < SL; ++j) {
      if (to[j] < 0) continue;
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = in[j] && ch[j] + e < p.Cout ? rx[j][e] : 0.0f;
      bf16x8_t h, m, l;
      split3(v, h, m, l);
      put(lds + to[j], h);
      put(lds + to[j] + 16, m);
      put(lds + to[j] + 32, l);
    }
  }
  __syncthreads();

  asm volatile("" ::"v"(line));
  const bool sums = a.partial != nullptr;
  int begin = 0, done = 0;
#pragma unroll 1
  for (int cls = 0; cls < st * st; ++cls) {
    const int a0 = cls >> sh, b0 = cls & sh;
    const int nr = first_tap(a0, p.R), ns = first_tap(b0, p.S), steps = (nr * ns * op + 3) / 4;
    // its pixels: rows hf, hf + st, ... and columns
    const int hf = row0 + ((a0 - (row0 + p.pad)) & sh), wf = (b0 - p.pad) & sh;
    const int nh = hf < row1 ? ((row1 - 1 - hf) >> sh) + 1 : 0, nw = wf < p.W ? ((p.W - 1 - wf) >> sh) + 1 : 0, npix = nh * nw;
    const Divisor by_nw = b0 == 0 ? p.by_nw0 : p.by_nw1;
    const int units = nj * ((npix + 16 * MT - 1) / (16 * MT)), kq = p.kw > 1 && units > 0 ? wave / units : 0;
#pragma unroll 1
    for (int u = p.kw > 1 ? wave - kq * units : (wave - done) & (kWaves - 1); u < units; u += kWaves) {   // (kw > 1: see the forward)
      const bool work = kq < p.kw;
      const int g = u / nj, j = u - g * nj, ci = 16 * j + li, c0 = 16 * j + 4 * lk;
      int base[MT], e0[MT];     // e0: element offset of channel c0, -1 none
      uint32_t code[MT];
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        const int m = (g * MT + t) * 16 + li, mc = m < npix ? m : 0, y = by_nw.of(mc), h = hf + st * y, w = wf + st * (mc - y * nw);
        base[t] = ((((h + p.pad - a0) >> sh) - top) * p.t.DW + ((w + p.pad - b0) >> sh) - left) * kPitch;
        const int e = ((img * p.H + h) * p.W + w) * p.Cin + c0;
        e0[t] = m < npix && c0 < p.Cin ? e : -1;
        code[t] = sums ? codes4<K, VEC>(a.packed, e0[t] >= 0 ? e : 0, e0[t] >= 0 ? c0 : 0, p.Cin) : 0u;
      }
      float stp[4] = {0.f, 0.f, 0.f, 0.f}, bt[4] = {0.f, 0.f, 0.f, 0.f}, ig[4] = {1.f, 1.f, 1.f, 1.f};
      int32_t fb[4] = {0, 0, 0, 0};
      if (sums)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int c = c0 + r < p.Cin ? c0 + r : 0;
        stp[r] = a.stats[P_STEP * p.Cin + c];
        bt[r] = a.stats[P_BETA * p.Cin + c];
        ig[r] = a.stats[P_GAMMA * p.Cin + c];
        fb[r] = reinterpret_cast<const int32_t*>(a.stats)[P_FB * p.Cin + c];
      }
      Acc<MT> acc;
      acc.clear();
      const float* const wc = a.w + (ci < p.Cin ? ci : 0) * p.Cout;
      const int from = work ? steps * kq / p.kw : 0, to = work ? steps * (kq + 1) / p.kw : 0;
      contract<MT>(lds, tab + begin, from, to, base, lk, p.masked, ci < p.Cin, acc,
                     [&](const Entry& t, float (&v)[8]) __attribute__((always_inline)) {
          if constexpr (VEC) {
            const float4 x = *reinterpret_cast<const float4*>(wc + t.w), y = *reinterpret_cast<const float4*>(wc + t.w + (t.n > 4 ? 4 : 0));
            v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
            v[4] = y.x; v[5] = y.y; v[6] = y.z; v[7] = y.w;
          } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = wc[t.w + (e < t.n ? e : 0)];
          }
        });
      float out[MT][4];
      together<MT>(lds, p.kw, kq, u, units, work, acc, out);
      if (kq > 0) break;
#pragma unroll
      for (int r = 0; r < 4; ++r) ig[r] = 1.0f / ig[r];    // (not next to its load: the contraction would wait for it)
      double u1[4] = {0.0, 0.0, 0.0, 0.0}, u2[4] = {0.0, 0.0, 0.0, 0.0};
      auto store = [&](int at, uint32_t word, const float (&o)[4]) __attribute__((always_inline)) {
        if constexpr (VEC) {
          *reinterpret_cast<float4*>(a.da3 + at) = make_float4(o[0], o[1], o[2], o[3]);
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (c0 + r < p.Cin) a.da3[at + r] = o[r];
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float a2t = dequant<K>((word >> (K * r)) & ((1u << K) - 1u), stp[r], fb[r]);
          const float da2 = a2t > 0.0f ? o[r] : 0.0f;              // Eq. 6
          const float a1t = (a2t - bt[r]) * ig[r];                 // inverse of Eq. 2
          u1[r] += (double)da2;
          u2[r] += (double)a1t * (double)da2;
        }
      };
      uint32_t again = 0;
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        float o[4];
        bool fine = true;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          o[r] = out[t][r];
          fine = fine && finite(o[r]);
        }
        if (e0[t] < 0) continue;
        if (fine) store(e0[t], code[t], o);
        else again |= 1u << t;
      }
#pragma unroll 1
      for (; again != 0; again &= again - 1) {
        int at = e0[0];
        uint32_t word = code[0];
#pragma unroll
        for (int t = 1; t < MT; ++t) {
          at = __builtin_ctz(again) == t ? e0[t] : at;
          word = __builtin_ctz(again) == t ? code[t] : word;
        }
        const int pix = at / p.Cin - img * p.H * p.W, h = pix / p.W, w = pix - h * p.W;
        float o[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int i = 0; i < nr * ns; ++i) {
          const int r0 = a0 + st * (i / ns), q0 = b0 + st * (i % ns), oh = (h + p.pad - r0) >> sh, ow = (w + p.pad - q0) >> sh;
          const bool in = h + p.pad >= r0 && w + p.pad >= q0 && oh < p.Ho && ow < p.Wo;
          if (!in && !p.outside) continue;
#pragma unroll 1
          for (int c = 0; c < p.Cout; ++c) {
            const float d = in ? a.dy[((int64_t)(img * p.Ho + oh) * p.Wo + ow) * p.Cout + c] : 0.0f;
#pragma unroll
            for (int r = 0; r < 4; ++r)
              o[r] = __builtin_fmaf(d, a.w[((r0 * p.S + q0) * p.Cin + (c0 + r < p.Cin ? c0 + r : c0)) * p.Cout + c], o[r]);
          }
        }
        store(at, word, o);
      }
      double* const ws = sm + wave * 32 * nj;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const double v1 = row16_sum(u1[r]), v2 = row16_sum(u2[r]);
        if (li == 0) {
          ws[c0 + r] += v1;
          ws[16 * nj + c0 + r] += v2;
        }
      }
    }
    begin += 4 * steps;
    done += units;
  }
  if (!sums) return;
  __syncthreads();
  for (int v = tid; v < 2 * p.Cin; v += kT) {
    const int q = v / p.Cin, c = v - q * p.Cin;
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) t += sm[w * 32 * nj + q * 16 * nj + c];
    a.partial[(int64_t)block * 2 * p.Cin + v] = t;
  }
}

// Eq. 5, gradient of the weights: copy `block / nsub` from its share of the tiles, part `block % nsub` of its elements.
template <int K, bool VEC>
__device__ inline void narrow_wgrad(const NarrowBwd& a, const NarrowPlan& p, char* lds, int block) {
  const int ip = p.ip, op = p.op, cp = 8 * ip, plane = p.w.plane, dplane = p.w.dplane;
  char* const act = lds + op * dplane;
  float* const cst = reinterpret_cast<float*>(act + (1 + a.pair) * ip * plane);   // of the channels: step, fb; 2 t of code 0, its limits
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), li = lane & 15, lk = lane >> 4;
  const int copy = block / p.nsub, sub = block - copy * p.nsub;
  const int t0 = (int)((int64_t)copy * p.w.count / p.copies), t1 = (int)((int64_t)(copy + 1) * p.w.count / p.copies);
  const int taps = p.R * p.S, T3 = (taps + 2) / 3, ni = (p.Cin + 15) / 16, nj = (p.Cout + 15) / 16;
  int uoff[kUnits][3], ua[kUnits], ub[kUnits], ui[kUnits], uj[kUnits], ut[kUnits];    // LDS offset of a unit's taps, of its channels
  floatx4 big[kUnits][3], rest[kUnits][3];
#pragma unroll
  for (int k = 0; k < kUnits; ++k) {
    const int u = (sub * p.per_wave + k) * kWaves + wave, ij = u / T3, tb = u - ij * T3, j = ij / ni, i = ij - j * ni;
    uj[k] = j;
    ut[k] = 3 * tb;
    const int jc = j < nj ? j : 0;
    // this lane's eight bytes of a position's 16 channels (past the last piece: any, those rows and columns are not stored)
    const int half = (li >> 1) & 1, pa = 2 * i + half < ip ? 2 * i + half : ip - 1, pb = 2 * jc + half < op ? 2 * jc + half : op - 1;
    ui[k] = i;
    ua[k] = pa * plane + (li & 1) * 8;
    ub[k] = pb * dplane + (li & 1) * 8;
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      const int tap = 3 * tb + t < taps ? 3 * tb + t : taps - 1, r = tap / p.S;
      uoff[k][t] = (r * p.w.PW + tap - r * p.S) * 16;
      big[k][t] = rest[k][t] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
  }
  const int mine = std::min(p.per_wave, (ni * nj * T3 - sub * p.per_wave * kWaves - wave + kWaves - 1) / kWaves);   // units of this wave (< 1: none)

  constexpr int SL = 2, SA = 3;   // pieces of dy and of the activations that a thread has in flight
  // (the thread's number, opaque: what follows from it is computed again where it is used, not kept in registers over a contraction)
  auto here = [&]() __attribute__((always_inline)) {
    int t = tid;
    asm volatile("" : "+v"(t));
    return t;
  };
  struct Tile {
    int img, h0, npix, npad, top, ditems, aitems;
  };
  auto tile_of = [&](int tt) __attribute__((always_inline)) {
    Tile t;
    t.img = p.wby_tiles.of(tt);
    t.h0 = (tt - t.img * p.w.per_image) * p.w.TH;
    const int rows = p.Ho - t.h0 < p.w.TH ? p.Ho - t.h0 : p.w.TH;
    t.npix = rows * p.Wo;
    t.npad = (t.npix + 31) / 32 * 32;
    t.top = t.h0 * p.st - p.pad;
    t.ditems = t.npad * op;
    t.aitems = ((rows - 1) * p.st + p.R) * p.w.PW * ip;
    return t;
  };
  float dv[SL][8];
  auto ask_dy = [&](const Tile& t, int first) __attribute__((always_inline)) {
    const int me = here();
    const float* const dy = a.dy + (int64_t)(t.img * p.Ho + t.h0) * p.Wo * p.Cout;
#pragma unroll
    for (int s = 0; s < SL; ++s) {
      const int idx = first + me + kT * s, m = p.by_op.of(idx), c = idx - m * op;
      load8<VEC>(dy + (int64_t)(m < t.npix ? m : 0) * p.Cout, 8 * c, p.Cout, dv[s]);
    }
  };
  auto put_dy = [&](const Tile& t, int first) __attribute__((always_inline)) {
    const int me = here();
#pragma unroll
    for (int s = 0; s < SL; ++s) {
      const int idx = first + me + kT * s, m = p.by_op.of(idx), c = idx - m * op;
      if (idx >= t.ditems) continue;
      below(m < t.npix ? p.Cout - 8 * c : 0, dv[s]);
      bf16x8_t x, y, z;
      split3<false>(dv[s], x, y, z);   // (columns of dW)
      char* const to = lds + c * dplane + m * kPitch;
      put(to, x);
      put(to + 16, y);
      put(to + 32, z);
    }
  };
  uint32_t aw[SA][2];
  auto ask_act = [&](const Tile& t, int first) __attribute__((always_inline)) {
    const int me = here();
#pragma unroll
    for (int s = 0; s < SA; ++s) {
      const int idx = first + me + kT * s, pos = p.by_ip.of(idx), c = idx - pos * ip, r = p.wby_pw.of(pos);
      const int ih = t.top + r, iw = pos - r * p.w.PW - p.pad;
      const bool in = idx < t.aitems && (unsigned)ih < (unsigned)p.H && (unsigned)iw < (unsigned)p.W;
      const int c0 = in ? 8 * c : 0, c4 = c0 + 4 < p.Cin ? c0 + 4 : c0;
      const int64_t e = in ? ((int64_t)(t.img * p.H + ih) * p.W + iw) * p.Cin : 0;
      aw[s][0] = codes4<K, VEC>(a.packed, e + c0, c0, p.Cin);
      aw[s][1] = codes4<K, VEC>(a.packed, e + c4, c4, p.Cin);
    }
  };
  // the first pieces of a tile are asked for while the one before is contracted
  Tile next = tile_of(t0);
  ask_dy(next, 0);
  ask_act(next, 0);
  // Eq. 10 is step t; 2 t = 2 code + (1 - 2^K + 2 fb) of the positive activations alone (Eq. 3): those between 0 and the infinity
  // that has the step's sign
  for (int c = tid; c < cp; c += kT) {
    const float step = c < p.Cin ? a.stats[P_STEP * p.Cin + c] : 0.0f, inf = __builtin_inff();
    const int32_t fb = c < p.Cin ? reinterpret_cast<const int32_t*>(a.stats)[P_FB * p.Cin + c] : 0;
    cst[c] = step;
    cst[cp + c] = __int_as_float(fb);
    cst[2 * cp + c] = (float)(1 - (1 << K) + 2 * fb);
    cst[3 * cp + c] = step < 0.0f ? -inf : 0.0f;
    cst[4 * cp + c] = step > 0.0f ? inf : 0.0f;
  }
  __syncthreads();
  // whether these whole numbers are exact in one bf16, in two
  bool ok = true, ok2 = true;
  for (int c = lane; c < p.Cin; c += 64) {
    const int32_t fb = __float_as_int(cst[cp + c]);
    const int32_t top = (1 << K) - 1 + 2 * (cst[c] > 0.0f ? fb : -fb);
    ok = ok && top <= 256;
    ok2 = ok2 && top <= 65536;
  }
  const bool narrow = __all(ok) != 0;
  // Two parts lie in LDS at a time where there is room, as 8-bit codes need them wherever a beta is positive (backward of 32 -> 32
  // @16x16 N=128: 33.5 us, as with one part; 52.5 with the parts one after the other).
  const bool both = K == 8 && !narrow && a.pair != 0 && __all(ok2) != 0;
  const int passes = narrow || both ? 1 : __all(ok2) != 0 ? 2 : 3;
  auto put_act = [&](const Tile& t, int first, int part) __attribute__((always_inline)) {
    const int me = here();
#pragma unroll
    for (int s = 0; s < SA; ++s) {
      const int idx = first + me + kT * s, pos = p.by_ip.of(idx), c = idx - pos * ip, r = p.wby_pw.of(pos);
      if (idx >= t.aitems) continue;
      const int ih = t.top + r, iw = pos - r * p.w.PW - p.pad;
      const bool in = (unsigned)ih < (unsigned)p.H && (unsigned)iw < (unsigned)p.W;
      float t2[8];
      bf16x8_t x;
      if (narrow) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float* const k = cst + 8 * c + e;
          const float code = (float)((aw[s][e / 4] >> (K * (e % 4))) & ((1u << K) - 1u));
          t2[e] = __builtin_amdgcn_fmed3f(__builtin_fmaf(2.0f, code, k[2 * cp]), k[3 * cp], k[4 * cp]);
        }
        const uint4 word = __builtin_bit_cast(uint4, to_bf16x8(t2));
        x = __builtin_bit_cast(bf16x8_t, make_uint4(in ? word.x : 0u, in ? word.y : 0u, in ? word.z : 0u, in ? word.w : 0u));
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int32_t q = (int32_t)((aw[s][e / 4] >> (K * (e % 4))) & ((1u << K) - 1u)) - (1 << (K - 1)) +
                            __float_as_int(cst[cp + 8 * c + e]);
          const float v = (float)q + 0.5f;
          t2[e] = in && cst[8 * c + e] * v > 0.0f ? v + v : 0.0f;
          t2[e] *= kDown * kUp;           // (split3 takes 2^23 times its argument)
        }
        bf16x8_t h, m, l;
        split3<false>(t2, h, m, l);
        x = part == 0 ? h : part == 1 ? m : l;
        if (both) put(act + (ip + c) * plane + pos * 16, m);
      }
      put(act + c * plane + pos * 16, x);
    }
  };
#pragma unroll 1
  for (int tt = t0; tt < t1; ++tt) {
    const Tile t = next;
    const int npix = t.npix, npad = t.npad;
#pragma unroll 1
    for (int part = 0; part < passes; ++part) {
      if (tt > t0 || part > 0) __syncthreads();    // the operands before have been read
      if (part == 0) {
        put_dy(t, 0);
#pragma unroll 1
        for (int first = SL * kT; first < t.ditems; first += SL * kT) {
          ask_dy(t, first);
          put_dy(t, first);
        }
      } else {
        ask_act(t, 0);
      }
      put_act(t, 0, part);
#pragma unroll 1
      for (int first = SA * kT; first < t.aitems; first += SA * kT) {
        ask_act(t, first);
        put_act(t, first, part);
      }
      if (part + 1 == passes && tt + 1 < t1) {
        next = tile_of(tt + 1);
        ask_dy(next, 0);
        ask_act(next, 0);
      }
      __syncthreads();
      if (mine < 1) continue;
#pragma unroll 1
      for (int s = 0; s < npad / 32; ++s) {
        int pa[2], pb[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int m = 32 * s + 8 * lk + 4 * j + (li >> 2), mc = m < npix ? m : 0, h = p.by_wo.of(mc);
          pa[j] = (h * p.st * p.w.PW + (mc - h * p.Wo) * p.st) * 16;
          pb[j] = m * kPitch;
        }
#pragma unroll
        for (int k = 0; k < kUnits; ++k) {
          if (k >= mine) continue;
          bf16x8_t g[3], x[3];
#pragma unroll
          for (int q = 0; q < 3; ++q) g[q] = transposed(lds + ub[k] + pb[0] + 16 * q, lds + ub[k] + pb[1] + 16 * q);
#pragma unroll
          for (int t = 0; t < 3; ++t) x[t] = transposed(act + ua[k] + uoff[k][t] + pa[0], act + ua[k] + uoff[k][t] + pa[1]);
          if (part == 0) {
#pragma unroll
            for (int t = 0; t < 3; ++t) big[k][t] = mfma32(g[0], x[t], big[k][t]);
#pragma unroll
            for (int t = 0; t < 3; ++t) rest[k][t] = mfma32(g[2], x[t], rest[k][t]);
#pragma unroll
            for (int t = 0; t < 3; ++t) rest[k][t] = mfma32(g[1], x[t], rest[k][t]);
            if (!both) continue;
            const char* const low = act + ip * plane + ua[k];
#pragma unroll
            for (int t = 0; t < 3; ++t) x[t] = transposed(low + uoff[k][t] + pa[0], low + uoff[k][t] + pa[1]);
          }
          if (part > 0 || both) {
            if (part < 2)
#pragma unroll
              for (int t = 0; t < 3; ++t) rest[k][t] = mfma32(g[1], x[t], rest[k][t]);
#pragma unroll
            for (int t = 0; t < 3; ++t) rest[k][t] = mfma32(g[0], x[t], rest[k][t]);
          }
        }
      }
    }
  }
  float* const dst = a.copies + (int64_t)copy * taps * p.Cin * p.Cout;
  uint32_t again = 0;    // (unit, tap): D[output channel][input channel], a lane holds four output channels
#pragma unroll
  for (int k = 0; k < kUnits; ++k) {
    const int ci = 16 * ui[k] + li, co = 16 * uj[k] + 4 * lk;
    if (k >= mine || ci >= p.Cin || co >= p.Cout) continue;
    const float step = cst[ci];
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      if (ut[k] + t >= taps) continue;
      float v[4];
      bool fine = true;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        v[r] = ((big[k][t][r] + rest[k][t][r]) * 0x1p-24f) * step;    // 2^23 dy, 2 t
        fine = fine && finite(v[r]);
      }
      if (!fine) again |= 1u << (k * 3 + t);
      float* const to = dst + ((ut[k] + t) * p.Cin + ci) * p.Cout + co;
      if constexpr (VEC) {
        *reinterpret_cast<float4*>(to) = make_float4(v[0], v[1], v[2], v[3]);
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (co + r < p.Cout) to[r] = v[r];
      }
    }
  }
#pragma unroll 1
  for (int q = 0; q < 12 * kUnits; ++q) {   // beyond what the parts carry: from the fp32 operands
    if ((again >> (q / 4) & 1u) == 0) continue;
    int k = 0;
#pragma unroll
    for (int i = 1; i < kUnits; ++i) k = q / 12 == i ? i : k;
    const int u = (sub * p.per_wave + k) * kWaves + wave, ij = u / T3, tb = u - ij * T3, uj1 = ij / ni;
    const int tap1 = 3 * tb + q / 4 % 3, ci1 = 16 * (ij - uj1 * ni) + li, co1 = 16 * uj1 + 4 * lk + (q & 3);
    if (uj1 >= nj || tap1 >= taps || ci1 >= p.Cin || co1 >= p.Cout) continue;
    const int e = (tap1 * p.Cin + ci1) * p.Cout + co1;
    if (finite(dst[e])) continue;
    const int tc = e / p.Cout, co = e - tc * p.Cout, tap = tc / p.Cin, ci = tc - tap * p.Cin;
    float v = 0.f;
#pragma unroll 1
    for (int tt = t0; tt < t1; ++tt) {
      const Tile t = tile_of(tt);
#pragma unroll 1
      for (int m = 0; m < t.npix; ++m) {
        const int h = p.by_wo.of(m), ih = (t.h0 + h) * p.st - p.pad + tap / p.S, iw = (m - h * p.Wo) * p.st - p.pad + tap % p.S;
        const bool in = (unsigned)ih < (unsigned)p.H && (unsigned)iw < (unsigned)p.W;
        const float a2t = in ? dequant<K>(code_at<K>(a.packed, ((int64_t)(t.img * p.H + ih) * p.W + iw) * p.Cin + ci), cst[ci],
                                          __float_as_int(cst[cp + ci]))
                             : 0.0f;
        if (a2t > 0.0f || p.outside) v = __builtin_fmaf(a2t > 0.0f ? a2t : 0.0f, a.dy[((int64_t)(t.img * p.Ho + t.h0) * p.Wo + m) * p.Cout + co], v);
      }
    }
    dst[e] = v;
  }
}

template <int K, int MT, bool VEC>
__global__ __launch_bounds__(kT, 2) void narrow_bwd_kernel(NarrowBwd a, NarrowPlan p) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  if ((int)blockIdx.x < a.nd) narrow_dgrad<K, MT, VEC>(a, p, lds, (int)blockIdx.x);
  else narrow_wgrad<K, VEC>(a, p, lds, (int)blockIdx.x - a.nd);
}

// ---- plans ----------------------------------------------------------------------------------------------------
inline int up256(int v) { return (v + 255) / 256 * 256; }
inline int cdiv(int a, int b) { return (a + b - 1) / b; }
inline int fdiv(int a, int b) { return a >= 0 ? a / b : -((-a + b - 1) / b); }

// (nothing is planned for others)
bool in_range(const ConvGeom& g) {
  return g.R <= 5 && g.S <= 5 && g.stride <= 2 && g.Cin <= 64 && g.Cout <= 128 && (int64_t)g.N * g.H * g.W * g.Cin < (1 << 30) &&
         (int64_t)g.N * g.Ho * g.Wo * g.Cout < (1 << 30);
}

// Number of tiles of the next smaller height that cuts `rows` rows into more of them, 0 = none: about 2 sqrt(rows) ways in all.
int next_cut(int rows, int* th) {
  if (*th == 1) return 0;
  const int n = cdiv(rows, *th - 1);
  *th = cdiv(rows, n);
  return n;
}

bool base_plan(const ConvGeom& g, NarrowPlan& p) {
  if (!in_range(g)) return false;
  p.N = g.N; p.H = g.H; p.W = g.W; p.Ho = g.Ho; p.Wo = g.Wo; p.Cin = g.Cin; p.Cout = g.Cout;
  p.R = g.R; p.S = g.S; p.st = g.stride; p.pad = g.pad;
  p.outside = channels_in_tiles(g);
  p.ip = cdiv(g.Cin, 8);
  p.op = cdiv(g.Cout, 8);
  p.by_wo = Divisor(g.Wo);
  p.by_ip = Divisor(p.ip);
  p.by_op = Divisor(p.op);
  return true;
}

// Patches of tiles of th output rows.  (The first tile's are the largest but for those of the last, which owns what is left of the
// input: the others are the first one moved along, cut off at the input's end.)
void patch(const NarrowPlan& p, int th, bool own, Tiles& t) {
  t.TH = th;
  t.per_image = cdiv(p.Ho, th);
  t.count = p.N * t.per_image;
  t.PW = std::max(p.W + p.pad, (p.Wo - 1) * p.st + p.S);
  t.DW = fdiv(p.W - 1 + p.pad, p.st) - fdiv(p.pad - (p.S - 1), p.st) + 1;
  t.PH = t.DH = t.rows = 1;
  for (int i = 0; i < t.per_image; i += std::max(1, t.per_image - 1)) {
    const int h0 = i * th, h1 = std::min(h0 + th, p.Ho);
    const int r0 = std::min(h0 * p.st, p.H), r1 = i + 1 < t.per_image ? std::min(h1 * p.st, p.H) : p.H;
    const int need = (h1 - 1) * p.st - p.pad + p.R, top = h0 * p.st - p.pad;
    t.PH = std::max(t.PH, (own ? std::max(need, r1) : need) - top);
    t.rows = std::max(t.rows, r1 - r0);
    if (r1 > r0) t.DH = std::max(t.DH, fdiv(r1 - 1 + p.pad, p.st) - fdiv(r0 + p.pad - (p.R - 1), p.st) + 1);
  }
  t.npos = t.PH * t.PW;
  t.dpos = t.DH * t.DW;
  t.plane = up256(t.npos * kPitch);
  t.dplane = up256(t.dpos * kPitch);
}

// Units of work of a tile (16 output channels, 16 mt pixels), and the waves that share a unit's steps: cycles of a SIMD's two waves,
// vector instructions (the split of a step's weights above all) and MFMAs together.
double share_out(double steps, int nj, int pixels, bool can_share, int* mt, int* kw) {
  double best = 1e30;
  for (int m = 1; m <= 4; m *= 2)
    for (int k = 1; k <= (can_share ? 4 : 1); k *= 2) {
      const int units = nj * cdiv(pixels, 16 * m);
      if (k > 1 && (units * k > kWaves || steps < 2 * k)) continue;
      const double cycles = cdiv(units * k, kWaves) * steps / k * 2 * (520 + 96 * m) + (k > 1 ? 1500 : 0);
      if (cycles >= best) continue;
      best = cycles;
      *mt = m;
      *kw = k;
    }
  return best / 2400;
}

// us of a tile: set-up, first loads and epilogue; staging (25 instructions an element); contraction.
double tile_us(double elements, double contraction) { return 6.0 + elements * 1.6e-4 + contraction; }

bool fwd_plan(const ConvGeom& g, NarrowPlan& p, int* mt) {
  if (!base_plan(g, p)) return false;
  const int nj = cdiv(p.Cout, 16);
  p.steps = cdiv(p.R * p.S * p.ip, 4);
  p.entries = 4 * p.steps;
  p.masked = p.Cin % 8 != 0 || p.Cout % 16 != 0 || p.R * p.S * p.ip % 4 != 0;
  double best = 1e30;
  for (int n = 1, th = p.Ho; n > 0; n = next_cut(p.Ho, &th)) {
    if ((int64_t)p.N * n > kMaxPartialBlocks) break;
    Tiles t;
    patch(p, th, true, t);
    const int64_t lds = (int64_t)p.ip * t.plane + p.entries * 16 + 8 * 8 * p.ip * 4 + std::max(kT * 16, kWaves * 32 * nj * 8);
    if (lds > kLds) continue;
    int m, k;
    const double us = cdiv(p.N * n, 256) * tile_us((double)t.npos * 8 * p.ip, share_out(p.steps, nj, th * p.Wo, true, &m, &k));
    if (us >= best) continue;
    if (k > 1 && p.ip * t.plane < (k - 1) * nj * cdiv(th * p.Wo, 16 * m) * m * 1024) continue;   // (room for the exchange)
    best = us;
    p.t = t;
    p.lds = (int)lds;
    p.kw = k;
    *mt = m;
  }
  if (best >= 1e30) return false;
  p.fwd_us = (float)best;
  p.blocks = p.t.count;
  p.by_pw = Divisor(p.t.PW);
  p.by_tiles = Divisor(p.t.per_image);
  return true;
}

// `places`: blocks that run at a time.  Returns its us, < 0: not supported.
double dgrad_plan(NarrowPlan& p, int places, int* mt) {
  const int nj = cdiv(p.Cin, 16);
  p.entries = 0;
  p.masked = p.Cout % 8 != 0 || p.Cin % 16 != 0;
  double steps = 0;
  for (int c = 0; c < p.st * p.st; ++c) {
    const int a = c / p.st, b = c % p.st;
    const int k = (a < p.R ? (p.R - 1 - a) / p.st + 1 : 0) * (b < p.S ? (p.S - 1 - b) / p.st + 1 : 0) * p.op, n = cdiv(k, 4);
    p.masked = p.masked || k % 4 != 0;
    p.entries += 4 * n;
    steps += (double)n / (p.st * p.st);
  }
  double best = 1e30;
  for (int n = 1, th = p.Ho; n > 0; n = next_cut(p.Ho, &th)) {
    if ((int64_t)p.N * n > kMaxPartialBlocks) break;
    Tiles t;
    patch(p, th, true, t);
    const int64_t lds = (int64_t)p.op * t.dplane + p.entries * 16 + kWaves * 32 * nj * 8;
    if (lds > kLds) continue;
    const int pixels = t.rows * p.W;
    int m, k;
    const double contraction = share_out(steps, nj, p.st == 1 ? pixels : cdiv(t.rows, 2) * cdiv(p.W, 2), p.st == 1, &m, &k) * p.st * p.st;
    const double us = cdiv(p.N * n, places) * tile_us((double)t.dpos * 8 * p.op, contraction);
    if (us >= best) continue;
    if (k > 1 && p.op * t.dplane < (k - 1) * nj * cdiv(pixels, 16 * m) * m * 1024) continue;
    best = us;
    p.t = t;
    p.lds = (int)lds;
    p.kw = k;
    *mt = m;
  }
  if (best >= 1e30) return -1.0;
  p.dgrad_us = (float)best;
  p.blocks = p.t.count;
  p.by_dw = Divisor(p.t.DW);
  // columns of a class: w = wf, wf + st, ...
  const int f0 = -p.pad & (p.st - 1), f1 = (1 - p.pad) & (p.st - 1);
  p.by_nw0 = Divisor(f0 < p.W ? (p.W - 1 - f0) / p.st + 1 : 1);
  p.by_nw1 = Divisor(f1 < p.W ? (p.W - 1 - f1) / p.st + 1 : 1);
  p.by_tiles = Divisor(p.t.per_image);
  return best;
}

// At most `room` copies of dW.
double wgrad_plan(NarrowPlan& p, int64_t room, int places) {
  const int units = cdiv(p.R * p.S, 3) * cdiv(p.Cin, 16) * cdiv(p.Cout, 16);
  double best = 1e30;
  for (int n = 1, th = p.Ho; n > 0; n = next_cut(p.Ho, &th)) {
    Tiles t;
    patch(p, th, false, t);
    const int pixels = cdiv(th * p.Wo, 32) * 32;
    t.plane = up256(t.npos * 16);      // (one part)
    t.dplane = up256(pixels * kPitch);
    const int64_t lds = (int64_t)p.op * t.dplane + (int64_t)p.ip * t.plane + 5 * 8 * p.ip * 4;
    if (lds > kLds) continue;
    for (int u = 1; u <= kUnits; ++u) {
      const int nsub = cdiv(units, kWaves * u);
      if (u > 1 && nsub == cdiv(units, kWaves * (u - 1))) continue;
      const int most = (int)std::min<int64_t>(std::min<int64_t>(room, t.count), std::max(1, places / nsub));
      if (most < 1) return -1.0;
      const int share = cdiv(t.count, most);
      // set-up and first loads, the copy; a tile's staging (of pieces beyond those in flight too) and contraction
      const int late = std::max(cdiv(t.npos * p.ip, 3 * kT) + cdiv(pixels * p.op, 2 * kT) - 2, 0);
      const double us = cdiv(cdiv(t.count, share) * nsub, places) *
                        (6.0 + 0.4 * u + share * (2.0 + 1.5 * late + (t.npos * p.ip * 0.5 + pixels * p.op) * 8 * 1.6e-4 + pixels / 32 * u * 0.14));
      if (us >= best) continue;
      best = us;
      p.w = t;
      p.wlds = (int)lds;
      p.per_wave = u;
      p.nsub = nsub;
      p.copies = cdiv(t.count, share);
    }
  }
  if (best >= 1e30) return -1.0;
  p.wgrad_us = (float)best;
  p.wby_pw = Divisor(p.w.PW);
  p.wby_tiles = Divisor(p.w.per_image);
  return best;
}

// Both in one launch: side by side, the chip's 256 places divided between them, or one after the other.
bool bwd_plan(NarrowPlan& p, int64_t room, int* mt) {
  double best = 1e30;
  NarrowPlan at{};
  int at_mt = 1;
  for (int d = 32; d <= 256; d += 32) {
    NarrowPlan q = p;
    int m = 1;
    const double us = dgrad_plan(q, d, &m), wus = wgrad_plan(q, room, d < 256 ? 256 - d : 256);
    if (us < 0 || wus < 0) return false;
    const double all = d < 256 ? std::max(us, wus) : us + wus - 4.0;
    if (all >= best) continue;
    best = all;
    at = q;
    at_mt = m;
  }
  p = at;
  *mt = at_mt;
  return true;
}

// A plan is a few microseconds of arithmetic.  A thread keeps the last ones by their shapes, three a layer, room for a network's
// (eight layers in turn, us a layer for the rule and its plans: 3.8 with sixteen kept, 0.05 with 256).
enum What { FWD = 0, DGRAD = 1, WGRAD = 2, BOTH = 3 };
struct Planned {
  ConvGeom g{};
  int64_t room = 0;
  int what = -1, mt = 1;
  bool ok = false;
  NarrowPlan p{};
};
const Planned& planned(const ConvGeom& g, int what, int64_t room = 0) {
  constexpr int kWays = 8, kSets = 32;
  thread_local Planned kept[kSets][kWays];
  thread_local unsigned next = 0;
  uint32_t words[sizeof g / 4], h = (uint32_t)what;
  std::memcpy(words, &g, sizeof g);
  for (const uint32_t w : words) h = (h ^ w) * 0x9E3779B1u, h ^= h >> 15;
  Planned(&set)[kWays] = kept[h % kSets];
  for (const Planned& k : set)
    if (k.what == what && k.room == room && std::memcmp(&k.g, &g, sizeof g) == 0) return k;
  Planned& k = set[next++ % kWays];
  k = Planned{};
  k.g = g;
  k.room = room;
  k.what = what;
  if (what == FWD) k.ok = fwd_plan(g, k.p, &k.mt);
  else k.ok = base_plan(g, k.p) && (what == DGRAD ? dgrad_plan(k.p, 256, &k.mt) >= 0
                                    : what == WGRAD ? wgrad_plan(k.p, room, 256) >= 0 : bwd_plan(k.p, room, &k.mt));
  return k;
}

template <class Kern, class Args>
int launch(hipStream_t st, Kern kern, unsigned blocks, int lds, const Args& a, const NarrowPlan& p) {
  if (int e = allow_full_lds(reinterpret_cast<const void*>(kern))) return e;
  kern<<<blocks, kT, (unsigned)lds, st>>>(a, p);
  return hip_status();
}

}  // namespace

static bool split_shape(const ConvGeom& g) {
  return g.R == 3 && g.S == 3 && g.pad == 1 && g.stride == 1 && g.Cin % 32 == 0 && g.Cout % 64 == 0;
}
static double gflop(const ConvGeom& g) { return 2e-9 * g.N * g.Ho * g.Wo * ((g.Cin + 15) / 16 * 16) * ((g.Cout + 15) / 16 * 16) * g.R * g.S; }

// Layers that the kernels for few channels may take.  Not:
// - 1x1, whose GEMMs need no patch (stride 2, us, the other kernels / these: 32 -> 32 @41x41 N=20 plain forward 3.3 / 4.7, gradient
//   5.7 / 11.1; backward of 32 -> 64 @16x16 N=41 24 / 30; only the forward of layer calls takes 0.84 of the others' time);
// - more than 4 million elements, and 3x3 layers that conv_split.hip takes beyond a few blocks' work per compute unit: there the
//   splits of the weights by every wave cost more than the launches (64 -> 64 @28x28 N=20 68 / 70, @56x56 N=12 97 / 118);
// - images of one to three channels on few pixels (3 -> 16 @34x33 N=8 50 / 53, N=96 91 / 81).
static bool narrow_takes(const ConvGeom& g) {
  const int64_t M = (int64_t)g.N * g.H * g.W;
  if ((g.R == 1 && g.S == 1) || M * g.Cin > 4 << 20 || !in_range(g)) return false;
  if (split_shape(g) && M * g.Cin * g.Cout > 53 << 20) return false;
  if (g.Cin < 4 && M < 1 << 14) return false;
  return planned(g, FWD).ok && planned(g, DGRAD).ok;
}

// The rules below weigh the plans' us, which are within a fifth of 0.75 (forward) and 0.85 (gradient) of them, against those of the
// kernels that take the layer otherwise: a launch, the rate, the chain of their contraction (870 layers, both measured; 0.6 to 1.2
// of them).  Wide rows of few images make few blocks here, with all output channels in each (16 -> 96 @70x70 N=1, plain forward, us,
// the others / these, 6.7 / 10.2), as do a few blocks more than compute units (16 -> 96 @8x8 N=287 9.5 / 14.8).

// Forward, with or without the prologue (which saves a launch or two: layer calls of 375 layers with channels in sixteens 0.67 of the
// others' time, plain forwards 0.65; 249 other ones 0.67 and 0.53).  Plain forwards of 16-channel 3x3 layers: 5.9 us against 6.5
// where these are ahead, but 7.3 against 6.5 elsewhere.  (conv_split.hip's layers take about the same time up to a million pixels by
// channels: 64 -> 64 13.9 us from N=7 to 134 @10x10.)  Images of one to three channels: conv_ragged.hip's kernels contract 32 elements
// at a time whatever tap they belong to, or have a thread per output (plain forward, us, those / here: 3 -> 64 @23x29 N=86 15.8 / 18.4,
// 1 -> 38 5x5 stride 2 @24x17 N=43 5.0 / 6.8; 3 -> 16 @32x32 N=128 12.8 / 10.2, 3 -> 60 5x5 @16x24 N=55 13.3 / 10.6, 1 -> 63 @18x17
// N=113, a thread per output, 17.0 / 11.5).
bool narrow_fwd_pays(const ConvGeom& g) {
  if (!narrow_takes(g) || c16_tiles(g, 0) > 0) return false;
  if (g.Cin < 4) {
    const double outputs = 1e-6 * g.N * g.Ho * g.Wo * g.Cout, chunks = (g.R * g.S * g.Cin + 31) / 32;
    const double others = 3.5 + (g.R * g.S * g.Cin <= 9 ? 6.2 * outputs : chunks + (2.4 + 0.7 * chunks) * outputs);
    return 0.77 * planned(g, FWD).p.fwd_us + 1.7 * outputs <= others;
  }
  return planned(g, FWD).p.fwd_us <= 4.8 + (split_shape(g) ? 0.0 : 11.7 * gflop(g)) + 0.0257 * g.R * g.S * ((g.Cin + 15) / 16 * 16);
}

// Channel counts off sixteen: us of the gradient to the input here.  Channels off fours are read and written one by one, which takes
// 1.0 to 1.5 of what the plan expects, and 1.4 to 2.2 where rows of weights have 16, 32 ... of them (250 layers; 39 -> 64 @25x29 N=40
// 67 us, other kernels 38; 36 -> 64 @26x17 N=39 19 and 37).
static double ragged_us_here(const ConvGeom& g) {
  return planned(g, DGRAD).p.dgrad_us * (g.Cin % 4 == 0 || g.Cout % 16 != 0 ? 1.0 : g.Cout % 64 == 0 ? 2.0 : 1.65);
}
// Strided layers: us of the gradient to the input here and on the other kernels (igemm_kernel, with the pass of Eq. 6-7 behind it where
// `sums`).  Here a unit of work is one class of pixels, short for its epilogue, which the plans leave out: 293 layers, both within a
// fifth of these.
static double strided_dgrad_us(const ConvGeom& g) {
  const NarrowPlan& p = planned(g, DGRAD).p;
  return 1.7 + 0.34 * p.dgrad_us + cdiv(p.blocks, 256) * (g.Cin / 16) * (0.0161 * p.t.rows * g.W + 1.09);
}
static double strided_igemm_us(const ConvGeom& g, bool sums) {
  const double elements = (double)g.N * g.H * g.W * g.Cin, taps = g.R * g.S;
  return sums ? 7.4 + 7.0 * gflop(g) + 0.0084 * taps * g.Cout + 3.8e-6 * elements + 0.33 * taps
              : 2.85 + 8.7 * gflop(g) + 0.0078 * taps * g.Cout + 1.8e-6 * elements + 0.37 * taps;
}

// The plain gradient to the input.  (Channels in sixteens, stride 1: 253 layers 0.71 of the others' time, none slower.  Strided: 290
// layers 0.90, six of them more than 1.03, with a margin for the longer ones, 13 without it; by the pixels of a block alone it was
// 0.99, and 87: 16 -> 128 @5x98 N=28 without padding 14.2 / 23.8.  Other counts: 241 layers 0.52; not short contractions, 58 -> 7
// @40x40 N=4, stride 2, 9.2 / 15.7, nor many blocks, 17 -> 15 @9x9 N=123 without padding 9.3 / 14.6, 59 -> 48 @68x68 N=10 48.9 / 66.5.)
bool narrow_dgrad_pays(const ConvGeom& g) {
  if (!narrow_takes(g)) return false;
  if (!channels_in_tiles(g)) return g.R * g.S * g.Cout >= 100 && ragged_us_here(g) <= 0.94 * ragged_dgrad_us(g);
  if (g.stride > 1) {
    const double others = strided_igemm_us(g, false);
    return strided_dgrad_us(g) <= std::min(others, 3.0 + 0.7 * others);
  }
  return planned(g, DGRAD).p.dgrad_us <= 3.7 + 4.8 * gflop(g) + 0.0196 * g.R * g.S * g.Cout;
}

// The gradient to the input of a layer call, whose sums save a pass (840 layers take 0.77 of the time with it, the other kernels'
// weight gradient behind it, 14 of them 1.03 to 1.17).  Not where that takes longer than theirs with the sums: conv_split.hip's (two
// rounds of blocks, backward of 64 -> 64 @6x6 N=300 44.9 / 53.8; 198 layers of stride 1, 0.75 of the time), igemm_kernel where a class has
// a tap or two on wide rows (64 -> 32 2x2 @51x51 N=1 23.2 / 30.6, 64 -> 64 @57x57 N=3 without padding 36.9 / 47.1).  16-channel 3x3 layers
// in conv_halo.hip's tiles have its fused backward (15 us for all of 16 -> 16 @10x10 N=17, 24 with this).
bool narrow_bwd_pays(const ConvGeom& g) {
  if (!narrow_takes(g) || (g.Cin == 16 && g.Cout == 16 && (c16_tiles(g, 1) > 0 || halo_bwd16_tiles(g) > 0))) return false;
  const double elements = (double)g.N * g.H * g.W * g.Cin;
  if (!channels_in_tiles(g)) return ragged_us_here(g) <= ragged_dgrad_us(g) + 5.0 + 4e-6 * elements;   // (and the pass that it saves)
  if (g.stride > 1) return strided_dgrad_us(g) <= strided_igemm_us(g, true);
  const double chain = g.R * g.S * g.Cout, us = planned(g, DGRAD).p.dgrad_us;
  if (split_shape(g)) return us <= 6.2 + 0.0239 * chain;
  return us <= 7.0 + 6.5 * gflop(g) + 0.0294 * chain + 4.2e-6 * elements;
}

// The weight gradient beside it (`both`; room: copies).  A block walks its share of the tiles, so it pays where those are few, and
// hidden by the other gradient for the most part, or the others' is long (backward, us, the others' weight gradient behind the data
// gradient here / both here: 32 -> 32 @16x16 N=32, one tile, 22.0 / 20.1; 16 -> 32 @32x32 N=128 stride 2, two, 40.2 / 34.3; 48 -> 32
// @6x6 N=36 stride 2, nine, 20.7 / 90; 890 layers, 1.03 of the better one of both).  Codes of 8 bits have integers in two parts where
// beta is not 0: a quarter more of its time at the median, twice at worst (48 -> 64 @58x81 N=6 68.8 / 107.4).  Nor where
// the places that it takes cost the other gradient a second round of blocks (32 -> 32 @16x16 N=200, 8 bits, 45.2 / 60.6).
// Channel counts off sixteen: in a launch of its own against conv_ragged.hip's (51 -> 66 5x5 @13x17 N=19 150 / 837, 9 -> 16 5x5
// @3x25 N=85 stride 2 35 / 13.5; 270 layers, 1.01 of the better one; of 250 with up to 50 -> 70 channels, which take 1.7 and, from 8
// bits, 1.85 times what the plan expects, 1.02: backward of 45 -> 64 5x5 @23x26 N=23, 8 bits, 232 / 302).
bool narrow_wgrad_pays(const ConvGeom& g, int K, int64_t room, bool both) {
  const Planned& k = planned(g, both ? BOTH : WGRAD, room);
  if (!k.ok) return false;
  const double w = k.p.wgrad_us, d = k.p.dgrad_us;
  if (!both) return (K == 8 ? 1.85 : 1.7) * w + 4.0 <= ragged_wgrad_us(g, (size_t)g.N * g.H * g.W * g.Cin * sizeof(float));
  if (k.p.w.count > 3 * k.p.copies || d > 1.9 * planned(g, DGRAD).p.dgrad_us) return false;
  const double others = 7.0 + 17.6 * gflop(g) + 0.65e-6 * ((double)g.N * g.H * g.W * g.Cin * 0.5 + 4.0 * g.N * g.Ho * g.Wo * g.Cout);
  return std::max((K == 8 ? 1.45 : 1.2) * w, d) + 2.0 <= planned(g, DGRAD).p.dgrad_us + others;
}

int narrow_fwd_rows(const ConvGeom& g) { return std::min(kMaxPartialBlocks, std::max(32, 4096 / g.Cin)); }

#define ABL_MT(kern, K, VEC) (mt == 1 ? kern<K, 1, VEC> : mt == 2 ? kern<K, 2, VEC> : kern<K, 4, VEC>)

int narrow_fwd_blocks(const ConvGeom& g) {
  const Planned& k = planned(g, FWD);
  return k.ok ? k.p.blocks : 0;
}

int launch_narrow_fwd(hipStream_t st, const ConvGeom& g, int K, const float* x, const float* w, const double* partial, int nb,
                      const float* shift, const float* gamma, const float* beta, void* stats, const float* skip, float* y, void* packed,
                      double* out_partial) {
  const Planned& plan = planned(g, FWD);
  if (!plan.ok) return ABL_ERR_SHAPE;
  if (nb > 0 && partial == out_partial) return ABL_ERR_ARG;   // (a block reads all rows and leaves its own before others begin)
  const NarrowPlan& p = plan.p;
  const int mt = plan.mt;
  const int64_t M = (int64_t)g.N * g.H * g.W, raw = (M * g.Cin * K + 7) / 8;
  const NarrowFwd a{x, w, skip, partial, nb, shift, gamma, beta, static_cast<float*>(stats), y, static_cast<uint8_t*>(packed),
                    (int)((raw + 127) / 128 * 128 - raw), out_partial, M};
  const bool vec = g.Cin % 4 == 0 && g.Cout % 4 == 0;
  if (K != 0 && !vec) return ABL_ERR_SHAPE;
  auto kern = K == 4 ? ABL_MT(narrow_fwd_kernel, 4, true)
            : K == 8 ? ABL_MT(narrow_fwd_kernel, 8, true)
            : vec    ? ABL_MT(narrow_fwd_kernel, 0, true)
                     : ABL_MT(narrow_fwd_kernel, 0, false);
  return launch(st, kern, (unsigned)p.blocks, p.lds, a, p);
}

bool narrow_bwd_blocks(const ConvGeom& g, int64_t room, bool both, int* rows, int* copies) {
  const Planned& w = planned(g, both ? BOTH : WGRAD, room);
  if (!w.ok) return false;
  *copies = w.p.copies;
  const Planned& d = both ? w : planned(g, DGRAD);
  *rows = d.ok ? d.p.blocks : 0;
  return d.ok;
}

int narrow_dgrad_rows(const ConvGeom& g) {
  const Planned& k = planned(g, DGRAD);
  return k.ok ? k.p.blocks : 0;
}

int launch_narrow_bwd(hipStream_t st, const ConvGeom& g, int K, int what, const float* dy, const float* w, const void* packed,
                      const void* stats, float* da3, double* partial, float* copies, int64_t room) {
  const Planned& plan = planned(g, what, (what & 2) != 0 ? room : 0);
  if (!plan.ok) return ABL_ERR_SHAPE;
  const NarrowPlan& p = plan.p;
  const int mt = plan.mt;
  const int second = p.ip * p.w.plane, pair = (what & 2) != 0 && K == 8 && p.wlds + second <= kLds ? 1 : 0;
  const NarrowBwd a{dy, w, static_cast<const uint8_t*>(packed), static_cast<const float*>(stats), da3, partial, copies,
                    (what & 1) != 0 ? p.blocks : 0, pair};
  const unsigned blocks = (unsigned)(a.nd + ((what & 2) != 0 ? p.copies * p.nsub : 0));
  const bool vec = g.Cin % 4 == 0 && g.Cout % 4 == 0;
  auto kern = vec ? (K == 4 ? ABL_MT(narrow_bwd_kernel, 4, true)
                            : ABL_MT(narrow_bwd_kernel, 8, true))
                  : (K == 4 ? ABL_MT(narrow_bwd_kernel, 4, false)
                            : ABL_MT(narrow_bwd_kernel, 8, false));
  return launch(st, kern, blocks, std::max((what & 1) != 0 ? p.lds : 0, (what & 2) != 0 ? p.wlds + pair * second : 0), a, p);
}

}  // namespace abl
