// Internal declarations shared by the HIP translation units of libabl (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "abl.h"

namespace abl {

// Planes of the per-channel `stats` block, each C 4-byte values.
enum StatPlane { P_MEAN = 0, P_VAR, P_RSTD, P_GAMMA, P_BETA, P_CQ, P_STEP, P_FB };

constexpr int kMaxPartialBlocks = 512;  // upper bound on per-block reduction partials

// Bytes of partial-sum workspace for the per-channel reductions over [M,C].
size_t bn_partial_bytes(int64_t M, int C);

// Division by a number that the host knows: 0 <= n < 2^31, exact.  (n m / 2^(31 + l) with m = 2^(31 + l) / d rounded up and
// 2^l >= d is off by less than n 2^-(31 + l) < 1 / d.)
struct Divisor {
  uint32_t mul = 0x80000000u, shift = 0;
  Divisor() = default;
  explicit Divisor(int d) {
    while (((int64_t)1 << shift) < d) ++shift;
    mul = (uint32_t)((((uint64_t)1 << (31 + shift)) + (uint64_t)d - 1) / (uint64_t)d);
  }
  __device__ inline int of(int n) const { return (int)(__umulhi((uint32_t)n << 1, mul) >> shift); }
};

// ---- weights of the split-operand convolutions, split once per call -------------------------------------------
// Parts of all weights in the order in which a wave of split_conv_kernel reads them: [tap][32 contraction channels][16
// output channels][part][lane] 16-byte pieces, eight consecutive contraction channels of one output channel each.  (The
// kernel splits its weights itself where no workspace is at hand; every block does so then.)
struct SplitWeights {
  const float* w;   // [R][S][Cin][Cout]
  uint4* out;       // nullptr: nothing to do
  int mode, np;     // 0 forward, 1 gradient to the input; 3 parts, or 1 = rounded to bf16
  int taps, Cin, Cout;
  __host__ __device__ int64_t items() const { return out != nullptr ? (int64_t)taps * Cin * Cout / 8 : 0; }
};
struct DwSum;
// dwsum (nullable): copies of a weight gradient to be summed by the same launch.
int launch_split_weights(hipStream_t st, const SplitWeights& sw, const DwSum* dwsum = nullptr);

// ---- batch-norm / quantizer kernels (bn_kernels.hip) ----
// sw / next: weights to be split by the launch as well, in blocks of their own.
int launch_bn_stats(hipStream_t st, const float* x, int64_t M, int C, const float* gamma,
                    const float* beta, int K, void* scratch, void* stats, const SplitWeights& sw = SplitWeights{});
// naive: a3 = ReLU of the dequantized code instead of the exact A3 (the baseline of Sec. 4).
// slope: 0 = ReLU (Eq. 3); > 0 = leaky ReLU (Sec. 3.4), in every launcher below that takes one.
int launch_bn_relu_pack(hipStream_t st, const float* x, int64_t M, int C, int K, const void* stats,
                        float* a3, void* packed, bool naive = false, float slope = 0.0f);
int launch_pack(hipStream_t st, const float* a2, int64_t M, int C, int K, const void* stats,
                void* packed);
// act: apply the non-linearity to the dequantized values (the A3~ the weight gradient contracts).
int launch_unpack(hipStream_t st, const void* packed, int64_t M, int C, int K, const void* stats,
                  float* a2t, bool act = false, float slope = 0.0f);
// The first pass of launch_bn_stats alone: *nb rows of sums around x's first row, in scratch.
int launch_bn_stats_partial(hipStream_t st, const float* x, int64_t M, int C, void* scratch, int* nb,
                            int max_rows = kMaxPartialBlocks);
// The second halves of the two reductions, for partial sums produced elsewhere (conv epilogues).
size_t bn_means_offset(int C);
int launch_bn_stats_finalize(hipStream_t st, const double* partial, int nb, const float* shift_row, int64_t M,
                             int C, const float* gamma, const float* beta, int K, void* stats,
                             const SplitWeights& sw = SplitWeights{});
// dwsum (nullable): a weight gradient left as `copies` partial copies of n floats by the conv
// backward kernel; the finalize launch also sums them into dw (fixed order).
struct DwSum {
  const float* partial;
  int copies;
  int64_t n;
  float* dw;
};
int launch_sgd_momentum(hipStream_t st, int64_t n, float lr, float mu, float wd, float* w, const float* grad,
                        float* v);
// Backward of BN + ReLU from dA3 and the codes (Eq. 6-8): both passes.
int launch_bn_bwd(hipStream_t st, const void* packed, const void* stats, const float* da3, int64_t M,
                  int C, int K, bool accum, void* scratch, float* dx, float* dgamma, float* dbeta,
                  const DwSum* dwsum = nullptr, float slope = 0.0f, const SplitWeights& next = SplitWeights{});
int launch_bn_bwd_finish(hipStream_t st, const void* packed, const void* stats, const float* da3, int64_t M,
                         int C, int K, bool accum, void* scratch, int nb, float* dx, float* dgamma,
                         float* dbeta, const DwSum* dwsum = nullptr, float slope = 0.0f, const SplitWeights& next = SplitWeights{});
// Its last launch: Eq. 8 with the means [2][C] at hand.
int launch_bn_bwd_apply(hipStream_t st, const void* packed, const void* stats, const float* da3, int64_t M, int C, int K, bool accum,
                        const float* means, float* dx, float slope = 0.0f, const SplitWeights& next = SplitWeights{});
// Inspection copy of a layer's input (or incoming gradient); trace and its entries may be null.
int trace_copy(hipStream_t st, float* const* trace, int i, const float* src, size_t floats);

// Convolution geometry passed to the kernels by value.
struct ConvGeom {
  int N, H, W, Cin, Cout, R, S, stride, pad, Ho, Wo;
};

inline int out_dim(int in, int pad, int f, int stride) { return (in + 2 * pad - f) / stride + 1; }

inline ConvGeom geom_of(const abl_shape& s) {
  ConvGeom g;
  g.N = s.N; g.H = s.H; g.W = s.W; g.Cin = s.Cin; g.Cout = s.Cout;
  g.R = s.R; g.S = s.S; g.stride = s.stride; g.pad = s.pad;
  g.Ho = out_dim(s.H, s.pad, s.R, s.stride);
  g.Wo = out_dim(s.W, s.pad, s.S, s.stride);
  return g;
}

// ---- stride-1 convolutions with the input tile staged once in LDS (conv_halo.hip) ----
// mode 0: forward, mode 1: gradient to the input.
bool halo_conv_supported(const ConvGeom& g);
int launch_halo_conv(hipStream_t st, const ConvGeom& g, int mode, bool bf16, const float* in, const float* w,
                     const float* skip, float* out, double* out_partial = nullptr);
// Forward with Eq. 1-3 and Eq. 9 applied while the input patch is staged: reads x, writes y and
// the packed codes; A3 never reaches memory.  Supported for 'same' stride-1 convolutions.
bool halo_fused_supported(const ConvGeom& g);
// out_partial (nullable): [tiles][2][Cout] doubles = per-tile sum(y), sum(y^2) of the output,
// the first pass of the next layer's statistics.  halo_tile_count gives `tiles` (0: unsupported).
int halo_tile_count(const ConvGeom& g, int mode);
// Pixels of its tiles and its blocks for this layer; false: not supported.
bool halo_grid(const ConvGeom& g, int mode, int* pixels, int64_t* blocks);
int launch_halo_fwd_fused(hipStream_t st, const ConvGeom& g, int K, bool bf16, const float* x,
                          const void* stats, const float* w, const float* skip, float* y, void* packed,
                          double* out_partial);
// Gradient to the conv input with the first pass of the BN backward (Eq. 6-7 sums from the
// layer's packed codes) in the epilogue: partial = [tiles][2][Cin] doubles.
int launch_halo_dgrad_reduce(hipStream_t st, const ConvGeom& g, int K, bool bf16, const float* dy,
                             const float* w, const void* packed, const void* stats, float* da3,
                             double* partial);

// Weight gradient of stride-1 3x3 convolutions from the packed activation, all taps per pass.
// halo_wgrad_partial_bytes returns 0 when the shape is not supported.
size_t halo_wgrad_partial_bytes(const ConvGeom& g);
int launch_halo_wgrad(hipStream_t st, const ConvGeom& g, int K, bool bf16, const void* packed, const float* stats,
                      const float* dy, void* scratch, float* dw);

// Whole conv backward of a 3x3 'same' stride-1 layer with 16 input and 16 output channels:
// dA3, the Eq. 6-7 partial sums ([tiles][2][16] doubles) and dW in one pass over dy and the codes.
// halo_bwd16_tiles returns 0 when the shape is not supported.  wscratch: as for launch_halo_wgrad.
int halo_bwd16_tiles(const ConvGeom& g);
// dw == nullptr: the per-tile copies of dW ([tiles][3][3][16][16]) are left in wscratch unsummed.
int launch_halo_bwd16(hipStream_t st, const ConvGeom& g, int K, bool bf16, const float* dy, const float* w,
                      const void* packed, const void* stats, float* da3, double* partial, void* wscratch,
                      float* dw);

// ---- the same layers on split operands, fp32 (conv_c16.hip) ----
// Blocks of the forward (mode 0) or of the backward of a layer: rows of sums, copies of dW; 0: not supported.
int c16_tiles(const ConvGeom& g, int mode);
// Forward with Eq. 1's second pass (nb > 0 rows of sums around `shift`, nullable; nb = 0: `stats` is given) and Eq. 1-3, 9.  y is not
// x, out_partial (nullable) not partial.
int launch_c16_fwd(hipStream_t st, const ConvGeom& g, int K, const float* x, const float* w, const double* partial, int nb,
                   const float* shift, const float* gamma, const float* beta, void* stats, const float* skip, float* y, void* packed,
                   double* out_partial);
// As launch_halo_bwd16 without the sum of dW's copies.
int launch_c16_bwd(hipStream_t st, const ConvGeom& g, int K, const float* dy, const float* w, const void* packed, const void* stats,
                   float* da3, double* partial, float* copies);
// The backward of a stack of equal such layers in pairs with a shortcut around each, up to Eq. 7-8 of the bottom layer (its rows
// are in rows[0], its dA3 in da3, its copies of dW in front): Eq. 7-8 of the others go along with the layer below.
// c16_stack_tiles: blocks, 0 = not such a stack; room: bytes for two sets of copies.  means: room for 4 x 16 floats.  trace (nullable):
// where each layer's dy goes (nullable).
int c16_stack_tiles(const abl_layer* layers, int L, int K, int skip_every, size_t room);
int launch_c16_stack_bwd(hipStream_t st, const abl_layer* layers, int L, int K, float* s, float* t, float* da3, double* const (&rows)[2],
                         float* copies, float* means, float* const* trace);

// ---- layers of few channels on split operands, fp32 (conv_narrow.hip) ----
// Where these are the faster kernels: forward with or without the prologue; gradient to the input; the same with the sums of a layer
// call; the weight gradient beside that in one launch, or (both = false, channel counts off sixteen) in its own, of `room` copies.
bool narrow_fwd_pays(const ConvGeom& g);
bool narrow_dgrad_pays(const ConvGeom& g);
bool narrow_bwd_pays(const ConvGeom& g);
bool narrow_wgrad_pays(const ConvGeom& g, int K, int64_t room, bool both);
// Blocks of the forward (rows of its sums of y); 0: not supported.
int narrow_fwd_blocks(const ConvGeom& g);
// Rows of the statistics' sums that its blocks should have to add up at most.
int narrow_fwd_rows(const ConvGeom& g);
// As launch_c16_fwd (K = 4 / 8: both channel counts in fours), or the convolution of a given A3 (K = 0; x is A3).  y is not x.
int launch_narrow_fwd(hipStream_t st, const ConvGeom& g, int K, const float* x, const float* w, const double* partial, int nb,
                      const float* shift, const float* gamma, const float* beta, void* stats, const float* skip, float* y, void* packed,
                      double* out_partial);
// Rows of the Eq. 6-7 sums, and copies of dW, at most `room` of them, of both in one launch or of one after the other; false: not
// supported.
bool narrow_bwd_blocks(const ConvGeom& g, int64_t room, bool both, int* rows, int* copies);
int narrow_dgrad_rows(const ConvGeom& g);   // rows of what = 1
// what: 1 = dA3 and the Eq. 6-7 sums (partial = nullptr: dA3), 2 = the copies of dW, 3 = both.
int launch_narrow_bwd(hipStream_t st, const ConvGeom& g, int K, int what, const float* dy, const float* w, const void* packed,
                      const void* stats, float* da3, double* partial, float* copies, int64_t room);

// ---- convolution kernels (conv_kernels.hip) ----
size_t wgrad_partial_bytes(const abl_shape& s);
// sums / rows (nullable): where the kernel can, it leaves per-block fp64 sums of y and y^2
// ([rows][2][Cout], *rows <= kMaxPartialBlocks) for the next layer's statistics; *rows = 0 if not.
int launch_conv_fwd(hipStream_t st, const abl_shape& s, bool bf16, const float* a3, const float* w,
                    const float* skip, float* y, double* sums = nullptr, int* rows = nullptr, const void* parts = nullptr);
// Parts of the weights that launch_conv_fwd can read (SplitWeights::np), 0 = none.
int conv_fwd_parts(const ConvGeom& g, bool bf16);
int launch_conv_dgrad(hipStream_t st, const abl_shape& s, bool bf16, const float* dy, const float* w,
                      float* da3);
// Forward of a 1x1 stride-1 convolution without padding with Eq. 1-3 and Eq. 9 applied while the
// A tile is staged: reads x, writes y and the packed codes; A3 never reaches memory.  y must not
// alias x.
// 1x1 stride-1 convolutions without padding whose channel counts allow it (contraction a
// multiple of 64, outputs a multiple of 16) run as plain GEMMs with the activation operand
// loaded straight into MFMA layout.  mode 0 forward (skip nullable), 1 dgrad.
bool pointwise_supported(const ConvGeom& g, int mode);
int launch_pointwise_conv(hipStream_t st, const ConvGeom& g, int mode, bool bf16, const float* in, const float* w,
                          const float* skip, float* out, double* sums = nullptr, int* rows = nullptr);
int launch_pointwise_fwd_fused(hipStream_t st, const ConvGeom& g, int K, bool bf16, const float* x, const float* stats,
                               const float* w, const float* skip, float* y, void* packed, double* sums = nullptr,
                               int* rows = nullptr);
// dgrad (Eq. 5) with the Eq. 6-7 sums taken in its epilogue from the layer's codes: one row of
// [2][Cin] doubles per block, *rows of them (<= kMaxPartialBlocks), for launch_bn_bwd_finish.
int launch_pointwise_dgrad_reduce(hipStream_t st, const ConvGeom& g, int K, bool bf16, const float* dy, const float* w,
                                  const void* packed, const void* stats, float* da3, double* sums, int* rows);
bool igemm_fused_supported(const abl_shape& s);
int launch_conv_fwd_fused(hipStream_t st, const abl_shape& s, int K, bool bf16, const float* x, const void* stats,
                          const float* w, const float* skip, float* y, void* packed, double* sums = nullptr,
                          int* rows = nullptr);
// K = 32: `packed` is an fp32 tensor, used as it is or (relu32) as the pre-ReLU activation A2.
// defer (nullable): where the kernel leaves split partial copies, describe them there instead of
// summing them (copies = 0 when dw is already complete) - for launch_bn_bwd_finish.
// room: bytes at `scratch`; channel counts that are not multiples of 16 need it, the split kernels make more copies of more
// (wgrad_partial_bytes at least are taken to be there).
int launch_conv_wgrad_packed(hipStream_t st, const abl_shape& s, int K, bool bf16, const void* packed,
                             const void* stats, const float* dy, void* scratch, float* dw, bool relu32 = false,
                             DwSum* defer = nullptr, size_t room = 0);

// ---- channel counts that are not multiples of 16 (conv_ragged.hip), fp32 ----
// What launch_ragged_conv (mode 1, filters) and launch_conv_wgrad_packed take on up to 64 channels, us.
double ragged_dgrad_us(const ConvGeom& g);
double ragged_wgrad_us(const ConvGeom& g, size_t room);
inline bool channels_in_tiles(const ConvGeom& g) { return g.Cin % 16 == 0 && g.Cout % 16 == 0; }
int launch_ragged_conv(hipStream_t st, const ConvGeom& g, int mode, const float* in, const float* w, const float* skip,
                       float* out);
// Copies of dW ([copies][R][S][Cin][Cout] floats, 1 = dW itself) that launch_ragged_wgrad writes with `room` bytes
// for them; 0: the kernel with a block per element of dW is the faster one.
int ragged_wgrad_copies(const ConvGeom& g, size_t room);
int launch_ragged_wgrad(hipStream_t st, const ConvGeom& g, int K, const void* packed, const float* stats,
                        const float* dy, int copies, float* dst, bool relu32);

// ---- ABL_MATH_BF16 contractions on the 32-deep bf16 matrix instruction (conv_bf16.hip) ----
// Forward (mode 0) / gradient to the input (mode 1) of any stride, filter and padding whose
// contraction channels are a multiple of 32 and output channels a multiple of 64.
bool bf16_gemm_supported(const ConvGeom& g, int mode);
// sums / rows (nullable, mode 0): [*rows][2][Cout] doubles = per-block sum(y), sum(y^2) of the output;
// *rows = 0 when the kernel leaves none (more blocks than kMaxPartialBlocks).
int launch_bf16_gemm(hipStream_t st, const ConvGeom& g, int mode, const float* in, const float* w, const float* skip,
                     float* out, double* sums = nullptr, int* rows = nullptr);
// Gradient to the conv input with the Eq. 6-7 sums from the layer's codes (K = 4 / 8) in the epilogue of
// whichever bf16 kernel takes the shape: partial = [rows][2][Cin] doubles; bf16_dgrad_reduce_rows = 0 if none does.  parts:
// whether the weights come in parts as well.
int bf16_dgrad_reduce_rows(const ConvGeom& g, bool parts);
int launch_bf16_dgrad_reduce(hipStream_t st, const ConvGeom& g, int K, const float* dy, const float* w,
                             const void* packed, const void* stats, float* da3, double* partial,
                             const void* parts = nullptr);
// Whether that is split_conv_kernel with one part, which can read `parts`.
bool bf16_dgrad_reduce_splits(const ConvGeom& g, bool parts);
// 3x3 'same' stride-1 convolutions whose whole image fits in LDS as bf16 (up to 208 pixels, e.g.
// 14x14 with 256 channels): one block per image and 64 output channels.
// sums (nullable, mode 0): [N][2][Cout] doubles = per-image sum(y), sum(y^2) of the output.
// parts: the weights come in parts as well, which split_conv_kernel reads.
bool image_bf16_supported(const ConvGeom& g, int mode, bool parts = false);
int launch_image_bf16(hipStream_t st, const ConvGeom& g, int mode, const float* in, const float* w,
                      const float* skip, float* out, double* sums);

// ---- fp32 contractions on the bf16 matrix cores, operands split into three bf16 parts (conv_split.hip) ----
// 'same' stride-1 3x3 and 1x1 layers with contraction channels in multiples of 32 (1x1: 64) and output channels
// in multiples of 64, where they are the faster ones.  split_conv_blocks: rows of the sums ([rows][2][C] doubles: of y in mode
// 0, Eq. 6-7 in launch_split_dgrad_reduce), 0 = not supported.
// bf16: operands rounded to bf16 instead.
// sums: with the Eq. 6-7 sums (launch_split_dgrad_reduce).
// parts (nullable, in the launchers): the weights as SplitWeights leaves them, same mode and operands.
int split_conv_blocks(const ConvGeom& g, int mode, bool bf16 = false, bool sums = false);
// Whether splitting the weights of a layer that split_conv_kernel takes once per call (SplitWeights) is faster than in the kernel.
// own_launch: no other launch can do it (the gradient of abl_backward, and of a stack's last layer).
bool parts_pay(const ConvGeom& g, int mode, bool bf16, bool own_launch);
// Whether split_conv_kernel with bf16 operands is faster than the image-resident kernel on a 3x3 layer that both take.
bool split_beats_image(const ConvGeom& g, int mode);
bool split_parts_beat_image(const ConvGeom& g, int mode);   // ... with the weights in parts
// The fp32 forward of a 1x1 layer with a pass of its own for Eq. 1-3 and 9 in front is faster than the pointwise kernel's
// prologue.
bool split_beats_prologue(const ConvGeom& g);
int launch_split_conv(hipStream_t st, const ConvGeom& g, int mode, bool bf16, const float* in, const float* w,
                      const float* skip, float* out, double* sums, const void* parts = nullptr);
// The 3x3 forward with Eq. 1-3 and Eq. 9 (fp32 operands, y not x): 1 = launch_split_fwd_fused, which applies them while the
// patch is staged (*rows = rows of its sums), -1 = launch_split_conv with a pass of its own in front, 0 = other kernels.
int split_forward3(const ConvGeom& g, int* rows);
int launch_split_fwd_fused(hipStream_t st, const ConvGeom& g, int K, const float* x, const void* stats, const float* w,
                           const float* skip, float* y, void* packed, double* sums, const void* parts = nullptr);
int launch_split_dgrad_reduce(hipStream_t st, const ConvGeom& g, int K, bool bf16, const float* dy, const float* w,
                              const void* packed, const void* stats, float* da3, double* partial,
                              const void* parts = nullptr);

// Weight gradient of 'same' stride-1 3x3 and 1x1 layers from the codes, dy split into three bf16 parts
// (wgrad_split.hip; Cin a multiple of 32 - 1x1: 64 - and Cout of 64).  split_wgrad_copies: copies of dW that
// launch_split_wgrad leaves in dst, at most `room` bytes of them ([copies][R][S][Cin][Cout] floats); 0 = not supported or
// not the faster kernel.  bf16: both operands rounded to bf16 instead.
int split_wgrad_copies(const ConvGeom& g, int K, bool bf16, size_t room);
int launch_split_wgrad(hipStream_t st, const ConvGeom& g, int K, bool bf16, const void* packed, const float* stats,
                       const float* dy, float* dst, size_t room);

// ---- fp32 3x3 'same' stride-1 convolutions with the whole image resident in LDS (conv_image.hip) ----
// Images of up to 208 pixels (14x14, 7x7 ...), 16, 32 or a multiple of 64 contraction channels,
// output channels a multiple of 64, at most kMaxPartialBlocks images and at least 224 blocks: one
// block per image and 64 output channels.
// sums (nullable, mode 0): [N][2][Cout] doubles = per-image sum(y), sum(y^2) of the output.
bool image_f32_supported(const ConvGeom& g, int mode);
int launch_image_f32(hipStream_t st, const ConvGeom& g, int mode, const float* in, const float* w,
                     const float* skip, float* out, double* sums);
// Gradient to the conv input with the Eq. 6-7 sums from the layer's packed codes (K = 4 / 8) in the
// epilogue: partial = [N][2][Cin] doubles, one row per image.
int launch_image_dgrad_reduce(hipStream_t st, const ConvGeom& g, int K, const float* dy, const float* w,
                              const void* packed, const void* stats, float* da3, double* partial);

// Copies of dW that the workspace of a 3x3 layer on 14-pixel-wide images has room for (0: the tiled kernel's).
int image_wgrad_copies(const ConvGeom& g, int K);

// Weight gradient of a 1x1 stride-1 layer from its K-bit codes with operands rounded to bf16 and the block's 64 x 256
// tile of dW in registers (Cin a multiple of 64, Cout of 256, N H W of 32).  Each share of the pixels writes its own
// copy of dW in `copies` ([rows_wgrad_copies][Cin][Cout] floats) for the caller to sum.  rows_wgrad_copies returns 0
// when the shape is not supported; with bf16 = false it counts N H W in multiples of 16 (the workspace's size).
int rows_wgrad_copies(const ConvGeom& g, int K, bool bf16);
int launch_rows_wgrad(hipStream_t st, const ConvGeom& g, int K, const void* packed, const float* stats,
                      const float* dy, float* copies);

// ---- Eq. 9 / Eq. 10 for one value.  Callers must be compiled with floating-point contraction
// off: the codes are compared bit for bit with an IEEE fp32 evaluation.
// floor() limited to +-2^24 so that the integer conversion is defined for any input.
__device__ inline float limit_floor(float u) {
  const float lim = 16777216.0f;
  // one instruction: the median of (u, -lim, lim); a NaN input gives the smallest of the other
  // two, -lim, as the comparison form (u >= -lim ? u : -lim) does
  return __builtin_amdgcn_fmed3f(floorf(u), -lim, lim);
}

// Eq. 9 for one value (cq = 2^K/(6 gamma), fb = floor(beta*cq)).  K = 32 is exact storage: the
// "code" is the value's bit pattern.
template <int K>
__device__ inline uint32_t quant_code(float a2, float cq, int32_t fb) {
  if constexpr (K == 32) {
    return __float_as_uint(a2);
  } else {
    const float u = limit_floor(a2 * cq);
    int32_t v = (int32_t)u + (1 << (K - 1)) - fb;
    v = v < 0 ? 0 : v;
    v = v > (1 << K) - 1 ? (1 << K) - 1 : v;
    return (uint32_t)v;
  }
}

// The planes of one channel's statistics (StatPlane; fb as its bits) from its two sums, taken around `shift`.
__device__ inline void channel_constants(double t0, double t1, float shift, int64_t M, float gm, float bt, int K, float (&out)[8]) {
  const double k = (double)shift;
  const double mk = t0 / (double)M;
  double var = t1 / (double)M - mk * mk;
  var = var > 0.0 ? var : 0.0;
  const float var_f = (float)var;
  out[P_MEAN] = (float)(k + mk);
  out[P_VAR] = var_f;
  out[P_RSTD] = (float)(1.0 / sqrt((double)var_f + (double)ABL_BN_EPS));
  // K = 32 (exact storage) has no quantizer: the constants are written as zeros
  const float two_k = K < 32 ? (float)(1 << K) : 0.0f;
  const float six_g = 6.0f * gm;
  // double division then one rounding == correctly rounded fp32 division
  const float cq = K < 32 ? (float)((double)two_k / (double)six_g) : 0.0f;
  out[P_GAMMA] = gm;
  out[P_BETA] = bt;
  out[P_CQ] = cq;
  out[P_STEP] = K < 32 ? (float)((double)six_g / (double)two_k) : 0.0f;
  out[P_FB] = __int_as_float(K < 32 ? (int32_t)limit_floor(bt * cq) : 0);
}

// Eq. 10 for one code.
template <int K>
__device__ inline float dequant(uint32_t q, float step, int32_t fb) {
  if constexpr (K == 32) {
    return __uint_as_float(q);
  } else {
    const int32_t j = (int32_t)q - (1 << (K - 1)) + fb;
    const float t = (float)j + 0.5f;
    return step * t;
  }
}

// Sum over the 16 lanes of a row (lanes that differ in bits 0-3); every lane gets the total.
// (Data-parallel-primitive moves within the row: swap neighbours, swap pairs, mirror each half,
// mirror the row.)
template <int CTRL>
__device__ inline double dpp_move(double v) {
  const unsigned long long u = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, 0xf, 0xf, false);
  return __longlong_as_double(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}
__device__ inline double row16_sum(double v) {
  v += dpp_move<0xB1>(v);   // quad_perm [1,0,3,2]
  v += dpp_move<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dpp_move<0x141>(v);  // row_half_mirror
  v += dpp_move<0x140>(v);  // row_mirror
  return v;
}

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef short shortx4 __attribute__((ext_vector_type(4)));

// D = A(16x4) * B(4x16) + C on the fp32 matrix cores; lane l supplies A[l%16][l/16] and
// B[l/16][l%16] and holds D[4*(l/16) + r][l%16], r = 0..3.
__device__ inline floatx4 mfma16(float a, float b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// fp32 -> bf16, round to nearest even, by the hardware's packed convert (v_cvt_pk_bf16_f32).
typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
// eight floats -> the 8-deep bf16 operand of one lane of v_mfma_f32_16x16x32_bf16
__device__ inline bf16x8_t to_bf16x8(const float (&v)[8]) {
  return bf16x8_t{(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3],
                  (__bf16)v[4], (__bf16)v[5], (__bf16)v[6], (__bf16)v[7]};
}
// ---- 16-byte pieces of eight bf16 values in LDS (conv_c16.hip, conv_narrow.hip) ----
typedef short short4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) short4_t lds_short4;

__device__ inline floatx4 mfma32(const bf16x8_t& a, const bf16x8_t& b, const floatx4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ inline bf16x8_t piece(const char* p) { return *reinterpret_cast<const bf16x8_t*>(p); }
__device__ inline void put(char* p, const bf16x8_t& v) { *reinterpret_cast<bf16x8_t*>(p) = v; }
// Eight positions of one channel: 16 lanes fetch four positions' 16 channels each time and receive one channel's four.
__device__ inline bf16x8_t transposed(const char* p, const char* q) {
  struct two { short4_t a, b; };
  const two t{__builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)p), __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)q)};
  return __builtin_bit_cast(bf16x8_t, t);
}
__device__ inline bool finite(float v) { return __builtin_fabsf(v) <= 3.402823466e38f; }
// ---- fp32 operands in three bf16 parts (conv_split.hip) ----
constexpr float kUp = 0x1p23f, kDown = 0x1p-46f;   // both operands are split as 2^23 times their values
// u holds two bf16 values: a minus the lower or the upper one in one instruction (fp32 result of exact products, here exact).  The
// selector stays in a scalar register: as a literal constant of the instruction the lower one came out as zero.
__device__ inline float less_low(float a, uint32_t u) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  uint32_t minus_one = 0x0000BF80u;
  asm("" : "+s"(minus_one));
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, u), __builtin_bit_cast(bf16x2, minus_one), a, false);
}
__device__ inline float less_high(float a, uint32_t u) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  uint32_t minus_one = 0xBF800000u;
  asm("" : "+s"(minus_one));
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, u), __builtin_bit_cast(bf16x2, minus_one), a, false);
}
// 2^23 x = h + m + l, eight values at a time (the parts of two values share a 32-bit word).
// TOGETHER: the eight go into the same sums.  Then the remainders of a pair may share an instruction's operand, where an infinity
// of one makes the other NaN: 9 instead of 13 instructions a pair (a loop of splits 2.10 -> 1.45 ms), the same bits otherwise.
template <bool TOGETHER = true>
__device__ inline void split3(const float (&x)[8], bf16x8_t& h, bf16x8_t& m, bf16x8_t& l) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  uint4 hw, mw, lw;
  auto two = [](float a, float b, uint32_t& u, uint32_t& v, uint32_t& w) __attribute__((always_inline)) {
    a *= kUp;
    b *= kUp;
    u = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)a, (__bf16)b});
    if constexpr (TOGETHER) {
      const float ra = less_low(a, u), rb = less_high(b, u);
      v = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)ra, (__bf16)rb});
      w = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)less_low(ra, v), (__bf16)less_high(rb, v)});
    } else {
      const float ra = a - __uint_as_float(u << 16), rb = b - __uint_as_float(u & 0xFFFF0000u);
      v = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)ra, (__bf16)rb});
      w = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)(ra - __uint_as_float(v << 16)),
                                              (__bf16)(rb - __uint_as_float(v & 0xFFFF0000u))});
    }
  };
  two(x[0], x[1], hw.x, mw.x, lw.x);
  two(x[2], x[3], hw.y, mw.y, lw.y);
  two(x[4], x[5], hw.z, mw.z, lw.z);
  two(x[6], x[7], hw.w, mw.w, lw.w);
  h = __builtin_bit_cast(bf16x8_t, hw);
  m = __builtin_bit_cast(bf16x8_t, mw);
  l = __builtin_bit_cast(bf16x8_t, lw);
}

__device__ inline void split_weights_item(const SplitWeights& s, int64_t it) {
  const int Cg = s.mode == 0 ? s.Cin : s.Cout, Ng = s.mode == 0 ? s.Cout : s.Cin;
  const int lane = (int)(it & 63), li = lane & 15, lk = lane >> 4;
  const uint32_t tile = (uint32_t)(it >> 6);
  const uint32_t step = tile / (uint32_t)(Ng / 16), n = 16 * (tile - step * (uint32_t)(Ng / 16)) + li;
  const uint32_t tap = step / (uint32_t)(Cg / 32), c = 32 * (step - tap * (uint32_t)(Cg / 32)) + 8 * lk;
  float x[8];
  if (s.mode == 0) {
    const float* p = s.w + ((size_t)tap * s.Cin + c) * s.Cout + n;
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = p[(size_t)e * s.Cout];
  } else {
    const float* p = s.w + ((size_t)(s.taps - 1 - tap) * s.Cin + n) * s.Cout + c;
#pragma unroll
    for (int q = 0; q < 8; q += 4) {
      const floatx4 v = *reinterpret_cast<const floatx4*>(p + q);
#pragma unroll
      for (int e = 0; e < 4; ++e) x[q + e] = v[e];
    }
  }
  uint4* to = s.out + (size_t)tile * 64 * s.np + lane;
  if (s.np == 3) {
    bf16x8_t h, m, l;
    split3(x, h, m, l);
    to[0] = __builtin_bit_cast(uint4, h);
    to[64] = __builtin_bit_cast(uint4, m);
    to[128] = __builtin_bit_cast(uint4, l);
  } else {
    to[0] = __builtin_bit_cast(uint4, to_bf16x8(x));
  }
}

__device__ inline shortx4 to_bf16x4(const float4& v) {
  const bf16x4_t b = {(__bf16)v.x, (__bf16)v.y, (__bf16)v.z, (__bf16)v.w};
  return __builtin_bit_cast(shortx4, b);
}

// Contract four consecutive k (one float4 per lane and operand row) into every accumulator
// tile.  fp32: four 16x16x4 MFMAs per tile, component e of the float4 = k-step e, the lane
// group l/16 = k within the step.  bf16: operands rounded to bf16, ONE 16x16x16 MFMA per
// tile, lane group l/16 supplies k = 4*(l/16) + e; accumulation stays fp32.
template <bool BF16, int MT, int NT>
__device__ inline void mma_k4(const float4 (&af)[MT], const float4 (&bf)[NT], floatx4 (&acc)[MT][NT]) {
  if constexpr (BF16) {
    shortx4 a[MT], b[NT];
#pragma unroll
    for (int i = 0; i < MT; ++i) a[i] = to_bf16x4(af[i]);
#pragma unroll
    for (int j = 0; j < NT; ++j) b[j] = to_bf16x4(bf[j]);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a[i], b[j], acc[i][j], 0, 0, 0);
  } else {
    // k-step outermost: consecutive MFMAs write different accumulators
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[i][j] = mfma16(af[i].x, bf[j].x, acc[i][j]);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[i][j] = mfma16(af[i].y, bf[j].y, acc[i][j]);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[i][j] = mfma16(af[i].z, bf[j].z, acc[i][j]);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[i][j] = mfma16(af[i].w, bf[j].w, acc[i][j]);
  }
}

// The same contraction for the first NB (compile-time, <= NT) tiles of the second operand only;
// the others are left untouched and cost no matrix-core time.
template <bool BF16, int MT, int NT, int NB>
__device__ inline void mma_k4_first(const float4 (&af)[MT], const float4 (&bf)[NT], floatx4 (&acc)[MT][NT]) {
  static_assert(NB <= NT, "at most all tiles");
  if constexpr (BF16) {
    shortx4 a[MT], b[NB > 0 ? NB : 1];
#pragma unroll
    for (int i = 0; i < MT; ++i) a[i] = to_bf16x4(af[i]);
#pragma unroll
    for (int j = 0; j < NB; ++j) b[j] = to_bf16x4(bf[j]);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a[i], b[j], acc[i][j], 0, 0, 0);
  } else {
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) acc[i][j] = mfma16(af[i].x, bf[j].x, acc[i][j]);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) acc[i][j] = mfma16(af[i].y, bf[j].y, acc[i][j]);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) acc[i][j] = mfma16(af[i].z, bf[j].z, acc[i][j]);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) acc[i][j] = mfma16(af[i].w, bf[j].w, acc[i][j]);
  }
}

// v where ok, zeros elsewhere - written per component so that it stays in registers
__device__ inline float4 keep_if(bool ok, const float4& v) {
  return make_float4(ok ? v.x : 0.f, ok ? v.y : 0.f, ok ? v.z : 0.f, ok ? v.w : 0.f);
}

// Grids of one dimension: more than 2^22 blocks go on in y, since a dimension holds fewer than 2^32 work-items (a larger
// one is cut off without an error).  The last row of blocks may go past the end; up to 2^31 blocks in all.
inline dim3 grid_of(int64_t blocks) {
  const int64_t x = (int64_t)1 << 22;
  return blocks <= x ? dim3((unsigned)blocks) : dim3((unsigned)x, (unsigned)((blocks + x - 1) / x));
}
__device__ inline uint32_t block_of_grid() { return blockIdx.x + gridDim.x * blockIdx.y; }

// More than the default 64 KB of LDS per block has to be asked for, once per kernel and device (the full 160 KB, so that
// the answer does not depend on the first shape seen); any thread.  An ABL_ code.
int allow_full_lds(const void* kern);

inline int hip_status() { return hipGetLastError() == hipSuccess ? ABL_OK : ABL_ERR_HIP; }

}  // namespace abl
