// Shared by the CNN gradient translation units: bf16 helpers, layer descriptors, dispatch.
#pragma once

#include <vector>

#include "dpsgd_internal.h"

namespace dpsgd {

typedef unsigned short bf16_t;

__device__ __forceinline__ bf16_t f2bf(float f)
{   // round to nearest, ties to even (v_cvt_pk_bf16_f32)
    const __bf16 h = (__bf16)f;
    return __builtin_bit_cast(unsigned short, h);
}
__device__ __forceinline__ unsigned f2bf_pack(float lo, float hi)
{
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    const f32x2_t v = {lo, hi};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2_t));
}
__device__ __forceinline__ float bf2f(bf16_t h) { return __uint_as_float((unsigned)h << 16); }
__device__ __forceinline__ bool bf16_positive(bf16_t h) { return (h & 0x7fffu) != 0 && (h & 0x8000u) == 0; }

// One 3x3 convolution (zero padding 1): input Ci x H x W, output Co x Ho x Wo, weights at w_off
// ([Co][Ci][3][3] fp32) and one scalar bias at b_off inside a worker's parameter vector.
// How its tensors lie in memory: stored channels, rows and columns of the input (Cis x His x Wis) and of the output
// (Cos x Hos x Wos), each at least the real extent.  What lies beyond the real extent of a stored activation or delta
// holds zeros.  (The network's input image is the caller's and is stored as it is; the stem's His x Wis are those of
// the copies the MFMA stem makes of it.)
struct ConvDesc {
    int Ci, Co, H, W, Ho, Wo, stride;
    long long w_off, b_off;
    int Cis, His, Wis, Cos, Hos, Wos;
    bool padded_out() const { return Cos != Co || Hos != Ho || Wos != Wo; }
};

struct ResnetPlan {
    std::vector<ConvDesc> convs;   // [0] stem, then conv1, conv2 of each block
    long long fcw_off = 0, fcb_off = 0;
    int classes = 0, C_last = 0, H_last = 0, W_last = 0, nblocks = 0;
    int Cs_last = 0, Hs_last = 0, Ws_last = 0;   // stored extents of the last stage
};

// pad: store the stages that fit them in the shapes the MFMA kernels take (see stored_stage); else every tensor has its
// real extents.
ResnetPlan make_resnet_plan(const dpsgd_model_desc &m, bool pad);

// An activation or delta tensor: bf16, channel-major [n][B][C][H][W] (stored extents).  The weight gradient contracts
// over pixels and reads them contiguously; forward and data gradient contract over channels and
// transpose their source rows on the way into LDS; epilogues read and write 4 consecutive pixels
// of one channel.
// `sign` (may be null): one bit per element of an activation, stored per band of 8 rows:
// [n][B][H / 8][C][8 rows][W / 8] bytes, bit i of a byte = pixel 8 k + i of that row is positive.  The MFMA forward kernel writes it next to the activation and the MFMA data gradient reads
// it as its ReLU mask instead of the 16 times larger activation.
struct Tensor {
    bf16_t *t = nullptr;
    unsigned char *sign = nullptr;
};
// Forward: the block input added to the block output at (y*S, x*S) for the first C channels.
// Backward: the delta of the block output added to the block input's delta at multiples of S.
struct ShortcutRef {
    const bf16_t *t;
    int C, H, W, S;
};

// out = round(ReLU(conv(in) + bias + shortcut)).  wpack: this conv's packed bf16 weights (see conv_pack_weights).
// For the stem on MFMA (conv_stem_uses_mfma) `in` is the image padded to 8 channels, pixel-major.
dpsgd_status conv_forward(dpsgd_ctx *ctx, const ConvDesc &c, int B, Tensor in, const float *X, const bf16_t *wpack,
                          ShortcutRef sc, Tensor out);
// A residual block that keeps the resolution, both convolutions in one launch: u = conv_forward(c1, in),
// out = conv_forward(c2, u, shortcut = in), the same bits, without reading u back from memory.  _ok: whether the
// shapes allow it (stride 1; 16 channels on images of 16 or 32 pixels by a multiple of 8 rows, 32 channels on images of
// 16 x 16 pixels, 64 channels on images of 8 x 8 pixels; "conv_block" option on).
bool conv_block_forward_ok(const dpsgd_ctx *ctx, const ConvDesc &c1, const ConvDesc &c2);
dpsgd_status conv_block_forward(dpsgd_ctx *ctx, const ConvDesc &c1, const ConvDesc &c2, int B, Tensor in, const float *X,
                                const bf16_t *wpack1, const bf16_t *wpack2, Tensor u, Tensor out);
// Consecutive residual blocks of that kind, all convolutions convs[first .. first + nconv) in one launch (conv_fwd.hip); _ok: whether
// the shape (the same for all) and the number of images allow it ("conv_block" option on).  Same bits; leaves no sign bitmap (out[..].sign becomes null) but the last one's.
bool conv_chain_ok(const dpsgd_ctx *ctx, const ConvDesc &c, int B);
// ... and whether the block of c1 (stride 2) and c2, which opens a stage, may be the first of them ("conv_down" option on)
bool conv_chain_down_ok(const dpsgd_ctx *ctx, const ConvDesc &c1, const ConvDesc &c2, int B);
// ... and whether the stem c may come before them (first == 0; in: the image, bf16, channel-major, stored extents), next: the
// first block's convolutions
bool conv_chain_stem_ok(const dpsgd_ctx *ctx, const ConvDesc &c, const ConvDesc &next, int B, const void *image);
dpsgd_status conv_chain_forward(dpsgd_ctx *ctx, const std::vector<ConvDesc> &convs, int first, int nconv, int B, Tensor in, const float *X,
                                const std::vector<bf16_t *> &wpack, std::vector<Tensor> &out);
// din = round([act > 0] * (conv^T(dout) + shortcut delta)).
dpsgd_status conv_data_grad(dpsgd_ctx *ctx, const ConvDesc &c, int B, Tensor dout, const float *X, const bf16_t *wpack_d,
                            ShortcutRef scd, Tensor act, Tensor din);
// The weight-gradient kernels of the MFMA path leave partial sums (several workgroups per worker), in accumulator order:
// [co tile][ci tile][tap][lane][4] floats, then one or more sums of the deltas.  What turns them into G is collected here and done
// for all convolutions of the network by ONE launch, conv_weight_grad_finish.
// Floats of one partial sum: whole cache lines, so that the 16-byte stores of every one of them are aligned.
constexpr int wgrad_partial_size(int tiles, int biases) { return (tiles * 9 * 256 + biases + 31) / 32 * 32; }
struct WgradReduceJob {
    const float *part;         // the conv's partial sums, [n][splits][psz]
    long long w_off, b_off;    // where the conv's weights and its scalar bias sit in a worker's parameter vector
    int splits, psz, tiles, biases, ci_tiles, CIr, COr;   // psz: floats of a partial sum; CIr, COr: the conv's real channels
    int block0;                // first blockIdx.x of this job
};
constexpr int kMaxReduceJobs = 48;
struct WgradReduceTable {      // an argument of the reduction kernel
    WgradReduceJob job[kMaxReduceJobs];
    int njobs;
};
struct WgradReduceList {
    WgradReduceTable table;
    int njobs = 0, blocks = 0;
};
// Adds a job (its block0 is set here); what is pending goes out first where the table is full.
dpsgd_status conv_weight_grad_add(dpsgd_ctx *ctx, WgradReduceList *pending, const WgradReduceJob &job, float *G);
// G[w_off..] = dout (*) in, G[b_off] = sum(dout).  partials: this conv's own scratch of conv_wgrad_partial_bytes(ctx, c, B) * n
// bytes, which must stay untouched until conv_weight_grad_finish(pending) has run on the same stream; G holds the
// result only after that call.  Without partials or pending (or for shapes the MFMA kernel does not take) G is
// written directly.
dpsgd_status conv_weight_grad(dpsgd_ctx *ctx, const ConvDesc &c, int B, Tensor in, Tensor dout, float *G, float *partials,
                              WgradReduceList *pending);
dpsgd_status conv_weight_grad_finish(dpsgd_ctx *ctx, WgradReduceList *pending, float *G);

// Whether this conv has packed weights for the forward, or packed weights for the data gradient and partial sums for the weight
// gradient: what the kernels that keep whole images in LDS take from the workspace.
bool conv_has_forward_operands(const ConvDesc &c);
bool conv_has_backward_operands(const ConvDesc &c);
// Bytes per worker of the packed weights of one conv (forward operand, or data-gradient operand).
size_t conv_pack_bytes(const ConvDesc &c, bool dgrad);
size_t conv_wgrad_partial_bytes(const dpsgd_ctx *ctx, const ConvDesc &c, int B);
// Rounds the fp32 weights of every conv and worker to bf16 in MFMA operand order (forward and data-gradient
// operands, wpack_f[q] / wpack_d[q] for convs[q]; nothing is written for convs the MFMA kernels do not take).
dpsgd_status conv_pack_weights(dpsgd_ctx *ctx, const std::vector<ConvDesc> &convs, const float *X,
                               const std::vector<bf16_t *> &wpack_f, const std::vector<bf16_t *> &wpack_d);

// Stem support: whether the first conv runs on MFMA, and the image copies it then needs: a bf16
// channel-major copy (made from fp32 images and where the stored extents differ; may be null) and the image padded to
// 8 channels (NHWC8).
bool conv_stem_uses_mfma(const ConvDesc &c);
// Whether conv_forward fills out.sign for this conv (the stem counts only when it runs on MFMA).
bool conv_forward_writes_sign(const ConvDesc &c, bool is_stem);
// chw_bf16 and nhwc8 are His x Wis pixels, zero beyond H x W.
dpsgd_status conv_prep_image(dpsgd_ctx *ctx, const ConvDesc &c, int B, const void *image, bool image_is_bf16,
                             bf16_t *chw_bf16, bf16_t *nhwc8);

// Weight and data gradient of a 3x3 convolution of stride 1 in one launch (conv_bwd.hip), or of both convolutions of a
// residual block that keeps the resolution, whose inner delta then stays in LDS.  _ok: whether the shapes allow it.
bool conv_bwd_ok(const dpsgd_ctx *ctx, const ConvDesc &c);
bool conv_block_bwd_ok(const dpsgd_ctx *ctx, const ConvDesc &c1, const ConvDesc &c2);
// workgroups per worker (and partial sums of its weight gradient; C: their channels, 0 where there are none)
int conv_image_splits(int n, int B, int slots, int C);
// whether conv_bwd divides a worker's work by channels as well, and the partial sums it leaves
bool conv_bwd_by_channels(const dpsgd_ctx *ctx, const ConvDesc &c, int B, int *splits);
// din = round([act > 0] * (conv^T(dout) + scd)), dW and bias gradient from (act, dout); scd may be null
dpsgd_status conv_bwd(dpsgd_ctx *ctx, const ConvDesc &c, int B, Tensor dout, const bf16_t *wpack_d, const bf16_t *scd, Tensor act,
                      Tensor din, float *G, float *partials, WgradReduceList *pending);
// conv_bwd(c2, dv, u -> du), conv_bwd(c1, du, in -> din, shortcut dv)
dpsgd_status conv_block_bwd(dpsgd_ctx *ctx, const ConvDesc &c1, const ConvDesc &c2, int B, Tensor dv, const bf16_t *wpack_d1,
                            const bf16_t *wpack_d2, Tensor u, Tensor in, Tensor din, float *G, float *partials1, float *partials2,
                            WgradReduceList *pending);

// The same for the convolution of stride 2 that opens a stage (conv_down.hip), scd: the delta of the block output (its channels beyond
// the input's are the shortcut's zeros).
bool conv_down_bwd_ok(const dpsgd_ctx *ctx, const ConvDesc &c);
dpsgd_status conv_down_bwd(dpsgd_ctx *ctx, const ConvDesc &c, int B, Tensor dout, const bf16_t *wpack_d, const bf16_t *scd, Tensor act,
                           Tensor din, float *G, float *partials, WgradReduceList *pending);

dpsgd_status conv_forward_generic(dpsgd_ctx *ctx, const ConvDesc &c, int B, Tensor in, const float *X, ShortcutRef sc,
                                  Tensor out);
dpsgd_status conv_data_grad_generic(dpsgd_ctx *ctx, const ConvDesc &c, int B, Tensor dout, const float *X,
                                    ShortcutRef scd, Tensor act, Tensor din);
dpsgd_status conv_weight_grad_generic(dpsgd_ctx *ctx, const ConvDesc &c, int B, Tensor in, Tensor dout, float *G);

}  // namespace dpsgd
