// Declarations shared by the gradient translation units.
#pragma once

#include "dpsgd_internal.h"

namespace dpsgd {

typedef float f32x4 __attribute__((ext_vector_type(4)));
// The same in memory, at any float: 16-byte accesses need no more alignment than that, rows may have any length or stride.
typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));

// Four consecutive elements of a row of which only the first `have` exist, as a load whose first element was clamped to
// the row's last four left them: element i sits 4 - have places further on when 0 < have < 4.  Zeros for the rest.
__device__ __forceinline__ f32x4 mend4(f32x4 v, int have)
{
    f32x4 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float x = v[i];
        if (have == 3) x = i < 3 ? v[i + 1 < 4 ? i + 1 : 3] : 0.f;
        if (have == 2) x = i < 2 ? v[i + 2 < 4 ? i + 2 : 3] : 0.f;
        if (have == 1) x = i < 1 ? v[3] : 0.f;
        if (have <= 0) x = 0.f;
        o[i] = x;
    }
    return o;
}

// logits [n][B][C] -> dz = (softmax - onehot)/B and loss[w] (may be null); grid n, block 256.
// Labels outside [0, C) are clamped into range.  With G set, also the bias gradient of the class layer:
// G[w * ld + boff + c] = sum_b dz[w][b][c].
__global__ void softmax_xent_kernel(const float *__restrict__ z, const int *__restrict__ labels, int B, int C,
                                    float *__restrict__ dz, float *__restrict__ loss, float *__restrict__ G,
                                    long long ld, long long boff);

size_t f32_workspace_bytes(const dpsgd_ctx *ctx, const dpsgd_model_desc &m);
dpsgd_status launch_grad_f32(dpsgd_ctx *ctx, const dpsgd_model_desc &m, const float *X, const void *inputs,
                             const void *targets, float *G, float *loss);

bool launch_step_lsq(dpsgd_ctx *ctx, const dpsgd_model_desc &m, float *X, const void *inputs, const void *targets, float *G,
                     float *loss, float *consensus, dpsgd_status *st);

size_t mlp_bf16_workspace_bytes(const dpsgd_ctx *ctx, const dpsgd_model_desc &m);
dpsgd_status launch_grad_mlp_bf16(dpsgd_ctx *ctx, const dpsgd_model_desc &m, const float *X, const void *inputs,
                                  const void *targets, float *G, float *loss);

// One whole iteration in place for bf16 MLPs on a ring: weight gradients of the large layers are formed inside
// the mix kernel and never written to G.
dpsgd_status launch_step_mlp_bf16(dpsgd_ctx *ctx, const dpsgd_model_desc &m, float *X, const void *inputs,
                                  const void *targets, float *G, float *loss, float *consensus);

size_t resnet_workspace_bytes(const dpsgd_ctx *ctx, const dpsgd_model_desc &m);
dpsgd_status launch_grad_resnet(dpsgd_ctx *ctx, const dpsgd_model_desc &m, const float *X, const void *inputs,
                                const void *targets, float *G, float *loss);

}  // namespace dpsgd
