// What the kernels that keep whole images of the CNN pixel-major in LDS share (conv_fwd.hip, conv_bwd.hip).
#pragma once

#include "resnet_common.h"

namespace dpsgd {
namespace {

typedef long long i64;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

constexpr int ksteps(int ci) { return (9 * ci + 31) / 32; }

// Pixels per LDS row: the image and its halo; rows of 8 pixels are padded so that a row is a multiple of 256 bytes
// (the pixel right of a row and the one left of the next are the same: both are zero)
__host__ __device__ constexpr int row_pixels(int C, int W) { return W >= 16 ? W + 1 : (C == 16 ? 16 : C == 32 ? 12 : 10); }
__host__ __device__ constexpr int image_lds(int C, int W, int H) { return ((H + 2) * row_pixels(C, W) + (W >= 16 ? 1 : 0)) * 2 * C; }

// A group of 8 channels goes to 16-byte unit (group ^ swizzle(column)) of its pixel.  An LDS access of 16 bytes per lane is
// served in four phases, lanes 0-3, 12-15 and 20-27 first, 4-11, 16-19 and 28-31 second, the other half alike; with these, lanes
// reading the same channels of 16 consecutive pixels (or of 8 pixels in each of two rows) at any column meet in no bank, nor
// do the 16-channel rows of 8 consecutive pixels that 32 lanes of a transposing read touch.
template <int C>
__device__ __forceinline__ int swizzle(int col) { return C == 16 ? 0 : C == 32 ? ((col >> 2) & 1) << 1 : ((col >> 1) & 3) << 1; }

// Four pixels of four channels per lane: 16 lanes fetch 4 pixels x 16 channels at p0 (and at p1) and each ends up with the
// pixels of one channel.
__device__ __forceinline__ u32x4 read_transposed(const unsigned char *p0, const unsigned char *p1)
{
    typedef __attribute__((address_space(3))) s16x4 *lds_ptr;
    const s16x4 l = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p0)), h = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p1));
    const u32x2 x = __builtin_bit_cast(u32x2, l), y = __builtin_bit_cast(u32x2, h);
    return (u32x4){x.x, x.y, y.x, y.y};
}

// Images a workgroup of 512 threads takes at a time: as many as give every thread a staging task (32 elements), where their size
// is a usual one
inline int images_at_once(int C, int H, int W) { return (C == 32 && H == 16 && W == 16) || (C == 64 && H == 8 && W == 8) ? 2 : 1; }

// The stages those kernels take: 16, 32 or 64 channels, rows of 8, 16 or (16 channels) 32 pixels, a multiple of 8 rows, at most
// 512 staging tasks an image
inline bool image_shape_ok(const ConvDesc &c)
{
    if (c.stride != 1 || c.Ci != c.Co || c.Cis != c.Cos || c.His != c.Hos || c.Wis != c.Wos) return false;
    const int C = c.Cos, W = c.Wos, H = c.Hos;
    if (H < 8 || H % 8 || H * W * C > 512 * 32) return false;
    return (C == 16 && (W == 8 || W == 16 || W == 32)) || ((C == 32 || C == 64) && (W == 8 || W == 16));
}
}  // namespace
}  // namespace dpsgd
