// Kernels of the pose-proposal network (BF16 MFMA convolutions, FP32 head,
// loss and Adam) and the launchers the proposal object and the layer-level
// C entry points share.
#pragma once

#include <algorithm>
#include <cmath>

#include "ups_internal.hpp"

namespace ups {

constexpr int kCnnOut = 6;  // (omega, t) of the proposed pose

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// round to nearest even
__device__ __forceinline__ uint16_t f2bf(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// four values rounded to nearest even (two per v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint2 bf16x4_of(float4 v) {
    typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
    typedef float f32x4_t __attribute__((ext_vector_type(4)));
    return __builtin_bit_cast(uint2, __builtin_convertvector((f32x4_t{v.x, v.y, v.z, v.w}), bf16x4_t));
}

// Vector accesses to memory that is aligned to its elements only.
struct __attribute__((packed, aligned(2))) PackedU4 { uint32_t x, y, z, w; };
struct __attribute__((packed, aligned(2))) PackedU2 { uint32_t x, y; };
struct __attribute__((packed, aligned(4))) PackedF4 { float x, y, z, w; };
__device__ __forceinline__ uint4 load_u4(const uint16_t *p) {
    const PackedU4 v = *(const PackedU4 *)p;
    return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ uint2 load_u2(const uint16_t *p) {
    const PackedU2 v = *(const PackedU2 *)p;
    return make_uint2(v.x, v.y);
}
__device__ __forceinline__ float4 load_f4(const float *p) {
    const PackedF4 v = *(const PackedF4 *)p;
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void store_f4(float *p, f32x4 v) { *(PackedF4 *)p = PackedF4{v[0], v[1], v[2], v[3]}; }

// A buffer descriptor: loads through it at or past `bytes` read 0.
typedef __amdgpu_buffer_rsrc_t Rsrc;
__device__ __forceinline__ Rsrc rsrc_of(const void *p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, 0x00027000);
}

// A 3x3 convolution on NHWC tensors: width circular, height zero-padded,
// output (h-1)/stride+1 x (w-1)/stride+1.
struct ConvShape {
    int n, h, w, cin, cout, stride, ho, wo;
};

// A walk over the output pixels in steps of `unit`: a step in mixed radix
// (rows and columns; whole images are in step_add), what it adds to the
// offset in x of a window's centre, and what a wrap to the next row or image adds.
struct WalkArgs {
    ConvShape c;
    int step_oy, step_ox;
    uint32_t step_add, row_add, image_add;
};
WalkArgs walk_args(const ConvShape &c, int unit);

// An output pixel (oy, ox) of some image and the offset in x of its window's
// centre, moved along without divisions (each of which costs
// more than the rest of a pixel's staging).
struct PixelWalk {
    int oy, ox;
    uint32_t centre;
    __device__ __forceinline__ void start(const ConvShape &c, int p) {
        const int b = p / (c.ho * c.wo), q = p - b * c.ho * c.wo;
        oy = q / c.wo, ox = q - oy * c.wo;
        centre = (uint32_t)((b * c.h + c.stride * oy) * c.w + c.stride * ox) * (uint32_t)c.cin;
    }
    __device__ __forceinline__ void wrap(const WalkArgs &a) {
        if (ox >= a.c.wo) ox -= a.c.wo, oy++, centre += a.row_add;
        if (oy >= a.c.ho) oy -= a.c.ho, centre += a.image_add;
    }
    __device__ __forceinline__ void step(const WalkArgs &a) {
        ox += a.step_ox, oy += a.step_oy, centre += a.step_add;
        wrap(a);
    }
    __device__ __forceinline__ void next(const WalkArgs &a) {
        ox++, centre += a.c.stride * a.c.cin;
        wrap(a);
    }
};

// Where tap (ky, kx) of a window lies: `off` from the centre, `wrap_add` more
// on output column `wrap_ox` (the width is circular), nowhere on output row
// `no_oy` (the height is zero-padded).
struct Tap {
    int off, wrap_add, wrap_ox, no_oy;
    __device__ __forceinline__ Tap(const ConvShape &c, int ky, int kx) {
        off = ((ky - 1) * c.w + kx - 1) * c.cin;
        wrap_add = kx == 0 ? c.w * c.cin : -c.w * c.cin;
        wrap_ox = kx == 0 ? 0 : (kx == 2 && c.stride * (c.wo - 1) + 1 == c.w) ? c.wo - 1 : -1;
        no_oy = ky == 0 ? 0 : (ky == 2 && c.stride * (c.ho - 1) + 1 >= c.h) ? c.ho - 1 : -1;
    }
    __device__ __forceinline__ bool inside(const PixelWalk &w) const { return w.oy != no_oy; }
    __device__ __forceinline__ uint32_t at(const PixelWalk &w) const {
        return w.centre + off + (w.ox == wrap_ox ? wrap_add : 0);
    }
};

// Four masked gradients in bfloat16: dy where y > 0.
__device__ __forceinline__ uint2 masked_grad4(uint2 y, float4 g) {
    const uint2 h = bf16x4_of(g);
    auto keep = [](uint32_t y2, uint32_t h2) {  // y as a signed integer is positive where it is not a zero and has no sign
        return ((int)(y2 << 16) > 0 ? h2 & 0xFFFFu : 0) | ((int)y2 > 0xFFFF ? h2 & 0xFFFF0000u : 0);
    };
    return make_uint2(keep(y.x, h.x), keep(y.y, h.y));
}

ConvShape conv_shape(int n, int h, int w, int cin, int cout, int stride);
ups_status conv_check(const ConvShape &c);
int64_t conv_wgt_work_floats(const ConvShape &c);  // of this shape
int64_t conv_wgt_work_limit(const ConvShape &c);   // of this one with any number of images up to its own
ups_status launch_conv_fwd(const ConvShape &c, const uint16_t *x, const uint16_t *w_nk, const float *b, uint16_t *y,
                           hipStream_t s);
ups_status launch_conv_bwd_data(const ConvShape &c, const uint16_t *y, const float *dy, const uint16_t *w_kn,
                                float *dx, hipStream_t s);
// The forward pass and the data gradient of layers whose contracted channels
// come in eights, and the forward pass of at most three input channels
// (ups_cnn_conv.hip); false: the tile engine of ups_cnn.hip takes them.
bool conv_gather_fits(const ConvShape &c, bool grad);
bool conv_narrow_fits(const ConvShape &c);
ups_status launch_conv_gather_fwd(const ConvShape &c, const uint16_t *x, const uint16_t *w_nk, const float *b,
                                  uint16_t *y, hipStream_t s);
ups_status launch_conv_narrow_fwd(const ConvShape &c, const uint16_t *x, const uint16_t *w_nk, const float *b,
                                  uint16_t *y, hipStream_t s);
ups_status launch_conv_gather_bwd_data(const ConvShape &c, const uint16_t *y, const float *dy, const uint16_t *w_kn,
                                       float *dx, hipStream_t s);
ups_status launch_conv_bwd_weight(const ConvShape &c, const uint16_t *x, const uint16_t *y, const float *dy,
                                  float *dw, float *db, float *work, int64_t work_floats, hipStream_t s);
ups_status launch_fc_fwd(int n, int feat, const uint16_t *f, const float *Wfc, const float *bfc, float *out,
                         hipStream_t s);
ups_status launch_head_bwd(int n, int feat, const uint16_t *f, const float *y, const float *target, const float *Wfc,
                           float *dWfc, float *dbfc, float *df, float *loss, hipStream_t s);

// A run of consecutive parameters in an update: a convolution's weights
// [9 cin][N] and bias [N], whose gradients are the sums of `splits` partial
// ones, or (sums null) parameters whose gradients are there already.
struct UpdatePart {
    int64_t offset, n;
    int N, splits, block0;
    const float *sums;
    uint16_t *w_kn, *w_nk;
};
struct UpdateArgs {
    UpdatePart part[6];
    int count;
    float *p, *g, *m, *v;
    float lr, beta1, beta2, eps, c1, c2;
};
// The splits' partial sums of the weight gradient into `work`
// (conv_wgt_work_floats), and their number; then the update they enter.
ups_status launch_conv_wgrad_sums(const ConvShape &c, const uint16_t *x, const uint16_t *y, const float *dy, float *work,
                                  int *splits, hipStream_t s);
ups_status launch_conv_update(UpdateArgs &a, float lr, int64_t step, hipStream_t s);
ups_status launch_pack_weight(int K, int N, const float *W, uint16_t *w_kn, uint16_t *w_nk, hipStream_t s);

}  // namespace ups
