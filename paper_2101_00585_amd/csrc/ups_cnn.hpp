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

// A 3x3 convolution on NHWC tensors: width circular, height zero-padded,
// output (h-1)/stride+1 x (w-1)/stride+1.
struct ConvShape {
    int n, h, w, cin, cout, stride, ho, wo;
};

ConvShape conv_shape(int n, int h, int w, int cin, int cout, int stride);
ups_status conv_check(const ConvShape &c);
int64_t conv_wgt_work_floats(const ConvShape &c);
ups_status launch_conv_fwd(const ConvShape &c, const uint16_t *x, const uint16_t *w_nk, const float *b, uint16_t *y,
                           hipStream_t s);
ups_status launch_conv_bwd_data(const ConvShape &c, const uint16_t *y, const float *dy, const uint16_t *w_kn,
                                float *dx, hipStream_t s);
ups_status launch_conv_bwd_weight(const ConvShape &c, const uint16_t *x, const uint16_t *y, const float *dy,
                                  float *dw, float *db, float *work, int64_t work_floats, hipStream_t s);
ups_status launch_fc_fwd(int n, int feat, const uint16_t *f, const float *Wfc, const float *bfc, float *out,
                         hipStream_t s);
ups_status launch_loss(int n, const float *y, const float *target, float *dout, float *loss, hipStream_t s);
ups_status launch_fc_bwd(int n, int feat, const uint16_t *f, const float *dout, const float *Wfc, float *dWfc,
                         float *dbfc, float *df, hipStream_t s);
ups_status launch_adam(int64_t n, float *p, const float *g, float *m, float *v, float lr, int64_t step,
                       hipStream_t s);
ups_status launch_pack_weight(int K, int N, const float *W, uint16_t *w_kn, uint16_t *w_nk, hipStream_t s);

}  // namespace ups
