// Weight and bias gradients of the 3x3 convolutions:
//   dW[r][co] = sum over output pixels p of X_col[p][r] G[p][co],  r = (tap, ci),
//   db[co]    = sum over p of G[p][co],
// G = dL/dy masked by y > 0 (ReLU) and rounded to bfloat16.  The contraction
// runs over pixels while both operands lie in memory with their channels
// contiguous, so the blocks stage them as they lie ([pixel][row] and
// [pixel][co] in LDS, 16-byte loads and stores) and the matrix-core fragments
// come from gfx950's transposing LDS read (ds_read_b64_tr_b16): the lanes of a
// 16-lane group supply the addresses of four pixels' 16-element rows and each
// receives the four pixels of one row element.
//
// The order of every sum is that of the flattened contraction: a split's pixels
// in ascending slices of 32, a slice's pixels in order within the instruction,
// the splits as sum_splits says.  A training step's weights are rounded to
// bfloat16, so a sum added in another order is not a difference of 1e-7 in the
// steps after it: one weight that rounds the other way moved the gradients by
// 4e-4.
#include "ups_cnn.hpp"

namespace ups {

namespace {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

struct WgradArgs {
    WalkArgs walk;
    const uint16_t *x, *y;
    const float *dy;
    float *w_sums, *b_sums;  // [9 cin][cout] and [cout] of the first split
    int64_t split_stride;    // from a split's sums to the next one's
    int chunk;               // output pixels of a split
};

// Fragment of rows e0 .. e0+15 over the 32 pixels from row p0 of an LDS image
// [pixel][element] of `pitch` bytes whose rows are in the order of lds_row: lane
// group g holds pixels 8g .. 8g+7, which lie in rows 4g .. 4g+3 and 16+4g ..
// 16+4g+3, so the sixteen 32-byte rows of one read fall on different banks when
// the pitch is an odd multiple of 32 bytes.
__device__ __forceinline__ int lds_row(int pixel) {
    return (pixel & ~31) + ((pixel & 24) >> 1) + ((pixel & 4) << 2) + (pixel & 3);
}
__device__ __forceinline__ bf16x8 tr_fragment(const uint8_t *base, int pitch, int p0, int e0) {
    const int l = threadIdx.x & 63, px = p0 + 4 * (l >> 4) + ((l & 15) >> 2);
    const uint8_t *p = base + px * pitch + 2 * e0 + 8 * (l & 3);
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)p);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p + 16 * pitch));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

constexpr int kRowTile = 288, kPix = 64, kWideThreads = 576;

// Wide form: a block of nine wavefronts owns kRowTile rows r and NF * 16
// output channels (each wavefront 32 rows) over one split of the pixels, 64
// pixels a step; 288 rows are all nine taps of 32 channels, so few blocks
// read a gradient.  Bound by a step's round trips (window loads, LDS, barrier)
// with about one block a CU, which the workspace of the splits' sums sets; so
// two steps' loads are in flight and two LDS buffers leave one barrier a step.
// Layers of 32 -> 64, 64 -> 96, 96 -> 128 and 128 -> 128 channels at batch
// 256: 26.5, 27.7, 17.8 and 18.0 us with the reduction, against 177.5, 165.6,
// 68.6 and 78 on 64 x 64 tiles gathered along pixels by 2-byte loads.  UNIT:
// elements per load of x (8 where cin is a multiple of 8, 2 where it is even,
// else 1, whose 32 loads a step leave registers for one step in flight).
// Window elements shorter than a vector load come through a buffer descriptor,
// no load behind a branch: a load whose result joins another's in one
// register inside a branch waits there (65536 pixels of 5, 33 and 4 -> 64
// channels: 22.8, 59.8 and 18.4 us so; 53.7, 119.8 and 30.7 with branches and a
// division an element).
template <int NF, int UNIT>
__global__ __launch_bounds__(kWideThreads) void k_conv_wgrad(WgradArgs a) {
    constexpr int kXP = kRowTile * 2 + 32;                      // 19 x 32 bytes
    constexpr int kGP = (NF % 2) ? NF * 32 + 64 : NF * 32 + 32;  // an odd multiple of 32 bytes
    __shared__ __align__(16) uint8_t xs[2][kPix * kXP];
    __shared__ __align__(16) uint8_t gs[2][kPix * kGP];
    const ConvShape &c = a.walk.c;
    // the wavefront's number as a scalar: MFMA ignores the execution mask, so what it guards has to be a scalar branch
    const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    const int rows = 9 * c.cin, row0 = blockIdx.x * kRowTile, co0 = blockIdx.y * NF * 16;
    const int p_begin = blockIdx.z * a.chunk, p_end = min(c.n * c.ho * c.wo, p_begin + a.chunk);
    // staging: 8 rows of four consecutive pixels of each step, and 8 channels of one pixel
    const int r8 = t % 36, pr = 4 * (t / 36), r = row0 + 8 * r8;
    const int tap = r / c.cin, ci = r - tap * c.cin;
    const Tap at(c, tap / 3, tap % 3);
    // the same for single elements: window row ky0, element k0 of its 3 cin in memory order
    const int row_k = 3 * c.cin, ky0 = r / row_k, k0 = r - ky0 * row_k;
    const Tap at0(c, ky0, 0), at1(c, ky0 + 1, 0);
    const int last_ox = c.stride * (c.wo - 1) + 1 == c.w ? c.wo - 1 : -1;
    const Rsrc xr = rsrc_of(a.x, 2 * (uint32_t)(c.n * c.h * c.w) * (uint32_t)c.cin);
    constexpr uint32_t kNowhere = UNIT == 2 ? 0xFFFFFFFCu : 0xFFFFFFFEu;  // past every tensor
    PixelWalk px;
    px.start(c, p_begin + pr);
    const int gp = t / (2 * NF), gc = co0 + 8 * (t % (2 * NF));
    constexpr int kStages = UNIT == 1 ? 1 : 2;
    struct Staged {
        uint32_t x[4][8 / UNIT * (UNIT == 8 ? 4 : 1)];
        float4 dy[2];
        uint2 y[2];
    } st[kStages];
    auto fetch = [&](Staged &f, int p0) {
        PixelWalk w = px;
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int p = p0 + pr + i;
            if constexpr (UNIT == 8) {
                uint4 v = make_uint4(0, 0, 0, 0);
                if (p < p_end && r < rows && at.inside(w)) v = load_u4(a.x + at.at(w) + ci);
                f.x[i][0] = v.x, f.x[i][1] = v.y, f.x[i][2] = v.z, f.x[i][3] = v.w;
            } else {
                const bool on0 = p < p_end && ky0 < 3 && at0.inside(w), on1 = p < p_end && ky0 < 2 && at1.inside(w);
                const int left = w.ox == 0 ? c.w * c.cin : 0, right = w.ox == last_ox ? c.w * c.cin : 0;
#pragma unroll
                for (int e = 0; e < 8; e += UNIT) {
                    const bool next = k0 + e >= row_k;  // of the next window row
                    const int k = k0 + e - (next ? row_k : 0);
                    const uint32_t o = w.centre + (next ? at1.off : at0.off) + k + (k < c.cin ? left : k >= 2 * c.cin ? -right : 0);
                    const uint32_t b = (next ? on1 : on0) ? 2 * o : kNowhere;
                    f.x[i][e / UNIT] = UNIT == 2 ? (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(xr, b, 0, 0)
                                                 : (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(xr, b, 0, 0);
                }
            }
            if (i < 3) w.next(a.walk);
        }
        px.step(a.walk);
        if (gp < kPix)
#pragma unroll
            for (int hh = 0; hh < 2; hh++) {
                const int p = p0 + gp, co = gc + 4 * hh;
                f.dy[hh] = make_float4(0.f, 0.f, 0.f, 0.f);
                f.y[hh] = make_uint2(0, 0);
                if (p < p_end && co < c.cout) {
                    const size_t o = (size_t)p * c.cout + co;
                    f.dy[hh] = load_f4(a.dy + o);
                    f.y[hh] = load_u2(a.y + o);
                }
            }
    };
    f32x4 acc[2][NF], accb = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int m = 0; m < 2; m++)
#pragma unroll
        for (int f = 0; f < NF; f++) acc[m][f] = f32x4{0.f, 0.f, 0.f, 0.f};
    const bool bias = blockIdx.x == 0 && wave < NF;  // this wavefront also sums channels 16 wave ..
    constexpr uint16_t one = 0x3F80;
    const bf16x8 ones = __builtin_bit_cast(bf16x8, s16x8{one, one, one, one, one, one, one, one});
    auto step = [&](Staged &f, int buf, int p0) {
        uint8_t *x = xs[buf], *g = gs[buf];
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const uint32_t *v = f.x[i];
            *(uint4 *)(x + (lds_row(pr) + i) * kXP + 16 * r8) =
                UNIT == 1 ? make_uint4(v[0] | v[1] << 16, v[2] | v[3] << 16, v[4] | v[5] << 16, v[6] | v[7] << 16)
                          : make_uint4(v[0], v[1], v[2], v[3]);
        }
        if (gp < kPix) {
            const uint2 lo = masked_grad4(f.y[0], f.dy[0]), hi = masked_grad4(f.y[1], f.dy[1]);
            *(uint4 *)(g + lds_row(gp) * kGP + 16 * (t % (2 * NF))) = make_uint4(lo.x, lo.y, hi.x, hi.y);
        }
        // the buffer's readers of two steps ago passed the last step's barrier
        __syncthreads();
        if (p0 + kStages * kPix < p_end) fetch(f, p0 + kStages * kPix);
#pragma unroll
        for (int kc = 0; kc < kPix; kc += 32) {
            bf16x8 fx[2], fg[NF];
#pragma unroll
            for (int m = 0; m < 2; m++) fx[m] = tr_fragment(x, kXP, kc, 32 * wave + 16 * m);
#pragma unroll
            for (int k = 0; k < NF; k++) fg[k] = tr_fragment(g, kGP, kc, 16 * k);
            // channels as the result's rows: a lane ends with four consecutive channels of one r
#pragma unroll
            for (int k = 0; k < NF; k++) {
#pragma unroll
                for (int m = 0; m < 2; m++)
                    acc[m][k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fg[k], fx[m], acc[m][k], 0, 0, 0);
                if (bias && k == wave) accb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fg[k], ones, accb, 0, 0, 0);
            }
        }
    };
    if (p_begin < p_end) fetch(st[0], p_begin);
    if (kStages > 1 && p_begin + kPix < p_end) fetch(st[kStages - 1], p_begin + kPix);
    for (int p0 = p_begin; p0 < p_end; p0 += 2 * kPix) {
        step(st[0], 0, p0);
        if (p0 + kPix < p_end) step(st[kStages - 1], 1, p0 + kPix);
    }
    float *part = a.w_sums + blockIdx.z * a.split_stride;
#pragma unroll
    for (int m = 0; m < 2; m++) {
        const int row = row0 + 32 * wave + 16 * m + (lane & 15);
        if (row < rows)
#pragma unroll
            for (int f = 0; f < NF; f++) {
                const int co = co0 + 16 * f + 4 * (lane >> 4);
                if (co < c.cout) store_f4(part + (size_t)row * c.cout + co, acc[m][f]);
            }
    }
    if (bias && (lane & 15) == 0) {
        const int co = co0 + 16 * wave + 4 * (lane >> 4);
        if (co < c.cout) store_f4(a.b_sums + blockIdx.z * a.split_stride + co, accb);
    }
}

// Narrow form, for cin <= 3 (at most 27 rows, and the bias as one more row of
// ones, so that the 288-row tile would be nine tenths empty): bound by reading
// the gradients, so each wavefront streams its own 32 pixels of a step through
// 6 KB of LDS, the next step's loads in flight, and four of them then multiply
// the step's slices in order, a quarter of the result each.  2 -> 32 channels,
// 524288 pixels: 20.3 us (109 MB at 5.4 TB/s) without the reduction's 5 us,
// against 335 with it on 64 x 64 tiles.
template <int CIN, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void k_conv_wgrad_narrow(WgradArgs a) {
    constexpr int kP = 96;                // bytes per pixel: 32 elements, an odd multiple of 32
    constexpr int kWaveBytes = 64 * kP;   // 32 pixels of x, 32 of the gradient
    __shared__ __align__(16) uint8_t lds[WAVES * kWaveBytes];
    const ConvShape &c = a.walk.c;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    uint8_t *xs = lds + wave * kWaveBytes, *gs = xs + 32 * kP;
    constexpr int rows = 9 * CIN;
    const int co0 = blockIdx.y * 32;
    const int p_begin = blockIdx.z * a.chunk, p_end = min(c.n * c.ho * c.wo, p_begin + a.chunk);
    // staging: lane's pixel lane % 32, taps 0-4 (lower half) or 5-8 and the row of ones; gradients 4 channels at a time
    const int px = lane & 31, half = lane >> 5;
    for (int i = lane; i < kWaveBytes / 16; i += 64) *(uint4 *)(xs + 16 * i) = make_uint4(0, 0, 0, 0);
    uint16_t xv[5][CIN];
    float4 gd[4];
    uint2 gy[4];
    PixelWalk w;
    w.start(c, p_begin + 32 * wave + px);
    auto fetch = [&](int p0) {
        const int p = p0 + px;
#pragma unroll
        for (int k = 0; k < 5; k++) {
            const int tap = 5 * half + k;
            const Tap at(c, tap / 3, tap % 3);
            const bool on = p < p_end && tap < 9 && at.inside(w);
            if constexpr (CIN == 2) {
                const uint32_t v = on ? *(const uint32_t *)(a.x + at.at(w)) : 0;
                xv[k][0] = v & 0xFFFF, xv[k][1] = v >> 16;
            } else {
#pragma unroll
                for (int e = 0; e < CIN; e++) xv[k][e] = on ? a.x[at.at(w) + e] : 0;
            }
        }
        w.step(a.walk);
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const int pg = p0 + (lane >> 3) + 8 * k, co = co0 + 4 * (lane & 7);
            gd[k] = make_float4(0.f, 0.f, 0.f, 0.f);
            gy[k] = make_uint2(0, 0);
            if (pg < p_end && co < c.cout) {
                const size_t o = (size_t)pg * c.cout + co;
                gd[k] = load_f4(a.dy + o);
                gy[k] = load_u2(a.y + o);
            }
        }
    };
    // the quarter of the result that this wavefront multiplies
    const int m = wave & 1, f = (wave >> 1) & 1;
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
    constexpr int kStep = 32 * WAVES;
    if (p_begin + 32 * wave < p_end) fetch(p_begin + 32 * wave);
    for (int p0 = p_begin; p0 < p_end; p0 += kStep) {
        if (p0 + 32 * wave < p_end) {
            uint16_t *row = (uint16_t *)(xs + lds_row(px) * kP);
#pragma unroll
            for (int k = 0; k < 5; k++) {
                const int tap = 5 * half + k;
                if (tap < 9) {
                    uint16_t *d = row + tap * CIN;
                    if constexpr (CIN == 2) *(uint32_t *)d = xv[k][0] | ((uint32_t)xv[k][1] << 16);
                    else
#pragma unroll
                        for (int e = 0; e < CIN; e++) d[e] = xv[k][e];
                } else {
                    row[rows] = 0x3F80;
                }
            }
#pragma unroll
            for (int k = 0; k < 4; k++)
                *(uint2 *)(gs + lds_row((lane >> 3) + 8 * k) * kP + 8 * (lane & 7)) = masked_grad4(gy[k], gd[k]);
        }
        __syncthreads();
        if (p0 + kStep + 32 * wave < p_end) fetch(p0 + kStep + 32 * wave);
        if (WAVES == 4 || wave < 4) {
            const int slices = min(WAVES, (p_end - p0 + 31) / 32);
            const uint8_t *x = lds;
#pragma unroll 4
            for (int k = 0; k < slices; k++, x += kWaveBytes)
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tr_fragment(x + 32 * kP, kP, 0, 16 * f),
                                                              tr_fragment(x, kP, 0, 16 * m), acc, 0, 0, 0);
        }
        __syncthreads();
    }
    const int r = 16 * m + (lane & 15), co = co0 + 16 * f + 4 * (lane >> 4);
    if (wave < 4 && r <= rows && co < c.cout)
        store_f4((r < rows ? a.w_sums + r * c.cout : a.b_sums) + blockIdx.z * a.split_stride + co, acc);
}

// The sum over the splits of output threadIdx.x of a block's 256 (count in all,
// a multiple of 4, rows of which are `first` onward).  At least 64 splits of few
// outputs are added as 64 sums, of every 64th split, and these in halves (sum l
// and sum l + 32, then 16, .. 1); the others one after the other.  Bound by the
// latency of the loads, of which sixteen are in flight (64, in 256 registers a
// thread: 6 us more a training step of 256 pairs, 2.5 for 128 -> 128 channels).
constexpr int kReduceThreads = 256;

// (at most 256 splits: split_limit)
__device__ __forceinline__ bool splits_in_halves(int64_t count, int splits) { return count <= 32768 && splits >= 64; }

__device__ __forceinline__ float sum_splits(const float *part, int64_t count, int splits, int64_t first,
                                            float4 (*red)[64]) {
    if (!splits_in_halves(count, splits)) {
        const float *p = part + min(first + (int64_t)threadIdx.x, count - 1);
        constexpr int kAhead = 16;
        float s = 0.f;
        for (int z0 = 0; z0 < splits; z0 += kAhead) {
            float v[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; u++) v[u] = p[min(z0 + u, splits - 1) * count];
#pragma unroll
            for (int u = 0; u < kAhead; u++) s += z0 + u < splits ? v[u] : 0.f;
        }
        return s;
    }
    // a thread makes 16 of the 64 sums (4 j + its wavefront) of four outputs, in the order in which the halves meet
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const float *p = part + min(first + 4 * lane, count - 4);
    auto add = [](float4 a, float4 b) { return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w); };
    auto quarter = [&](int j0) {  // sums j0, j0 + 4, j0 + 8, j0 + 12
        float4 v[4][4], s[4];
#pragma unroll
        for (int k = 0; k < 4; k++)
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const int z = wave + 4 * (j0 + 4 * k) + 64 * u;
                v[k][u] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (z < splits) v[k][u] = load_f4(p + z * count);
            }
#pragma unroll
        for (int k = 0; k < 4; k++) s[k] = add(add(add(v[k][0], v[k][1]), v[k][2]), v[k][3]);
        return add(add(s[0], s[2]), add(s[1], s[3]));
    };
    float4 half, sum;
#pragma unroll 1
    for (int h = 0; h < 2; h++) {
#pragma unroll 1
        for (int g = 0; g < 2; g++) {
            const float4 q = quarter(h + 2 * g);
            half = g ? add(half, q) : q;
        }
        sum = h ? add(sum, half) : half;
    }
    red[wave][lane] = sum;
    __syncthreads();
    const float *r = (const float *)red + threadIdx.x;
    return (r[0] + r[512]) + (r[256] + r[768]);
}

__global__ __launch_bounds__(kReduceThreads) void k_conv_wgrad_reduce(int M, int N, int splits,
                                                                      const float *__restrict__ part,
                                                                      float *__restrict__ dw, float *__restrict__ db) {
    __shared__ float4 red[4][64];
    const int64_t first = (int64_t)blockIdx.x * kReduceThreads, count = (int64_t)M * N, last = count - N;
    const float s = sum_splits(part, count, splits, first, red);
    const int64_t i = first + threadIdx.x;
    if (i < count) *(i < last ? dw + i : db + (i - last)) = s;
}

// The whole parameter update of a training step in one launch: the layers'
// gradients from their splits' sums, Adam (Kingma and Ba) with c1 = 1 / (1 -
// beta1^t) and c2 = 1 / (1 - beta2^t), and the bfloat16 copies of the
// convolutions' weights; a parameter a thread, its moments on their way during
// the sums.  Blocks of four wavefronts are all resident at once for the
// network's 360000 parameters: 15.4 us for the 60 MB of sums of 256 pairs, against
// 18.4 with sixteen wavefronts (2.75 rounds of blocks, the moments after the
// sums by one wavefront).
__global__ __launch_bounds__(kReduceThreads) void k_conv_update(UpdateArgs a) {
    __shared__ float4 red[4][64];
    int l = 0;
    while (l + 1 < a.count && (int)blockIdx.x >= a.part[l + 1].block0) l++;
    const UpdatePart &p = a.part[l];
    const int64_t j = (int64_t)(blockIdx.x - p.block0) * kReduceThreads + threadIdx.x;  // in the part
    const int64_t i = p.offset + min(j, p.n - 1);
    float g = p.sums ? 0.f : a.g[i];
    const float m = a.m[i], v = a.v[i], w0 = a.p[i];
    if (p.sums) {
        g = sum_splits(p.sums, p.n, p.splits, (int64_t)(blockIdx.x - p.block0) * kReduceThreads, red);
    }
    if (j >= p.n) return;
    if (p.sums) a.g[i] = g;
    // written out, so that the rounding does not depend on what the compiler contracts
    const float mi = fmaf(1.f - a.beta1, g, a.beta1 * m);
    const float vi = fmaf((1.f - a.beta2) * g, g, a.beta2 * v);
    a.m[i] = mi;
    a.v[i] = vi;
    const float w = w0 - a.lr * (mi * a.c1) / (sqrtf(vi * a.c2) + a.eps);
    a.p[i] = w;
    const int64_t weights = p.n - p.N;  // the last row is the bias
    if (!p.w_kn || j >= weights) return;
    const uint16_t h = f2bf(w);
    const int k = (int)(j / p.N), n = (int)(j - (int64_t)k * p.N), K = (int)(weights / p.N);
    p.w_kn[j] = h;
    p.w_nk[(size_t)n * K + k] = h;
}

int cdiv(int a, int b) { return (a + b - 1) / b; }

// Splits of the pixels: about 1024 of the 64 x 64 tiles that the workspace's
// size was laid out for, at least 64 pixels each.  split_limit: the most that
// a layer of these channels takes for any number of images up to c.n.
int split_limit(const ConvShape &c) {
    const int tiles = cdiv(9 * c.cin + 1, 64) * cdiv(c.cout, 64), P = std::max(c.n * c.ho * c.wo, 1);
    return std::min(std::max(1, std::min(256, cdiv(1024, tiles))), cdiv(P, 64));
}
// Output pixels of a split.
int split_chunk(const ConvShape &c) {
    return std::max(64, cdiv(cdiv(std::max(c.n * c.ho * c.wo, 1), split_limit(c)), 16) * 16);
}
int max_splits(const ConvShape &c) { return cdiv(std::max(c.n * c.ho * c.wo, 1), split_chunk(c)); }

template <int WAVES>
void launch_narrow(const WgradArgs &a, dim3 grid, hipStream_t s) {
    if (a.walk.c.cin == 1) hipLaunchKernelGGL((k_conv_wgrad_narrow<1, WAVES>), grid, dim3(64 * WAVES), 0, s, a);
    else if (a.walk.c.cin == 2) hipLaunchKernelGGL((k_conv_wgrad_narrow<2, WAVES>), grid, dim3(64 * WAVES), 0, s, a);
    else hipLaunchKernelGGL((k_conv_wgrad_narrow<3, WAVES>), grid, dim3(64 * WAVES), 0, s, a);
}

template <int NF>
void launch_wide(const WgradArgs &a, dim3 grid, hipStream_t s) {
    if (a.walk.c.cin % 8 == 0) hipLaunchKernelGGL((k_conv_wgrad<NF, 8>), grid, dim3(kWideThreads), 0, s, a);
    else if (a.walk.c.cin % 2 == 0) hipLaunchKernelGGL((k_conv_wgrad<NF, 2>), grid, dim3(kWideThreads), 0, s, a);
    else hipLaunchKernelGGL((k_conv_wgrad<NF, 1>), grid, dim3(kWideThreads), 0, s, a);
}

}  // namespace

int64_t conv_wgt_work_limit(const ConvShape &c) { return (int64_t)split_limit(c) * (9 * c.cin + 1) * c.cout; }
int64_t conv_wgt_work_floats(const ConvShape &c) { return (int64_t)max_splits(c) * (9 * c.cin + 1) * c.cout; }

// dw, db: where a single split's sums go, which are the gradients; null: into `work` like the others.
static ups_status wgrad_sums(const ConvShape &c, const uint16_t *x, const uint16_t *y, const float *dy, float *work,
                             float *dw, float *db, int *splits, hipStream_t s) {
    const int P = c.n * c.ho * c.wo, M = 9 * c.cin + 1;
    *splits = 0;
    if (P == 0) return UPS_OK;
    const bool narrow = c.cin <= 3;
    const int row_tiles = narrow ? 1 : cdiv(9 * c.cin, kRowTile);
    // 64 channels a block: half the staged windows of 32 for the same products (batch 256, 32 -> 64 and 64 -> 96
    // channels: 26.5 and 27.7 us against 36.0 and 36.9); 32 where there are no more
    const int nf = narrow || c.cout <= 32 ? 2 : 4;
    const int chunk = split_chunk(c);
    // narrow form: four wavefronts a block where a split is one step of theirs, or where several blocks share a split
    // and so a CU (us with 4 / 16, two channels: 16384 pixels to 32 and 128 channels 10.0/10.3 and 12.1/19.0, 131072
    // pixels 14.6/13.6 and 29.4/35.9)
    const int waves = chunk <= 128 || c.cout > 32 ? 4 : 16, unit = narrow ? 32 * waves : kPix;
    *splits = cdiv(P, chunk);
    const bool direct = *splits == 1 && dw;
    const WgradArgs a{walk_args(c, unit), x, y, dy, direct ? dw : work, direct ? db : work + (int64_t)(M - 1) * c.cout,
                      (int64_t)M * c.cout, chunk};
    const dim3 grid(row_tiles, cdiv(c.cout, 16 * nf), *splits);
    if (narrow && waves == 4) launch_narrow<4>(a, grid, s);
    else if (narrow) launch_narrow<16>(a, grid, s);
    else if (nf == 2) launch_wide<2>(a, grid, s);
    else launch_wide<4>(a, grid, s);
    UPS_CHECK_HIP(hipGetLastError());
    return UPS_OK;
}

ups_status launch_conv_wgrad_sums(const ConvShape &c, const uint16_t *x, const uint16_t *y, const float *dy, float *work,
                                  int *splits, hipStream_t s) {
    return wgrad_sums(c, x, y, dy, work, nullptr, nullptr, splits, s);
}

ups_status launch_conv_bwd_weight(const ConvShape &c, const uint16_t *x, const uint16_t *y, const float *dy,
                                  float *dw, float *db, float *work, int64_t work_floats, hipStream_t s) {
    const int M = 9 * c.cin + 1;
    UPS_REQUIRE(conv_wgt_work_floats(c) <= work_floats, "weight-gradient workspace too small");
    int splits = 0;
    const ups_status st = wgrad_sums(c, x, y, dy, work, dw, db, &splits, s);
    if (st != UPS_OK || splits == 1) return st;
    hipLaunchKernelGGL(k_conv_wgrad_reduce, dim3((unsigned)(((int64_t)M * c.cout + kReduceThreads - 1) / kReduceThreads)),
                       dim3(kReduceThreads), 0, s, M, c.cout, splits, work, dw, db);
    UPS_CHECK_HIP(hipGetLastError());
    return UPS_OK;
}

ups_status launch_conv_update(UpdateArgs &a, float lr, int64_t step, hipStream_t s) {
    const double b1 = 0.9, b2 = 0.999;
    a.lr = lr, a.beta1 = (float)b1, a.beta2 = (float)b2, a.eps = 1e-8f;
    a.c1 = (float)(1.0 / (1.0 - std::pow(b1, (double)step)));
    a.c2 = (float)(1.0 / (1.0 - std::pow(b2, (double)step)));
    int blocks = 0;
    for (int l = 0; l < a.count; l++) {
        a.part[l].block0 = blocks;
        blocks += (int)((a.part[l].n + 255) / 256);
    }
    hipLaunchKernelGGL(k_conv_update, dim3(blocks), dim3(kReduceThreads), 0, s, a);
    UPS_CHECK_HIP(hipGetLastError());
    return UPS_OK;
}

}  // namespace ups
