// Convolution, fully connected, loss and Adam kernels of the pose-proposal
// network (BF16 operands on the matrix cores, FP32 accumulation).
//
// The convolution passes here take the shapes that the streaming kernels of
// ups_cnn_conv.hip do not (contracted channels that are no multiple of 8,
// tensors past 2 GiB, a data gradient of stride 2 over more than 128 channels):
// implicit GEMMs on one tile engine, where a 256-thread block computes a 64 x
// 64 tile of C = A B, staging 64 x 32 slices of A and B through LDS as
// bfloat16 and issuing gfx950's v_mfma_f32_16x16x32_bf16 (each wavefront owns
// a 32 x 32 quarter: 2 x 2 MFMA tiles, 32 k per instruction).
// The K loop loads the next slice into registers while the matrix cores work
// on the current one.  Operand loaders gather A and B
// straight from the NHWC activations, so no im2col buffer exists:
//   forward          C[pixel_out][cout] = X_col[pixel_out][(tap,ci)] W[(tap,ci)][cout]
//   backward (data)  C[pixel_in][ci]    = G_col[pixel_in][(tap,co)]  W[(tap,ci)][co]^T
// with G = dL/dy masked by y > 0 (ReLU), taps (ky, kx) of a 3x3 window, the
// width circular and the height zero-padded.  The weight gradient contracts
// over pixels and has kernels of its own (ups_cnn_wgrad.hip).
#include <cstdint>

#include "ups_cnn.hpp"

namespace ups {

constexpr int kBM = 64, kBN = 64;

// One 64 x 64 tile: A rows m0.., B columns n0.., K range [k_begin, k_end).
// LA::load(row, k, out[4]) / LB::load(col, k, out[4]) return bf16 values of
// A(row, k..k+3) / B(k..k+3, col), zero outside the operand; ST::store(row,
// col, v) writes one result.
template <class LA, class LB, class ST>
__device__ __forceinline__ void mfma_tile(const LA &la, const LB &lb, const ST &st, int m0, int n0, int M, int N,
                                          int k_begin, int k_end) {
    constexpr int KB = 32;
    // LDS row pitch (elements), padded to spread the rows over the banks and
    // keeping each row 16-byte aligned for the 8-element fragment loads
    constexpr int kLP = KB + 8;
    constexpr int kQ = KB / 16;  // k quads per thread and operand in one slice
    __shared__ __align__(16) uint16_t As[kBM * kLP];
    __shared__ __align__(16) uint16_t Bs[kBN * kLP];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int lr = tid >> 2, lq = tid & 3;  // loader: row / column lr of the tile, k quads lq + 4 q
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    uint16_t a[kQ][4], b[kQ][4];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int q = 0; q < kQ; q++) {
            const int k = k0 + 4 * (lq + 4 * q);
            la.load(m0 + lr, k, k_end, a[q]);
            lb.load(n0 + lr, k, k_end, b[q]);
        }
    };
    if (k_begin < k_end) fetch(k_begin);
    for (int k0 = k_begin; k0 < k_end; k0 += KB) {
#pragma unroll
        for (int q = 0; q < kQ; q++) {
            const int o = lr * kLP + 4 * (lq + 4 * q);
            *(uint2 *)&As[o] = make_uint2(a[q][0] | ((uint32_t)a[q][1] << 16), a[q][2] | ((uint32_t)a[q][3] << 16));
            *(uint2 *)&Bs[o] = make_uint2(b[q][0] | ((uint32_t)b[q][1] << 16), b[q][2] | ((uint32_t)b[q][3] << 16));
        }
        __syncthreads();
        // the next slice's loads are in flight while this slice is multiplied
        if (k0 + KB < k_end) fetch(k0 + KB);
        // lane l carries row (A) or column (B) l % 16 and the slice's k =
        // 8 (l / 16) .. + 7: the same k in the same slot of both operands
        bf16x8 fa[2], fb[2];
#pragma unroll
        for (int i = 0; i < 2; i++)
            fa[i] = *(const bf16x8 *)&As[(32 * wm + 16 * i + (lane & 15)) * kLP + 8 * (lane >> 4)];
#pragma unroll
        for (int j = 0; j < 2; j++)
            fb[j] = *(const bf16x8 *)&Bs[(32 * wn + 16 * j + (lane & 15)) * kLP + 8 * (lane >> 4)];
#pragma unroll
        for (int i = 0; i < 2; i++)
#pragma unroll
            for (int j = 0; j < 2; j++)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
        __syncthreads();
    }
    // D[4 (lane/16) + e][lane % 16] of each 16 x 16 tile
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const int row = m0 + 32 * wm + 16 * i + 4 * (lane >> 4) + e;
                const int col = n0 + 32 * wn + 16 * j + (lane & 15);
                if (row < M && col < N) st.store(row, col, acc[i][j][e]);
            }
}

// ------------------------------------------------------------ forward

// A = the 3x3 windows of the input: row = output pixel (b, oy, ox), column
// k = tap * cin + ci with tap = 3 ky + kx.
struct LoadIm2col {
    ConvShape c;
    const uint16_t *x;
    float inv_cin;  // 1 / cin
    // k / cin without an integer division: (k + 1/2) / cin lies at least
    // 1 / (2 cin) away from an integer, and the FP32 product (below 9, as
    // k < 9 cin) is within 9 * 2^-22 of it, so the truncation is exact for
    // any cin below 2^17
    __device__ __forceinline__ int tap_of(int k) const { return (int)(((float)k + 0.5f) * inv_cin); }
    __device__ __forceinline__ uint16_t at(int b, int oy, int ox, int k) const {
        const int tap = tap_of(k), ci = k - tap * c.cin;
        const int ky = tap / 3, kx = tap - 3 * ky;
        const int iy = c.stride * oy + ky - 1;
        if (iy < 0 || iy >= c.h) return 0;
        int ix = c.stride * ox + kx - 1;
        ix = ix < 0 ? ix + c.w : (ix >= c.w ? ix - c.w : ix);
        return x[((size_t)(b * c.h + iy) * c.w + ix) * c.cin + ci];
    }
    __device__ __forceinline__ void load(int m, int k, int k_end, uint16_t *o) const {
        const int P = c.n * c.ho * c.wo;
        if (m >= P) {
            o[0] = o[1] = o[2] = o[3] = 0;
            return;
        }
        const int b = m / (c.ho * c.wo), r = m - b * c.ho * c.wo, oy = r / c.wo, ox = r - oy * c.wo;
        if ((c.cin & 3) == 0 && k + 3 < k_end) {
            // four channels of one tap: one 8-byte load
            const int tap = tap_of(k), ci = k - tap * c.cin;
            const int ky = tap / 3, kx = tap - 3 * ky;
            const int iy = c.stride * oy + ky - 1;
            if (iy < 0 || iy >= c.h) {
                o[0] = o[1] = o[2] = o[3] = 0;
                return;
            }
            int ix = c.stride * ox + kx - 1;
            ix = ix < 0 ? ix + c.w : (ix >= c.w ? ix - c.w : ix);
            const uint2 v = *(const uint2 *)&x[((size_t)(b * c.h + iy) * c.w + ix) * c.cin + ci];
            o[0] = v.x & 0xFFFF, o[1] = v.x >> 16, o[2] = v.y & 0xFFFF, o[3] = v.y >> 16;
            return;
        }
        if ((c.cin & 1) == 0 && k + 3 < k_end) {
            // even cin (k is a multiple of 4): two channel pairs, each of one tap
#pragma unroll
            for (int p = 0; p < 2; p++) {
                const int kk = k + 2 * p, tap = tap_of(kk), ci = kk - tap * c.cin;
                const int ky = tap / 3, kx = tap - 3 * ky;
                const int iy = c.stride * oy + ky - 1;
                uint32_t v = 0;
                if (iy >= 0 && iy < c.h) {
                    int ix = c.stride * ox + kx - 1;
                    ix = ix < 0 ? ix + c.w : (ix >= c.w ? ix - c.w : ix);
                    v = *(const uint32_t *)&x[((size_t)(b * c.h + iy) * c.w + ix) * c.cin + ci];
                }
                o[2 * p] = v & 0xFFFF, o[2 * p + 1] = v >> 16;
            }
            return;
        }
#pragma unroll
        for (int e = 0; e < 4; e++) o[e] = (k + e < k_end) ? at(b, oy, ox, k + e) : 0;
    }
};

// B^T rows: W^T[cout][K] (bf16, K contiguous).
struct LoadRowsBf16 {
    const uint16_t *w;
    int rows, K;
    __device__ __forceinline__ void load(int n, int k, int k_end, uint16_t *o) const {
        if (n >= rows) {
            o[0] = o[1] = o[2] = o[3] = 0;
            return;
        }
        const uint16_t *p = w + (size_t)n * K;
        if ((K & 3) == 0 && k + 3 < k_end) {
            // rows start on 8-byte boundaries: one 8-byte load
            const uint2 v = *(const uint2 *)&p[k];
            o[0] = v.x & 0xFFFF, o[1] = v.x >> 16, o[2] = v.y & 0xFFFF, o[3] = v.y >> 16;
            return;
        }
#pragma unroll
        for (int e = 0; e < 4; e++) o[e] = (k + e < k_end) ? p[k + e] : 0;
    }
};

struct StoreReluBf16 {
    const float *bias;
    uint16_t *y;
    int N;
    __device__ __forceinline__ void store(int m, int n, float v) const {
        y[(size_t)m * N + n] = f2bf(fmaxf(v + bias[n], 0.f));
    }
};

__global__ __launch_bounds__(256) void k_conv_fwd(ConvShape c, const uint16_t *__restrict__ x,
                                                  const uint16_t *__restrict__ w_nk, const float *__restrict__ bias,
                                                  uint16_t *__restrict__ y) {
    const int M = c.n * c.ho * c.wo, N = c.cout, K = 9 * c.cin;
    mfma_tile(LoadIm2col{c, x, 1.f / (float)c.cin}, LoadRowsBf16{w_nk, N, K}, StoreReluBf16{bias, y, N}, blockIdx.x * kBM,
              blockIdx.y * kBN, M, N, 0, K);
}

// ------------------------------------------------------ backward (data)

// A row = input pixel (b, iy, ix), column k = tap * cout + co: the output
// gradient at the output pixel whose tap (ky, kx) reads (iy, ix), if any.
struct LoadGradCol {
    ConvShape c;
    const float *dy;
    const uint16_t *y;
    float inv_cout;  // 1 / cout: k / cout as in LoadIm2col::tap_of
    __device__ __forceinline__ void load(int m, int k, int k_end, uint16_t *o) const {
        o[0] = o[1] = o[2] = o[3] = 0;
        if (m >= c.n * c.h * c.w || k >= k_end) return;
        const int b = m / (c.h * c.w), r = m - b * c.h * c.w, iy = r / c.w, ix = r - iy * c.w;
        // cout is a multiple of 4: the four columns share a tap
        const int tap = (int)(((float)k + 0.5f) * inv_cout), co = k - tap * c.cout;
        const int ky = tap / 3, kx = tap - 3 * ky;
        const int sh = c.stride >> 1;  // stride 1 or 2
        const int ty = iy + 1 - ky;
        if (ty < 0 || (ty & sh) != 0 || (ty >> sh) >= c.ho) return;
        int tx = ix + 1 - kx;
        tx = tx < 0 ? tx + c.w : (tx >= c.w ? tx - c.w : tx);
        if ((tx & sh) != 0 || (tx >> sh) >= c.wo) return;
        const size_t base = ((size_t)(b * c.ho + (ty >> sh)) * c.wo + (tx >> sh)) * c.cout + co;
        // four consecutive channels: one 8-byte load of y, one 16-byte load of dy
        const uint2 yv = *(const uint2 *)&y[base];
        const float4 g = *(const float4 *)&dy[base];
        const uint16_t yy[4] = {(uint16_t)(yv.x & 0xFFFF), (uint16_t)(yv.x >> 16), (uint16_t)(yv.y & 0xFFFF),
                                (uint16_t)(yv.y >> 16)};
        const float gg[4] = {g.x, g.y, g.z, g.w};
#pragma unroll
        for (int e = 0; e < 4; e++) o[e] = (yy[e] != 0 && !(yy[e] & 0x8000)) ? f2bf(gg[e]) : (uint16_t)0;
    }
};

// B^T row n = ci: W[(tap, ci)][co] over k = tap * cout + co (4 co contiguous).
struct LoadWkn {
    ConvShape c;
    const uint16_t *w_kn;
    float inv_cout;
    __device__ __forceinline__ void load(int n, int k, int k_end, uint16_t *o) const {
        o[0] = o[1] = o[2] = o[3] = 0;
        if (n >= c.cin || k >= k_end) return;
        const int tap = (int)(((float)k + 0.5f) * inv_cout), co = k - tap * c.cout;
        const uint2 v = *(const uint2 *)&w_kn[((size_t)tap * c.cin + n) * c.cout + co];
        o[0] = v.x & 0xFFFF, o[1] = v.x >> 16, o[2] = v.y & 0xFFFF, o[3] = v.y >> 16;
    }
};

struct StoreF32 {
    float *out;
    int N;
    __device__ __forceinline__ void store(int m, int n, float v) const { out[(size_t)m * N + n] = v; }
};

__global__ __launch_bounds__(256) void k_conv_bwd_data(ConvShape c, const uint16_t *__restrict__ y,
                                                       const float *__restrict__ dy,
                                                       const uint16_t *__restrict__ w_kn, float *__restrict__ dx) {
    const int M = c.n * c.h * c.w, N = c.cin, K = 9 * c.cout;
    const float inv_cout = 1.f / (float)c.cout;
    mfma_tile(LoadGradCol{c, dy, y, inv_cout}, LoadWkn{c, w_kn, inv_cout}, StoreF32{dx, N}, blockIdx.x * kBM,
              blockIdx.y * kBN, M, N, 0, K);
}

// ------------------------------------------------------------ host side

static int cdiv(int a, int b) { return (a + b - 1) / b; }

ConvShape conv_shape(int n, int h, int w, int cin, int cout, int stride) {
    ConvShape c;
    c.n = n, c.h = h, c.w = w, c.cin = cin, c.cout = cout, c.stride = stride;
    c.ho = (h - 1) / stride + 1;
    c.wo = (w - 1) / stride + 1;
    return c;
}

WalkArgs walk_args(const ConvShape &c, int unit) {
    const int b = unit / (c.ho * c.wo), oy = unit / c.wo % c.ho, ox = unit % c.wo;
    WalkArgs a{c, oy, ox, 0, 0, 0};
    a.step_add = ((uint32_t)(b * c.h + c.stride * oy) * c.w + c.stride * ox) * (uint32_t)c.cin;
    a.row_add = (uint32_t)(c.stride * (c.w - c.wo)) * (uint32_t)c.cin;
    a.image_add = (uint32_t)((c.h - c.stride * c.ho) * c.w) * (uint32_t)c.cin;
    return a;
}

ups_status conv_check(const ConvShape &c) {
    UPS_REQUIRE(c.n >= 0 && c.h >= 1 && c.w >= 2 && c.cin >= 1 && c.cin <= 65536 && c.cout >= 4 &&
                    c.cout <= 65536 && (c.cout & 3) == 0,
                "conv shape: need n >= 0, h >= 1, w >= 2, 1 <= cin <= 65536, cout a multiple of 4 in [4, 65536]");
    UPS_REQUIRE(c.stride == 1 || c.stride == 2, "conv stride must be 1 or 2");
    UPS_REQUIRE(c.w % c.stride == 0, "conv width must be a multiple of the stride");
    UPS_REQUIRE((int64_t)c.n * c.h * c.w * (c.cin > c.cout ? c.cin : c.cout) < ((int64_t)1 << 31),
                "conv tensors too large");
    return UPS_OK;
}

ups_status launch_conv_fwd(const ConvShape &c, const uint16_t *x, const uint16_t *w_nk, const float *b, uint16_t *y,
                           hipStream_t s) {
    const int M = c.n * c.ho * c.wo;
    if (M == 0) return UPS_OK;
    if (conv_gather_fits(c, false)) return launch_conv_gather_fwd(c, x, w_nk, b, y, s);
    if (conv_narrow_fits(c)) return launch_conv_narrow_fwd(c, x, w_nk, b, y, s);
    hipLaunchKernelGGL(k_conv_fwd, dim3(cdiv(M, kBM), cdiv(c.cout, kBN)), dim3(256), 0, s, c, x, w_nk, b, y);
    UPS_CHECK_HIP(hipGetLastError());
    return UPS_OK;
}

ups_status launch_conv_bwd_data(const ConvShape &c, const uint16_t *y, const float *dy, const uint16_t *w_kn,
                                float *dx, hipStream_t s) {
    const int M = c.n * c.h * c.w;
    if (M == 0) return UPS_OK;
    if (conv_gather_fits(c, true)) return launch_conv_gather_bwd_data(c, y, dy, w_kn, dx, s);
    hipLaunchKernelGGL(k_conv_bwd_data, dim3(cdiv(M, kBM), cdiv(c.cin, kBN)), dim3(256), 0, s, c, y, dy, w_kn, dx);
    UPS_CHECK_HIP(hipGetLastError());
    return UPS_OK;
}

// ------------------------------------------------- head, loss, optimiser

// Sum of one value of each of 256 threads, halves added onto each other (t +
// (t + 128), then 64, .. 1); the first thread has it.  `red`: LDS of this sum.
__device__ __forceinline__ float tree_sum_256(float v, int t, float (*red)[64]) {
    red[t >> 6][t & 63] = v;
    __syncthreads();
    float s = (red[0][t & 63] + red[2][t & 63]) + (red[1][t & 63] + red[3][t & 63]);
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) s += __shfl_down(s, w, 64);
    return s;
}

// y[b][o] = bfc[o] + sum_k f[b][k] Wfc[o][k]; one block per sample, fixed-order
// sums.  Bound by the round trips of the loads, so eight k's loads of a thread
// are in flight (256 samples of 4096 features: 8.2 us one after the other, 6.0 so).
__global__ __launch_bounds__(256) void k_fc_fwd(int feat, const uint16_t *__restrict__ f, const float *__restrict__ Wfc,
                                                const float *__restrict__ bfc, float *__restrict__ out) {
    __shared__ float red[kCnnOut][4][64];
    const int b = blockIdx.x, t = threadIdx.x;
    float s[kCnnOut] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    constexpr int kAhead = 8;
    for (int k0 = t; k0 < feat; k0 += 256 * kAhead) {
        // loads without a condition (past the end, of the last feature), so that none waits for another
        uint16_t v[kAhead];
        float w[kAhead][kCnnOut];
#pragma unroll
        for (int i = 0; i < kAhead; i++) {
            const int k = min(k0 + 256 * i, feat - 1);
            v[i] = f[(size_t)b * feat + k];
#pragma unroll
            for (int o = 0; o < kCnnOut; o++) w[i][o] = Wfc[(size_t)o * feat + k];
        }
#pragma unroll
        for (int i = 0; i < kAhead; i++)
            if (k0 + 256 * i < feat)
#pragma unroll
                for (int o = 0; o < kCnnOut; o++) s[o] = fmaf(bf2f(v[i]), w[i][o], s[o]);
    }
#pragma unroll
    for (int o = 0; o < kCnnOut; o++) {
        const float q = tree_sum_256(s[o], t, red[o]);
        if (t == 0) out[b * kCnnOut + o] = q + bfc[o];
    }
}

// The loss sum (y - target)^2 / (2 n) and the head's gradients in one launch,
// with d[b][o] = (y - target) / n:
//   df[b][k] = sum_o d[b][o] Wfc[o][k],  dWfc[o][k] = sum_b d[b][o] f[b][k],  dbfc[o] = sum_b d[b][o].
// A block owns 64 features and brings their activations of 256 samples and
// the samples' d into LDS, all loads in flight.  Six wavefronts then each add
// one output's dWfc over the samples in order, the others write df.  (A thread
// that waited for each sample's load took 75 us for 256 samples of 4096
// features, the loss 4.2 and df 5.2 as launches of their own; 8.5 us for all
// three so.)  In block 0 the seventh wavefront adds dbfc, and four add the loss.
constexpr int kHeadWaves = 16, kHeadChunk = 256;

__global__ __launch_bounds__(64 * kHeadWaves) void k_head_bwd(int n, int feat, const uint16_t *__restrict__ f,
                                                              const float *__restrict__ y,
                                                              const float *__restrict__ target,
                                                              const float *__restrict__ Wfc, float *__restrict__ dWfc,
                                                              float *__restrict__ dbfc, float *__restrict__ df,
                                                              float *__restrict__ loss) {
    __shared__ __align__(16) float d[kCnnOut][kHeadChunk];
    __shared__ uint16_t fs[kHeadChunk][64];
    __shared__ float red[4][64];
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int k = blockIdx.x * 64 + lane;
    const bool on = k < feat;
    const float inv = 1.f / (float)n;
    float w[kCnnOut], s = 0.f, sb = 0.f;
#pragma unroll
    for (int o = 0; o < kCnnOut; o++) w[o] = Wfc[(size_t)o * feat + min(k, feat - 1)];
    for (int b0 = 0; b0 < n; b0 += kHeadChunk) {
        const int m = min(kHeadChunk, n - b0);
        __syncthreads();
        constexpr int kRows = kHeadChunk / kHeadWaves;
        uint16_t v[kRows];
#pragma unroll
        for (int i = 0; i < kRows; i++)
            v[i] = f[(size_t)(b0 + min(wave + kHeadWaves * i, m - 1)) * feat + min(k, feat - 1)];
        for (int i = t; i < m * kCnnOut; i += 64 * kHeadWaves)
            d[i % kCnnOut][i / kCnnOut] = (y[b0 * kCnnOut + i] - target[b0 * kCnnOut + i]) * inv;
#pragma unroll
        for (int i = 0; i < kRows; i++) fs[wave + kHeadWaves * i][lane] = v[i];
        __syncthreads();
        if (wave < kCnnOut) {
            const float *dw = d[wave];
            int i = 0;
            for (; i + 16 <= m; i += 16)
#pragma unroll
                for (int j = 0; j < 16; j++) s = fmaf(dw[i + j], bf2f(fs[i + j][lane]), s);
            for (; i < m; i++) s = fmaf(dw[i], bf2f(fs[i][lane]), s);
        } else {
            if (wave == kCnnOut && blockIdx.x == 0 && lane < kCnnOut)
#pragma unroll 16
                for (int i = 0; i < m; i++) sb += d[lane][i];
#pragma unroll 2
            for (int i = wave - kCnnOut; i < m; i += kHeadWaves - kCnnOut) {
                float g = 0.f;
#pragma unroll
                for (int o = 0; o < kCnnOut; o++) g = fmaf(d[o][i], w[o], g);
                if (on) df[(size_t)(b0 + i) * feat + k] = g;
            }
        }
    }
    if (wave < kCnnOut && on) dWfc[(size_t)wave * feat + k] = s;
    if (blockIdx.x != 0) return;
    if (wave == kCnnOut && lane < kCnnOut) dbfc[lane] = sb;
    float l = 0.f;
    if (t < 256)
#pragma unroll 4
        for (int i = t; i < n * kCnnOut; i += 256) {
            const float e = y[i] - target[i];
            l = fmaf(e, e, l);
        }
    __syncthreads();
    if (t < 256) red[t >> 6][lane] = l;
    __syncthreads();
    if (wave != 0) return;
    l = (red[0][lane] + red[2][lane]) + (red[1][lane] + red[3][lane]);
#pragma unroll
    for (int h = 32; h > 0; h >>= 1) l += __shfl_down(l, h, 64);
    if (t == 0 && loss) *loss = l * 0.5f * inv;
}

// bf16 copies of a conv weight W[K][N] (FP32): w_kn = W, w_nk = W^T
__global__ __launch_bounds__(256) void k_pack_weight(int K, int N, const float *__restrict__ W,
                                                     uint16_t *__restrict__ w_kn, uint16_t *__restrict__ w_nk) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= K * N) return;
    const int k = i / N, nn = i - k * N;
    const uint16_t h = f2bf(W[i]);
    w_kn[i] = h;
    w_nk[(size_t)nn * K + k] = h;
}

ups_status launch_fc_fwd(int n, int feat, const uint16_t *f, const float *Wfc, const float *bfc, float *out,
                         hipStream_t s) {
    if (n == 0) return UPS_OK;
    hipLaunchKernelGGL(k_fc_fwd, dim3(n), dim3(256), 0, s, feat, f, Wfc, bfc, out);
    UPS_CHECK_HIP(hipGetLastError());
    return UPS_OK;
}

ups_status launch_head_bwd(int n, int feat, const uint16_t *f, const float *y, const float *target, const float *Wfc,
                           float *dWfc, float *dbfc, float *df, float *loss, hipStream_t s) {
    hipLaunchKernelGGL(k_head_bwd, dim3(cdiv(feat, 64)), dim3(64 * kHeadWaves), 0, s, n, feat, f, y, target, Wfc, dWfc,
                       dbfc, df, loss);
    UPS_CHECK_HIP(hipGetLastError());
    return UPS_OK;
}

ups_status launch_pack_weight(int K, int N, const float *W, uint16_t *w_kn, uint16_t *w_nk, hipStream_t s) {
    hipLaunchKernelGGL(k_pack_weight, dim3(cdiv(K * N, 256)), dim3(256), 0, s, K, N, W, w_kn, w_nk);
    UPS_CHECK_HIP(hipGetLastError());
    return UPS_OK;
}

}  // namespace ups
