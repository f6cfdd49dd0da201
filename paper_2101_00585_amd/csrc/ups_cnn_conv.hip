// Forward pass and data gradient of the 3x3 convolutions, where the
// contraction runs over (tap, channel) and both operands lie in memory with
// their channels contiguous.  A block stages the weights of its output
// channels once in LDS in fragment order; every wavefront then streams its own
// pixels' channels, several loads ahead, through a small LDS buffer of its own
// into matrix-core fragments, without block barriers.  The detour through LDS
// is for the load's shape: with a fragment's own layout (consecutive lanes on
// consecutive pixels) each lane is a cache access of its own, and these
// accesses bounded the kernel (9.3 M for 32 -> 64 channels at batch 256: 15 of
// its 20 us); four lanes on the 64 bytes of one pixel are one access.
//
// Taps and channels are added in the order of the flattened contraction
// index, 32 channels to an instruction.
//
// Batch 256, each layer's pass on 64 x 64 tiles (ups_cnn.hip) -> here, us:
//   channels, stride   2->32,2    32->64,2   64->96,2   96->128,2   128->128,1
//   forward            30.5->11.2 28.1->14.9 24.8->11.4 23.0->8.9   28.2->10.4
//   data gradient                 155->29.8  79.9->17.7 52.0->11.5  42.2->14.5
// The first layers move 42 and 50 MB forward (8 and 10 us of a device copy);
// the last are bound by a wavefront's chain of round trips.
#include "ups_cnn.hpp"

namespace ups {

namespace {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct GatherArgs {
    ConvShape c;
    int hs, ws, ck;          // source grid and channels (contracted)
    int chunks;              // 32-channel chunks of a tap
    int N;                   // output channels
    int wn, wt;              // weight strides of an output channel and of a tap
    const uint16_t *src;     // forward: x; data gradient: y (with dy)
    const float *dy;
    const uint16_t *w;
    const float *bias;
    void *out;
};

// Loads through a buffer descriptor: an offset at or past its size reads 0,
// which serves the pixels and channels that do not exist.  `kNone`: an element
// offset whose byte offset is past every tensor that conv_gather_fits admits.
constexpr uint32_t kMaxBytes = 0x80000000u;
template <bool GRAD>
constexpr uint32_t kNone = kMaxBytes / (GRAD ? 4 : 2);
__device__ __forceinline__ u32x4 load_b128(Rsrc r, uint32_t offset, uint32_t uniform = 0) {
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, offset, uniform, 0));
}

// Between LDS accesses by which a wavefront's lanes hand values to each other,
// and before a buffer so read is written again: the hardware takes a
// wavefront's accesses in order, the compiler knows only each lane's own.
__device__ __forceinline__ void lds_handover() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local"); }

// The weights of output channels n0 .. n0 + 16 NF - 1 for chunks c0 .. c0 +
// count - 1 of the flattened (tap, chunk) list, as fragments of 1 KB: a
// wavefront fetches every WAVES-th fragment, kBatch of them before it stores the
// first; four lanes read 64 bytes of one channel's row.
template <int NF, int WAVES>
__device__ __forceinline__ void stage_weights(const GatherArgs &a, u32x4 *wf, int n0, int c0, int count, int wave,
                                              int lane) {
    static_assert(WAVES % NF == 0, "a wavefront's fragments are of one channel group");
    constexpr int kBatch = 6;
    const Rsrc w = rsrc_of(a.w, (uint32_t)(18 * a.N) * (uint32_t)a.ck);
    const int row = lane >> 2, k8 = lane & 3, n = n0 + 16 * (wave % NF) + row;
    int tap = 0, chunk = c0 + wave / NF;
    while (chunk >= a.chunks) chunk -= a.chunks, tap++;
    for (int j0 = wave; j0 < count * NF; j0 += WAVES * kBatch) {
        u32x4 v[kBatch];
#pragma unroll
        for (int i = 0; i < kBatch; i++) {
            const int ch = 32 * chunk + 8 * k8;
            const bool on = n < a.N && ch < a.ck && j0 + WAVES * i < count * NF;
            v[i] = load_b128(w, on ? 2 * (uint32_t)(n * a.wn + tap * a.wt + ch) : kMaxBytes);
            chunk += WAVES / NF;
            while (chunk >= a.chunks) chunk -= a.chunks, tap++;
        }
#pragma unroll
        for (int i = 0; i < kBatch; i++)
            if (j0 + WAVES * i < count * NF) wf[(j0 + WAVES * i) * 64 + 16 * k8 + row] = v[i];
    }
}

// A source chunk of 16 pixels on its way: lane l holds 8 channels of pixel
// l / 4, the four lanes of a pixel in an order turned with the pixel, so that
// the fragment reads below fall on different banks.
template <bool GRAD>
struct Chunk {
    u32x4 v, lo, hi;
    __device__ __forceinline__ void load(Rsrc src, Rsrc dy, uint32_t at, int chunk) {
        v = load_b128(src, 2 * at, 64 * chunk);
        if constexpr (GRAD) lo = load_b128(dy, 4 * at, 128 * chunk), hi = load_b128(dy, 4 * at + 16, 128 * chunk);
    }
    __device__ __forceinline__ void store(u32x4 *buf, int lane) const {
        if constexpr (GRAD) {
            const uint2 l = masked_grad4(make_uint2(v[0], v[1]), __builtin_bit_cast(float4, lo));
            const uint2 h = masked_grad4(make_uint2(v[2], v[3]), __builtin_bit_cast(float4, hi));
            buf[lane] = u32x4{l.x, l.y, h.x, h.y};
        } else buf[lane] = v;
    }
};
__device__ __forceinline__ int chunk_channel(int lane) { return 8 * ((lane & 3) ^ ((lane >> 4) & 3)); }
__device__ __forceinline__ bf16x8 chunk_fragment(const u32x4 *buf, int lane) {
    const int px = lane & 15, k8 = lane >> 4;
    return __builtin_bit_cast(bf16x8, buf[4 * px + (k8 ^ ((px >> 2) & 3))]);
}

// At most so many weight fragments of 1 KB in LDS, beside 2 MT KB a wavefront
// of source chunks: two blocks of four wavefronts a CU, or one of eight.
constexpr int kFragments = 72;

// relu(sums + bias) of pixels m0 .. m0+15 and channels n0 .. n0 + 16 NF - 1 in
// bfloat16, laid out in `tile` (512 NF bytes of LDS of this wavefront) and
// stored from there 16 bytes a lane, the lanes along a pixel's channels.  sums:
// lane l holds channels 16 f + 4 (l / 16) .. of pixel l % 16.  N is a multiple
// of 4.
template <int NF>
__device__ __forceinline__ void store_relu(const f32x4 *sums, const float *bias, uint16_t *out, int m0, int M, int n0,
                                           int N, uint16_t *tile, int lane) {
    constexpr int kPitch = 16 * NF, kUnits = 2 * NF;  // elements of a pixel, 8-channel units
    // pixels whose units share banks keep them in different order (32 -> 64 channels at batch 256: 13.8 us, 15.3 without)
    auto at = [](int px, int unit) { return px * kPitch + 8 * (unit ^ (px / (8 / NF) & (kUnits - 1))); };
    lds_handover();
#pragma unroll
    for (int f = 0; f < NF; f++) {
        const int k = 16 * f + 4 * (lane >> 4);
        const float4 b = load_f4(bias + min(n0 + k, N - 4));
        *(uint2 *)(tile + at(lane & 15, k >> 3) + (k & 4)) =
            bf16x4_of(make_float4(fmaxf(sums[f][0] + b.x, 0.f), fmaxf(sums[f][1] + b.y, 0.f),
                                  fmaxf(sums[f][2] + b.z, 0.f), fmaxf(sums[f][3] + b.w, 0.f)));
    }
    lds_handover();
#pragma unroll
    for (int i = 0; i < kUnits / 4; i++) {
        const int u = 64 * i + lane, m = m0 + u / kUnits, n = n0 + 8 * (u % kUnits);
        const uint4 v = *(const uint4 *)(tile + at(u / kUnits, u % kUnits));
        if (m >= M || n >= N) continue;
        uint16_t *o = out + (size_t)m * N + n;
        if (n + 8 <= N) *(PackedU4 *)o = PackedU4{v.x, v.y, v.z, v.w};
        else *(PackedU2 *)o = PackedU2{v.x, v.y};
    }
}

// Forward pass (any stride), or with GRAD the data gradient of stride 1 (the
// same sum over the output gradient, the offsets mirrored).  A block computes
// WAVES * 16 MT pixels x 16 NF output channels.
template <bool GRAD, int NF, int MT, int WAVES, int DEPTH>
__global__ __launch_bounds__(64 * WAVES, 4) void k_conv_gather(GatherArgs a) {
    extern __shared__ u32x4 lds[];
    static_assert(DEPTH % 2 == 0, "the source buffers alternate");
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    u32x4 *buf = lds + wave * 2 * MT * 64, *wf = lds + WAVES * 2 * MT * 64;
    const int n0 = blockIdx.y * NF * 16, total = 9 * a.chunks;
    const uint32_t src_n = (uint32_t)(a.c.n * a.hs * a.ws) * (uint32_t)a.ck;
    const Rsrc src = rsrc_of(a.src, 2 * src_n), dy = rsrc_of(GRAD ? (const void *)a.dy : a.src, GRAD ? 4 * src_n : 0);
    const int ph = GRAD ? a.c.h : a.c.ho, pw = GRAD ? a.c.w : a.c.wo, ss = GRAD ? 1 : a.c.stride;
    const int m0 = (blockIdx.x * WAVES + wave) * MT * 16, M = a.c.n * ph * pw, kq = chunk_channel(lane);
    // this lane's pixel of each chunk: offset of the centre tap, what the side columns add, which rows exist
    uint32_t centre[MT], left[MT], right[MT], rows[MT], at[MT];
#pragma unroll
    for (int t = 0; t < MT; t++) {
        const int m = m0 + 16 * t + (lane >> 2), b = m / (ph * pw), q = m - b * ph * pw, my = q / pw;
        const int sy = ss * my, sx = ss * (q - my * pw);
        centre[t] = (uint32_t)((b * a.hs + sy) * a.ws + sx) * (uint32_t)a.ck + kq;
        left[t] = (sx == 0 ? a.ws - 1 : -1) * a.ck, right[t] = (sx + 1 == a.ws ? 1 - a.ws : 1) * a.ck;
        rows[t] = m < M ? 2u | (sy > 0 ? 1u : 0u) | (sy + 1 < a.hs ? 4u : 0u) : 0u;
    }
    int ty = -1, tx = -1, chunk = 0;
    auto enter_tap = [&]() {
        const int oy = GRAD ? -ty : ty, ox = GRAD ? -tx : tx;
#pragma unroll
        for (int t = 0; t < MT; t++) {
            const uint32_t o = centre[t] + oy * a.ws * a.ck + (ox < 0 ? left[t] : ox > 0 ? right[t] : 0u);
            at[t] = (rows[t] >> (oy + 1)) & 1 ? o : kNone<GRAD>;
        }
    };
    Chunk<GRAD> raw[DEPTH][MT];
    auto issue = [&](int d) {
        // channels past the last (a count that is no multiple of 32) do not exist
        const bool partial = 32 * chunk + 32 > a.ck;
#pragma unroll
        for (int t = 0; t < MT; t++)
            raw[d][t].load(src, dy, partial && 32 * chunk + kq >= a.ck ? kNone<GRAD> : at[t], chunk);
        // the loads past the last chunk repeat the last tap and are not used
        if (++chunk == a.chunks) {
            chunk = 0;
            if (tx < 1) tx++, enter_tap();
            else if (ty < 1) tx = -1, ty++, enter_tap();
        }
    };
    enter_tap();
#pragma unroll
    for (int d = 0; d < DEPTH; d++) issue(d);
    f32x4 acc[MT][NF];
#pragma unroll
    for (int t = 0; t < MT; t++)
#pragma unroll
        for (int f = 0; f < NF; f++) acc[t][f] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto put = [&](int d) {
#pragma unroll
        for (int t = 0; t < MT; t++) raw[d][t].store(buf + ((d & 1) * MT + t) * 64, lane);
    };
    // multiply the chunk in buffer d & 1 by weight chunk q while the next one is put into the other
    auto use = [&](int d, int q) {
        bf16x8 fw[NF], fs[MT];
#pragma unroll
        for (int f = 0; f < NF; f++) fw[f] = __builtin_bit_cast(bf16x8, wf[(q * NF + f) * 64 + lane]);
        lds_handover();
#pragma unroll
        for (int t = 0; t < MT; t++) fs[t] = chunk_fragment(buf + ((d & 1) * MT + t) * 64, lane);
        put((d + 1) % DEPTH);
        issue((d + 1) % DEPTH);
        // gradient: pixels as the result's rows, a lane's neighbours hold the next channels (64 bytes of FP32);
        // forward: channels as the rows, a lane holds four channels of a pixel for the store through LDS
#pragma unroll
        for (int f = 0; f < NF; f++)
#pragma unroll
            for (int t = 0; t < MT; t++)
                acc[t][f] = GRAD ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(fs[t], fw[f], acc[t][f], 0, 0, 0)
                                 : __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[f], fs[t], acc[t][f], 0, 0, 0);
    };
    constexpr int kHeld = kFragments / NF, kSegment = kHeld / DEPTH * DEPTH;  // chunks whose weights LDS holds
    for (int c0 = 0; c0 < total; c0 += kSegment) {
        const int seg = total - c0 <= kHeld ? total - c0 : kSegment;
        if (c0) __syncthreads();
        stage_weights<NF, WAVES>(a, wf, n0, c0, seg, wave, lane);
        __syncthreads();
        if (c0 == 0) {
            put(0);
            issue(0);
        }
        int q = 0;
        for (; q + DEPTH <= seg; q += DEPTH)
#pragma unroll
            for (int d = 0; d < DEPTH; d++) use(d, q + d);
        // the last segment's remainder
#pragma unroll
        for (int d = 0; d < DEPTH - 1; d++)
            if (q + d < seg) use(d, q + d);
        if (seg != kSegment) break;
    }
    if constexpr (!GRAD) {
#pragma unroll
        for (int t = 0; t < MT; t++)
            store_relu<NF>(acc[t], a.bias, (uint16_t *)a.out, m0 + 16 * t, M, n0, a.N, (uint16_t *)(buf + t * 64 * NF / 2), lane);
        return;
    }
#pragma unroll
    for (int f = 0; f < NF; f++) {
        const int n = n0 + 16 * f + (lane & 15);
        if (n >= a.N) continue;
#pragma unroll
        for (int t = 0; t < MT; t++)
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const int m = m0 + 16 * t + 4 * (lane >> 4) + e;
                if (m < M) ((float *)a.out)[(size_t)m * a.N + n] = acc[t][f][e];
            }
    }
}

// Data gradient of stride 2: an input pixel is reached by 1, 2 or 4 of the
// taps, by the parity of its row and column.  A wavefront computes all four
// parity classes of 16 MT positions (2 my + py, 2 mx + px) from the four
// output pixels (my + 0/1, mx + 0/1): nine products a position instead of 36,
// and each gradient loaded four times instead of nine.  The output pixels are
// taken in the order that adds each class's taps in ascending order.
template <int CHUNKS, int NF, int MT, int WAVES, int DEPTH>
__global__ __launch_bounds__(64 * WAVES) void k_conv_bwd_data_s2(GatherArgs a) {
    extern __shared__ u32x4 lds[];
    static_assert(9 * CHUNKS * NF <= kFragments, "all weights of the block in LDS");
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    u32x4 *buf = lds + wave * 2 * MT * 64, *wf = lds + WAVES * 2 * MT * 64;
    const int n0 = blockIdx.y * NF * 16;
    const uint32_t src_n = (uint32_t)(a.c.n * a.hs * a.ws) * (uint32_t)a.ck;
    const Rsrc src = rsrc_of(a.src, 2 * src_n), dy = rsrc_of(a.dy, 4 * src_n);
    const int m0 = (blockIdx.x * WAVES + wave) * MT * 16, M = a.c.n * a.hs * a.ws, kq = chunk_channel(lane);
    constexpr uint32_t kNoPixel = 0x7FFFFFFFu, kOddRow = 0x80000000u;
    uint32_t centre[MT], right[MT], below[MT], pixel[MT];  // pixel: of class (0, 0), and whether the odd row exists
#pragma unroll
    for (int t = 0; t < MT; t++) {
        const int m = m0 + 16 * t + (lane >> 2), b = m / (a.hs * a.ws), q = m - b * a.hs * a.ws, my = q / a.ws;
        const int mx = q - my * a.ws;
        centre[t] = m < M ? (uint32_t)m * (uint32_t)a.ck + kq : kNone<true>;
        right[t] = m < M ? (mx + 1 == a.ws ? 1 - a.ws : 1) * a.ck : 0;
        below[t] = m < M && my + 1 < a.hs ? centre[t] + a.ws * a.ck : kNone<true>;
        pixel[t] = m < M ? (uint32_t)((b * a.c.h + 2 * my) * a.c.w + 2 * mx) | (2 * my + 1 < a.c.h ? kOddRow : 0u)
                         : kNoPixel;
    }
    Chunk<true> raw[DEPTH][MT];
    // step s: chunk s % CHUNKS of the output pixel (my + oy, mx + ox), (oy, ox) = (1,1), (1,0), (0,1), (0,0)
    auto issue = [&](int s) {
        if (s >= 4 * CHUNKS) return;
        const int shift = s / CHUNKS, chunk = s % CHUNKS, oy = shift < 2, ox = shift % 2 == 0;
        const bool on = 32 * chunk + kq < a.ck;
#pragma unroll
        for (int t = 0; t < MT; t++) {
            const uint32_t row = oy ? below[t] : centre[t], at = row == kNone<true> ? row : row + (ox ? right[t] : 0u);
            raw[s % DEPTH][t].load(src, dy, on ? at : kNone<true>, chunk);
        }
    };
#pragma unroll
    for (int s = 0; s < DEPTH; s++) issue(s);
    stage_weights<NF, WAVES>(a, wf, n0, 0, 9 * CHUNKS, wave, lane);
    f32x4 acc[4][MT][NF];
#pragma unroll
    for (int k = 0; k < 4; k++)
#pragma unroll
        for (int t = 0; t < MT; t++)
#pragma unroll
            for (int f = 0; f < NF; f++) acc[k][t][f] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto put = [&](int s) {
#pragma unroll
        for (int t = 0; t < MT; t++) raw[s % DEPTH][t].store(buf + ((s & 1) * MT + t) * 64, lane);
        issue(s + DEPTH);
    };
    __syncthreads();
    put(0);
#pragma unroll
    for (int s = 0; s < 4 * CHUNKS; s++) {
        const int shift = s / CHUNKS, chunk = s % CHUNKS, oy = shift < 2, ox = shift % 2 == 0;
        bf16x8 fs[MT];
        lds_handover();
#pragma unroll
        for (int t = 0; t < MT; t++) fs[t] = chunk_fragment(buf + ((s & 1) * MT + t) * 64, lane);
        if (s + 1 < 4 * CHUNKS) put(s + 1);
#pragma unroll
        for (int py = oy; py < 2; py++)
#pragma unroll
            for (int px = ox; px < 2; px++) {
                const int ky = py ? (oy ? 0 : 2) : 1, kx = px ? (ox ? 0 : 2) : 1;
#pragma unroll
                for (int f = 0; f < NF; f++) {
                    const bf16x8 fw = __builtin_bit_cast(bf16x8, wf[(((3 * ky + kx) * CHUNKS + chunk) * NF + f) * 64 + lane]);
#pragma unroll
                    for (int t = 0; t < MT; t++)
                        acc[2 * py + px][t][f] =
                            __builtin_amdgcn_mfma_f32_16x16x32_bf16(fs[t], fw, acc[2 * py + px][t][f], 0, 0, 0);
                }
            }
    }
#pragma unroll
    for (int t = 0; t < MT; t++)
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const uint32_t u = (uint32_t)__shfl((int)pixel[t], 4 * (4 * (lane >> 4) + e), 64), p = u & ~kOddRow;
            if (u == kNoPixel) continue;
#pragma unroll
            for (int k = 0; k < 4; k++) {
                if (k >= 2 && !(u & kOddRow)) continue;
                float *o = (float *)a.out + (size_t)(p + (k & 1) + (k >= 2 ? a.c.w : 0)) * a.N;
#pragma unroll
                for (int f = 0; f < NF; f++) {
                    const int n = n0 + 16 * f + (lane & 15);
                    if (n < a.N) o[n] = acc[k][t][f][e];
                }
            }
        }
}

// Forward pass of at most three input channels (at most 27 products an
// output, two instructions of 16): bound by writing the outputs, so each
// wavefront keeps the weights of 32 output channels in registers and walks
// over groups of 16 pixels, the next group's windows in flight.
template <int CIN>
__global__ __launch_bounds__(256) void k_conv_fwd_narrow(WalkArgs a, const uint16_t *__restrict__ x,
                                                         const uint16_t *__restrict__ w_nk,
                                                         const float *__restrict__ bias, uint16_t *__restrict__ y) {
    constexpr int K = 9 * CIN, KC = (K + 15) / 16;
    constexpr int UNIT = CIN == 2 ? 2 : 1, LOADS = 4 / UNIT;  // elements a load, loads a lane and instruction
    const ConvShape &c = a.c;
    const int lane = threadIdx.x & 63, wave = blockIdx.x * 4 + (threadIdx.x >> 6), waves = gridDim.x * 4;
    const int n0 = blockIdx.y * 32, P = c.n * c.ho * c.wo, k0 = 4 * (lane >> 4);
    bf16x4 fw[KC][2];
#pragma unroll
    for (int kc = 0; kc < KC; kc++)
#pragma unroll
        for (int f = 0; f < 2; f++)
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const int n = n0 + 16 * f + (lane & 15), k = 16 * kc + k0 + e;
                fw[kc][f][e] = (n < c.cout && k < K) ? (short)w_nk[n * K + k] : (short)0;
            }
    const Rsrc src = rsrc_of(x, 2 * (uint32_t)(c.n * c.h * c.w) * CIN);
    int p = 16 * wave + (lane & 15);
    PixelWalk w;
    w.start(c, p);
    uint32_t v[KC][LOADS];
    auto fetch = [&]() {
#pragma unroll
        for (int kc = 0; kc < KC; kc++)
#pragma unroll
            for (int i = 0; i < LOADS; i++) {
                const int k = 16 * kc + k0 + UNIT * i, tap = k / CIN;
                const Tap at(c, tap / 3, tap % 3);
                const uint32_t o = p < P && k < K && at.inside(w) ? 2 * (at.at(w) + k - tap * CIN) : kMaxBytes;
                v[kc][i] = UNIT == 2 ? (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(src, o, 0, 0)
                                     : (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(src, o, 0, 0);
            }
    };
    __shared__ __align__(16) uint16_t tiles[4][16 * 32];
    if (16 * wave < P) fetch();
    for (int g = 16 * wave; g < P; g += 16 * waves) {
        bf16x4 fx[KC];
#pragma unroll
        for (int kc = 0; kc < KC; kc++)
#pragma unroll
            for (int e = 0; e < 4; e++) fx[kc][e] = (short)(v[kc][e / UNIT] >> (16 * (e % UNIT)));
        p += 16 * waves;
        w.step(a);
        if (g + 16 * waves < P) fetch();
        f32x4 r[2];
#pragma unroll
        for (int f = 0; f < 2; f++) {
            r[f] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kc = 0; kc < KC; kc++)
                r[f] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(fw[kc][f], fx[kc], r[f], 0, 0, 0);
        }
        store_relu<2>(r, bias, y, g, P, n0, c.cout, tiles[threadIdx.x >> 6], lane);
    }
}

// The same for two input channels at stride 2 on images whose rows are whole
// segments of 128 outputs (256 inputs): a wavefront takes a segment, its three
// input rows by one 16-byte load each (and the pixel to the left of them,
// around the panorama's seam for the first segment, by a fourth) into LDS, and
// reads the windows there.  The gathers above cost five loads of 64 scattered
// words for every 16 pixels, 21 lines a load: 16.1 us for 256 images of 32 x
// 256, 11.2 so.
constexpr int kSegment = 128;

__global__ __launch_bounds__(256) void k_conv_fwd_rows(ConvShape c, const uint16_t *__restrict__ x,
                                                       const uint16_t *__restrict__ w_nk,
                                                       const float *__restrict__ bias, uint16_t *__restrict__ y) {
    constexpr int K = 18, kPitch = 2 * kSegment + 8;  // words of a row; input column j of the segment at word j + 4
    __shared__ __align__(16) uint32_t rows[4][3 * kPitch];
    __shared__ __align__(16) uint16_t tiles[4][16 * 32];
    const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), i = lane & 15, q = lane >> 4;
    const int n0 = blockIdx.y * 32, per_row = c.wo / kSegment, segments = c.n * c.ho * per_row;
    uint32_t *r = rows[wid];
    const Rsrc src = rsrc_of(x, 4 * (uint32_t)(c.n * c.h * c.w));
    u32x4 v[3];
    uint32_t left;
    auto fetch = [&](int seg) {
        const int row = seg / per_row, j0 = (seg - row * per_row) * 2 * kSegment, b = row / c.ho, i0 = 2 * (row - b * c.ho) - 1;
        auto at = [&](int t, int j) { return i0 + t >= 0 && i0 + t < c.h ? 4 * (uint32_t)((b * c.h + i0 + t) * c.w + j) : kMaxBytes; };
#pragma unroll
        for (int t = 0; t < 3; t++) v[t] = load_b128(src, at(t, j0 + 4 * lane));
        left = __builtin_amdgcn_raw_buffer_load_b32(src, lane < 3 ? at(lane, j0 > 0 ? j0 - 1 : c.w - 1) : kMaxBytes, 0, 0);
    };
    int seg = blockIdx.x * 4 + wid;
    if (seg < segments) fetch(seg);
    const Rsrc weights = rsrc_of(w_nk, 2 * K * (uint32_t)c.cout);  // zeros past the last channel
    bf16x4 fw[2][2];
#pragma unroll
    for (int f = 0; f < 2; f++) {
        const uint32_t at = 2 * K * (uint32_t)(n0 + 16 * f + i);
        fw[0][f] = __builtin_bit_cast(bf16x4, __builtin_amdgcn_raw_buffer_load_b64(weights, at + 8 * q, 0, 0));
        const uint32_t tap8 = __builtin_amdgcn_raw_buffer_load_b32(weights, q == 0 ? at + 32 : kMaxBytes, 0, 0);
        fw[1][f] = __builtin_bit_cast(bf16x4, make_uint2(tap8, 0u));
    }
    // taps 2q and 2q + 1 of the lane's output, and tap 8 (the other products of the second instruction are zero)
    const uint32_t *t0 = r + (2 * q) / 3 * kPitch + (2 * q) % 3 + 2 * i + 3,
                   *t1 = r + (2 * q + 1) / 3 * kPitch + (2 * q + 1) % 3 + 2 * i + 3, *t8 = r + 2 * kPitch + 2 + 2 * i + 3;
    for (; seg < segments; seg += 4 * gridDim.x) {
        lds_handover();
#pragma unroll
        for (int t = 0; t < 3; t++) *(u32x4 *)(r + t * kPitch + 4 + 4 * lane) = v[t];
        if (lane < 3) r[lane * kPitch + 3] = left;
        lds_handover();
        if (seg + 4 * (int)gridDim.x < segments) fetch(seg + 4 * gridDim.x);
#pragma unroll
        for (int g = 0; g < kSegment / 16; g++) {
            const uint32_t a = t0[32 * g], b = t1[32 * g], e = q == 0 ? t8[32 * g] : 0;
            const bf16x4 fx[2] = {__builtin_bit_cast(bf16x4, make_uint2(a, b)), __builtin_bit_cast(bf16x4, make_uint2(e, 0u))};
            f32x4 s[2];
#pragma unroll
            for (int f = 0; f < 2; f++) {
                s[f] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kc = 0; kc < 2; kc++)
                    s[f] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(fw[kc][f], fx[kc], s[f], 0, 0, 0);
            }
            store_relu<2>(s, bias, y, seg * kSegment + 16 * g, segments * kSegment, n0, c.cout, tiles[wid], lane);
        }
    }
}

template <bool GRAD, int NF, int MT, int WAVES, int DEPTH>
void launch_gather(const GatherArgs &a, int M, hipStream_t s) {
    const int px = 16 * MT * WAVES, ch = 16 * NF, fragments = std::min(kFragments, 9 * a.chunks * NF);
    hipLaunchKernelGGL((k_conv_gather<GRAD, NF, MT, WAVES, DEPTH>), dim3((M + px - 1) / px, (a.N + ch - 1) / ch),
                       dim3(64 * WAVES), (fragments + 2 * MT * WAVES) * 1024, s, a);
}

template <int CHUNKS, int MT>
void launch_s2(const GatherArgs &a, int M, hipStream_t s) {
    constexpr int WAVES = 4, px = 16 * MT * WAVES;
    hipLaunchKernelGGL((k_conv_bwd_data_s2<CHUNKS, 2, MT, WAVES, 2>), dim3((M + px - 1) / px, (a.N + 31) / 32),
                       dim3(64 * WAVES), (18 * CHUNKS + 2 * MT * WAVES) * 1024, s, a);
}

}  // namespace

// Eight channels a load; byte offsets below kMaxBytes; with stride 2 a data
// gradient's weights of 32 input channels in LDS; with stride 1 more than eight
// output channels, whose chunks of 32 would be three quarters empty (524288
// pixels of 40 -> 8 channels: 89.9 us, 45.1 on 64 x 64 tiles).
bool conv_gather_fits(const ConvShape &c, bool grad) {
    const int64_t ck = grad ? c.cout : c.cin, pixels = (int64_t)c.n * (grad ? c.ho * c.wo : c.h * c.w);
    return ck % 8 == 0 && pixels * ck * (grad ? 4 : 2) <= (int64_t)kMaxBytes &&
           18 * (int64_t)c.cin * c.cout <= (int64_t)kMaxBytes && (!grad || (c.stride == 1 ? ck > 8 : ck <= 128));
}

bool conv_narrow_fits(const ConvShape &c) {
    return c.cin <= 3 && 2 * (int64_t)c.n * c.h * c.w * c.cin <= (int64_t)kMaxBytes;
}

ups_status launch_conv_gather_fwd(const ConvShape &c, const uint16_t *x, const uint16_t *w_nk, const float *b,
                                  uint16_t *y, hipStream_t s) {
    const GatherArgs a{c, c.h, c.w, c.cin, (c.cin + 31) / 32, c.cout, 9 * c.cin, c.cin, x, nullptr, w_nk, b, y};
    const int M = c.n * c.ho * c.wo;
    // tiles of 256 pixels share a block's weights among eight wavefronts and give each weight fragment two uses, where
    // they still cover every CU (32 -> 64 channels: 14.9 us; before the output tiles' order 16.7, and 20.3 with four
    // wavefronts, three blocks a CU and so a second round of them); else tiles of 64 pixels (96 -> 128 channels, 8192
    // pixels: 8.9 us)
    if (a.N > 32 && M / 256 * ((a.N + 63) / 64) >= 256) launch_gather<false, 4, 2, 8, 2>(a, M, s);
    else if (M / 256 * ((a.N + 31) / 32) >= 256) launch_gather<false, 2, 2, 8, 4>(a, M, s);
    else launch_gather<false, 2, 1, 4, 8>(a, M, s);
    UPS_CHECK_HIP(hipGetLastError());
    return UPS_OK;
}

ups_status launch_conv_narrow_fwd(const ConvShape &c, const uint16_t *x, const uint16_t *w_nk, const float *b,
                                  uint16_t *y, hipStream_t s) {
    if (c.cin == 2 && c.stride == 2 && c.w % (2 * kSegment) == 0) {
        // one segment a wavefront up to eight blocks a CU
        const int blocks = std::max(1, std::min(2048, (c.n * c.ho * (c.wo / kSegment) + 3) / 4));
        hipLaunchKernelGGL(k_conv_fwd_rows, dim3(blocks, (c.cout + 31) / 32), dim3(256), 0, s, c, x, w_nk, b, y);
        UPS_CHECK_HIP(hipGetLastError());
        return UPS_OK;
    }
    // at most five blocks a CU (what the registers leave room for at three channels), each wavefront several groups; at
    // three channels at most two rounds of them over all output channels (131072 pixels, 128 and 256 channels: 25.8 and
    // 46.7 us with 1280 for every 32 channels, 21.5 and 30.6 so; at one and two channels the same or up to 16 % slower)
    const int P = c.n * c.ho * c.wo, ny = (c.cout + 31) / 32;
    const int blocks = std::max(1, std::min(1280 / (c.cin == 3 ? std::max(1, ny / 2) : 1), (P + 127) / 128));
    const WalkArgs a = walk_args(c, 64 * blocks);
    const dim3 grid(blocks, ny), block(256);
    if (c.cin == 1) hipLaunchKernelGGL(k_conv_fwd_narrow<1>, grid, block, 0, s, a, x, w_nk, b, y);
    else if (c.cin == 2) hipLaunchKernelGGL(k_conv_fwd_narrow<2>, grid, block, 0, s, a, x, w_nk, b, y);
    else hipLaunchKernelGGL(k_conv_fwd_narrow<3>, grid, block, 0, s, a, x, w_nk, b, y);
    UPS_CHECK_HIP(hipGetLastError());
    return UPS_OK;
}

ups_status launch_conv_gather_bwd_data(const ConvShape &c, const uint16_t *y, const float *dy, const uint16_t *w_kn,
                                       float *dx, hipStream_t s) {
    const GatherArgs a{c, c.ho, c.wo, c.cout, (c.cout + 31) / 32, c.cin, c.cout, c.cin * c.cout, y, dy, w_kn, nullptr, dx};
    const int M = c.n * c.ho * c.wo;  // positions: pixels, or 2 x 2 pixels
    const bool many = M / 128 * ((a.N + 31) / 32) >= 512;
    if (c.stride == 1) {
        // us for blocks of 64 pixels x 32 channels / 128 x 32 / 128 x 64 / 64 x 64 tiles:
        //   32768 px, 128->128   71.0/101.8/ 56.6/ 82.9     16384 px, 64->64 (too few blocks)  10.2/12.2/10.7/23.3
        //   524288 px, 40->16   107.7/ 92.1/ 62.1/ 67.6     524288 px, 16->16                  54.9/47.4/59.4/62.0
        //                                                   524288 px, 2->128                 271.2/368.2/340.2/632.0
        // 64 channels a block mask and round each gradient half as often; 128 pixels use each weight fragment twice, but
        // with the weights of more than 64 channels LDS holds one block a CU
        if (a.N > 32 && M / 128 * ((a.N + 63) / 64) >= 256) launch_gather<true, 4, 1, 8, 4>(a, M, s);
        else if (many && a.chunks <= 2) launch_gather<true, 2, 2, 4, 2>(a, M, s);
        else launch_gather<true, 2, 1, 4, 4>(a, M, s);
    } else if (many && a.chunks <= 3) {
        if (a.chunks == 1) launch_s2<1, 2>(a, M, s);
        else if (a.chunks == 2) launch_s2<2, 2>(a, M, s);
        else launch_s2<3, 2>(a, M, s);
    } else {
        if (a.chunks == 1) launch_s2<1, 1>(a, M, s);
        else if (a.chunks == 2) launch_s2<2, 1>(a, M, s);
        else if (a.chunks == 3) launch_s2<3, 1>(a, M, s);
        else launch_s2<4, 1>(a, M, s);
    }
    UPS_CHECK_HIP(hipGetLastError());
    return UPS_OK;
}

}  // namespace ups
