// Surface normals of a panoramic range image (UPSLAM Section III-A): a rough
// normal from the cross product of the vectors to two image neighbours, then
// an edge-aware a-trous wavelet filter over LDS-staged tiles.
#include "ups_internal.hpp"

namespace ups {

// Raw normal of pixel (i, j) from its range rc and the ranges of its right
// neighbour (i, j+1 mod cols) and lower neighbour (i+1, j) -- (i-1, j) on the
// last row: the normalised cross product of the two difference vectors,
// oriented towards the sensor; zero when a range is invalid, a neighbour jumps
// by more than max_rel_jump * rc, or the cross product is degenerate.
// The same from usable ranges (or NaN) and the rays of the three pixels (uc:
// the pixel, ua: its right neighbour, ub: the lower one).
__device__ __forceinline__ float3 raw_normal_ranges(float rc, float ra, float rb, float3 uc, float3 ua, float3 ub,
                                                    float max_rel_jump) {
    const float jump = max_rel_jump * rc;
    bool ok = !((fabsf(ra - rc) > jump) | (fabsf(rb - rc) > jump));
    const float3 pc = make_float3(rc * uc.x, rc * uc.y, rc * uc.z);
    const float3 a = make_float3(ra * ua.x - pc.x, ra * ua.y - pc.y, ra * ua.z - pc.z);
    const float3 b = make_float3(rb * ub.x - pc.x, rb * ub.y - pc.y, rb * ub.z - pc.z);
    const float3 n = cross3(a, b);
    const float nn = __builtin_amdgcn_sqrtf(dot3(n, n));
    ok &= nn > 1e-6f * __builtin_amdgcn_sqrtf(dot3(a, a) * dot3(b, b));
    const float inv = __builtin_amdgcn_rcpf(nn);
    const float s = (dot3(n, pc) > 0.f) ? -inv : inv;
    return make_float3(ok ? n.x * s : 0.f, ok ? n.y * s : 0.f, ok ? n.z * s : 0.f);
}

__device__ __forceinline__ float3 raw_normal(const DGeom &g, int i, int j, int ib, float rc, float ra, float rb,
                                             float max_rel_jump) {
    if (!(range_ok(g, rc) && ib >= 0 && range_ok(g, ra) && range_ok(g, rb))) return make_float3(0.f, 0.f, 0.f);
    const int ja = (j + 1 == g.cols) ? 0 : j + 1;
    return raw_normal_ranges(rc, ra, rb, ray(g, i, j), ray(g, i, ja), ray(g, ib, j), max_rel_jump);
}

// Ray of a pixel from its row's (cos el, sin el) and its column's (cos az, sin az).
__device__ __forceinline__ float3 ray_of(float2 e, float2 a) { return make_float3(e.x * a.x, e.x * a.y, e.y); }

// Raw normals only (no smoothing): one thread per pixel; the neighbour reads
// are served from L1/L2.
__global__ __launch_bounds__(kBlock) void k_normals_raw(DGeom g, const float *__restrict__ depth,
                                                        float4 *__restrict__ out, float max_rel_jump) {
    const int npix = g.rows * g.cols;
    const int p = blockIdx.x * kBlock + threadIdx.x;
    if (p >= npix) return;
    const int i = p / g.cols, j = p - i * g.cols;
    const float rc = depth[p];
    const int ja = (j + 1 == g.cols) ? 0 : j + 1;
    const int ib = (i + 1 < g.rows) ? i + 1 : i - 1;
    const float ra = depth[i * g.cols + ja], rb = ib >= 0 ? depth[ib * g.cols + j] : 0.f;
    const float3 n = raw_normal(g, i, j, ib, rc, ra, rb, max_rel_jump);
    out[p] = make_float4(n.x, n.y, n.z, range_ok(g, rc) ? rc : 0.f);
}

// Output tiles of the a-trous passes: 64 pixels wide, 4 R rows high.  A
// wavefront makes R rows of the tile, one pixel of each per lane: rows that
// share their taps' rows (spaced as the taps are), so each tap is read from LDS
// once for up to five of them.  The passes are bound by vector instructions:
// 225 a pixel for the taps, the rest for staging, raw normals and ends.
// Batches take 16 rows, whose halo is the smaller part of a tile: the two
// passes over 256 scans of 64 x 512 to 128 x 2048 (31.7 million pixels) take
// 275 and 249 us, against 365 and 325 with a row a time per lane and pixels
// staged one by one (370 and 279 instructions a pixel, against 424 and 304).
// A single panorama has too few
// rows to fill the chip with that: 4 rows a tile take 4.4 + 3.4 us at 64 x
// 1024 where 8 take 5.1 + 4.0 and 16 take 6.6 + 5.2, and at 256 x 2048 all
// lie within 7 % (25.4, 25.0 and 26.7 us for three passes).
constexpr int kRowsBatch = 4, kRowsOne = 1;
constexpr int kTileW = 64, kWaves = kBlock / 64;
constexpr int kTileHBatch = kWaves * kRowsBatch, kTileHOne = kWaves * kRowsOne;

// First row in the tile of a wavefront's outputs b + STEP k, k < R.
template <int R, int STEP>
__device__ __forceinline__ int first_row(int wave) {
    static_assert(kWaves % STEP == 0, "the wavefronts' rows fill the tile");
    return wave % STEP + R * STEP * (wave / STEP);
}

// R a-trous outputs of a lane from an LDS surfel tile of row pitch LW: `tile`
// points to the first tap of the first output, output k lies STEP k rows lower.
// 5x5 B3-spline taps spaced STEP, weight
// h[dy] h[dx] exp(-(dr^2 + (2 - 2 n_p.n_q)/sigma_n^2))
// with dr = (r_q - r_p)/(sigma_r r_p), renormalised; the range is unchanged.
// The whole weight is one exp2: log2 e and 1/sigma_n^2 are folded into a
// scaled copy of the centre normal, sqrt(log2 e)/(sigma_r r_p) into the range
// difference and log2(h[dy] h[dx]) into the exponent, so a tap costs three
// FMAs for the normal term, two for the range term and three to accumulate.
// Taps without a normal need no test: their zero normal adds nothing to the
// weighted sum, and the sum is renormalised rather than divided by the total
// weight.
template <int R, int STEP, int LW>
__device__ __forceinline__ void atrous_tap_sums(const float4 *tile, float inv_sigma_r, float inv_sigma_n2,
                                                float4 (&o)[R]) {
    constexpr float kLog2e = 1.4426950408889634f;
    // log2 of h = (1, 4, 6, 4, 1) / 16
    constexpr float lh[5] = {-4.f, -2.f, -1.4150374992788437f, -2.f, -4.f};
    // log2 e (2 - 2 n_p.n_q) / sigma_n^2 = kn - kn n_p.n_q
    const float kn = 2.f * kLog2e * inv_sigma_n2;
    float cx[R], cy[R], cz[R], sr[R], csr[R], ax[R], ay[R], az[R];
    bool any = false;
#pragma unroll
    for (int k = 0; k < R; k++) {
        const float4 c = tile[(k + 2) * STEP * LW + 2 * STEP];
        o[k] = make_float4(0.f, 0.f, 0.f, c.w);
        any |= normal_ok(c);
        cx[k] = kn * c.x, cy[k] = kn * c.y, cz[k] = kn * c.z;
        // log2 e ((r_q - r_p) / (sigma_r r_p))^2 = (r_q sr - r_p sr)^2
        sr[k] = 1.2011224087864498f * inv_sigma_r * __builtin_amdgcn_rcpf(c.w);  // sqrt(log2 e) / (sigma_r r_p)
        csr[k] = -c.w * sr[k];
        ax[k] = ay[k] = az[k] = 0.f;
    }
    if (!__builtin_amdgcn_ballot_w64(any)) return;
#pragma unroll
    for (int m = 0; m < R + 4; m++) {
        const float4 *row = tile + m * STEP * LW;
        float4 q[5];
#pragma unroll
        for (int dx = 0; dx < 5; dx++) q[dx] = row[dx * STEP];
#pragma unroll
        for (int k = 0; k < R; k++) {
            const int dy = m - k;
            if (dy < 0 || dy > 4) continue;
#pragma unroll
            for (int dx = 0; dx < 5; dx++) {
                float e = fmaf(cx[k], q[dx].x, lh[dy] + lh[dx] - kn);
                e = fmaf(cy[k], q[dx].y, e);
                e = fmaf(cz[k], q[dx].z, e);
                const float d = fmaf(q[dx].w, sr[k], csr[k]);
                e = fmaf(-d, d, e);
                const float w = __builtin_amdgcn_exp2f(e);
                ax[k] = fmaf(w, q[dx].x, ax[k]);
                ay[k] = fmaf(w, q[dx].y, ay[k]);
                az[k] = fmaf(w, q[dx].z, az[k]);
            }
        }
    }
#pragma unroll
    for (int k = 0; k < R; k++) {
        // summed in this order in every kernel
        const float nn2 = fmaf(az[k], az[k], fmaf(ay[k], ay[k], ax[k] * ax[k]));
        // an output without a normal of its own has none
        if (normal_ok(tile[(k + 2) * STEP * LW + 2 * STEP]) && nn2 > 0.f) {
            const float s = __builtin_amdgcn_rsqf(nn2);
            o[k].x = ax[k] * s;
            o[k].y = ay[k] * s;
            o[k].z = az[k] * s;
        }
    }
}

// Pyramid levels 1-3 of an image from its level-0 pixel (i, j): level-l pixel
// (i >> l, j >> l) when i and j are multiples of 2^l (every 2^l-th row and
// column; pyr[l - 1] null past the last level).
__device__ __forceinline__ void store_pyramid(const DGeom &g, float4 *const *pyr, int i, int j, float4 v) {
#pragma unroll
    for (int l = 1; l <= 3; l++) {
        float4 *dst = pyr[l - 1];
        if (dst && (i & ((1 << l) - 1)) == 0 && (j & ((1 << l) - 1)) == 0)
            stg_u(dst + (size_t)(i >> l) * (g.cols >> l), (uint32_t)j >> l, v);
    }
}

// The outputs of a wavefront: rows first_row + STEP k of the tile at (x0, y0),
// from its LDS tile of pitch LW.
template <int R, int STEP, int LW>
__device__ __forceinline__ void atrous_rows(const DGeom &g, const float4 *tile, float4 *__restrict__ out, int x0, int y0,
                                            float inv_sigma_r, float inv_sigma_n2, float4 *const *pyr) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int b = first_row<R, STEP>(wave);
    if (y0 + b >= g.rows) return;
    float4 v[R];
    atrous_tap_sums<R, STEP, LW>(tile + b * LW + lane, inv_sigma_r, inv_sigma_n2, v);
#pragma unroll
    for (int k = 0; k < R; k++) {
        const int gy = y0 + b + STEP * k;
        if (gy >= g.rows) break;
        stg_u(out + (size_t)gy * g.cols, (uint32_t)(x0 + lane), v[k]);
        if (pyr) store_pyramid(g, pyr, gy, x0 + lane, v[k]);
    }
}

__device__ __forceinline__ int wrap_col(const DGeom &g, int gx) {
    return gx < 0 ? gx + g.cols : (gx >= g.cols ? gx - g.cols : gx);
}

template <int R, int STEP>
constexpr int atrous_tile_elems() { return (kTileW + 4 * STEP) * (4 * R + 4 * STEP); }

// One a-trous level with taps spaced STEP for the 4R x 64 output tile at
// (x0, y0): the block stages the (4R + 4 STEP) x (64 + 4 STEP) surfel tile
// around it in LDS (rows outside the image empty, columns wrapped), each
// wavefront R + STEP rows of it: 64 columns of a row by one load, the others of
// its rows together.  STEP is a template parameter so that every tap reads LDS
// at a constant offset from the output's address.
template <int R, int STEP>
__device__ __forceinline__ void atrous_tile(const DGeom &g, const float4 *__restrict__ in, float4 *__restrict__ out,
                                            int x0, int y0, float inv_sigma_r, float inv_sigma_n2, float4 *tile,
                                            float4 *const *pyr) {
    constexpr int halo = 2 * STEP, LW = kTileW + 2 * halo;
    constexpr int NR = R + STEP;                   // rows staged by a wavefront
    constexpr int SC = 2 * halo;                   // columns past the first 64
    constexpr int NS = (NR * SC + 63) / 64;        // loads of these for all its rows
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int ly0 = wave * NR, gx = wrap_col(g, x0 - halo + lane);
    float4 v[NR], w[NS];
#pragma unroll
    for (int k = 0; k < NR; k++) {
        const int gy = min(max(y0 - halo + ly0 + k, 0), g.rows - 1);
        v[k] = ldg_u(in + (size_t)gy * g.cols, (uint32_t)gx);
    }
#pragma unroll
    for (int k = 0; k < NS; k++) {
        const int q = min(lane + 64 * k, NR * SC - 1);
        const int gy = min(max(y0 - halo + ly0 + q / SC, 0), g.rows - 1);
        w[k] = ldg(in, gy * g.cols + wrap_col(g, x0 - halo + 64 + q % SC));
    }
    if (y0 < halo || y0 + 4 * R + halo > g.rows) {
        auto clear = [&](float4 &f, int gy) {
            const bool in = (gy >= 0) & (gy < g.rows);
            f.x = in ? f.x : 0.f, f.y = in ? f.y : 0.f, f.z = in ? f.z : 0.f, f.w = in ? f.w : 0.f;
        };
#pragma unroll
        for (int k = 0; k < NR; k++) clear(v[k], y0 - halo + ly0 + k);
#pragma unroll
        for (int k = 0; k < NS; k++) clear(w[k], y0 - halo + ly0 + (lane + 64 * k) / SC);
    }
#pragma unroll
    for (int k = 0; k < NR; k++) tile[(ly0 + k) * LW + lane] = v[k];
#pragma unroll
    for (int k = 0; k < NS; k++) {
        const int q = lane + 64 * k;
        if (q < NR * SC) tile[(ly0 + q / SC) * LW + 64 + q % SC] = w[k];
    }
    __syncthreads();
    atrous_rows<R, STEP, LW>(g, tile, out, x0, y0, inv_sigma_r, inv_sigma_n2, pyr);
}

template <int STEP>
__global__ __launch_bounds__(kBlock) void k_atrous(DGeom g, const float4 *__restrict__ in, float4 *__restrict__ out,
                                                   float inv_sigma_r, float inv_sigma_n2) {
    __shared__ float4 tile[atrous_tile_elems<kRowsOne, STEP>()];
    atrous_tile<kRowsOne, STEP>(g, in, out, blockIdx.x * kTileW, blockIdx.y * kTileHOne, inv_sigma_r, inv_sigma_n2,
                                tile, nullptr);
}

// Raw normals and the first a-trous level (step 1) in one pass: the raw
// normals of the (4R + 4) x 68 tile around the outputs into LDS, then the
// filter.  A lane walks down R + 1 rows of one column, so it keeps the
// column's ray tables and passes a pixel's range and ray on as the next row's;
// the ranges come straight from the image.  The tile's last four columns are
// the work of other lanes, a pixel each (of wavefronts that change from block
// to block, since a block's first wavefront often starts on the same SIMD).
template <int R>
__device__ __forceinline__ void normals_atrous_tile(const DGeom &g, const float *__restrict__ depth,
                                                    float4 *__restrict__ out, int x0, int y0, float max_rel_jump,
                                                    float inv_sigma_r, float inv_sigma_n2, float4 *const *pyr) {
    constexpr int FH = 4 * R + 4, FW = kTileW + 4;
    static_assert(4 * FH <= kBlock, "one pixel of the last columns per thread");
    __shared__ float4 raw[FH * FW];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const float nan = __int_as_float(0x7fc00000);
    // an unusable range as NaN: the normals it is part of fail their last test, as they must
    auto range = [&](float r, bool ok) { return range_ok(g, r) & ok ? r : nan; };
    // the lower neighbour's row, the one above on the last row; clamped for rows outside the image
    auto clamp_row = [&](int i) { return min(max(i, 0), g.rows - 1); };
    auto below = [&](int i) { return clamp_row(i + 1 < g.rows ? i + 1 : i - 1); };
    auto row_ray = [&](int i) { return ldg_u(g.lut_row, (uint32_t)i << g.lshift); };
    auto col_ray = [&](int j) { return ldg_u(g.lut_col, (uint32_t)j << g.lshift); };
    auto put = [&](int ly, int lx, float rc, float ra, float rb, float3 uc, float3 ua, float3 ub) {
        const int gy = y0 - 2 + ly;
        const bool in = (gy >= 0) & (gy < g.rows);  // a row outside the image is empty
        const float3 n = raw_normal_ranges(rc, range(ra, in), rb, uc, ua, ub, max_rel_jump);
        raw[ly * FW + lx] = make_float4(n.x, n.y, n.z, in & (rc == rc) ? rc : 0.f);
    };
    // the last columns' pixel of this thread
    const int q0 = 64 * ((wave + (int)blockIdx.x) & (kWaves - 1)), q = min(q0 + lane, 4 * FH - 1);
    const int qy = q >> 2, qx = 64 + (q & 3);
    float q_rc = nan, q_ra = nan, q_rb = nan;
    float2 q_e0, q_e1, q_ac, q_ar;
    if (q0 < 4 * FH) {
        const int i = clamp_row(y0 - 2 + qy), ib = below(y0 - 2 + qy);
        const int j = wrap_col(g, x0 - 2 + qx), jr = wrap_col(g, x0 - 1 + qx);
        q_rc = ldg(depth, i * g.cols + j), q_ra = ldg(depth, i * g.cols + jr), q_rb = ldg(depth, ib * g.cols + j);
        q_e0 = row_ray(i), q_e1 = row_ray(ib);
        q_ac = col_ray(j), q_ar = col_ray(jr);
    }
    const int ly0 = wave * (R + 1), j = wrap_col(g, x0 - 2 + lane), jr = wrap_col(g, x0 - 1 + lane);
    float rc[R + 2], ra[R + 1];
    float2 e[R + 2];
    const float2 ac = col_ray(j), ar = col_ray(jr);
#pragma unroll
    for (int k = 0; k < R + 2; k++) {
        const int i = k ? below(y0 - 2 + ly0 + k - 1) : clamp_row(y0 - 2 + ly0);
        const float *row = depth + (size_t)i * g.cols;
        rc[k] = ldg_u(row, (uint32_t)j);
        if (k <= R) ra[k] = ldg_u(row, (uint32_t)jr);
        e[k] = lds_uniform(g.lut_row, i << g.lshift);
    }
    float3 uc = ray_of(e[0], ac);
#pragma unroll
    for (int k = 0; k < R + 2; k++) rc[k] = range(rc[k], true);
#pragma unroll
    for (int k = 0; k <= R; k++) {
        const float3 ub = ray_of(e[k + 1], ac);
        put(ly0 + k, lane, rc[k], ra[k], rc[k + 1], uc, ray_of(e[k], ar), ub);
        uc = ub;
    }
    if (q0 < 4 * FH)
        put(qy, qx, range(q_rc, true), q_ra, range(q_rb, true), ray_of(q_e0, q_ac), ray_of(q_e0, q_ar),
            ray_of(q_e1, q_ac));
    __syncthreads();
    atrous_rows<R, 1, FW>(g, raw, out, x0, y0, inv_sigma_r, inv_sigma_n2, pyr);
}

__global__ __launch_bounds__(kBlock) void k_normals_atrous(DGeom g, const float *__restrict__ depth,
                                                           float4 *__restrict__ out, float max_rel_jump,
                                                           float inv_sigma_r, float inv_sigma_n2) {
    normals_atrous_tile<kRowsOne>(g, depth, out, blockIdx.x * kTileW, blockIdx.y * kTileHOne, max_rel_jump,
                                  inv_sigma_r, inv_sigma_n2, nullptr);
}

// ---- batched: block -> (image, tile) from a table, one word per tile:
// (image << kNormTileBits) | tile of the image
__global__ __launch_bounds__(kBlock) void k_normals_atrous_batch(const NormImg *__restrict__ imgs,
                                                                 const unsigned *__restrict__ tile_of,
                                                                 int out_tmp, int write_pyr, float max_rel_jump,
                                                                 float inv_sigma_r, float inv_sigma_n2) {
    const unsigned v = tile_of[blockIdx.x];
    const NormImg im = imgs[v >> kNormTileBits];
    const int t = (int)(v & ((1u << kNormTileBits) - 1)), tx = im.g.cols / kTileW;
    const int by = t / tx, bx = t - by * tx;
    normals_atrous_tile<kRowsBatch>(im.g, im.depth, out_tmp ? im.tmp : im.out, bx * kTileW, by * kTileHBatch,
                                    max_rel_jump, inv_sigma_r, inv_sigma_n2, write_pyr ? im.pyr : nullptr);
}

template <int STEP>
__global__ __launch_bounds__(kBlock) void k_atrous_batch(const NormImg *__restrict__ imgs,
                                                         const unsigned *__restrict__ tile_of, int src_tmp,
                                                         int write_pyr, float inv_sigma_r, float inv_sigma_n2) {
    __shared__ float4 tile[atrous_tile_elems<kRowsBatch, STEP>()];
    const unsigned v = tile_of[blockIdx.x];
    const NormImg im = imgs[v >> kNormTileBits];
    const int t = (int)(v & ((1u << kNormTileBits) - 1)), tx = im.g.cols / kTileW;
    const int by = t / tx, bx = t - by * tx;
    atrous_tile<kRowsBatch, STEP>(im.g, src_tmp ? im.tmp : im.out, src_tmp ? im.out : im.tmp, bx * kTileW,
                                  by * kTileHBatch, inv_sigma_r, inv_sigma_n2, tile, write_pyr ? im.pyr : nullptr);
}

// Tiles of a panorama in the batched a-trous launches.
int normal_tiles(const DGeom &g) { return (g.cols / kTileW) * ((g.rows + kTileHBatch - 1) / kTileHBatch); }

ups_status launch_normals_batch(const NormImg *imgs, const unsigned *tile_of, int total_tiles,
                                const ups_normal_params &p, int write_pyr, hipStream_t s) {
    const int L = p.atrous_levels;
    const float inv_sr = 1.f / p.sigma_r, inv_sn2 = 1.f / (p.sigma_n * p.sigma_n);
    if (L == 0 || total_tiles == 0) {
        if (total_tiles > 0) {
            set_error("batched normals need at least one a-trous level");
            return UPS_ERR_UNSUPPORTED;
        }
        return UPS_OK;
    }
    // ping-pong between out and tmp so that the last level writes out
    int in_tmp = (L - 1) % 2;
    // the last pass writes the surfel images (and, with write_pyr, their pyramids)
    hipLaunchKernelGGL(k_normals_atrous_batch, dim3(total_tiles), dim3(kBlock), 0, s, imgs, tile_of, in_tmp,
                       (L == 1) ? write_pyr : 0, p.max_rel_jump, inv_sr, inv_sn2);
    UPS_CHECK_HIP(hipGetLastError());
    for (int l = 1; l < L; l++) {
        // levels 1 and 2 (taps spaced 2 and 4); the caller limits the levels to 3
        const int last = (l == L - 1) ? write_pyr : 0;
        if (l == 1)
            hipLaunchKernelGGL(k_atrous_batch<2>, dim3(total_tiles), dim3(kBlock), 0, s, imgs, tile_of, in_tmp,
                               last, inv_sr, inv_sn2);
        else
            hipLaunchKernelGGL(k_atrous_batch<4>, dim3(total_tiles), dim3(kBlock), 0, s, imgs, tile_of, in_tmp,
                               last, inv_sr, inv_sn2);
        UPS_CHECK_HIP(hipGetLastError());
        in_tmp ^= 1;
    }
    return UPS_OK;
}

ups_status launch_normals(ups_context *ctx, const DGeom &g, const float *depth, float4 *surfel,
                          const ups_normal_params &p, hipStream_t s) {
    const int npix = g.rows * g.cols;
    const int L = p.atrous_levels;
    const float inv_sr = 1.f / p.sigma_r, inv_sn2 = 1.f / (p.sigma_n * p.sigma_n);
    if (L == 0) {
        hipLaunchKernelGGL(k_normals_raw, dim3((npix + kBlock - 1) / kBlock), dim3(kBlock), 0, s, g, depth, surfel,
                           p.max_rel_jump);
        UPS_CHECK_HIP(hipGetLastError());
        return UPS_OK;
    }
    const dim3 grid(g.cols / kTileW, (g.rows + kTileHOne - 1) / kTileHOne);
    // ping-pong so that the last level writes `surfel`
    float4 *bufs[2] = {surfel, ctx->tmp_surfel};
    float4 *dst = bufs[(L - 1) % 2];
    hipLaunchKernelGGL(k_normals_atrous, grid, dim3(kBlock), 0, s, g, depth, dst, p.max_rel_jump, inv_sr, inv_sn2);
    UPS_CHECK_HIP(hipGetLastError());
    const float4 *src = dst;
    for (int l = 1; l < L; l++) {
        dst = bufs[(L - 1 - l) % 2];
        // levels 1 and 2 (taps spaced 2 and 4); the caller limits the levels to 3
        if (l == 1) hipLaunchKernelGGL(k_atrous<2>, grid, dim3(kBlock), 0, s, g, src, dst, inv_sr, inv_sn2);
        else hipLaunchKernelGGL(k_atrous<4>, grid, dim3(kBlock), 0, s, g, src, dst, inv_sr, inv_sn2);
        UPS_CHECK_HIP(hipGetLastError());
        src = dst;
    }
    return UPS_OK;
}

}  // namespace ups
