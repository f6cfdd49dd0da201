// Loop-closure grid search (UPSLAM Section III-C): a few hundred candidate
// transforms of every registration of a batch are compared by a coarse
// projective alignment test -- the number of Omega inliers at a subsampled
// pyramid level -- and the best candidate becomes the start of the
// full-resolution registration.
//
// Candidates: c = (a, u, v) with yaw index a < n_yaw and grid indices
// u, v < n_xy; G_c = (Rz(2 pi a / n_yaw), ((u - h) s, (v - h) s, 0)) with
// h = (n_xy - 1) / 2 and s the grid step; the scored pose is base_k G_c.
//
// Scores are integer sums (block counts added with atomics), so they do not
// depend on the order in which blocks finish.
#include <type_traits>

#include "ups_icp.hpp"

namespace ups {

// Candidate pose base * G_c in FP64 (row-major R, then t).
__device__ __forceinline__ void candidate_pose(const ups_pose &base, const GridArgs &g, int c, double *R,
                                               double *t) {
    const int per_yaw = g.n_xy * g.n_xy;
    const int a = c / per_yaw, u = (c / g.n_xy) % g.n_xy, v = c % g.n_xy;
    const double yaw = 6.283185307179586 * (double)a / (double)g.n_yaw;
    const double h = 0.5 * (double)(g.n_xy - 1);
    const double cy = cos(yaw), sy = sin(yaw);
    const double Gr[9] = {cy, -sy, 0.0, sy, cy, 0.0, 0.0, 0.0, 1.0};
    const double Gt[3] = {((double)u - h) * g.xy_step, ((double)v - h) * g.xy_step, 0.0};
    for (int r = 0; r < 3; r++) {
        for (int q = 0; q < 3; q++)
            R[3 * r + q] = base.R[3 * r] * Gr[q] + base.R[3 * r + 1] * Gr[3 + q] + base.R[3 * r + 2] * Gr[6 + q];
        t[r] = base.R[3 * r] * Gt[0] + base.R[3 * r + 1] * Gt[1] + base.R[3 * r + 2] * Gt[2] + base.t[r];
    }
}

typedef float v4fa __attribute__((ext_vector_type(4), aligned(8)));

// (int)floorf(v) in one instruction (0 for a NaN).
__device__ __forceinline__ int floor_int(float v) {
    int r;
    asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(r) : "v"(v));
    return r;
}

// project() to entry i pitch + j of a table whose rows also hold column cols
// (the column is not wrapped), for a panorama that is `NARROW` or not: the
// same angles, with fewer instructions around them.  The azimuth's sign and
// turn are one step (2 pi - r where y is negative; a zero r then gives column
// cols for 0, the same column), the row is tested as an integer.  An elevation
// that is no number (the origin, a point of denormal coordinates) has no pixel.
// Next to the vertical axis the reciprocal overflows and the column is any
// integer: callers bound the entry, except where `NARROW`, whose directions
// have |z| < rho and so an x or y whose square is no zero.
template <bool NARROW>
__device__ __forceinline__ bool project_at(const DGeom &g, float3 q, uint32_t pitch, uint32_t &at) {
    const float rho = __builtin_amdgcn_sqrtf(q.x * q.x + q.y * q.y);
    bool ok;
    float el;
    if constexpr (NARROW) {
        ok = fabsf(q.z) < rho;
        el = atan_unit(q.z * __builtin_amdgcn_rcpf(rho));
    } else {
        el = atan2_fast(q.z, rho);
        ok = el == el;
    }
    const float ax = fabsf(q.x), ay = fabsf(q.y);
    const bool steep = ay > ax;
    float r = atan_unit((steep ? ax : ay) * __builtin_amdgcn_rcpf(steep ? ay : ax));
    if (steep) r = 1.57079632679489662f - r;
    if (q.x < 0.f) r = 3.14159265358979324f - r;
    const float az = __float_as_int(q.y) < 0 ? kTwoPi - r : r;
    float below;
    {
        // project() branches on g.narrow before this difference, so the arctangent's last product is rounded by itself
#pragma clang fp contract(off)
        below = g.el_top - el;
    }
    const uint32_t i = (uint32_t)floor_int(below * g.inv_d_el + 0.5f);
    const uint32_t j = (uint32_t)floor_int(az * g.az_scale + 0.5f);
    at = __umul24(i, pitch) + j;
    return ok & (i < (uint32_t)g.rows);
}

// blockIdx.x: a tile of the batch at the grid level (the level's prefix table
// of tiles of kBlock * K pixels); blockIdx.y: the candidate.
__global__ __launch_bounds__(kBlock) void k_grid_score(const Inst *__restrict__ insts,
                                                       const int *__restrict__ tile_start, int n, int K,
                                                       const ups_pose *__restrict__ base, GridArgs g,
                                                       int *__restrict__ scores) {
    __shared__ float Ts[12];
    __shared__ int block_count;
    const int b = blockIdx.x, c = blockIdx.y, tid = threadIdx.x;
    int lo = 0, hi = n;  // the last k with tile_start[k] <= b
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (tile_start[mid] <= b) lo = mid;
        else hi = mid;
    }
    const Inst &I = insts[lo];
    const int tile = b - tile_start[lo];
    const int l = g.level;
    const DGeom sg = I.sg[l], kg = I.kg[l];
    const float4 *__restrict__ scan = I.scan[l];
    const float4 *__restrict__ kf = I.kf[l];
    if (tid == 0) {
        double R[9], t[3];
        candidate_pose(base[lo], g, c, R, t);
        for (int q = 0; q < 9; q++) Ts[q] = (float)R[q];
        for (int q = 0; q < 3; q++) Ts[9 + q] = (float)t[q];
        block_count = 0;
    }
    __syncthreads();
    Rt32 T;
#pragma unroll
    for (int q = 0; q < 9; q++) T.r[q] = Ts[q];
#pragma unroll
    for (int q = 0; q < 3; q++) T.t[q] = Ts[9 + q];
    const int npix = sg.rows * sg.cols;
    int count = 0;
    for (int k = 0; k < K; k++) {
        // the 64 pixels of a wavefront lie in one row (cols is a multiple of 64)
        const int pw = __builtin_amdgcn_readfirstlane(tile * kBlock * K + k * kBlock + (tid & ~63));
        if (pw >= npix) break;
        const int p = pw + (tid & 63);
        const int i = pw / sg.cols, j = p - i * sg.cols;
        float4 s2 = ldg_u(scan, (uint32_t)min(p, npix - 1));
        s2.w = p < npix ? s2.w : 0.f;
        const float2 e = lds_uniform(sg.lut_row, i << sg.lshift);
        const float2 ca = ldg_u(sg.lut_col, (uint32_t)j << sg.lshift);
        const Gather G = scan_side(sg, s2, e, ca, kg, kf, T);
        bool inl;
        float r;
        float3 n1;
        kf_side(kg, G, g.d_max2, g.cos_theta, inl, r, n1);
        count += inl ? 1 : 0;
    }
    if (count) atomicAdd(&block_count, count);
    __syncthreads();
    if (tid == 0 && block_count) atomicAdd(&scores[lo * g.C + c], block_count);
}

// What a candidate needs of a keyframe surfel, per pixel of the grid level:
// its point x1 = range * ray and its normal, so that a candidate gathers 24
// bytes from one place and forms neither the ray nor the point, nor tests the
// surfel (an unusable one has a NaN point, which no distance test passes).
// Rows are one entry longer than the image (entry cols repeats column 0, for
// an azimuth that rounds up to it), and one more NaN entry after the last row
// serves the candidates that project outside.
struct GridPoint {
    float x[3], n[3];
};

// blockIdx.y: the registration.  The table of its keyframe, and its scores zeroed.
__global__ __launch_bounds__(kBlock) void k_grid_points(const Inst *__restrict__ insts, GridArgs g,
                                                        int *__restrict__ scores) {
    const Inst &I = insts[blockIdx.y];
    const int l = g.level, first = blockIdx.x * kBlock + threadIdx.x, stride = gridDim.x * kBlock;
    for (int c = first; c < g.C; c += stride) scores[(size_t)blockIdx.y * g.C + c] = 0;
    if (!g.points) return;
    const DGeom kg = I.kg[l];
    const int pitch = kg.cols + 1, total = kg.rows * pitch;
    GridPoint *out = (GridPoint *)(g.points + g.points_off[blockIdx.y]);
    for (int q = first; q <= total; q += stride) {
        const int i = q / pitch, j = q - i * pitch;
        const float nan = __int_as_float(0x7fc00000);
        GridPoint o = {{nan, nan, nan}, {0.f, 0.f, 0.f}};
        if (q < total) {
            const int jj = j == kg.cols ? 0 : j;
            const float4 s1 = ldg_u(I.kf[l], (uint32_t)(i * kg.cols + jj));
            if (surfel_ok(kg, s1)) {
                // the products of kf_side, rounded the same
#pragma clang fp contract(off)
                const float2 e = ldg_u(kg.lut_row, (uint32_t)i << kg.lshift);
                const float2 ca = ldg_u(kg.lut_col, (uint32_t)jj << kg.lshift);
                const float3 uk = make_float3(e.x * ca.x, e.x * ca.y, e.y);
                o = GridPoint{{s1.w * uk.x, s1.w * uk.y, s1.w * uk.z}, {s1.x, s1.y, s1.z}};
            }
        }
        out[q] = o;
    }
}

// The scoring kernel for n_xy <= 5: blockIdx.x = a chunk of YB yaws (all
// NXY^2 translations of each), blockIdx.y = a tile of the level.  The scan
// pixels of the tile are loaded once per block and the rotated point and
// normal once per yaw; each candidate then costs a translation, the
// projection, the keyframe gather and the Omega test.  Inlier counts are wave
// ballots accumulated in wave-uniform registers.  The same FP32 pose values
// and operations as k_grid_score, so the scores are the same.  Consecutive
// blocks share a tile, so its keyframe image is fetched into L2 once for all
// chunks that run together.
// Bound by the vector instructions of a candidate, mostly the two arctangents.
// POINTS: the keyframe comes from the table of k_grid_points (levels 1 and up,
// where the batch's sizes and the candidates are such that it pays): no ray
// tables, no surfel test, one address: 227 us against 300 for 64 registrations
// x 324 candidates at level 2, with 7.7 us to fill the table.
template <int NXY, int YB, bool POINTS>
__global__ __launch_bounds__(kBlock) void k_grid_score_yaw(const Inst *__restrict__ insts,
                                                           const unsigned *__restrict__ tile_of, int K,
                                                           const ups_pose *__restrict__ base, GridArgs g,
                                                           int *__restrict__ scores) {
    constexpr int NT = NXY * NXY;
    __shared__ float Rs[YB][9];
    __shared__ float Ts[NT][3];
    __shared__ int wcount[kBlock / 64][YB * NT];
    const int chunk = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const unsigned of = tile_of[blockIdx.y];
    const int reg = (int)(of >> 16), tile = (int)(of & 0xFFFFu);
    const Inst &I = insts[reg];
    const int l = g.level;
    const DGeom sg = I.sg[l], kg = I.kg[l];
    const float4 *__restrict__ scan = I.scan[l];
    const float4 *__restrict__ kf = I.kf[l];
    const char *points = g.points + (POINTS ? g.points_off[reg] : 0);
    const int pitch = kg.cols + 1;
    const uint32_t nowhere = (uint32_t)(kg.rows * pitch);
    const int a0 = chunk * YB;
    const int ny = min(YB, g.n_yaw - a0);  // yaws of this chunk
    // the FP64 candidate poses of candidate_pose, split: rotation base.R Rz(yaw)
    // per yaw, translation base.R Gt + base.t per grid cell, each rounded to FP32
    if (tid < ny) {
        double R[9], t[3];
        candidate_pose(base[reg], g, (a0 + tid) * NT, R, t);
        for (int q = 0; q < 9; q++) Rs[tid][q] = (float)R[q];
    }
    if (tid >= 64 && tid < 64 + NT) {
        double R[9], t[3];
        candidate_pose(base[reg], g, tid - 64, R, t);
        for (int q = 0; q < 3; q++) Ts[tid - 64][q] = (float)t[q];
    }
    __syncthreads();
    int cnt[YB * NT];
#pragma unroll
    for (int c = 0; c < YB * NT; c++) cnt[c] = 0;
    const int npix = sg.rows * sg.cols;
    for (int k = 0; k < K; k++) {
        // the 64 pixels of a wavefront lie in one row (cols is a multiple of 64)
        const int pw = __builtin_amdgcn_readfirstlane(tile * kBlock * K + k * kBlock + (tid & ~63));
        if (pw >= npix) break;
        const int p = pw + lane;
        const int i = pw / sg.cols, j = p - i * sg.cols;
        float4 s2 = ldg_u(scan, (uint32_t)min(p, npix - 1));
        s2.w = p < npix ? s2.w : 0.f;
        const float2 e = lds_uniform(sg.lut_row, i << sg.lshift);
        const float2 ca = ldg_u(sg.lut_col, (uint32_t)j << sg.lshift);
        const bool sok = surfel_ok(sg, s2);
        if constexpr (POINTS)
            if (!__builtin_amdgcn_ballot_w64(sok)) continue;  // no surfel in this wavefront's pixels
        const float3 u = make_float3(e.x * ca.x, e.x * ca.y, e.y);
        const float3 p3 = make_float3(s2.w * u.x, s2.w * u.y, s2.w * u.z);
        const float3 n2 = make_float3(s2.x, s2.y, s2.z);
        auto yaws = [&](auto narrow) {
            // POINTS: a candidate's gather is tested after the next candidate's projection, which covers its latency
            float3 q_of[2], m_of[2];
            v4f v_of[2];
            v2f w_of[2];
            auto test = [&](int c) {
                const v4f v = v_of[c & 1];
                const v2f w = w_of[c & 1];
                const float3 d = sub3(q_of[c & 1], make_float3(v.x, v.y, v.z)), n1 = make_float3(v.w, w.x, w.y);
                const bool inl = (dot3(d, d) <= g.d_max2) & (dot3(m_of[c & 1], n1) >= g.cos_theta);
                cnt[c] += __builtin_popcountll(__builtin_amdgcn_ballot_w64(inl));
            };
#pragma unroll
            for (int y = 0; y < YB; y++) {
                if (y >= ny) break;
                Rt32 T;
#pragma unroll
                for (int q = 0; q < 9; q++) T.r[q] = Rs[y][q];
                const float3 rp = rotate(T, p3), m = rotate(T, n2);
#pragma unroll
                for (int t = 0; t < NT; t++) {
                    const float3 q = make_float3(rp.x + Ts[t][0], rp.y + Ts[t][1], rp.z + Ts[t][2]);
                    const int c = y * NT + t;
                    if constexpr (POINTS) {
                        uint32_t at;
                        const bool ok = project_at<decltype(narrow)::value>(kg, q, (uint32_t)pitch, at) & sok;
                        at = ok ? at : nowhere;
                        if constexpr (!decltype(narrow)::value) at = min(at, nowhere);
                        at = __umul24(at, 24u);
                        const UPS_AS_GLOBAL char *gp = (const UPS_AS_GLOBAL char *)points + at;
                        v_of[c & 1] = *(const UPS_AS_GLOBAL v4fa *)gp;
                        w_of[c & 1] = *(const UPS_AS_GLOBAL v2f *)(gp + 16);
                        q_of[c & 1] = q, m_of[c & 1] = m;
                        __builtin_amdgcn_sched_barrier(0);
                        if (c > 0) test(c - 1);
                    } else {
                        Gather G;
                        G.q = q, G.m = m;
                        int ki, kj;
                        const bool ok = project(kg, q, ki, kj) & sok;
                        ki = ok ? ki : 0;
                        kj = ok ? kj : 0;
                        const uint32_t idx = __umul24((uint32_t)ki, (uint32_t)kg.cols) + (uint32_t)kj;
                        G.kf_index = ok ? (int)idx : -1;
                        G.s1 = ldg_u(kf, idx);
                        G.e = ldg_u(kg.lut_row, (uint32_t)ki << kg.lshift);
                        G.a = ldg_u(kg.lut_col, (uint32_t)kj << kg.lshift);
                        bool inl;
                        float r;
                        float3 n1;
                        kf_side(kg, G, g.d_max2, g.cos_theta, inl, r, n1);
                        cnt[c] += __builtin_popcountll(__builtin_amdgcn_ballot_w64(inl));
                    }
                }
                if constexpr (POINTS)
                    if (y + 1 == YB || y + 1 >= ny) test((y + 1) * NT - 1);
            }
        };
        // a branch of its own for each kind of panorama, so that candidates follow each other without one
        if (POINTS && kg.narrow) yaws(std::true_type{});
        else yaws(std::false_type{});
    }
    if (lane == 0) {
#pragma unroll
        for (int c = 0; c < YB * NT; c++) wcount[wave][c] = cnt[c];
    }
    __syncthreads();
    if (tid < ny * NT) {
        int s = 0;
#pragma unroll
        for (int w = 0; w < kBlock / 64; w++) s += wcount[w][tid];
        if (s) atomicAdd(&scores[reg * g.C + a0 * NT + tid], s);
    }
}

// One block per registration: the candidate with the most inliers (the
// lowest index among equals) and its pose.
__global__ __launch_bounds__(256) void k_grid_best(int C, const int *__restrict__ scores,
                                                    const ups_pose *__restrict__ base, GridArgs g,
                                                    ups_pose *__restrict__ best, int *__restrict__ best_score) {
    __shared__ int bs[256], bc[256];
    const int k = blockIdx.x, tid = threadIdx.x;
    int s = -1, ci = 0;
    for (int c = tid; c < C; c += 256) {
        const int v = scores[k * C + c];
        if (v > s) {
            s = v;
            ci = c;
        }
    }
    bs[tid] = s;
    bc[tid] = ci;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (tid < w) {
            const int s2 = bs[tid + w], c2 = bc[tid + w];
            if (s2 > bs[tid] || (s2 == bs[tid] && c2 < bc[tid])) {
                bs[tid] = s2;
                bc[tid] = c2;
            }
        }
        __syncthreads();
    }
    if (tid == 0) {
        double R[9], t[3];
        candidate_pose(base[k], g, bc[0], R, t);
        for (int q = 0; q < 9; q++) best[k].R[q] = R[q];
        for (int q = 0; q < 3; q++) best[k].t[q] = t[q];
        if (best_score) best_score[k] = bs[0];
    }
}

size_t grid_points_bytes(const DGeom &kg) { return ((size_t)kg.rows * (kg.cols + 1) + 1) * sizeof(GridPoint); }

ups_status launch_grid_search(const Inst *insts, const int *tile_start_l, const unsigned *tile_of, int n, int K,
                              int tiles, const ups_pose *base, const GridArgs &g, int *scores, ups_pose *best,
                              int *best_score, hipStream_t s) {
    const int fill = g.points ? 32 : (std::min(g.C, 8192) + kBlock - 1) / kBlock;  // or only the scores to clear
    hipLaunchKernelGGL(k_grid_points, dim3(fill, n), dim3(kBlock), 0, s, insts, g, scores);
    UPS_CHECK_HIP(hipGetLastError());
    if (tiles > 0) {
        // yaws per block: as many as keep 36 or fewer candidates per block
#define UPS_GRID_CASE(NXY, YB)                                                                                        \
    case NXY: {                                                                                                       \
        const dim3 grid((g.n_yaw + YB - 1) / YB, tiles);                                                              \
        if (g.points)                                                                                                 \
            hipLaunchKernelGGL((k_grid_score_yaw<NXY, YB, true>), grid, dim3(kBlock), 0, s, insts, tile_of, K, base, g, scores); \
        else                                                                                                          \
            hipLaunchKernelGGL((k_grid_score_yaw<NXY, YB, false>), grid, dim3(kBlock), 0, s, insts, tile_of, K, base, g, scores); \
    } break;
        switch (g.n_xy) {
            UPS_GRID_CASE(1, 8)
            UPS_GRID_CASE(2, 4)
            UPS_GRID_CASE(3, 2)
            UPS_GRID_CASE(4, 1)
            UPS_GRID_CASE(5, 1)
            default:
                hipLaunchKernelGGL(k_grid_score, dim3(tiles, g.C), dim3(kBlock), 0, s, insts, tile_start_l, n, K,
                                   base, g, scores);
        }
#undef UPS_GRID_CASE
        UPS_CHECK_HIP(hipGetLastError());
    }
    hipLaunchKernelGGL(k_grid_best, dim3(n), dim3(256), 0, s, g.C, scores, base, g, best, best_score);
    UPS_CHECK_HIP(hipGetLastError());
    return UPS_OK;
}

}  // namespace ups
