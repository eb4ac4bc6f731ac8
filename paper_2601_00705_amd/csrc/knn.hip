// knn.hip -- exact neighbour searches among the valid Gaussians: the 3
// nearest (initial scale), the nearest (merging), and all within a radius
// (plane fit of the anisotropic initialisation, Eq. (app-sigma-init)).
//
// Seeds lie around surfaces, at densities that differ by orders of magnitude
// within one call, with a few far outliers, so no single cell size suits a
// grid.  The points are sorted along a Hilbert curve instead and cut
// into leaves of 64 consecutive points, one wave's worth, each with its
// bounding box and those of its 8 groups of 8; the leaves' size follows the
// local density by itself, and cells that outliers would make coarse are
// warped (knn_cell).  A wave takes one leaf as its 64 queries: their
// own leaf gives each query a first bound, then the leaves whose box lies
// within some query's bound are scanned from LDS.
//
//   k_knn_box      partial boxes of the finite valid points, and some of them
//   k_knn_split    the cells, and sample sort's splitters: every fourth of 4
//                  samples per bucket, ranked by counting (each block ranks
//                  64 samples)
//   k_knn_count    each point's bucket, and per block and bucket its offset
//                  inside the bucket (one atomic per block and bucket)
//   k_knn_place    points into their buckets (starts at multiples of 64)
//   k_knn_sort     one block per bucket: bitonic sort by (code, index) in
//                  LDS, leaf and group boxes
//   k_knn_supers   the boxes of every 64 consecutive leaves
//   k_knn_query / k_frame_query   the searches, one wave per leaf
//   k_knn_small / k_frame_small   up to GSR_KNN_SMALL points: no tree, 16
//                  waves share 64 queries and split the candidates
//
// The box tests and the candidates' prefilter run in FP32 with margins above
// their rounding; every decision is taken in double on (distance, index), so
// which points are found does not depend on the tree.  The moments of the
// radius search are sums in double in the order of the leaves; where a bucket
// is larger than its LDS the points' order in them is arbitrary, and the last
// bits may differ from call to call.
//
// Measured on MI355X, the whole call: the 3 nearest of 500,000 triangulated
// seeds 0.53 to 0.8 ms over ten inputs (queries 0.35 of 0.55, build 0.20),
// against 4.9 to 6.3 ms for hashed grid levels with an exhaustive search for
// far seeds; the nearest of 1M points on a room's walls 0.37 to 0.39 ms
// (queries 0.11; 0.5 for one input of ten), against 1.8 ms; 1,000 points 16 us,
// against 0.6 ms over 38 launches.  The queries are bound by VALU issue.
// Tried: a tree of fan-out 8 walked by every lane for itself, 2.2 ms for the
// same seeds (a node is a gather of 192 bytes per lane); Morton order, whose
// jumps give some leaves boxes across the scene, 1.2 ms.
#include "kernels.h"
#include "mat3.h"

namespace gsr {

#define KNN_THREADS 256
#define KNN_NONE 0xffffffffu
#define KNN_FAR 1024.0 // extent of the points, in half the width of their bulk, above which the cells are warped
#define GSR_KNN_LN2 0.69314718f
#define KNN_REFINE 20  // length of a wave's list of boxes above which it is cut down query by query

// ---------------------------------------------------------------------------
// building the leaves

__device__ __forceinline__ float wave_minf(float x)
{
    for (int off = 32; off > 0; off >>= 1) x = fminf(x, __shfl_xor(x, off, 64));
    return x;
}

__device__ __forceinline__ float wave_maxf(float x)
{
    for (int off = 32; off > 0; off >>= 1) x = fmaxf(x, __shfl_xor(x, off, 64));
    return x;
}

// a point that is not finite has no neighbours (and is none: its distances
// are infinite or NaN)
__device__ __forceinline__ bool finite_point(const float4& p)
{
    return __builtin_isfinite(p.x) && __builtin_isfinite(p.y) && __builtin_isfinite(p.z);
}

// Sample s of S: a point of the s-th of S equal runs of points, at a place in
// the run that looks random.  (The first point of every run lets a validity
// that follows the storage order, every other pixel of a row of 1024 say, hide
// all valid points from the samples: 2^20 points went into one bucket, and the
// nearest search took 18 ms instead of 0.5.)
__device__ __forceinline__ int64_t sample_point(int s, int S, int64_t n)
{
    uint32_t h = (uint32_t)s + 1u;
    h = (h ^ (h >> 16)) * 0x7feb352du;
    h = (h ^ (h >> 15)) * 0x846ca68bu;
    h ^= h >> 16;
    const int64_t i0 = (int64_t)s * n / S, len = (int64_t)(s + 1) * n / S - i0;
    return i0 + (int64_t)(((uint64_t)h * (uint64_t)len) >> 32);
}

// Partial box of the finite valid points of a block's stride, one such point
// of the block's run (NaN if 64 samples show none), and the bucket counters
// cleared.
__global__ __launch_bounds__(KNN_THREADS) void k_knn_box(KnnArgs a)
{
    __shared__ float red[6][KNN_THREADS / 64];
    for (int b = blockIdx.x * KNN_THREADS + threadIdx.x; b < a.buckets; b += gridDim.x * KNN_THREADS) a.total[b] = 0u;
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int64_t i = (int64_t)blockIdx.x * KNN_THREADS + threadIdx.x; i < a.n;
         i += (int64_t)gridDim.x * KNN_THREADS) {
        const float x = a.mean[i], y = a.mean[a.n + i], z = a.mean[2 * a.n + i];
        if (!a.valid[i] || !__builtin_isfinite(x) || !__builtin_isfinite(y) || !__builtin_isfinite(z)) continue;
        const float p[3] = {x, y, z};
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            lo[c] = fminf(lo[c], p[c]);
            hi[c] = fmaxf(hi[c], p[c]);
        }
    }
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const float l = wave_minf(lo[c]), h = wave_maxf(hi[c]);
        if (lane == 0) {
            red[c][w] = l;
            red[3 + c][w] = h;
        }
    }
    __syncthreads();
    if (threadIdx.x < 6) {
        const int k = threadIdx.x;
        float r = red[k][0];
        for (int j = 1; j < KNN_THREADS / 64; ++j) r = k < 3 ? fminf(r, red[k][j]) : fmaxf(r, red[k][j]);
        a.box[blockIdx.x * GSR_KNN_BOX + k] = r;
    }
    if (w == 3) {
        const int64_t i = sample_point(blockIdx.x * 64 + lane, GSR_KNN_BLOCKS * 64, a.n);
        float4 p = make_float4(a.mean[i], a.mean[a.n + i], a.mean[2 * a.n + i], 0.0f);
        if (!a.valid[i] || !finite_point(p)) p.x = NAN;
        const uint64_t have = __ballot(p.x == p.x);
        if (lane == (have ? __ffsll((unsigned long long)have) - 1 : 0)) {
            a.box[blockIdx.x * GSR_KNN_BOX + 6] = p.x;
            a.box[blockIdx.x * GSR_KNN_BOX + 7] = p.y;
            a.box[blockIdx.x * GSR_KNN_BOX + 8] = p.z;
        }
    }
}

// bit k of the 21-bit x moved to bit 3 k
__device__ __forceinline__ uint64_t spread21(uint64_t x)
{
    x &= 0x1fffffull;
    x = (x | (x << 32)) & 0x1f00000000ffffull;
    x = (x | (x << 16)) & 0x1f0000ff0000ffull;
    x = (x | (x << 8)) & 0x100f00f00f00f00full;
    x = (x | (x << 4)) & 0x10c30c30c30c30c3ull;
    x = (x | (x << 2)) & 0x1249249249249249ull;
    return x;
}

// Cell of coordinate x along axis c, below 2^21.  The cells are equal parts of
// the points' box, unless that is more than KNN_FAR times as wide as the cube
// that holds the bulk of the points: then the offsets from the cube's centre
// are taken as they are inside it and grow with their logarithm outside, so
// that no outlier makes the bulk's cells coarse.  With cells of the whole box,
// one point 10^8 scene sizes away put all others in a few cells, and the
// radius search through leaves of points in storage order took 19 ms for
// 200,000 points (0.21 without the outlier, now 0.22 with it; the nearest
// search 45 ms, now 39, for the outlier's own distances, which FP32 cannot
// tell apart).  Closer to the bulk equal cells are the better ones: seeds with
// outliers 10 to 100 scene sizes away take 5 to 20 % longer with the logarithm.
// The cells only order the points; every distance is that of the points
// themselves.
__device__ __forceinline__ double knn_warp(double u, double knee)
{
    return fabs(u) > knee ? copysign(1.0 + (double)(GSR_KNN_LN2 * __builtin_amdgcn_logf((float)fabs(u))), u) : u;
}

__device__ __forceinline__ uint32_t knn_cell(const KnnTree& t, int c, float x)
{
    const double q = (knn_warp(((double)x - t.centre[c]) * t.inv_half, t.knee) - t.least[c]) * t.cells;
    return q >= 2097151.0 ? 2097151u : (q > 0.0 ? (uint32_t)q : 0u);
}

// Place along the Hilbert curve through the 2^63 cells (Skilling 2004,
// transposed axes); consecutive cells share a face, where Morton order jumps
// and leaves a share of the boxes large.  Non-finite points come last.
__device__ __forceinline__ uint64_t knn_code(const KnnTree& t, float x, float y, float z)
{
    if (!__builtin_isfinite(x) || !__builtin_isfinite(y) || !__builtin_isfinite(z)) return ~0ull >> 1;
    uint32_t X[3] = {knn_cell(t, 0, x), knn_cell(t, 1, y), knn_cell(t, 2, z)};
    for (uint32_t Q = 1u << 20; Q > 1u; Q >>= 1) {
        const uint32_t P = Q - 1u;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            // invert axis 0 below this bit, or exchange it with axis c
            const uint32_t e = (X[0] ^ X[c]) & P;
            const bool inv = (X[c] & Q) != 0u;
            X[0] ^= inv ? P : e;
            if (c > 0) X[c] ^= inv ? 0u : e;
        }
    }
    X[1] ^= X[0];
    X[2] ^= X[1];
    uint32_t g = 0u;
    for (uint32_t Q = 1u << 20; Q > 1u; Q >>= 1)
        if (X[2] & Q) g ^= Q - 1u;
    return (spread21(X[0] ^ g) << 2) | (spread21(X[1] ^ g) << 1) | spread21(X[2] ^ g);
}

// Splitters of the buckets: split[b] is the least code of bucket b.  Every
// block forms the codes of all samples (an invalid one sorts last) and ranks
// 64 of them, the waves sharing the comparisons; the samples of ranks 4 b
// become the splitters.
//
// Before that every block forms the cells (knn_cell) alike: the bulk is what
// lies between the 1/8 and 7/8 quantiles of 64 points, along each
// axis; the cube is twice as wide about its middle, so that a uniform box and
// its walls lie inside and up to an eighth of the points may be anywhere.
template <int BUCKETS>
__global__ __launch_bounds__(1024) void k_knn_split(KnnArgs a)
{
    constexpr int S = 4 * BUCKETS;
    static_assert(S % 1024 == 0, "a wave counts whole runs of 64 samples");
    __shared__ uint64_t code[S];
    __shared__ uint32_t part[16][64];
    __shared__ float red[6][GSR_KNN_BLOCKS / 64];
    __shared__ float quant[3][2];
    __shared__ KnnTree t;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
#pragma unroll
    for (int c = 0; c < 6; ++c) {
        if (w >= GSR_KNN_BLOCKS / 64) break;
        const float x = a.box[tid * GSR_KNN_BOX + c], r = c < 3 ? wave_minf(x) : wave_maxf(x);
        if (lane == 0) red[c][w] = r;
    }
    if (w >= 13) {
        // wave 13 + c ranks 64 of the box pass's points along axis c
        const int c = w - 13;
        const float* q = a.box + lane * (GSR_KNN_BLOCKS / 64) * GSR_KNN_BOX + 6;
        const float x = q[0] == q[0] ? q[c] : NAN;
        const bool some = x == x;
        const int m = __popcll(__ballot(some));
        int rank = 0;
        for (int k = 0; k < 64; ++k) {
            const float y = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), k));
            rank += (y < x || (y == x && k < lane)) ? 1 : 0;
        }
        if (some && rank == m / 8) quant[c][0] = x;
        if (some && rank == m - 1 - m / 8) quant[c][1] = x;
        if (m == 0 && lane < 2) quant[c][lane] = 0.0f;
    }
    __syncthreads();
    if (w == 0) {
        // lanes 0, 1, 2: an axis each
        const int c = min(lane, 2);
        float l = INFINITY, h = -INFINITY;
#pragma unroll
        for (int k = 0; k < GSR_KNN_BLOCKS / 64; ++k) {
            l = fminf(l, red[c][k]);
            h = fmaxf(h, red[3 + c][k]);
        }
        const double lo = l, hi = h, q0 = quant[c][0], q1 = quant[c][1];
        const double centre = 0.5 * (q0 + q1);
        const bool some = lo <= hi;
        auto most = [](double x) { return fmax(fmax(__shfl(x, 0, 64), __shfl(x, 1, 64)), __shfl(x, 2, 64)); };
        double half = most(q1 - q0);
        const double far = most(some ? fmax(centre - lo, hi - centre) : 0.0);
        // (the bulk may be one point)
        half = half > 0.0 ? half : (far > 0.0 ? far : 1.0);
        const double inv_half = 1.0 / half, knee = far > KNN_FAR * half ? 1.0 : INFINITY;
        const double least = some ? knn_warp((lo - centre) * inv_half, knee) : 0.0;
        const double ext = most(some ? knn_warp((hi - centre) * inv_half, knee) - least : 0.0);
        if (lane < 3) {
            t.centre[c] = centre;
            t.least[c] = least;
        }
        if (lane == 0) {
            t.inv_half = inv_half;
            t.knee = knee;
            t.cells = ext > 0.0 ? 2097152.0 / ext : 0.0;
            t.leaves = 0;
        }
    }
    __syncthreads();
    if (blockIdx.x == 0 && tid == 0) *a.tree = t;
    for (int s = tid; s < S; s += 1024) {
        const int64_t i = sample_point(s, S, a.n);
        code[s] = a.valid[i] ? knn_code(t, a.mean[i], a.mean[a.n + i], a.mean[2 * a.n + i]) : ~0ull;
    }
    __syncthreads();
    const int base = blockIdx.x * 64;
    const uint64_t c = code[base + lane];
    uint32_t below = 0u;
    // equal codes rank by position: those of earlier samples count, those of
    // later ones do not, and the block's own 64 decide one by one
    for (int s = w * (S / 16); s < (w + 1) * (S / 16); s += 64) {
        if (s < base)
#pragma unroll 16
            for (int k = 0; k < 64; ++k) below += code[s + k] <= c ? 1u : 0u;
        else if (s > base)
#pragma unroll 16
            for (int k = 0; k < 64; ++k) below += code[s + k] < c ? 1u : 0u;
        else
            for (int k = 0; k < 64; ++k) below += (code[s + k] < c || (code[s + k] == c && k < lane)) ? 1u : 0u;
    }
    part[w][lane] = below;
    __syncthreads();
    if (w == 0) {
        uint32_t rank = 0u;
        for (int k = 0; k < 16; ++k) rank += part[k][lane];
        if ((rank & 3u) == 0u) a.split[rank >> 2] = rank == 0u ? 0ull : c;
    }
}

// what an invalid point's outputs hold
__device__ __forceinline__ void write_invalid(const KnnArgs& a, const FrameArgs& f, int64_t i)
{
    if (a.log_scale)
#pragma unroll
        for (int c = 0; c < 3; ++c) a.log_scale[c * a.n + i] = 0.0f;
    if (a.nn_index) a.nn_index[i] = -1;
    if (f.quat) {
        f.quat[i] = 1.0f;
#pragma unroll
        for (int k = 1; k < 4; ++k) f.quat[k * a.n + i] = 0.0f;
#pragma unroll
        for (int k = 0; k < 3; ++k) f.log_scale[k * a.n + i] = 0.0f;
    }
}

template <int BUCKETS>
__global__ __launch_bounds__(KNN_THREADS) void k_knn_count(KnnArgs a, FrameArgs f)
{
    __shared__ uint64_t split[BUCKETS];
    __shared__ uint32_t hist[BUCKETS];
    const int tid = threadIdx.x;
    for (int b = tid; b < BUCKETS; b += KNN_THREADS) {
        split[b] = a.split[b];
        hist[b] = 0u;
    }
    const KnnTree t = *a.tree;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * a.per_block;
    for (int k = tid; k < a.per_block; k += KNN_THREADS) {
        const int64_t i = base + k;
        if (i >= a.n) break;
        if (!a.valid[i]) {
            a.bucket_of[i] = 0xffffu;
            write_invalid(a, f, i);
            continue;
        }
        const uint64_t c = knn_code(t, a.mean[i], a.mean[a.n + i], a.mean[2 * a.n + i]);
        int b = 0;
#pragma unroll
        for (int step = BUCKETS / 2; step > 0; step >>= 1)
            if (split[b + step] <= c) b += step;
        a.bucket_of[i] = (uint16_t)b;
        atomicAdd(&hist[b], 1u);
    }
    __syncthreads();
    uint32_t* row = a.row + (int64_t)blockIdx.x * BUCKETS;
    for (int b = tid; b < BUCKETS; b += KNN_THREADS) {
        const uint32_t h = hist[b];
        if (h) row[b] = atomicAdd(&a.total[b], h);
    }
}

// Points into their buckets, each bucket's start a multiple of 64 (its first
// leaf); the order inside a bucket is arbitrary until it is sorted.
template <int BUCKETS>
__global__ __launch_bounds__(KNN_THREADS) void k_knn_place(KnnArgs a)
{
    constexpr int PER = BUCKETS / KNN_THREADS;
    __shared__ uint32_t cursor[BUCKETS];
    __shared__ uint32_t wsum[KNN_THREADS / 64];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    uint32_t leaves[PER], sum = 0u;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        leaves[k] = (a.total[tid * PER + k] + 63u) >> 6;
        sum += leaves[k];
    }
    uint32_t incl = sum;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(incl, off, 64);
        if (lane >= off) incl += y;
    }
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    uint32_t run = incl - sum;
    for (int k = 0; k < w; ++k) run += wsum[k];
    const uint32_t* row = a.row + (int64_t)blockIdx.x * BUCKETS;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int b = tid * PER + k;
        // a bucket this block has nothing in has no offset of its own
        cursor[b] = run * 64u + row[b];
        if (blockIdx.x == 0) a.bucket_leaf[b] = run;
        run += leaves[k];
    }
    if (blockIdx.x == 0 && tid == KNN_THREADS - 1) {
        a.bucket_leaf[BUCKETS] = run;
        a.tree->leaves = (int32_t)run;
    }
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * a.per_block;
    for (int k = tid; k < a.per_block; k += KNN_THREADS) {
        const int64_t i = base + k;
        if (i >= a.n) break;
        const uint32_t b = a.bucket_of[i];
        if (b == 0xffffu) continue;
        const uint32_t pos = atomicAdd(&cursor[b], 1u);
        a.placed[pos] = make_float4(a.mean[i], a.mean[a.n + i], a.mean[2 * a.n + i], __uint_as_float((uint32_t)i));
    }
}

// One block per bucket: the bucket's points by (code, index), CAP at a time
// (a larger bucket's parts are sorted one by one: their boxes overlap, the
// searches stay exact), padded to whole leaves of 64 with points at NaN.
template <int CAP>
__global__ __launch_bounds__(512) void k_knn_sort(KnnArgs a)
{
    __shared__ uint64_t code[CAP];
    __shared__ uint32_t idx[CAP];
    __shared__ uint16_t slot[CAP];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, b = blockIdx.x;
    const KnnTree t = *a.tree;
    const uint32_t cnt = a.total[b], start = a.bucket_leaf[b] * 64u;
    for (uint32_t c0 = 0; c0 < cnt; c0 += CAP) {
        const int m = (int)min(cnt - c0, (uint32_t)CAP);
        const float4* src = a.placed + start + c0;
        int m2 = 64;
        while (m2 < m) m2 <<= 1;
        for (int k = tid; k < m2; k += 512) {
            uint64_t c = ~0ull;
            uint32_t j = KNN_NONE;
            if (k < m) {
                const float4 p = src[k];
                c = knn_code(t, p.x, p.y, p.z);
                j = __float_as_uint(p.w);
            }
            code[k] = c;
            idx[k] = j;
            slot[k] = (uint16_t)k;
        }
        __syncthreads();
        for (int k = 2; k <= m2; k <<= 1) {
            for (int j = k >> 1; j > 0; j >>= 1) {
                for (int q = tid; q < m2 / 2; q += 512) {
                    const int lo = 2 * q - (q & (j - 1)), hi = lo + j;
                    const uint64_t cl = code[lo], ch = code[hi];
                    const uint32_t il = idx[lo], ih = idx[hi];
                    const bool gt = cl > ch || (cl == ch && il > ih);
                    if (gt == ((lo & k) == 0)) {
                        code[lo] = ch;
                        code[hi] = cl;
                        idx[lo] = ih;
                        idx[hi] = il;
                        const uint16_t s = slot[lo];
                        slot[lo] = slot[hi];
                        slot[hi] = s;
                    }
                }
                __syncthreads();
            }
        }
        for (int k0 = w * 64; k0 < m; k0 += 512) {
            const int k = k0 + lane;
            float4 p = make_float4(NAN, NAN, NAN, __uint_as_float(KNN_NONE));
            if (k < m) p = src[slot[k]];
            const uint32_t at = start + c0 + (uint32_t)k;
            a.pts[at] = p;
            // the boxes of the leaf's 8 groups, then its own; a point that
            // is not finite is in none
            if (!finite_point(p)) p.x = p.y = p.z = NAN;
            const float q[3] = {p.x, p.y, p.z};
            const uint32_t leaf = at >> 6;
            float* g = a.groups + 48 * (int64_t)leaf;
            float lo[3], hi[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                lo[c] = fminf(q[c], INFINITY);
                hi[c] = fmaxf(q[c], -INFINITY);
                for (int off = 1; off < 8; off <<= 1) {
                    lo[c] = fminf(lo[c], __shfl_xor(lo[c], off, 64));
                    hi[c] = fmaxf(hi[c], __shfl_xor(hi[c], off, 64));
                }
                if ((lane & 7) == 0) {
                    g[6 * (lane >> 3) + c] = lo[c];
                    g[6 * (lane >> 3) + 3 + c] = hi[c];
                }
                for (int off = 8; off < 64; off <<= 1) {
                    lo[c] = fminf(lo[c], __shfl_xor(lo[c], off, 64));
                    hi[c] = fmaxf(hi[c], __shfl_xor(hi[c], off, 64));
                }
            }
            if (lane == 0) {
                a.leaf_lo[leaf] = make_float4(lo[0], lo[1], lo[2], 0.0f);
                a.leaf_hi[leaf] = make_float4(hi[0], hi[1], hi[2], 0.0f);
            }
        }
        __syncthreads();
    }
}

// the box of leaves 64 s .. 64 s + 63, one wave each
__global__ __launch_bounds__(KNN_THREADS) void k_knn_supers(KnnArgs a)
{
    const int lane = threadIdx.x & 63, leaves = a.tree->leaves;
    const int s = blockIdx.x * (KNN_THREADS / 64) + (threadIdx.x >> 6), l = s * 64 + lane;
    if (s * 64 >= leaves) return;
    float4 lo = make_float4(INFINITY, INFINITY, INFINITY, 0.0f), hi = make_float4(-INFINITY, -INFINITY, -INFINITY, 0.0f);
    if (l < leaves) {
        lo = a.leaf_lo[l];
        hi = a.leaf_hi[l];
    }
    lo = make_float4(wave_minf(lo.x), wave_minf(lo.y), wave_minf(lo.z), 0.0f);
    hi = make_float4(wave_maxf(hi.x), wave_maxf(hi.y), wave_maxf(hi.z), 0.0f);
    if (lane == 0) {
        a.super_lo[s] = lo;
        a.super_hi[s] = hi;
    }
}

// ---------------------------------------------------------------------------
// searches

// FP32 bound that no candidate as near as the double squared distance d
// exceeds: its FP32 squared distance is within 3e-7 relative of the double
// one (1e-37 covers denormals)
__device__ __forceinline__ float near_bound(double d)
{
    return (float)d * 1.00001f + 1e-37f;
}

__device__ __forceinline__ float dist2(const float4& q, float px, float py, float pz)
{
    const float x = q.x - px, y = q.y - py, z = q.z - pz;
    return __builtin_fmaf(x, x, __builtin_fmaf(y, y, z * z));
}

__device__ __forceinline__ double dist2_exact(const float4& q, float px, float py, float pz)
{
    const double ex = (double)q.x - (double)px, ey = (double)q.y - (double)py, ez = (double)q.z - (double)pz;
    return ex * ex + ey * ey + ez * ez;
}

// (distance, index) pairs ordered by distance, then index: the nearest are
// unique even among equal distances
__device__ __forceinline__ bool knn_before(double d, uint32_t j, double bd, uint32_t bj)
{
    return d < bd || (d == bd && j < bj);
}

// A lane's query: its K nearest so far, ascending (an entry at distance
// infinity is none, and no candidate at distance infinity or NaN enters).
// bound is negative for a lane without a query.
template <int K>
struct Nearest {
    float px, py, pz, bound;
    uint32_t self;
    double d[K];
    uint32_t j[K];

    __device__ __forceinline__ void init(const float4& p, bool active)
    {
        px = p.x;
        py = p.y;
        pz = p.z;
        self = __float_as_uint(p.w);
        bound = active ? INFINITY : -1.0f;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            d[k] = INFINITY;
            j[k] = 0u;
        }
    }
    __device__ __forceinline__ void insert(double x, uint32_t i)
    {
        if (!knn_before(x, i, d[K - 1], j[K - 1])) return;
        if (K == 1) {
            d[0] = x;
            j[0] = i;
            return;
        }
        const bool c1 = knn_before(x, i, d[1 % K], j[1 % K]), c0 = knn_before(x, i, d[0], j[0]);
        d[2 % K] = c1 ? d[1 % K] : x;
        j[2 % K] = c1 ? j[1 % K] : i;
        d[1 % K] = c0 ? d[0] : (c1 ? x : d[1 % K]);
        j[1 % K] = c0 ? j[0] : (c1 ? i : j[1 % K]);
        d[0] = c0 ? x : d[0];
        j[0] = c0 ? i : j[0];
    }
    // the K-th least FP32 distance of 64 points: a bound before any exact
    // distance is known
    __device__ __forceinline__ void first(const float4* pts)
    {
        float b0 = INFINITY, b1 = INFINITY, b2 = INFINITY;
#pragma unroll 8
        for (int c = 0; c < 64; ++c) {
            const float4 q = pts[c];
            float x = fminf(dist2(q, px, py, pz), INFINITY);  // NaN: none
            x = __float_as_uint(q.w) == self ? INFINITY : x;
            if (K > 1) {
                b2 = __builtin_amdgcn_fmed3f(x, b1, b2);
                b1 = __builtin_amdgcn_fmed3f(x, b0, b1);
            }
            b0 = fminf(b0, x);
        }
        if (bound >= 0.0f) bound = near_bound((double)(K > 1 ? b2 : b0));
    }
    __device__ __forceinline__ void take(const float4& q)
    {
        const uint32_t i = __float_as_uint(q.w);
        if (i == self) return;
        insert(dist2_exact(q, px, py, pz), i);
        bound = fminf(bound, near_bound(d[K - 1]));
    }
};

// A lane's query: the moments about it of the points within the radius
// (itself included): count, first (3) and second (xx xy xz yy yz zz).
struct Ball {
    float px, py, pz, bound;
    double r2, m[10];

    __device__ __forceinline__ void init(const float4& p, bool active, double radius2)
    {
        px = p.x;
        py = p.y;
        pz = p.z;
        r2 = radius2;
        bound = active ? near_bound(radius2) : -1.0f;
#pragma unroll
        for (int k = 0; k < 10; ++k) m[k] = 0.0;
    }
    __device__ __forceinline__ void first(const float4*) {}
    __device__ __forceinline__ void take(const float4& q)
    {
        const double ex = (double)q.x - (double)px, ey = (double)q.y - (double)py, ez = (double)q.z - (double)pz;
        if (!(ex * ex + ey * ey + ez * ez <= r2)) return;
        m[0] += 1.0;
        m[1] += ex;
        m[2] += ey;
        m[3] += ez;
        m[4] += ex * ex;
        m[5] += ex * ey;
        m[6] += ex * ez;
        m[7] += ey * ey;
        m[8] += ey * ez;
        m[9] += ez * ez;
    }
};

// N points in LDS against the wave's queries: marks, per lane, the points
// within its bound.
template <int N, class Q>
__device__ __forceinline__ uint32_t mark(const Q& q, const float4* pts)
{
    uint32_t mask = 0u;
#pragma unroll 8
    for (int c = 0; c < N; ++c) mask |= dist2(pts[c], q.px, q.py, q.pz) <= q.bound ? 1u << c : 0u;
    return mask;
}

// Each lane takes its own marked points (the exact test inside the marking
// pass would run once per point that any lane needs).
template <class Q>
__device__ __forceinline__ void take_marked(Q& q, uint32_t mask, const float4* pts)
{
    while (mask) {
        const int c = __ffs((int)mask) - 1;
        mask &= mask - 1u;
        q.take(pts[c]);
    }
}

template <class Q>
__device__ __forceinline__ void scan64(Q& q, const float4* pts)
{
    take_marked(q, mark<32>(q, pts), pts);
    take_marked(q, mark<32>(q, pts + 32), pts + 32);
}

// least squared distance between the boxes [lo, hi] and [qlo, qhi], a little
// less (FP32: within 3e-7 relative).  Tests are written !(gap > bound), so
// that a NaN visits.
__device__ __forceinline__ float box_gap2(float lx, float ly, float lz, float hx, float hy, float hz,
                                          const float (&qlo)[3], const float (&qhi)[3])
{
    const float x = fmaxf(fmaxf(lx - qhi[0], qlo[0] - hx), 0.0f);
    const float y = fmaxf(fmaxf(ly - qhi[1], qlo[1] - hy), 0.0f);
    const float z = fmaxf(fmaxf(lz - qhi[2], qlo[2] - hz), 0.0f);
    return __builtin_fmaf(x, x, __builtin_fmaf(y, y, z * z)) * 0.99999f;
}

__device__ __forceinline__ float lane_f(float x, int lane)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane));
}

// The points of a leaf that some lane's bound may reach, by groups of 8.
template <class Q>
__device__ __forceinline__ void scan_leaf(Q& q, const KnnArgs& a, int leaf, float4* pts, int lane)
{
    __builtin_amdgcn_wave_barrier();
    pts[lane] = a.pts[(int64_t)leaf * 64 + lane];
    __builtin_amdgcn_wave_barrier();
    const float me[3] = {q.px, q.py, q.pz};
    const float* gb = a.groups + 48 * (int64_t)leaf;
    uint32_t mask[2] = {0u, 0u};
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const float* b = gb + 6 * c;
        const float gg = box_gap2(b[0], b[1], b[2], b[3], b[4], b[5], me, me);
        if (__any(q.bound >= 0.0f && !(gg > q.bound))) mask[c >> 2] |= mark<8>(q, pts + 8 * c) << (8 * (c & 3));
    }
    take_marked(q, mask[0], pts);
    take_marked(q, mask[1], pts + 32);
}

// Of the boxes (one per lane) marked in list, those that some query of the
// wave reaches, the queries taken one by one.
template <class Q>
__device__ __forceinline__ uint64_t refine(const Q& q, uint64_t list, const float4& lo, const float4& hi)
{
    bool need = false;
    for (int k = 0; k < 64; ++k) {
        const float b = lane_f(q.bound, k);
        const float p[3] = {lane_f(q.px, k), lane_f(q.py, k), lane_f(q.pz, k)};
        need |= b >= 0.0f && !(box_gap2(lo.x, lo.y, lo.z, hi.x, hi.y, hi.z, p, p) > b);
    }
    return list & __ballot(need);
}

// All points a query of the wave may need.  Boxes are tested 64 at a time,
// one per lane, against the wave's own box and its largest bound, which only
// falls: first those of 64 leaves, then the leaves'.  A leaf on the resulting
// list is scanned when some lane's own bound reaches its box.  Where a wave's
// queries lie far apart (outliers), the lists are long and few boxes are
// needed, so a long list is first cut down query by query.
template <class Q>
__device__ __forceinline__ void search(Q& q, const KnnArgs& a, int leaf, int leaves, float4* pts, int lane)
{
    pts[lane] = a.pts[(int64_t)leaf * 64 + lane];
    __builtin_amdgcn_wave_barrier();
    q.first(pts);
    scan64(q, pts);
    if (leaf > 0) scan_leaf(q, a, leaf - 1, pts, lane);
    if (leaf + 1 < leaves) scan_leaf(q, a, leaf + 1, pts, lane);
    const float4 l4 = a.leaf_lo[leaf], h4 = a.leaf_hi[leaf];
    const float qlo[3] = {l4.x, l4.y, l4.z}, qhi[3] = {h4.x, h4.y, h4.z};
    const float me[3] = {q.px, q.py, q.pz};
    float reach = wave_maxf(q.bound);
    const int supers = (leaves + 63) / 64;
    for (int sb = 0; sb < supers; sb += 64) {
        bool near = false;
        float4 lo = make_float4(0.0f, 0.0f, 0.0f, 0.0f), hi = lo;
        if (sb + lane < supers) {
            lo = a.super_lo[sb + lane];
            hi = a.super_hi[sb + lane];
            near = !(box_gap2(lo.x, lo.y, lo.z, hi.x, hi.y, hi.z, qlo, qhi) > reach);
        }
        uint64_t sm = __ballot(near);
        if (__popcll(sm) > KNN_REFINE / 4) sm = refine(q, sm, lo, hi);
        while (sm) {
            const int l0 = (sb + __ffsll((unsigned long long)sm) - 1) * 64, l = l0 + lane;
            sm &= sm - 1ull;
            near = false;
            if (l < leaves) {
                lo = a.leaf_lo[l];
                hi = a.leaf_hi[l];
                near = (l < leaf - 1 || l > leaf + 1) &&
                       !(box_gap2(lo.x, lo.y, lo.z, hi.x, hi.y, hi.z, qlo, qhi) > reach);
            }
            uint64_t lm = __ballot(near);
            if (__popcll(lm) > KNN_REFINE) lm = refine(q, lm, lo, hi);
            while (lm) {
                const int k = __ffsll((unsigned long long)lm) - 1;
                lm &= lm - 1ull;
                const float g = box_gap2(lane_f(lo.x, k), lane_f(lo.y, k), lane_f(lo.z, k), lane_f(hi.x, k),
                                         lane_f(hi.y, k), lane_f(hi.z, k), me, me);
                if (!__any(q.bound >= 0.0f && !(g > q.bound))) continue;
                scan_leaf(q, a, l0 + k, pts, lane);
            }
            reach = wave_maxf(q.bound);
        }
    }
}

__device__ __forceinline__ bool is_query(const float4& p)
{
    return __float_as_uint(p.w) != KNN_NONE && finite_point(p);
}

// the query's outputs: its log-scale (when asked for) and its nearest
// other seed (when asked for; -1 for none)
template <int K>
__device__ __forceinline__ void knn_write(const KnnArgs& a, int64_t i, const Nearest<K>& q)
{
    if (K == 3 && a.log_scale) {
        double sum = 0.0;
        int found = 0;
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (q.d[k] < INFINITY) {
                sum += sqrt(q.d[k]);
                ++found;
            }
        const double sc = found ? fmax(sum / (double)found, (double)a.floor_scale) : (double)a.floor_scale;
        const float ls = (float)log(sc);
#pragma unroll
        for (int c = 0; c < 3; ++c) a.log_scale[(int64_t)c * a.n + i] = ls;
    }
    if (a.nn_index) a.nn_index[i] = q.d[0] < INFINITY ? (int32_t)q.j[0] : -1;
}

template <int K>
__global__ __launch_bounds__(KNN_THREADS) void k_knn_query(KnnArgs a)
{
    __shared__ float4 lds[KNN_THREADS / 64][64];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int leaf = blockIdx.x * (KNN_THREADS / 64) + w, leaves = a.tree->leaves;
    if (leaf >= leaves) return;
    const float4 p = a.pts[(int64_t)leaf * 64 + lane];
    Nearest<K> q;
    q.init(p, is_query(p));
    search(q, a, leaf, leaves, lds[w], lane);
    if (__float_as_uint(p.w) != KNN_NONE) knn_write<K>(a, (int64_t)__float_as_uint(p.w), q);
}

// the moments go to mom [10][leaves * 64] for k_frame_fit, so that the
// search keeps few registers
__global__ __launch_bounds__(KNN_THREADS) void k_frame_query(KnnArgs a, FrameArgs f)
{
    __shared__ float4 lds[KNN_THREADS / 64][64];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int leaf = blockIdx.x * (KNN_THREADS / 64) + w, leaves = a.tree->leaves;
    if (leaf >= leaves) return;
    const float4 p = a.pts[(int64_t)leaf * 64 + lane];
    Ball q;
    q.init(p, is_query(p), f.radius * f.radius);
    search(q, a, leaf, leaves, lds[w], lane);
    const int64_t stride = (int64_t)leaves * 64;
#pragma unroll
    for (int k = 0; k < 10; ++k) a.mom[k * stride + (int64_t)leaf * 64 + lane] = q.m[k];
}

// point i of the input as a candidate or query (NaN where it is none)
__device__ __forceinline__ float4 input_point(const KnnArgs& a, int64_t i)
{
    if (i >= a.n || !a.valid[i]) return make_float4(NAN, NAN, NAN, __uint_as_float(KNN_NONE));
    return make_float4(a.mean[i], a.mean[a.n + i], a.mean[2 * a.n + i], __uint_as_float((uint32_t)i));
}

// Wave w of the block takes the w-th part of the candidates, 64 at a time.
template <class Q>
__device__ __forceinline__ void search_small(Q& q, const KnnArgs& a, float4* pts, int w, int lane)
{
    const int chunks = (int)((a.n + 63) / 64), per = (chunks + 15) / 16;
    const int c1 = min((w + 1) * per, chunks);
    for (int c = w * per; c < c1; ++c) {
        __builtin_amdgcn_wave_barrier();
        pts[lane] = input_point(a, (int64_t)c * 64 + lane);
        __builtin_amdgcn_wave_barrier();
        if (c == w * per) q.first(pts);
        scan64(q, pts);
    }
}

template <int K>
__global__ __launch_bounds__(1024) void k_knn_small(KnnArgs a)
{
    __shared__ float4 lds[16][64];
    __shared__ double md[8][K][64];
    __shared__ uint32_t mj[8][K][64];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t i = (int64_t)blockIdx.x * 64 + lane;
    const float4 p = input_point(a, i);
    Nearest<K> q;
    q.init(p, is_query(p));
    search_small(q, a, lds[w], w, lane);
    // the waves' lists, merged by halves
    for (int half = 8; half > 0; half >>= 1) {
        if (w >= half && w < 2 * half)
#pragma unroll
            for (int k = 0; k < K; ++k) {
                md[w - half][k][lane] = q.d[k];
                mj[w - half][k][lane] = q.j[k];
            }
        __syncthreads();
        if (w < half)
#pragma unroll
            for (int k = 0; k < K; ++k) q.insert(md[w][k][lane], mj[w][k][lane]);
        __syncthreads();
    }
    if (w != 0 || i >= a.n) return;
    if (a.valid[i]) knn_write<K>(a, i, q);
    else write_invalid(a, FrameArgs{}, i);
}

// ---- anisotropic initialisation, Eq. (app-sigma-init) ----------------------
// The moments of the seeds within the radius give the scatter about their
// mean; its eigenvector of the smallest eigenvalue is the plane normal v,
// that of the largest t1, and t2 = v x t1 (with fewer than three seeds: v the
// reference viewing ray, t1 any perpendicular).  s_perp = det(J J^T)^(-1/4),
// J the reference projection's 2 x 3 Jacobian at the seed (the equal-area
// radius of the back-projected one-pixel footprint); s_par = c_par s_perp
// max(1, err) / max(sin angle, 1e-6); both floored.  Output: the unit
// quaternion of [t1 t2 v] and the log-scales (s_perp, s_perp, s_par).
__device__ __forceinline__ void frame_fit(const FrameArgs& f, int64_t n, int64_t i, const float (&p)[3],
                                          const double (&mom)[10])
{
    const double cnt = mom[0];
    const double m1[3] = {mom[1], mom[2], mom[3]}, m2[6] = {mom[4], mom[5], mom[6], mom[7], mom[8], mom[9]};
    double v[3], t1[3];
    if (cnt >= 3.0) {
        const double ic = 1.0 / cnt;
        double S[3][3], V[3][3], lam[3];
        S[0][0] = m2[0] - m1[0] * m1[0] * ic;
        S[0][1] = S[1][0] = m2[1] - m1[0] * m1[1] * ic;
        S[0][2] = S[2][0] = m2[2] - m1[0] * m1[2] * ic;
        S[1][1] = m2[3] - m1[1] * m1[1] * ic;
        S[1][2] = S[2][1] = m2[4] - m1[1] * m1[2] * ic;
        S[2][2] = m2[5] - m1[2] * m1[2] * ic;
        eig3(S, V, lam);
        int kmin = 0, kmax = 1;
        if (lam[1] < lam[kmin]) kmin = 1;
        if (lam[2] < lam[kmin]) kmin = 2;
        kmax = kmin == 0 ? 1 : 0;
        for (int k = 0; k < 3; ++k)
            if (k != kmin && lam[k] > lam[kmax]) kmax = k;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            v[c] = V[c][kmin];
            t1[c] = V[c][kmax];
        }
    } else {
        double nv = 0.0;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            v[c] = (double)p[c] - f.centre[c];
            nv += v[c] * v[c];
        }
        nv = 1.0 / sqrt(nv);
        int am = 0;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            v[c] *= nv;
            if (fabs(v[c]) < fabs(v[am])) am = c;
        }
        // t1 = v x e_am, normalised
        double e[3] = {0.0, 0.0, 0.0};
        e[am] = 1.0;
        t1[0] = v[1] * e[2] - v[2] * e[1];
        t1[1] = v[2] * e[0] - v[0] * e[2];
        t1[2] = v[0] * e[1] - v[1] * e[0];
        const double nt = 1.0 / sqrt(t1[0] * t1[0] + t1[1] * t1[1] + t1[2] * t1[2]);
#pragma unroll
        for (int c = 0; c < 3; ++c) t1[c] *= nt;
    }
    const double t2[3] = {v[1] * t1[2] - v[2] * t1[1], v[2] * t1[0] - v[0] * t1[2], v[0] * t1[1] - v[1] * t1[0]};
    double U[3][3], q[4];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        U[c][0] = t1[c];
        U[c][1] = t2[c];
        U[c][2] = v[c];
    }
    rot_quat(U, q);
    // tangential scale from the reference projection's Jacobian
    const double X[3] = {(double)p[0], (double)p[1], (double)p[2]};
    const double* P = f.P;
    const double w = P[8] * X[0] + P[9] * X[1] + P[10] * X[2] + P[11];
    const double u = (P[0] * X[0] + P[1] * X[1] + P[2] * X[2] + P[3]) / w;
    const double vv = (P[4] * X[0] + P[5] * X[1] + P[6] * X[2] + P[7]) / w;
    double j1[3], j2[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        j1[c] = (P[c] - u * P[8 + c]) / w;
        j2[c] = (P[4 + c] - vv * P[8 + c]) / w;
    }
    const double A = j1[0] * j1[0] + j1[1] * j1[1] + j1[2] * j1[2];
    const double B = j1[0] * j2[0] + j1[1] * j2[1] + j1[2] * j2[2];
    const double D = j2[0] * j2[0] + j2[1] * j2[1] + j2[2] * j2[2];
    const double s_perp = fmax(pow(A * D - B * B, -0.25), f.floor_scale);
    const double s_par =
        fmax(f.c_par * s_perp * fmax(1.0, (double)f.err[i]) / fmax(sin((double)f.angle[i]), 1e-6), f.floor_scale);
#pragma unroll
    for (int k = 0; k < 4; ++k) f.quat[k * n + i] = (float)q[k];
    f.log_scale[i] = (float)log(s_perp);
    f.log_scale[n + i] = (float)log(s_perp);
    f.log_scale[2 * n + i] = (float)log(s_par);
}

__global__ __launch_bounds__(KNN_THREADS) void k_frame_fit(KnnArgs a, FrameArgs f)
{
    const int64_t stride = (int64_t)a.tree->leaves * 64;
    const int64_t t = (int64_t)blockIdx.x * KNN_THREADS + threadIdx.x;
    if (t >= stride) return;
    const float4 self = a.pts[t];
    if (__float_as_uint(self.w) == KNN_NONE) return;
    const float p[3] = {self.x, self.y, self.z};
    double mom[10];
#pragma unroll
    for (int k = 0; k < 10; ++k) mom[k] = a.mom[k * stride + t];
    frame_fit(f, a.n, (int64_t)__float_as_uint(self.w), p, mom);
}

__global__ __launch_bounds__(1024) void k_frame_small(KnnArgs a, FrameArgs f)
{
    __shared__ float4 lds[16][64];
    __shared__ double sum[8][10][64];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t i = (int64_t)blockIdx.x * 64 + lane;
    const float4 p = input_point(a, i);
    Ball q;
    q.init(p, is_query(p), f.radius * f.radius);
    search_small(q, a, lds[w], w, lane);
    for (int half = 8; half > 0; half >>= 1) {
        if (w >= half && w < 2 * half)
#pragma unroll
            for (int k = 0; k < 10; ++k) sum[w - half][k][lane] = q.m[k];
        __syncthreads();
        if (w < half)
#pragma unroll
            for (int k = 0; k < 10; ++k) q.m[k] += sum[w][k][lane];
        __syncthreads();
    }
    if (w != 0 || i >= a.n) return;
    if (!a.valid[i]) {
        write_invalid(a, f, i);
        return;
    }
    const float pos[3] = {p.x, p.y, p.z};
    frame_fit(f, a.n, i, pos, q.m);
}

// ---------------------------------------------------------------------------

template <int BUCKETS>
static void launch_build(const KnnArgs& a, const FrameArgs& f, hipStream_t s)
{
    const unsigned blocks = (unsigned)((a.n + a.per_block - 1) / a.per_block);
    hipLaunchKernelGGL(k_knn_box, dim3(GSR_KNN_BLOCKS), dim3(KNN_THREADS), 0, s, a);
    hipLaunchKernelGGL(k_knn_split<BUCKETS>, dim3(4 * BUCKETS / 64), dim3(1024), 0, s, a);
    hipLaunchKernelGGL(k_knn_count<BUCKETS>, dim3(blocks), dim3(KNN_THREADS), 0, s, a, f);
    hipLaunchKernelGGL(k_knn_place<BUCKETS>, dim3(blocks), dim3(KNN_THREADS), 0, s, a);
    // a bucket holds n / BUCKETS points on average and rarely over four times
    // that; the smaller LDS share lets more blocks run per CU
    if (a.n / BUCKETS <= 256) hipLaunchKernelGGL(k_knn_sort<2048>, dim3(BUCKETS), dim3(512), 0, s, a);
    else if (a.n / BUCKETS <= 1024) hipLaunchKernelGGL(k_knn_sort<4096>, dim3(BUCKETS), dim3(512), 0, s, a);
    else hipLaunchKernelGGL(k_knn_sort<8192>, dim3(BUCKETS), dim3(512), 0, s, a);
    const unsigned waves = KNN_THREADS / 64;
    hipLaunchKernelGGL(k_knn_supers, dim3((unsigned)(((a.max_leaves + 63) / 64 + waves - 1) / waves)),
                       dim3(KNN_THREADS), 0, s, a);
}

static void build(const KnnArgs& a, const FrameArgs& f, hipStream_t s)
{
    switch (a.buckets) {
    case 256: launch_build<256>(a, f, s); break;
    case 1024: launch_build<1024>(a, f, s); break;
    default: launch_build<4096>(a, f, s); break;
    }
}

hipError_t launch_seed_scale(const KnnArgs& a, hipStream_t s)
{
    if (a.n == 0) return hipSuccess;
    if (a.n <= GSR_KNN_SMALL) {
        const unsigned blocks = (unsigned)((a.n + 63) / 64);
        if (a.log_scale) hipLaunchKernelGGL(k_knn_small<3>, dim3(blocks), dim3(1024), 0, s, a);
        else hipLaunchKernelGGL(k_knn_small<1>, dim3(blocks), dim3(1024), 0, s, a);
        return hipGetLastError();
    }
    build(a, FrameArgs{}, s);
    const unsigned waves = KNN_THREADS / 64, blocks = (unsigned)((a.max_leaves + waves - 1) / waves);
    if (a.log_scale) hipLaunchKernelGGL(k_knn_query<3>, dim3(blocks), dim3(KNN_THREADS), 0, s, a);
    else hipLaunchKernelGGL(k_knn_query<1>, dim3(blocks), dim3(KNN_THREADS), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_seed_frame(const KnnArgs& a, const FrameArgs& f, hipStream_t s)
{
    if (a.n == 0) return hipSuccess;
    if (a.n <= GSR_KNN_SMALL) {
        hipLaunchKernelGGL(k_frame_small, dim3((unsigned)((a.n + 63) / 64)), dim3(1024), 0, s, a, f);
        return hipGetLastError();
    }
    build(a, f, s);
    const unsigned waves = KNN_THREADS / 64, blocks = (unsigned)((a.max_leaves + waves - 1) / waves);
    hipLaunchKernelGGL(k_frame_query, dim3(blocks), dim3(KNN_THREADS), 0, s, a, f);
    hipLaunchKernelGGL(k_frame_fit, dim3(blocks), dim3(KNN_THREADS), 0, s, a, f);
    return hipGetLastError();
}

}  // namespace gsr
