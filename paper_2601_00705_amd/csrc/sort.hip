// sort.hip -- per-tile ordering of the emitted pairs, and the tiles' order.
//
// k_seg_sort   one block per tile (longest first): sorts the segment's unique
//              64-bit keys (depth bits << 32 | Gaussian index) ascending and
//              writes the final pairs: key (tile << 32 | depth bits), value
//              slot = view * n + index.
// k_order_place  processing order of the tiles: descending pair count,
//              bucketed by floor(log2(count)), for the segment sort and
//              compositing (few tiles are placed where their ranges are formed).
//
// A list is placed, not ranked digit by digit: a histogram of its depth bits
// over GSR_SEG_COARSE linear bins gives its depth distribution, every coarse
// bin of c keys is cut into c fine bins, and a key's position is its fine
// bin's start (an LDS atomic and a scan) plus the smaller keys of its bin,
// one or two on average whatever surfaces the depths lie on.  The keys are
// unique, so no step needs to be stable.  Lists of more than 8 keys a thread
// are first spread over runs of whole coarse bins (one pass through memory)
// and these sorted one after another with the bins already known.  Where
// depths coincide (a key has more than GSR_SEG_CROWDED bin-mates on average)
// the keys are sorted by their digits instead; a long list that crowds one
// coarse bin is cut again within that bin (sort_segment).
//
// The kernel is bound by LDS traffic and, for the long lists, by the passes
// over memory (20 bytes a key, 24 more for a long list's three reads less
// what the caches hold).  It replaced four or more 8-bit digit passes of
// eight ballots each over three classes of lists on two streams: 4.8M pairs
// in lists of 290 (five 1200x680 views of 500k Gaussians) 431 -> 78 us, 41M
// pairs in lists of 1500 to 18500 (ten such views of 1M) 750 -> 380 us, 265M
// pairs in lists of 2800 to 48600 (36 views of 3M) about 5300 -> 2650 us,
// 194k pairs in lists of 150 76 -> 8 us.  Measured and worse: 512 threads and
// 4096 keys a block, 4 keys a thread (more, smaller runs of the long lists:
// 4930 us), 2048 coarse bins (2870 us), pairs written from the threads that
// ranked them instead of in order through LDS (3750 us).
//
// Lists that crowd a bin, 64 of 30,000 keys (spread depths 159 us): a wall
// with one near outlier 219 us, one depth for all 203, two walls and an outlier
// 209; as sorted chunks merged pairwise they took 517, 628 and 658, in the
// digit passes 285, 247 and 535.  One list of 200,000 keys at 419 depths and an
// outlier: 1.40 ms (spread 1.05); cut again by the key's bits instead of depth
// bits * n + index, which leaves equal depths to the digits, 2.62.
#include "kernels.h"

namespace gsr {

// lanes of the wave (valid ones) holding the same 8-bit digit as this lane:
// for every bit, keep the ballot of that bit where this lane's bit is 1 and
// its complement where it is 0, i.e. m &= ~(ballot ^ sign-extended bit), on
// the two 32-bit halves
__device__ __forceinline__ unsigned long long match_digit(uint32_t d, bool valid)
{
    const unsigned long long v = __ballot(valid);
    uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const uint32_t s = (uint32_t)((int32_t)(d << (31 - b)) >> 31);  // 0 or ~0
        const unsigned long long bb = __ballot(s != 0u);
        lo &= ~((uint32_t)bb ^ s);
        hi &= ~((uint32_t)(bb >> 32) ^ s);
    }
    return ((unsigned long long)hi << 32) | lo;
}

template <int WAVES>
struct SegLds {
    static constexpr int THREADS = WAVES * 64;
    static constexpr int ITEMS = THREADS * GSR_SEG_PER_THREAD;  // keys sorted at once
    static_assert(GSR_SEG_COARSE % THREADS == 0, "a thread scans the same number of coarse bins");
    // the digit scans of the radix sort give one thread to each digit
    static_assert(THREADS >= 256, "a sorting block needs at least 256 threads");
    union {
        unsigned long long sk[ITEMS];        // keys in fine-bin (digit) order
        uint32_t coarse[GSR_SEG_COARSE + 1]; // coarse counts, then starts (before sk is filled)
    };
    union {
        uint32_t fine[ITEMS + 1];            // fine counts, then starts
        uint32_t wcnt[WAVES][256];           // radix sort: per-wave digit counters, then wave offsets
    };
    uint32_t starts[GSR_SEG_COARSE + 1];     // a long list's coarse bins: counts, then starts
    uint32_t wsum[WAVES], wsum2[WAVES];
    uint32_t red[2][WAVES];
    unsigned long long red64[2][WAVES];
};

// Stable ranking of the block's items by digit (key >> shift) & 255.  Item
// (r, lane) of wave w has index w * R * 64 + r * 64 + lane; on return
// pos[r] is its position in digit order (digit-major, index order within a
// digit) or ~0 for an item past m.
template <int WAVES, int MAXR>
__device__ __forceinline__ void rank_items(const unsigned long long* key, int R, int m, int shift, uint32_t* pos,
                                           SegLds<WAVES>& L)
{
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    for (int k = tid; k < WAVES * 256; k += WAVES * 64) (&L.wcnt[0][0])[k] = 0u;
    __syncthreads();
    uint32_t dig[MAXR];
#pragma unroll
    for (int r = 0; r < MAXR; ++r) {
        if (r >= R) break;
        const int li = w * R * 64 + r * 64 + lane;
        const bool valid = li < m;
        const uint32_t d = valid ? (uint32_t)(key[r] >> shift) & 255u : 0u;
        const unsigned long long mk = match_digit(d, valid);
        // set bits of mk in the lanes below this one
        const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(mk >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mk, 0u));
        const uint32_t start = valid ? L.wcnt[w][d] : 0u;
        // every lane has read its counter before a leader updates it
        __builtin_amdgcn_wave_barrier();
        pos[r] = start + below;
        dig[r] = valid ? d : 256u;
        if (valid && below == 0u) L.wcnt[w][d] = start + (uint32_t)__popcll(mk);
    }
    __syncthreads();
    // threads 0..255 (one per digit): wave offsets inside the digit and the
    // block's digit starts
    uint32_t tot = 0, incl = 0;
    if (tid < 256) {
        for (int k = 0; k < WAVES; ++k) tot += L.wcnt[k][tid];
        incl = tot;
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = __shfl_up(incl, off, 64);
            if (lane >= off) incl += y;
        }
        if (lane == 63) L.wsum[w] = incl;
    }
    __syncthreads();
    if (tid < 256) {
        uint32_t ds = incl - tot;
        for (int k = 0; k < w; ++k) ds += L.wsum[k];
        for (int k = 0; k < WAVES; ++k) {
            const uint32_t c = L.wcnt[k][tid];
            L.wcnt[k][tid] = ds;
            ds += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < MAXR; ++r) {
        if (r >= R) break;
        pos[r] = dig[r] < 256u ? L.wcnt[w][dig[r]] + pos[r] : 0xffffffffu;
    }
}

__device__ __forceinline__ void write_pair(const SegArgs& a, uint32_t at, unsigned long long k, unsigned long long tile,
                                           uint32_t vbase)
{
    a.keys[at] = (tile << 32) | (k >> 32);
    a.vals[at] = vbase + (uint32_t)k;
}

// Stable LSD radix sort of the block's keys (item (r, lane) of wave w at
// index w * R * 64 + r * 64 + lane) by the digits in which they differ.
template <int WAVES>
__device__ __forceinline__ void radix_sort(unsigned long long (&key)[GSR_SEG_PER_THREAD], int m, SegLds<WAVES>& L)
{
    constexpr int THREADS = WAVES * 64, MAXR = GSR_SEG_PER_THREAD;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int R = (m + THREADS - 1) / THREADS;
    uint32_t pos[MAXR];
    unsigned long long o = 0ull, an = ~0ull;
#pragma unroll
    for (int r = 0; r < MAXR; ++r) {
        if (r >= R) break;
        if (w * R * 64 + r * 64 + lane < m) {
            o |= key[r];
            an &= key[r];
        }
    }
    for (int off = 32; off > 0; off >>= 1) {
        o |= __shfl_xor(o, off, 64);
        an &= __shfl_xor(an, off, 64);
    }
    if (lane == 0) {
        L.red64[0][w] = o;
        L.red64[1][w] = an;
    }
    __syncthreads();
    unsigned long long bor = 0ull, band = ~0ull;
    for (int k = 0; k < WAVES; ++k) {
        bor |= L.red64[0][k];
        band &= L.red64[1][k];
    }
    const unsigned long long diff = bor ^ band;
    for (int d = 0; d < 8; ++d) {
        if (((diff >> (8 * d)) & 255ull) == 0ull) continue;
        __syncthreads();
        rank_items<WAVES, MAXR>(key, R, m, 8 * d, pos, L);
#pragma unroll
        for (int r = 0; r < MAXR; ++r) {
            if (r >= R) break;
            if (pos[r] != 0xffffffffu) L.sk[pos[r]] = key[r];
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < MAXR; ++r) {
            if (r >= R) break;
            const int li = w * R * 64 + r * 64 + lane;
            if (li < m) key[r] = L.sk[li];
        }
    }
    __syncthreads();
}

// The linear map of depth bits (offset from the least, at most range) to
// GSR_SEG_COARSE coarse bins: the product's high word is the bin, its low
// word the place inside the bin.  mult = floor(bins 2^32 / (range + 1)), and
// range / (range + 1) <= 1 - 2^-32, so the bin is below GSR_SEG_COARSE
// whichever way the quotient rounds.
__device__ __forceinline__ unsigned long long coarse_mult(uint32_t range)
{
    return (unsigned long long)((double)GSR_SEG_COARSE * 4294967296.0 / ((double)range + 1.0));
}

// least and largest depth bits over the block
template <int WAVES>
__device__ __forceinline__ void block_min_max(uint32_t& lo, uint32_t& hi, SegLds<WAVES>& L)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int off = 32; off > 0; off >>= 1) {
        lo = min(lo, (uint32_t)__shfl_xor((int)lo, off, 64));
        hi = max(hi, (uint32_t)__shfl_xor((int)hi, off, 64));
    }
    if (lane == 0) {
        L.red[0][w] = lo;
        L.red[1][w] = hi;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < WAVES; ++k) {
        lo = min(lo, L.red[0][k]);
        hi = max(hi, L.red[1][k]);
    }
}

// Exclusive prefix of cnt[0, K THREADS) in place, K counters to a thread; the
// return value is the sum over all counters of f(counter), saturating.  Ends
// with a barrier.
template <int WAVES, int MAXK, class F>
__device__ __forceinline__ uint32_t scan_bins(uint32_t* cnt, int K, SegLds<WAVES>& L, F&& f, bool want_max)
{
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    uint32_t c[MAXK], sum = 0, q = 0;
#pragma unroll
    for (int k = 0; k < MAXK; ++k) {
        if (k >= K) break;
        c[k] = cnt[tid * K + k];
        sum += c[k];
        q = want_max ? max(q, c[k]) : q + f(c[k]);
    }
    uint32_t incl = sum;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(incl, off, 64);
        if (lane >= off) incl += y;
    }
    for (int off = 32; off > 0; off >>= 1) {
        const uint32_t y = (uint32_t)__shfl_xor((int)q, off, 64);
        q = want_max ? max(q, y) : q + y;
    }
    if (lane == 63) {
        L.wsum[w] = incl;
        L.wsum2[w] = q;
    }
    __syncthreads();
    uint32_t run = incl - sum;
    q = 0;
#pragma unroll
    for (int k = 0; k < WAVES; ++k) {
        run += k < w ? L.wsum[k] : 0u;
        q = want_max ? max(q, L.wsum2[k]) : q + L.wsum2[k];
    }
#pragma unroll
    for (int k = 0; k < MAXK; ++k) {
        if (k >= K) break;
        cnt[tid * K + k] = run;
        run += c[k];
    }
    __syncthreads();
    return q;
}

// A long list's coarse bins, as the fine bins need them: linear over (value -
// lo) >> shift of the keys' values.  A value is the key itself (gap 0, and
// shift 32 leaves the depth bits) or, gap being 2^32 - n, depth bits * n +
// index: as the indices are below n, the order is the same and the indices of
// one depth fill their range instead of its first part.
struct Coarse {
    unsigned long long lo;
    int shift;
    uint32_t gap;
    unsigned long long mult;  // coarse_mult of the range
};

__device__ __forceinline__ unsigned long long key_value(uint32_t gap, unsigned long long k)
{
    return k - (unsigned long long)(uint32_t)(k >> 32) * gap;
}

// place of a key among the bins: its bin in the high word of place * mult
__device__ __forceinline__ uint32_t place_in(const Coarse& c, unsigned long long k)
{
    return (uint32_t)((key_value(c.gap, k) - c.lo) >> c.shift);
}

__device__ __forceinline__ uint32_t bin_of(const Coarse& c, unsigned long long k)
{
    return (uint32_t)(((unsigned long long)place_in(c, k) * c.mult) >> 32);
}

// Sorts the m <= ITEMS unique keys src[0, m) with the whole block; on return
// (after a barrier) key[r] of thread (w, lane) holds the key of sorted
// position w * R * 64 + r * 64 + lane (R = ceil(m / THREADS)) when that is
// below m.  One pass places every key in one of m bins that follow the
// list's own depth distribution, about one key to a bin; a key's position is
// then its bin's start plus the smaller keys of its bin.  The distribution
// is measured on the keys, or (known) it is that of the long list they are
// a part of: the bins of L.starts, src starting at position `done`.
template <int WAVES>
__device__ __forceinline__ void lds_sort(const unsigned long long* src, int m, bool known, Coarse in_list, uint32_t done,
                                         unsigned long long (&key)[GSR_SEG_PER_THREAD], SegLds<WAVES>& L)
{
    constexpr int THREADS = WAVES * 64, MAXR = GSR_SEG_PER_THREAD, NC = GSR_SEG_COARSE / THREADS;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int R = (m + THREADS - 1) / THREADS;
#pragma unroll
    for (int r = 0; r < MAXR; ++r) {
        if (r >= R) break;
        const int li = w * R * 64 + r * 64 + lane;
        key[r] = li < m ? src[li] : ~0ull;
    }
    // a key's fine bin (high half) and its place among the bin's arrivals
    static_assert(SegLds<WAVES>::ITEMS <= 65536, "both fit in half a word");
    uint32_t slot[MAXR];
#pragma unroll
    for (int r = 0; r < MAXR; ++r) {
        if (r >= R) break;
        L.fine[tid + r * THREADS] = 0u;
    }
    // coarse bin b of c keys is cut into c fine bins, numbered from its
    // start
    if (known) {
        __syncthreads();
        auto place = [&](auto&& place_of) {
#pragma unroll
            for (int r = 0; r < MAXR; ++r) {
                if (r >= R) break;
                const int li = w * R * 64 + r * 64 + lane;
                if (li < m) {
                    const unsigned long long p = (unsigned long long)place_of(key[r]) * in_list.mult;
                    const uint32_t b = (uint32_t)(p >> 32), s = L.starts[b], e = L.starts[b + 1];
                    const uint32_t bin = s - done + __umulhi((uint32_t)p, e - s);
                    slot[r] = bin << 16 | atomicAdd(&L.fine[bin], 1u);
                }
            }
        };
        if (in_list.gap == 0u)
            place([&](unsigned long long k) { return (uint32_t)(k >> 32) - (uint32_t)(in_list.lo >> 32); });
        else
            place([&](unsigned long long k) { return place_in(in_list, k); });
    } else {
        uint32_t lo = 0xffffffffu, hi = 0u;
#pragma unroll
        for (int r = 0; r < MAXR; ++r) {
            if (r >= R) break;
            const int li = w * R * 64 + r * 64 + lane;
            if (li < m) {
                lo = min(lo, (uint32_t)(key[r] >> 32));
                hi = max(hi, (uint32_t)(key[r] >> 32));
            }
        }
#pragma unroll
        for (int k = 0; k < NC; ++k) L.coarse[tid + k * THREADS] = 0u;
        block_min_max<WAVES>(lo, hi, L);
        const unsigned long long mult = coarse_mult(hi - lo);
#pragma unroll
        for (int r = 0; r < MAXR; ++r) {
            if (r >= R) break;
            const int li = w * R * 64 + r * 64 + lane;
            if (li < m) atomicAdd(&L.coarse[((unsigned long long)((uint32_t)(key[r] >> 32) - lo) * mult) >> 32], 1u);
        }
        __syncthreads();
        scan_bins<WAVES, NC>(L.coarse, NC, L, [](uint32_t) { return 0u; }, true);
        if (tid == 0) L.coarse[GSR_SEG_COARSE] = (uint32_t)m;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < MAXR; ++r) {
            if (r >= R) break;
            const int li = w * R * 64 + r * 64 + lane;
            if (li < m) {
                const unsigned long long p = (unsigned long long)((uint32_t)(key[r] >> 32) - lo) * mult;
                const uint32_t b = (uint32_t)(p >> 32), s = L.coarse[b], e = L.coarse[b + 1];
                const uint32_t bin = s + __umulhi((uint32_t)p, e - s);
                slot[r] = bin << 16 | atomicAdd(&L.fine[bin], 1u);
            }
        }
    }
    __syncthreads();
    const uint32_t pairs = scan_bins<WAVES, MAXR>(L.fine, R, L, [](uint32_t c) { return c * c; }, false);
    if (pairs > GSR_SEG_CROWDED * (uint32_t)m) {
        // too many keys share (nearly) one depth: compared with each
        // other they would cost more than the digits do
        radix_sort<WAVES>(key, m, L);
        return;
    }
    if (tid == 0) L.fine[R * THREADS] = (uint32_t)m;
#pragma unroll
    for (int r = 0; r < MAXR; ++r) {
        if (r >= R) break;
        if (w * R * 64 + r * 64 + lane < m) L.sk[L.fine[slot[r] >> 16] + (slot[r] & 0xffffu)] = key[r];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < MAXR; ++r) {
        if (r >= R) break;
        if (w * R * 64 + r * 64 + lane < m) {
            const uint32_t s = L.fine[slot[r] >> 16], e = L.fine[(slot[r] >> 16) + 1];
            slot[r] = s;  // from here on its sorted position
            if (e - s > 1u)
                for (uint32_t j = s; j < e; ++j) slot[r] += L.sk[j] < key[r] ? 1u : 0u;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < MAXR; ++r) {
        if (r >= R) break;
        if (w * R * 64 + r * 64 + lane < m) L.sk[slot[r]] = key[r];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < MAXR; ++r) {
        if (r >= R) break;
        const int li = w * R * 64 + r * 64 + lane;
        if (li < m) key[r] = L.sk[li];
    }
    __syncthreads();
}

// f(key) for the keys src[0, m), the block's threads taking them in turn; eight
// loads are in flight per thread (a list's passes over memory are otherwise
// chains of one load's latency per THREADS keys).
template <int THREADS, class F>
__device__ __forceinline__ void for_keys(const unsigned long long* src, int m, F&& f)
{
    constexpr int K = 8;
    int i = threadIdx.x;
    for (; i + (K - 1) * THREADS < m; i += K * THREADS) {
        unsigned long long k[K];
#pragma unroll
        for (int j = 0; j < K; ++j) k[j] = src[i + j * THREADS];
#pragma unroll
        for (int j = 0; j < K; ++j) f(k[j]);
    }
    for (; i < m; i += THREADS) f(src[i]);
}

// A value that every lane holds alike, in a scalar register.
__device__ __forceinline__ uint32_t uniform(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }

__device__ __forceinline__ unsigned long long uniform(unsigned long long x)
{
    return ((unsigned long long)uniform((uint32_t)(x >> 32)) << 32) | uniform((uint32_t)x);
}

// The bins of a list of len keys by the range of their depth bits * n + index
// (as many leading bits as 32 hold), which cuts a list of one depth or of few
// by index; leaves their starts in L.starts.
template <int WAVES>
__device__ __forceinline__ Coarse key_bins(const unsigned long long* src, int len, int64_t n, SegLds<WAVES>& L)
{
    constexpr int THREADS = WAVES * 64, NC = GSR_SEG_COARSE / THREADS;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    unsigned long long lo = ~0ull, hi = 0ull;
    for_keys<THREADS>(src, len, [&](unsigned long long k) {
        lo = min(lo, k);
        hi = max(hi, k);
    });
    for (int off = 32; off > 0; off >>= 1) {
        lo = min(lo, (unsigned long long)__shfl_xor(lo, off, 64));
        hi = max(hi, (unsigned long long)__shfl_xor(hi, off, 64));
    }
    if (lane == 0) {
        L.red64[0][w] = lo;
        L.red64[1][w] = hi;
    }
#pragma unroll
    for (int k = 0; k < NC; ++k) L.starts[tid + k * THREADS] = 0u;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < WAVES; ++k) {
        lo = min(lo, L.red64[0][k]);
        hi = max(hi, L.red64[1][k]);
    }
    const uint32_t gap = 0u - (uint32_t)n;
    lo = uniform(key_value(gap, lo));
    const unsigned long long range = uniform(key_value(gap, hi)) - lo;
    const int shift = max(0, 32 - (int)__clzll((long long)range));
    const unsigned long long mult = uniform(coarse_mult((uint32_t)(range >> shift)));
    const Coarse bins{lo, shift, gap, mult};
    for_keys<THREADS>(src, len, [&](unsigned long long k) { atomicAdd(&L.starts[bin_of(bins, k)], 1u); });
    __syncthreads();
    scan_bins<WAVES, NC>(L.starts, NC, L, [](uint32_t) { return 0u; }, true);
    return bins;
}

// A list's keys from src to dst, bin by bin (their starts in L.starts).
template <int WAVES>
__device__ __forceinline__ void spread_keys(const unsigned long long* src, unsigned long long* dst, int len, const Coarse& bins,
                                            SegLds<WAVES>& L)
{
    constexpr int THREADS = WAVES * 64;
    static_assert(SegLds<WAVES>::ITEMS >= GSR_SEG_COARSE, "a cursor per bin");
    for (int b = threadIdx.x; b < GSR_SEG_COARSE; b += THREADS) L.fine[b] = L.starts[b];
    if (threadIdx.x == 0) L.starts[GSR_SEG_COARSE] = (uint32_t)len;
    __syncthreads();
    for_keys<THREADS>(src, len, [&](unsigned long long k) { dst[atomicAdd(&L.fine[bin_of(bins, k)], 1u)] = k; });
    __syncthreads();  // the block's own writes are visible to it
}

// Sorts the segment of one tile with the whole block.  A list of up to ITEMS
// keys is sorted in LDS.  A longer one is first spread over its coarse depth
// bins (emission buffer to output key array, the order inside a bin being
// arbitrary); whole bins are then taken together up to ITEMS keys at a time
// and sorted in LDS, in place.
//
// Where more keys than that (less an eighth, so that the bins can be taken
// together by their start) share one coarse bin, or a bin that is nearly as
// large leaves too many small chunks, as with surfaces seen head-on and an
// outlier, or with one depth for all, the list is spread bin by bin instead.
// A bin of more than ITEMS keys then becomes a list of its own with bins of
// its own range (key_bins), smaller by their number: seven rounds at most, two
// in practice.  Such lists wait in a chain: the first entries of a.vals in
// their places, which nothing else uses until they are sorted, hold the list's
// length, its buffer and the next list; in both buffers its places are its
// own, so the keys move back and forth between the two.
template <int WAVES>
__device__ __forceinline__ void sort_segment(const SegArgs& a, uint32_t tile, uint2 rg, SegLds<WAVES>& L)
{
    constexpr int THREADS = WAVES * 64, MAXR = GSR_SEG_PER_THREAD, ITEMS = SegLds<WAVES>::ITEMS;
    constexpr int NC = GSR_SEG_COARSE / THREADS;
    constexpr uint32_t NONE = 0xffffffffu;
    const int v = view_of_tile(a.views, (int)tile);
    const uint32_t vbase = (uint32_t)((int64_t)v * a.n);
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    uint32_t at = rg.x, head = NONE;     // the list in hand, those that wait
    int m = (int)(rg.y - rg.x);
    const unsigned long long* src = a.seg + at;
    Coarse bins{0ull, 32, 0u, 0ull};
    uint32_t per_start = 0u;
    bool in_keys = false;
    if (m > ITEMS) {
        uint32_t lo = 0xffffffffu, hi = 0u;
        for_keys<THREADS>(src, m, [&](unsigned long long k) {
            lo = min(lo, (uint32_t)(k >> 32));
            hi = max(hi, (uint32_t)(k >> 32));
        });
#pragma unroll
        for (int k = 0; k < NC; ++k) L.starts[tid + k * THREADS] = 0u;
        block_min_max<WAVES>(lo, hi, L);
        lo = uniform(lo);
        hi = uniform(hi);
        const unsigned long long mult = uniform(coarse_mult(hi - lo));
        for_keys<THREADS>(src, m, [&](unsigned long long k) {
            atomicAdd(&L.starts[((unsigned long long)((uint32_t)(k >> 32) - lo) * mult) >> 32], 1u);
        });
        __syncthreads();
        const uint32_t most = uniform(scan_bins<WAVES, NC>(L.starts, NC, L, [](uint32_t) { return 0u; }, true));
        bins = Coarse{(unsigned long long)lo << 32, 32, 0u, mult};
        // (the chunks' cursors need a place each, and tiny chunks do not pay)
        if (most <= (uint32_t)(ITEMS - ITEMS / 8) && (uint32_t)m / ((uint32_t)ITEMS - most) < (uint32_t)ITEMS) {
            unsigned long long* const bufB = a.keys + rg.x;  // output keys double as scratch
            // chunk of a coarse bin, by its start: the starts of one chunk's
            // bins differ by at most ITEMS - most, so it holds at most ITEMS
            per_start = 0xffffffffu / ((uint32_t)ITEMS - most);
            // the chunks' cursors, in the fine bins' place
            if (tid == 0) L.starts[GSR_SEG_COARSE] = (uint32_t)m;
            for (int b = tid; b < GSR_SEG_COARSE; b += THREADS) {
                const uint32_t c = __umulhi(L.starts[b], per_start);
                if (b == 0 || __umulhi(L.starts[b - 1], per_start) != c) L.fine[c] = L.starts[b];
            }
            __syncthreads();
            for_keys<THREADS>(src, m, [&](unsigned long long k) {
                const uint32_t b = (uint32_t)(((unsigned long long)((uint32_t)(k >> 32) - lo) * mult) >> 32);
                bufB[atomicAdd(&L.fine[__umulhi(L.starts[b], per_start)], 1u)] = k;
            });
            __syncthreads();  // the block's own writes are visible to it
            src = bufB;
        } else {
            src = nullptr;
            if (lo == hi) bins.mult = 0ull;
        }
    }
    for (int done = 0;;) {
        if (done == m) {
            if (head == NONE) return;
            __syncthreads();
            at = head;
            m = (int)uniform(a.vals[at]);
            in_keys = uniform(a.vals[at + 1]) != 0u;
            head = uniform(a.vals[at + 2]);
            done = 0;
            bins.mult = 0ull;
            src = nullptr;
        }
        if (!src) {
            src = (in_keys ? a.keys : a.seg) + at;
            unsigned long long* const dst = (in_keys ? a.seg : a.keys) + at;
            if (bins.mult == 0ull) bins = key_bins<WAVES>(src, m, a.n, L);
            spread_keys<WAVES>(src, dst, m, bins, L);
            src = dst;
        }
        int end = m;
        if (per_start != 0u) {
            // up to the first bin of a later chunk
            const uint32_t c = __umulhi((uint32_t)done, per_start);
            int b0 = 0, b1 = GSR_SEG_COARSE;
            while (b0 < b1) {
                const int mid = (b0 + b1) >> 1;
                if (__umulhi(L.starts[mid], per_start) > c) b1 = mid;
                else b0 = mid + 1;
            }
            end = (int)uniform(L.starts[b0]);
        } else if (bins.mult != 0ull) {
            // the last bin that starts within ITEMS keys
            int b0 = 0, b1 = GSR_SEG_COARSE;
            while (b0 < b1) {
                const int mid = (b0 + b1 + 1) >> 1;
                if (L.starts[mid] <= (uint32_t)(done + ITEMS)) b0 = mid;
                else b1 = mid - 1;
            }
            end = (int)uniform(L.starts[b0]);
            if (end == done) {  // it holds more
                end = (int)uniform(L.starts[b0 + 1]);
                const uint32_t p = at + (uint32_t)done;
                if (tid == 0) {
                    a.vals[p] = (uint32_t)(end - done);
                    a.vals[p + 1] = in_keys ? 0u : 1u;
                    a.vals[p + 2] = head;
                }
                head = p;
                done = end;
                continue;
            }
        }
        const int cm = end - done;
        unsigned long long key[MAXR];
        lds_sort<WAVES>(src + done, cm, bins.mult != 0ull, bins, (uint32_t)done, key, L);
        const int R = (cm + THREADS - 1) / THREADS;
#pragma unroll
        for (int r = 0; r < MAXR; ++r) {
            if (r >= R) break;
            const int li = w * R * 64 + r * 64 + lane;
            if (li < cm) write_pair(a, at + (uint32_t)(done + li), key[r], tile, vbase);
        }
        done = end;
    }
}

// One block per tile, in the processing order: the blocks of the longest
// lists start first, and the empty tiles' blocks, which end the order, exit.
__global__ __launch_bounds__(GSR_SEG_THREADS, GSR_SEG_WAVES) void k_seg_sort(SegArgs a)
{
    __shared__ SegLds<GSR_SEG_THREADS / 64> L;
    if (a.counters->overflow) return;
    const uint32_t tile = (uint32_t)__builtin_amdgcn_readfirstlane((int)a.order[blockIdx.x]);
    const uint2 r = a.ranges[tile];
    const uint2 rg = make_uint2((uint32_t)__builtin_amdgcn_readfirstlane((int)r.x),
                                (uint32_t)__builtin_amdgcn_readfirstlane((int)r.y));
    if (rg.y == rg.x) return;
    sort_segment<GSR_SEG_THREADS / 64>(a, tile, rg, L);
}

hipError_t launch_seg_sort(const SegArgs& a, int total_tiles, hipStream_t s)
{
    if (total_tiles == 0) return hipSuccess;
    hipLaunchKernelGGL(k_seg_sort, dim3((unsigned)total_tiles), dim3(GSR_SEG_THREADS), 0, s, a);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// processing order of the tiles: descending pair count, bucketed by
// floor(log2(count)) (count_bucket; counted with the tile ranges)

// places each tile at its bucket's base plus a block-aggregated cursor: one
// global atomic per (block, bucket)
__global__ void k_order_place(RangeArgs a)
{
    __shared__ uint32_t base[32], cnt[32], blk[32];
    if (threadIdx.x < 32) cnt[threadIdx.x] = 0u;
    if (threadIdx.x == 0) {
        uint32_t run = 0;
        for (int b = 0; b < 32; ++b) {
            base[b] = run;
            run += a.buckets[b];
        }
    }
    __syncthreads();
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    uint32_t b = 0, local = 0;
    if (t < a.total_tiles) {
        b = count_bucket(a.ranges[t]);
        local = atomicAdd(&cnt[b], 1u);
    }
    __syncthreads();
    if (threadIdx.x < 32) blk[threadIdx.x] = cnt[threadIdx.x] ? atomicAdd(&a.buckets[32 + threadIdx.x], cnt[threadIdx.x]) : 0u;
    __syncthreads();
    if (t < a.total_tiles) a.order[base[b] + blk[b] + local] = (uint32_t)t;
}

hipError_t launch_order(const RangeArgs& a, hipStream_t s)
{
    if (a.total_tiles <= GSR_ONE_TILES) return hipSuccess;  // placed by k_bin_tiles_one
    hipLaunchKernelGGL(k_order_place, dim3((unsigned)((a.total_tiles + 255) / 256)), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace gsr
