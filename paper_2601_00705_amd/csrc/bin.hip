// bin.hip -- the depth-ordered sets N(p) of Eq. (alpha), grouped by tile.
//
// For every live slot the conservative tile rectangle (tile_rect) gives the
// candidate tiles; a candidate is kept when the slot's ellipse reaches the
// tile's pixel-centre box (tile_hit).  Each kept (tile, slot) pair goes into
// the tile's segment of the pair array as one 64-bit key
//   (float bits of the camera depth << 32) | Gaussian index,
// which orders a segment by depth and breaks ties by index (positive floats
// order like their bit patterns).  The tile is the most significant part of
// the order, so it is resolved by counting instead of sorting.  A chunk is a
// run of consecutive entries of one view's list of live Gaussians (those whose
// rectangle is not empty), chunk_mult * GSR_BIN_CHUNK or fewer (chunk_len),
// staged GSR_BIN_CHUNK at a time:
//
//   k_bin_zero    clears the views' live counts and the order's buckets
//   k_bin_list    per view, the list of live Gaussians from the projection's
//                 liveness ballots (a block scans its words' popcounts and
//                 reserves its places with one atomic on the view's counter,
//                 so the list's order is arbitrary; every later step is exact
//                 whatever the order)
//   k_bin_count   per chunk: pairs per tile of the view, one row of the
//                 view's [chunk][tile] count matrix (LDS histogram; views
//                 with more than GSR_BIN_LDS_TILES tiles add straight into
//                 the row)
//   k_bin_colscan per tile: exclusive prefix of its column (the chunk's offset
//                 inside the tile's segment) and the tile's total, 32
//                 groups of threads to a column
//   k_bin_tiles   the tile ranges from the column scan's per-block prefixes
//                 and block sums, the pair count and the capacity flag, and
//                 the tiles per bucket of the processing order
//                 (k_bin_tiles_one: for few tiles, the order as well)
//   k_bin_emit    the chunk's pairs, each at its tile's cursor (LDS atomics:
//                 the order inside a chunk's group is arbitrary, and the
//                 per-tile sort of the unique keys makes it exact)
//
// The grid of the count and emit kernels covers the most chunks a view can
// have (rounded up to a multiple of GSR_XCDS); blocks past a view's list exit
// at once.  The emit pass maps blocks to chunks so that each die takes one
// contiguous range of a view's chunks: the runs that consecutive chunks
// write into a tile's segment are adjacent, and a cache line filled by
// several chunks is then filled inside one die's L2 instead of being
// written back in pieces by several (measured: 3.5x the key bytes written
// to HBM with chunks dealt round-robin).  Candidates of a staged
// group are numbered by the prefix of the rectangle areas over the group's
// owners (its slots with a non-empty rectangle, compacted); each thread
// walks a contiguous run of them, its first owner found by binary search.
// The walk has no branch per candidate: every step reloads its owner's
// 48-byte record from LDS (three 16-byte reads, the same for every lane
// wherever a lane stands in its run) and advances tile, row and owner by
// selects, so that the lanes of a wave never diverge over owner or row
// changes.
#include "kernels.h"

#include <algorithm>

#ifndef GSR_EMIT_BATCH
#define GSR_EMIT_BATCH 4
#endif

namespace gsr {

static_assert(GSR_BIN_CHUNK == 256, "one staged slot per thread");

// A staged owner: ellipse, reciprocals and rectangle (origin, width,
// height; the height's sign bit marks an ellipse with a non-finite term,
// which takes tile_hit itself).
struct __align__(16) Owner {
    float u, v, A, B;
    float C, q, iA, iC;
    int x0, y0, w, h;
};

struct ChunkLds {
    uint32_t excl[GSR_BIN_CHUNK + 1];  // prefix of the owners' rectangle areas
    Owner own[GSR_BIN_CHUNK];
    uint2 key[GSR_BIN_CHUNK];          // (depth bits, Gaussian index)
    uint32_t wsum[4], wnz[4];
};

// The records of one staged group, fetched into registers (thread t owns
// entry t).  All fields are loaded at once, so that one memory round trip
// serves the group; the next group's fetch is issued before the current
// group is walked.
struct GroupRegs {
    float4 gm, co;
    float q;
    uint32_t dbits, idx;
    bool in;
};

// entries of view v's live list
__device__ __forceinline__ uint32_t live_len(const BinArgs& a, int v)
{
    const uint32_t c = a.live_count[v * GSR_LIVE_STRIDE];
    return c < (uint64_t)a.n ? c : (uint32_t)a.n;
}

// Entries of one chunk of a view with len live Gaussians: chunk_mult *
// GSR_BIN_CHUNK, or fewer (a multiple of GSR_BIN_LEAST) where that would
// leave the views' chunks below GSR_BIN_BLOCKS, so that a sparse view's work
// still spreads over the chip: 8754 live of 100k Gaussians, 22 candidate
// tiles each, made 35 chunks of 256, counted in 24 us and emitted in 27;
// 137 of 64 take 16 and 17 (of 32: 13 and 14, and 2 more for their column
// scan).  The count matrix has a.chunks rows a view.
__device__ __forceinline__ uint32_t chunk_len(const BinArgs& a, uint32_t len)
{
    const uint32_t full = (uint32_t)a.chunk_mult * GSR_BIN_CHUNK;
    const uint32_t want = max(1u, (uint32_t)(GSR_BIN_BLOCKS / a.n_views));
    if (len / want >= full) return full;
    const uint32_t per = max((len + want - 1u) / want, (len + (uint32_t)a.chunks - 1u) / (uint32_t)a.chunks);
    return min(full, (max(per, 1u) + GSR_BIN_LEAST - 1u) / GSR_BIN_LEAST * GSR_BIN_LEAST);
}

__device__ __forceinline__ int view_chunks(const BinArgs& a, int v)
{
    const uint32_t len = live_len(a, v), per = chunk_len(a, len);
    return (int)((len + per - 1u) / per);
}

// entries base .. (below len, the chunk's end) of view v's live list
__device__ __forceinline__ void fetch_group(const BinArgs& a, int v, int64_t base, uint32_t len, bool want_depth,
                                            GroupRegs& R)
{
    const int64_t j = base + threadIdx.x;
    R.in = j < (int64_t)len;
    if (R.in) {
        const uint32_t i = a.live[(int64_t)v * a.n + j];
        R.idx = i;
        const int64_t slot = (int64_t)v * a.n + i;
        R.gm = a.geom[slot];
        R.co = a.conic_o[slot];
        R.q = a.qthr[slot];
        R.dbits = want_depth ? __float_as_uint(a.rgb_d[slot].w) : 0u;
    }
}

struct Staged {
    uint32_t total;   // candidates
    int owners;       // slots with a non-empty rectangle
};

// Stages a fetched group: the owners' records, compacted, and the scan of
// their rectangle areas.  Starts and ends with a block barrier.
__device__ Staged stage_group(const BinArgs& a, const ViewInfo& vw, const GroupRegs& R, bool want_key, ChunkLds& L)
{
    const float inv_tw = 1.0f / (float)a.cfg.tile_w, inv_th = 1.0f / (float)a.cfg.tile_h;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    __syncthreads();
    int x0 = 0, y0 = 0, x1 = -1, y1 = -1;
    const bool nz = R.in && tile_rect(R.gm.x, R.gm.y, R.gm.z, R.gm.w, inv_tw, inv_th, vw.tiles_x, vw.tiles_y, x0,
                                      y0, x1, y1);
    const uint32_t area = nz ? (uint32_t)((x1 - x0 + 1) * (y1 - y0 + 1)) : 0u;
    uint32_t ia = area, in_ = nz ? 1u : 0u;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t ya = __shfl_up(ia, off, 64), yn = __shfl_up(in_, off, 64);
        if (lane >= off) {
            ia += ya;
            in_ += yn;
        }
    }
    if (lane == 63) {
        L.wsum[w] = ia;
        L.wnz[w] = in_;
    }
    __syncthreads();
    uint32_t oa = 0, on = 0;
    for (int k = 0; k < w; ++k) {
        oa += L.wsum[k];
        on += L.wnz[k];
    }
    if (nz) {
        const uint32_t c = on + in_ - 1u;
        L.excl[c] = oa + ia - area;
        Owner o;
        o.u = R.gm.x;
        o.v = R.gm.y;
        o.A = R.co.x;
        o.B = R.co.y;
        o.C = R.co.z;
        o.q = R.q;
        o.iA = 1.0f / o.A;
        o.iC = 1.0f / o.C;
        const bool fast = __builtin_isfinite(o.A) && __builtin_isfinite(o.B) && __builtin_isfinite(o.C) &&
                          __builtin_isfinite(o.iA) && __builtin_isfinite(o.iC);
        o.x0 = x0;
        o.y0 = y0;
        o.w = x1 - x0 + 1;
        o.h = (y1 - y0 + 1) | (fast ? 0 : (int)0x80000000);
        L.own[c] = o;
        if (want_key) L.key[c] = make_uint2(R.dbits, R.idx);
    }
    Staged st;
    st.total = L.wsum[0] + L.wsum[1] + L.wsum[2] + L.wsum[3];
    st.owners = (int)(L.wnz[0] + L.wnz[1] + L.wnz[2] + L.wnz[3]);
    if (tid == 0) L.excl[st.owners] = st.total;
    __syncthreads();
    return st;
}

// tile_hit on a staged owner: the same float32 operations on the same
// operands, so the same decision, with 1/A and 1/C computed once per owner.
// Tile box corners come from exact values (float)(tx tw) + 0.5 (integers
// below 2^23 plus one half; the far corner adds tw - 1 exactly), the edge
// minimiser's clamp is a median of three and the minimum over the edges a
// float minimum: both equal tile_hit's comparisons when the clamped value
// is not NaN, which holds when A, B, C, 1/A, 1/C are finite (then
// -(B X) / C is a finite or infinite number, never NaN); a q that is NaN is
// skipped by both.  Owners with a non-finite term call tile_hit.
__device__ __forceinline__ bool owner_hit(const Owner& o, bool fast, int tx, int ty, int tw, int th)
{
    if (!fast) return tile_hit(o.u, o.v, o.A, o.B, o.C, o.iA, o.iC, o.q, tx, ty, tw, th);
    const float fx = (float)(tx * tw) + 0.5f, fy = (float)(ty * th) + 0.5f;
    const float x0 = fx - o.u, x1 = (fx + (float)(tw - 1)) - o.u;
    const float y0 = fy - o.v, y1 = (fy + (float)(th - 1)) - o.v;
    if (x0 <= 0.0f && x1 >= 0.0f && y0 <= 0.0f && y1 >= 0.0f) return true;
    const float B2 = 2.0f * o.B;
    float m = INFINITY;
    {
        const float ys = __builtin_amdgcn_fmed3f(-(o.B * x0) * o.iC, y0, y1);
        m = fminf(m, (o.A * x0) * x0 + (B2 * x0) * ys + (o.C * ys) * ys);
    }
    {
        const float ys = __builtin_amdgcn_fmed3f(-(o.B * x1) * o.iC, y0, y1);
        m = fminf(m, (o.A * x1) * x1 + (B2 * x1) * ys + (o.C * ys) * ys);
    }
    {
        const float xs = __builtin_amdgcn_fmed3f(-(o.B * y0) * o.iA, x0, x1);
        m = fminf(m, (o.A * xs) * xs + (B2 * xs) * y0 + (o.C * y0) * y0);
    }
    {
        const float xs = __builtin_amdgcn_fmed3f(-(o.B * y1) * o.iA, x0, x1);
        m = fminf(m, (o.A * xs) * xs + (B2 * xs) * y1 + (o.C * y1) * y1);
    }
    return m <= o.q;
}

// Walks this thread's contiguous run of the staged group's candidates,
// BATCH at a time: batch(tt, hit, key) gets, for each, the tile within the
// view, whether the tile test keeps it and (WANT_KEY) the owner's key.
template <int BATCH, bool WANT_KEY, class Batch>
__device__ __forceinline__ void walk_group(const ChunkLds& L, const Staged& st, const BinArgs& a, const ViewInfo& vw,
                                           Batch&& batch)
{
    const uint32_t per = (st.total + 255u) / 256u;
    uint32_t j = threadIdx.x * per;
    const uint32_t j1 = min(j + per, st.total);
    if (j >= j1) return;
    const int tw = a.cfg.tile_w, th = a.cfg.tile_h;
    // first owner: the largest s with excl[s] <= j
    int lo = 0, hi = st.owners - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (L.excl[mid] <= j) lo = mid; else hi = mid - 1;
    }
    int s = lo;
    const uint32_t r = j - L.excl[s];
    const uint32_t w0 = (uint32_t)L.own[s].w;
    int dx = (int)(r % w0), dy = (int)(r / w0);
    while (j < j1) {
        uint32_t tt[BATCH];
        bool hit[BATCH];
        uint2 key[BATCH];
#pragma unroll
        for (int e = 0; e < BATCH; ++e) {
            const bool valid = BATCH == 1 || j < j1;
            const int sl = BATCH == 1 ? s : min(s, st.owners - 1);
            const Owner o = L.own[sl];
            key[e] = WANT_KEY ? L.key[sl] : make_uint2(0u, 0u);
            const int h = o.h & 0x7fffffff;
            const int tx = o.x0 + dx, ty = o.y0 + dy;
            tt[e] = (uint32_t)(ty * vw.tiles_x + tx);
            hit[e] = valid && owner_hit(o, o.h >= 0, tx, ty, tw, th);
            // next candidate: along the row, then the next row, then the
            // next owner
            ++dx;
            const bool row_end = dx == o.w;
            dx = row_end ? 0 : dx;
            dy += row_end ? 1 : 0;
            const bool own_end = dy == h;
            dy = own_end ? 0 : dy;
            s += own_end ? 1 : 0;
            ++j;
        }
        batch(tt, hit, key);
    }
}

// the views' live counts and the processing order's bucket counts and cursors
__global__ __launch_bounds__(64) void k_bin_zero(BinArgs a)
{
    if (threadIdx.x == 0) a.live_count[blockIdx.x * GSR_LIVE_STRIDE] = 0u;
    if (blockIdx.x == 0) a.buckets[threadIdx.x] = 0u;
}

// Every wave holds the block's 64 WORDS ballot words (WORDS to a lane) and
// their prefix, and writes a quarter of them: 16 to a wave for one word a lane
// (128, at two words a lane and every wave its own, took 9 us at any size
// below 500k Gaussians, four blocks at 100k; now 5).  Past a million Gaussians
// the blocks' atomics on the view's counter would queue (36 views of 3M: 71
// us), so a lane takes four.
template <int WORDS>
__global__ __launch_bounds__(256) void k_bin_list(BinArgs a)
{
    __shared__ uint32_t base_s;
    const int v = blockIdx.y;
    const int lane = threadIdx.x & 63, w = (int)(threadIdx.x >> 6);
    const int64_t w0 = (int64_t)blockIdx.x * 64 * WORDS;
    uint64_t m[WORDS];
    uint32_t cnt = 0;
#pragma unroll
    for (int k = 0; k < WORDS; ++k) {
        const int64_t wd = w0 + lane * WORDS + k;
        m[k] = wd < a.mask_words ? a.live_mask[wd * a.n_views + v] : 0ull;
        // no Gaussian past n
        if (wd == a.mask_words - 1 && (a.n & 63)) m[k] &= (1ull << (a.n & 63)) - 1ull;
        cnt += (uint32_t)__popcll(m[k]);
    }
    uint32_t incl = cnt;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(incl, off, 64);
        if (lane >= off) incl += y;
    }
    if (threadIdx.x == 63) base_s = incl ? atomicAdd(&a.live_count[v * GSR_LIVE_STRIDE], incl) : 0u;
    __syncthreads();
    const uint32_t pos = base_s + incl - cnt;
    uint32_t* list = a.live + (int64_t)v * a.n;
    // a word's entries go out together: lane l keeps bit l of the word, so
    // the set bits are one coalesced run in index order
    const uint64_t below = (1ull << lane) - 1ull;
    for (int t = 0; t < 16; ++t) {
        const int j = w * 16 + t;
        uint32_t at = (uint32_t)__builtin_amdgcn_readlane((int)pos, j);
#pragma unroll
        for (int k = 0; k < WORDS; ++k) {
            const uint64_t word = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(m[k] >> 32), j) << 32) |
                                  (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)m[k], j);
            if (word == 0ull) continue;
            if ((word >> lane) & 1ull)
                list[at + (uint32_t)__popcll(word & below)] = (uint32_t)((w0 + j * WORDS + k) * 64 + lane);
            at += (uint32_t)__popcll(word);
        }
    }
}

// row of the count matrix of (view, chunk)
__device__ __forceinline__ uint32_t* count_row(const BinArgs& a, const ViewInfo& vw, int chunk)
{
    const int64_t tiles_v = (int64_t)vw.tiles_x * vw.tiles_y;
    return a.cnt + (int64_t)a.chunks * vw.tile_base + (int64_t)chunk * tiles_v;
}

template <bool LDS_HIST>
__global__ __launch_bounds__(256) void k_bin_count(BinArgs a)
{
    HIP_DYNAMIC_SHARED(uint32_t, hist)  // [tiles of the view] when LDS_HIST
    __shared__ ChunkLds L;
    const int v = blockIdx.y;
    if ((int)blockIdx.x >= view_chunks(a, v)) return;
    const uint32_t live = live_len(a, v), per_chunk = chunk_len(a, live);
    const uint32_t len = min(live, ((uint32_t)blockIdx.x + 1u) * per_chunk);  // the chunk's end
    const ViewInfo vw = a.views->v[v];
    const int tiles_v = vw.tiles_x * vw.tiles_y;
    uint32_t* row = count_row(a, vw, blockIdx.x);
    if (LDS_HIST)
        for (int t = threadIdx.x; t < tiles_v; t += 256) hist[t] = 0u;
    GroupRegs cur, nxt;
    int64_t base = (int64_t)blockIdx.x * per_chunk;
    fetch_group(a, v, base, len, false, nxt);
    for (int sub = 0; sub < a.chunk_mult; ++sub, base += GSR_BIN_CHUNK) {
        if (base >= (int64_t)len) break;
        cur = nxt;
        if (sub + 1 < a.chunk_mult) fetch_group(a, v, base + GSR_BIN_CHUNK, len, false, nxt);
        const Staged st = stage_group(a, vw, cur, false, L);
        walk_group<1, false>(L, st, a, vw, [&](const uint32_t(&tt)[1], const bool(&hit)[1], const uint2(&)[1]) {
            // a miss adds 0: no branch
            if (LDS_HIST) atomicAdd(&hist[tt[0]], hit[0] ? 1u : 0u);
            else if (hit[0]) atomicAdd(&row[tt[0]], 1u);
        });
    }
    if (LDS_HIST) {
        __syncthreads();
        for (int t = threadIdx.x; t < tiles_v; t += 256) row[t] = hist[t];
    }
}

__global__ void k_zero_u32(uint32_t* p, int64_t count)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0u;
}

// Column scan: a block takes GSR_COL_TILES (32: a cache line of counters)
// consecutive global tiles and scans their columns 256 chunks at a time, 32
// groups of threads with 8 rows each: the rows are read once into registers
// (the next pass's reads are issued before this one's barrier), the groups'
// sums meet in LDS, and the rows are rewritten as the exclusive prefix over
// chunks.  The column's total goes to ranges[].y.  Bound by the matrix's one
// read and one write; with 64 tiles a block, four waves and two reads the
// scan of one 1200x680 view (1954 chunks of 3225 tiles) kept 204 waves on 51
// CUs busy for 40 us, now (half the chunks, too) 18; five such views 92 -> 43,
// 36 views of 3M Gaussians 263 -> 98.
__global__ __launch_bounds__(1024) void k_bin_colscan(BinArgs a)
{
    constexpr int K = 8, GROUPS = 1024 / GSR_COL_TILES;
    static_assert(GSR_COL_TILES == 32, "the totals' scan runs over half a wave");
    __shared__ uint32_t part[GROUPS][GSR_COL_TILES];
    __shared__ int chunks_max;
    const int lt = threadIdx.x & (GSR_COL_TILES - 1), q = threadIdx.x / GSR_COL_TILES;
    const int g = blockIdx.x * GSR_COL_TILES + lt;
    const bool in = g < a.total_tiles;
    uint32_t* col = nullptr;
    int64_t stride = 0;
    int chunks_v = 0;
    if (threadIdx.x == 0) chunks_max = 0;
    __syncthreads();
    if (in) {
        const int v = view_of_tile(a.views, g);
        const ViewInfo& vw = a.views->v[v];
        stride = (int64_t)vw.tiles_x * vw.tiles_y;
        col = a.cnt + (int64_t)a.chunks * vw.tile_base + (g - vw.tile_base);
        chunks_v = view_chunks(a, v);
        if (q == 0) atomicMax(&chunks_max, chunks_v);
    }
    __syncthreads();
    const int last = chunks_max;
    uint32_t carry = 0u, x[K], nx[K];
#pragma unroll
    for (int k = 0; k < K; ++k) nx[k] = q * K + k < chunks_v ? col[(int64_t)(q * K + k) * stride] : 0u;
    for (int c0 = 0; c0 < last; c0 += K * GROUPS) {
        uint32_t sum = 0u;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            x[k] = nx[k];
            sum += x[k];
        }
        const int c = c0 + q * K, cn = c + K * GROUPS;
#pragma unroll
        for (int k = 0; k < K; ++k) nx[k] = cn + k < chunks_v ? col[(int64_t)(cn + k) * stride] : 0u;
        part[q][lt] = sum;
        __syncthreads();
        uint32_t run = carry, total = 0u;
#pragma unroll
        for (int k = 0; k < GROUPS; ++k) {
            const uint32_t y = part[k][lt];
            run += k < q ? y : 0u;
            total += y;
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (c + k < chunks_v) col[(int64_t)(c + k) * stride] = run;
            run += x[k];
        }
        carry += total;
        __syncthreads();
    }
    if (q == 0) {
        // the 32 tiles' totals: their exclusive prefix within the block goes
        // to ranges[].x, the block's pairs to tile_blocks (k_bin_tiles adds
        // the earlier blocks')
        unsigned long long incl = carry;
        for (int o = 1; o < GSR_COL_TILES; o <<= 1) {
            const unsigned long long y = __shfl_up(incl, o, GSR_COL_TILES);
            if (lt >= o) incl += y;
        }
        if (in) a.ranges[g] = make_uint2((uint32_t)(incl - carry), carry);
        if (lt == GSR_COL_TILES - 1) a.tile_blocks[blockIdx.x] = incl;
    }
}

// The tile ranges: each tile's start is the pairs of the earlier 32-tile
// blocks plus its prefix within its block; the pair count and the capacity
// flag come from the blocks' sum (every block forms it, so that all decide
// the overflow alike).  The tiles are also counted into the processing
// order's buckets.
__device__ __forceinline__ uint2 tile_range_of(uint2 r, unsigned long long pre, bool over)
{
    // empty tiles get [0, 0); on overflow every range is empty, so that no
    // kernel reads past the capacity
    const unsigned long long start = pre + r.x;
    return (over || r.y == 0u) ? make_uint2(0u, 0u) : make_uint2((uint32_t)start, (uint32_t)(start + r.y));
}

__global__ __launch_bounds__(256) void k_bin_tiles(BinArgs a)
{
    __shared__ unsigned long long red[2][4];
    __shared__ uint32_t hist[32];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int nb = (a.total_tiles + GSR_COL_TILES - 1) / GSR_COL_TILES;
    const int b0 = (int)blockIdx.x * (256 / GSR_COL_TILES);
    if (tid < 32) hist[tid] = 0u;
    unsigned long long pre = 0ull, tot = 0ull;
    for (int k = tid; k < nb; k += 256) {
        const unsigned long long x = a.tile_blocks[k];
        tot += x;
        if (k < b0) pre += x;
    }
    for (int o = 32; o > 0; o >>= 1) {
        pre += __shfl_xor(pre, o, 64);
        tot += __shfl_xor(tot, o, 64);
    }
    if (lane == 0) {
        red[0][w] = pre;
        red[1][w] = tot;
    }
    __syncthreads();
    pre = red[0][0] + red[0][1] + red[0][2] + red[0][3];
    tot = red[1][0] + red[1][1] + red[1][2] + red[1][3];
    const bool over = tot > a.counters->capacity;
    const int g = (int)blockIdx.x * 256 + tid;
    if (g < a.total_tiles) {
        for (int k = b0; k < b0 + tid / GSR_COL_TILES; ++k) pre += a.tile_blocks[k];
        const uint2 r = tile_range_of(a.ranges[g], pre, over);
        a.ranges[g] = r;
        atomicAdd(&hist[count_bucket(r)], 1u);
    }
    if (blockIdx.x == 0 && tid == 0) {
        a.counters->pairs = tot;
        a.counters->overflow = over ? 1u : 0u;
    }
    __syncthreads();
    if (tid < 32 && hist[tid]) atomicAdd(&a.buckets[tid], hist[tid]);
}

// The same for at most GSR_ONE_TILES tiles, in one block, which also places
// them in the processing order: one launch for this and k_order_place, each 4
// to 5 us of a 242 us step.
__global__ __launch_bounds__(1024) void k_bin_tiles_one(BinArgs a)
{
    constexpr int PER = GSR_ONE_TILES / 1024, NB = GSR_ONE_TILES / GSR_COL_TILES;
    static_assert(NB == 128, "the blocks' sums are scanned by two waves");
    __shared__ unsigned long long base[NB], half;
    __shared__ uint32_t hist[32], cursor[32];
    const int tid = threadIdx.x, lane = tid & 63;
    const int nb = (a.total_tiles + GSR_COL_TILES - 1) / GSR_COL_TILES;
    if (tid < 32) hist[tid] = 0u;
    unsigned long long incl = 0ull, own = 0ull;
    if (tid < NB) {
        own = incl = tid < nb ? a.tile_blocks[tid] : 0ull;
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned long long y = __shfl_up(incl, o, 64);
            if (lane >= o) incl += y;
        }
        if (tid == 63) half = incl;
    }
    __syncthreads();
    if (tid < NB) base[tid] = incl - own + (tid < 64 ? 0ull : half);
    __syncthreads();
    const unsigned long long tot = base[nb - 1] + a.tile_blocks[nb - 1];
    const bool over = tot > a.counters->capacity;
    uint32_t bucket[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int g = tid + k * 1024;
        bucket[k] = 0u;
        if (g < a.total_tiles) {
            const uint2 r = tile_range_of(a.ranges[g], base[g / GSR_COL_TILES], over);
            a.ranges[g] = r;
            bucket[k] = count_bucket(r);
            atomicAdd(&hist[bucket[k]], 1u);
        }
    }
    if (tid == 0) {
        a.counters->pairs = tot;
        a.counters->overflow = over ? 1u : 0u;
    }
    __syncthreads();
    if (tid < 32) {
        uint32_t run = 0;
        for (int k = 0; k < tid; ++k) run += hist[k];
        cursor[tid] = run;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int g = tid + k * 1024;
        if (g < a.total_tiles) a.order[atomicAdd(&cursor[bucket[k]], 1u)] = (uint32_t)g;
    }
}

template <bool LDS_HIST>
__global__ __launch_bounds__(256) void k_bin_emit(BinArgs a)
{
    HIP_DYNAMIC_SHARED(uint32_t, cursor)  // [tiles of the view] when LDS_HIST
    __shared__ ChunkLds L;
    if (a.counters->overflow) return;
    const int v = blockIdx.y;
    // block x runs on die x % GSR_XCDS (the grid's width is a multiple of
    // GSR_XCDS); die k takes chunks [k per, (k + 1) per)
    const int nc = view_chunks(a, v);
    const int per = (nc + GSR_XCDS - 1) / GSR_XCDS;
    const int chunk = (int)(blockIdx.x % GSR_XCDS) * per + (int)(blockIdx.x / GSR_XCDS);
    if ((int)(blockIdx.x / GSR_XCDS) >= per || chunk >= nc) return;
    const uint32_t live = live_len(a, v), per_chunk = chunk_len(a, live);
    const uint32_t len = min(live, ((uint32_t)chunk + 1u) * per_chunk);  // the chunk's end
    const ViewInfo vw = a.views->v[v];
    const int tiles_v = vw.tiles_x * vw.tiles_y;
    uint32_t* row = count_row(a, vw, chunk);
    const uint2* rng = a.ranges + vw.tile_base;
    if (LDS_HIST)
        for (int t = threadIdx.x; t < tiles_v; t += 256) cursor[t] = rng[t].x + row[t];
    GroupRegs cur, nxt;
    int64_t base = (int64_t)chunk * per_chunk;
    fetch_group(a, v, base, len, true, nxt);
    for (int sub = 0; sub < a.chunk_mult; ++sub, base += GSR_BIN_CHUNK) {
        if (base >= (int64_t)len) break;
        cur = nxt;
        if (sub + 1 < a.chunk_mult) fetch_group(a, v, base + GSR_BIN_CHUNK, len, true, nxt);
        const Staged st = stage_group(a, vw, cur, true, L);
        walk_group<GSR_EMIT_BATCH, true>(L, st, a, vw, [&](const uint32_t(&tt)[GSR_EMIT_BATCH],
                                                           const bool(&hit)[GSR_EMIT_BATCH],
                                                           const uint2(&key)[GSR_EMIT_BATCH]) {
            uint32_t pos[GSR_EMIT_BATCH];
            if (LDS_HIST) {
                // a miss adds 0 (its result is unused), so that the atomics
                // issue back to back and one wait covers them
#pragma unroll
                for (int e = 0; e < GSR_EMIT_BATCH; ++e) pos[e] = atomicAdd(&cursor[tt[e]], hit[e] ? 1u : 0u);
            } else {
#pragma unroll
                for (int e = 0; e < GSR_EMIT_BATCH; ++e)
                    pos[e] = hit[e] ? rng[tt[e]].x + atomicAdd(&row[tt[e]], 1u) : 0u;
            }
#pragma unroll
            for (int e = 0; e < GSR_EMIT_BATCH; ++e)
                if (hit[e]) a.seg[pos[e]] = ((unsigned long long)key[e].x << 32) | key[e].y;
        });
    }
}

hipError_t launch_bin(const BinArgs& a, int max_tiles_view, hipStream_t s)
{
    if (a.total_tiles == 0) return hipSuccess;
    hipLaunchKernelGGL(k_bin_zero, dim3((unsigned)a.n_views), dim3(64), 0, s, a);
    const int words = a.mask_words > 16384 ? 4 : 1;
    const dim3 lists((unsigned)std::max<int64_t>((a.mask_words + 64 * words - 1) / (64 * words), 1), (unsigned)a.n_views);
    if (words == 4) hipLaunchKernelGGL(k_bin_list<4>, lists, dim3(256), 0, s, a);
    else hipLaunchKernelGGL(k_bin_list<1>, lists, dim3(256), 0, s, a);
    dim3 grid((unsigned)((a.chunks + GSR_XCDS - 1) / GSR_XCDS * GSR_XCDS), (unsigned)a.n_views);
    const bool lds = max_tiles_view <= GSR_BIN_LDS_TILES;
    const size_t dyn = lds ? sizeof(uint32_t) * (size_t)max_tiles_view : 0;
    if (lds) {
        hipLaunchKernelGGL(k_bin_count<true>, grid, dim3(256), dyn, s, a);
    } else {
        const int64_t entries = (int64_t)a.chunks * a.total_tiles;
        hipLaunchKernelGGL(k_zero_u32, dim3(2048), dim3(256), 0, s, a.cnt, entries);
        hipLaunchKernelGGL(k_bin_count<false>, grid, dim3(256), 0, s, a);
    }
    hipLaunchKernelGGL(k_bin_colscan, dim3((unsigned)((a.total_tiles + GSR_COL_TILES - 1) / GSR_COL_TILES)), dim3(1024), 0,
                       s, a);
    if (a.total_tiles <= GSR_ONE_TILES) hipLaunchKernelGGL(k_bin_tiles_one, dim3(1), dim3(1024), 0, s, a);
    else hipLaunchKernelGGL(k_bin_tiles, dim3((unsigned)((a.total_tiles + 255) / 256)), dim3(256), 0, s, a);
    if (lds) hipLaunchKernelGGL(k_bin_emit<true>, grid, dim3(256), dyn, s, a);
    else hipLaunchKernelGGL(k_bin_emit<false>, grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace gsr
