// raster.hip -- per-tile alpha compositing, Eq. (alpha), forward and backward.
//
// One wavefront (64 lanes) per (view, tile); each lane owns PPT = tile
// pixels / 64 pixels of one column of the tile (rows l / tile_w + k * 64 /
// tile_w).  The tile's depth-sorted pair range is walked in batches of
// BATCH (64, 128 or 256) records: every lane stages BATCH / 64 records into
// LDS in exp2 form, the quadratic form expanded around the tile centre in
// double (power2 = c0 + g . d + a2 dx^2 + b2 dx dy + c2 dy^2 for the offset d
// of a pixel from the tile centre, the conic scaled by -log2(e)/2, and the
// alpha_min test as power2 < log2(alpha_min / o)); then the lane walks the
// batch for each of its pixels, sharing the per-entry terms of its column.
//
// Plans of few tiles deal a tile's pixels to several waves (k_raster_fwd_few,
// k_raster_bwd_few), with the same arithmetic.
//
// Forward: alpha = min(alpha_max, o 2^power2); entries below alpha_min are
// skipped; compositing stops before an entry that would take T below T_min;
// out = C + T bg, plus T_final and n_contrib (list position + 1 of the last
// blended entry) and, optionally, the number of blended entries.
//
// Backward: the range is replayed from the tile's largest n_contrib down.
// Each pixel recovers T before an entry as T / (1 - alpha) and keeps
// g . (colour behind) as a running scalar, so that
//   dL/dalpha_i = T_i g.c_i - (g.S_i + dL/dT_final T_final) / (1 - alpha_i).
// A lane sums its pixels' 9 screen-space partials of an entry, the wavefront
// reduces them on VALU cross-lane instructions (a transposed exchange of 8
// values in 7 swaps plus 3 DPP adds, and one full sum), and 9 lanes add the
// tile's totals to the slot's double accumulators with one atomic
// instruction (plus one).  Within a pixel the work is branch-free (selects);
// an entry no lane of the wave needs is skipped as a whole, and so are the
// lane's pixels (rows of the tile) that an entry reaches in no lane.
//
// Both passes are bound by VALU issue where the tiles fill the chip (an entry
// costs ~100 instructions of the forward's four pixels a lane, ~260 of the
// backward's, over half of which go to the nine sums of two pixels' partials
// and their reduction), and by one wave's serial chain where they do not.
// Everything about an entry that the lanes share (its tile, position, slot,
// whether it may clamp, whether a lane needs it) is therefore kept on the
// scalar unit, and decided once per batch where it can be: with loops and
// branches left divergent, predicates in vector registers and the clamp and
// position tests on every entry, the backward took 2804 us on ten 1200x680
// views of 1M Gaussians (then 2632) and 10325 us on 36 views of 3M (then
// 9346), the forward 1310 us (then 1277).
//
// An entry that reaches the tile reaches 85-90 % of its rows of pixels there
// (those views hold large Gaussians), but 46 % where Gaussians are small (five
// views of 500k: 27 of 256 pixels on average).  Skipping a row in which no
// lane blends adds nothing to any sum, so the backward always does (one
// scalar branch a row): 1123 -> 815 us on the five views, 2632 -> 2470 and
// 9346 -> 8450 us on the others, 367 -> 300 us on 12 tiles of a 64x48 view.
// The forward's row is half as long, and branches cost it more than they save
// where most rows are reached (1277 -> 1365 us; 8 pixels a lane 4130 -> 4757):
// it takes them in batches of mostly small entries (479 -> 419 us).
#include "kernels.h"

#include <type_traits>

namespace gsr {

#define GSR_LOG2E 1.4426950408889634f
#define GSR_LN2 0.69314718055994531f

// A value that every lane holds alike, in a scalar register: the compiler
// takes what a vector load returns as different between lanes, and the loops
// and branches that depend on it as divergent (exec-mask bookkeeping and
// register copies on every entry).
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

// Predicates of the lanes are kept as 64-bit masks in scalar registers and
// used by the selects from there; as bools they go through a vector register
// wherever two paths meet.
__device__ __forceinline__ uint64_t lanes(bool b) { return __builtin_amdgcn_ballot_w64(b); }
__device__ __forceinline__ bool in(uint64_t mask) { return __builtin_amdgcn_inverse_ballot_w64(mask); }

struct __align__(16) LdsRec {
    float4 p0;  // c0, gx, gy, a2   (power2 at the tile centre and its gradient; a2 = k A)
    float4 p1;  // b2, c2, o, thr   (b2 = 2 k B, c2 = k C, thr = log2(alpha_min / o))
    float4 p2;  // r, g, b, slot bits
    float4 p3;  // ox, oy, 1/o, 2 c2   ((ox, oy) = tile centre - projected centre)
};

// Stages the record of `slot` for the tile centred at (xc, yc).  With
// k = -log2(e) / 2 and o = (xc, yc) - (u, v), the exp2-space power at a pixel
// offset d from the tile centre is
//   power2(d) = k (o + d)^T conic (o + d)
//             = c0 + gx dx + gy dy + a2 dx^2 + b2 dx dy + c2 dy^2,
// c0 = k o^T conic o, (gx, gy) = 2 k conic o, formed here in double: the
// quadratic form of a Gaussian whose centre lies far from the tile cancels
// heavily, and |d| is at most half a tile.
// The staged fields of a slot, from either record format: MIXED reads the
// 32-byte record (float32 centre and conic, binary16 colour).
struct Staged {
    double u, v, A, B, C;
    float o, r, g, b;
};

template <bool MIXED>
__device__ __forceinline__ Staged load_staged(const RasterArgs& a, uint32_t slot)
{
    Staged t;
    if (MIXED) {
        const StageRecM sr = static_cast<const StageRecM*>(a.stage)[slot];
        t.u = sr.u;
        t.v = sr.v;
        t.A = sr.A;
        t.B = sr.B;
        t.C = sr.C;
        t.o = sr.o;
        t.r = __half2float(sr.r);
        t.g = __half2float(sr.g);
        t.b = __half2float(sr.b);
    } else {
        const StageRec sr = static_cast<const StageRec*>(a.stage)[slot];
        t.u = sr.u;
        t.v = sr.v;
        t.A = sr.A;
        t.B = sr.B;
        t.C = sr.C;
        t.o = sr.o;
        t.r = sr.r;
        t.g = sr.g;
        t.b = sr.b;
    }
    return t;
}

// What the batch loops ask of an entry before its batch is walked: its
// opacity, and whether a component of its colour is infinite or NaN.
struct Entry {
    float o;
    bool odd;
};

template <bool MIXED>
__device__ __forceinline__ Entry stage_record(const RasterArgs& a, uint32_t slot, double xc, double yc,
                                              LdsRec& r)
{
    const Staged sr = load_staged<MIXED>(a, slot);
    const double k = -0.5 * 1.4426950408889634;
    const double ox = xc - sr.u, oy = yc - sr.v;
    const double qx = sr.A * ox + sr.B * oy, qy = sr.B * ox + sr.C * oy;
    const float thr = a.cfg.alpha_min > 0.0f ? log2f(a.cfg.alpha_min / sr.o) : -INFINITY;
    r.p0 = make_float4((float)(k * (ox * qx + oy * qy)), (float)(2.0 * k * qx), (float)(2.0 * k * qy),
                       (float)(k * sr.A));
    r.p1 = make_float4((float)(2.0 * k * sr.B), (float)(k * sr.C), sr.o, thr);
    r.p2 = make_float4(sr.r, sr.g, sr.b, __uint_as_float(slot));
    r.p3 = make_float4((float)ox, (float)oy, 1.0f / sr.o, 2.0f * r.p1.y);
    return {sr.o, !(__builtin_isfinite(sr.r) && __builtin_isfinite(sr.g) && __builtin_isfinite(sr.b))};
}

// writes one colour value of the image (float32, or binary16 when MIXED)
template <bool MIXED>
__device__ __forceinline__ void put_rgb(void* rgb, int64_t i, float x)
{
    if (MIXED) static_cast<__half*>(rgb)[i] = __float2half_rn(x);
    else static_cast<float*>(rgb)[i] = x;
}

// The terms of power2 shared by the pixels of one lane (same column offset
// dx), and power2 at row offset dy; the same operation sequence in both
// passes, so that their decisions agree bit for bit.
struct ColTerms {
    float s0;  // c0 + gx dx + a2 dx^2
    float s1;  // gy + b2 dx
};

__device__ __forceinline__ ColTerms col_terms(const LdsRec& r, float dx)
{
    ColTerms t;
    t.s0 = __builtin_fmaf(__builtin_fmaf(r.p0.w, dx, r.p0.y), dx, r.p0.x);
    t.s1 = __builtin_fmaf(r.p1.x, dx, r.p0.z);
    return t;
}

__device__ __forceinline__ float power2(const ColTerms& t, float c2, float dy)
{
    return __builtin_fmaf(__builtin_fmaf(c2, dy, t.s1), dy, t.s0);
}

template <int PPT>
struct TileCtx {
    int tile;                 // global tile of this workgroup
    int px, py0, rs;          // column, first row, row stride
    int width, height, pix_base;
    int64_t base;             // index of row py0 into the concatenated [H][W] planes
    int64_t plane;            // H * W of the view
    double xc, yc;            // tile centre in view pixel coordinates
    float dx;                 // this lane's pixel-centre offset from it (column)
    float dy[PPT];            // and its rows'
    // the lane's k-th pixel: inside the view, its [H][W] index, and its
    // channel-0 index into the concatenated [3][H][W] images (derived when
    // needed rather than held in registers)
    __device__ __forceinline__ bool inside(int k) const { return px < width && py0 + k * rs < height; }
    __device__ __forceinline__ int64_t pix(int k) const { return base + (int64_t)(k * rs) * width; }
    __device__ __forceinline__ int64_t rgb0(int k) const { return pix(k) + 2 * (int64_t)pix_base; }
};

// The lane's PPT pixels of `tile`, starting at pixel k0 of the lane's
// column in the tile (rows (lane >> log2 tw) + (k0 + k) * rs); k0 = 0 and the
// tile's full PPT for a whole tile, a sub-range for a part of a split tile.
template <int PPT>
__device__ __forceinline__ TileCtx<PPT> tile_ctx_at(const RasterArgs& a, int tile, int k0)
{
    TileCtx<PPT> c;
    c.tile = tile;
    const int v = view_of_tile(a.views, tile);
    const ViewInfo& vw = a.views->v[v];
    const int lt = tile - vw.tile_base;
    const int ty = lt / vw.tiles_x;
    const int tx = lt - ty * vw.tiles_x;
    const int lane = threadIdx.x & 63;
    const int l2 = a.cfg.log2_tw;
    c.px = tx * a.cfg.tile_w + (lane & (a.cfg.tile_w - 1));
    c.rs = 64 >> l2;
    c.py0 = ty * a.cfg.tile_h + (lane >> l2) + k0 * c.rs;
    c.plane = (int64_t)vw.width * vw.height;
    c.xc = (double)(tx * a.cfg.tile_w) + 0.5 * a.cfg.tile_w;
    c.yc = (double)(ty * a.cfg.tile_h) + 0.5 * a.cfg.tile_h;
    c.dx = (float)(lane & (a.cfg.tile_w - 1)) + 0.5f - 0.5f * (float)a.cfg.tile_w;
    c.width = vw.width;
    c.height = vw.height;
    c.pix_base = vw.pix_base;
    c.base = (int64_t)vw.pix_base + (int64_t)c.py0 * vw.width + c.px;
#pragma unroll
    for (int k = 0; k < PPT; ++k)
        c.dy[k] = (float)((lane >> l2) + (k0 + k) * c.rs) + 0.5f - 0.5f * (float)a.cfg.tile_h;
    return c;
}

// the workgroup's tile (processing order) and all of its pixels
template <int PPT>
__device__ __forceinline__ TileCtx<PPT> tile_ctx(const RasterArgs& a)
{
    return tile_ctx_at<PPT>(a, uniform((int)a.order[blockIdx.x]), 0);
}

// the tile's pairs, empty after an overflow
__device__ __forceinline__ uint2 tile_range(const RasterArgs& a, int tile)
{
    const uint2 r = a.ranges[tile];
    return make_uint2((uint32_t)uniform((int)r.x), (uint32_t)uniform((int)r.y));
}

// Whether an entry of opacity o can have a clamped alpha anywhere (alpha =
// o G with G <= 1): !(o < alpha_max).  Both are positive floats, whose order
// is their bit patterns' order (a NaN of either sign is above all of them, as
// unsigned numbers), so the test runs on the scalar unit with the first
// lane's o (the staged record is the same for every lane).
__device__ __forceinline__ bool may_clamp(float o, float amax)
{
    return (uint32_t)__builtin_amdgcn_readfirstlane(__float_as_int(o)) >= __float_as_uint(amax);
}

// Whether the rows in which the entry can reach alpha_min lie within `half`
// of its centre: with power2 = -log2(e)/2 d^T conic d, the rows at which it
// is at least thr satisfy dy^2 <= -2 ln 2 thr A / (A C - B^2), and (a2, b2 / 2,
// c2) are (A, B, C) scaled by -log2(e)/2.  A rule for speed only.
__device__ __forceinline__ bool few_rows(const LdsRec& r, float half)
{
    const float det = r.p0.w * r.p1.y - 0.25f * r.p1.x * r.p1.x;
    return r.p1.w * r.p0.w <= half * half * det;
}

// Walks the batch in LDS for the lane's pixels.  A pixel that has stopped
// (or lies outside the view) carries a NaN row offset, so every later test
// power2 >= thr fails for it without a per-pixel flag.  Reaching T_min is
// rare (once per pixel at most), so the common step applies every passing
// entry and a wave-uniform branch undoes the blend of stopping pixels.
// CLAMPS: the batch holds an entry that may clamp, so every entry is asked.
// SMALL: most entries reach few of the lane's pixels' rows, and only the rows
// that an entry reaches are composited (each a branch).
template <int PPT, bool COUNT, bool CLAMPS, bool SMALL>
__device__ __forceinline__ void fwd_batch(const LdsRec* rec, int cnt, uint32_t pos0, float amax, float tmin,
                                          float dx, float (&dy)[PPT], float (&T)[PPT], float (&C0)[PPT],
                                          float (&C1)[PPT], float (&C2)[PPT], uint32_t (&last)[PPT],
                                          uint32_t (&nb)[PPT])
{
    for (int e = 0; e < cnt; ++e) {
        if ((e & 15) == 0) {
            uint64_t live = 0;
#pragma unroll
            for (int k = 0; k < PPT; ++k) live |= __builtin_amdgcn_ballot_w64(dy[k] == dy[k]);
            if (live == 0) break;
        }
        const LdsRec r = rec[e];
        const ColTerms ct = col_terms(r, dx);
        float p2[PPT];
        uint64_t pass[PPT], any = 0;
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            p2[k] = power2(ct, r.p1.y, dy[k]);
            pass[k] = lanes(p2[k] >= r.p1.w);
            any |= pass[k];
        }
        if (any == 0) continue;
        const uint32_t pos1 = pos0 + (uint32_t)e + 1u;
        uint64_t stop[PPT], any_stop = 0;
        if (SMALL) {
#pragma unroll
            for (int k = 0; k < PPT; ++k) {
                stop[k] = 0;
                if (pass[k] == 0) continue;
                const float a_raw = r.p1.z * __builtin_amdgcn_exp2f(p2[k]);
                const float al = CLAMPS ? fminf(amax, a_raw) : a_raw;
                const float Tn = __builtin_fmaf(-T[k], al, T[k]);
                stop[k] = lanes(Tn < tmin) & pass[k];
                any_stop |= stop[k];
                const uint64_t blend = pass[k] & ~stop[k];
                const float wgt = (in(blend) ? al : 0.0f) * T[k];
                C0[k] = __builtin_fmaf(r.p2.x, wgt, C0[k]);
                C1[k] = __builtin_fmaf(r.p2.y, wgt, C1[k]);
                C2[k] = __builtin_fmaf(r.p2.z, wgt, C2[k]);
                T[k] = in(blend) ? Tn : T[k];
                last[k] = in(blend) ? pos1 : last[k];
                if (COUNT) nb[k] += in(blend) ? 1u : 0u;
            }
            if (any_stop != 0) {
#pragma unroll
                for (int k = 0; k < PPT; ++k) dy[k] = in(stop[k]) ? __builtin_nanf("") : dy[k];
            }
            continue;
        }
        float ab[PPT], Tn[PPT];
        if (CLAMPS && may_clamp(r.p1.z, amax)) {
#pragma unroll
            for (int k = 0; k < PPT; ++k)
                ab[k] = in(pass[k]) ? fminf(amax, r.p1.z * __builtin_amdgcn_exp2f(p2[k])) : 0.0f;
        } else {
#pragma unroll
            for (int k = 0; k < PPT; ++k) ab[k] = in(pass[k]) ? r.p1.z * __builtin_amdgcn_exp2f(p2[k]) : 0.0f;
        }
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            Tn[k] = __builtin_fmaf(-T[k], ab[k], T[k]);
            stop[k] = lanes(Tn[k] < tmin);
            any_stop |= stop[k];
        }
        if (any_stop != 0) {
#pragma unroll
            for (int k = 0; k < PPT; ++k) {
                ab[k] = in(stop[k]) ? 0.0f : ab[k];
                Tn[k] = in(stop[k]) ? T[k] : Tn[k];
                dy[k] = in(stop[k]) ? __builtin_nanf("") : dy[k];
                pass[k] &= ~stop[k];
            }
        }
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            const float wgt = ab[k] * T[k];
            C0[k] = __builtin_fmaf(r.p2.x, wgt, C0[k]);
            C1[k] = __builtin_fmaf(r.p2.y, wgt, C1[k]);
            C2[k] = __builtin_fmaf(r.p2.z, wgt, C2[k]);
            T[k] = Tn[k];
            last[k] = in(pass[k]) ? pos1 : last[k];
            if (COUNT) nb[k] += in(pass[k]) ? 1u : 0u;
        }
    }
}

// The same walk four entries at a time, for waves that run (nearly) alone on
// their SIMD: the four alphas are independent, and only T passes from one to
// the next.  T never grows, so no pixel stops within the four unless it ends
// below T_min (or NaN); then they are taken one by one.  Records cnt .. up to
// a multiple of four must be null (thr = +inf).
template <int PPT, bool COUNT>
__device__ __forceinline__ void fwd_batch4(const LdsRec* rec, int cnt, uint32_t pos0, float amax, float tmin,
                                           float dx, float (&dy)[PPT], float (&T)[PPT], float (&C0)[PPT],
                                           float (&C1)[PPT], float (&C2)[PPT], uint32_t (&last)[PPT],
                                           uint32_t (&nb)[PPT])
{
    constexpr int U = 4;
    for (int e = 0; e < cnt; e += U) {
        if ((e & 15) == 0) {
            uint64_t live = 0;
#pragma unroll
            for (int k = 0; k < PPT; ++k) live |= __builtin_amdgcn_ballot_w64(dy[k] == dy[k]);
            if (live == 0) break;
        }
        LdsRec r[U];
#pragma unroll
        for (int u = 0; u < U; ++u) r[u] = rec[e + u];
        float ab[U][PPT];
        uint64_t pass[U][PPT], any = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const ColTerms ct = col_terms(r[u], dx);
#pragma unroll
            for (int k = 0; k < PPT; ++k) {
                ab[u][k] = power2(ct, r[u].p1.y, dy[k]);
                pass[u][k] = lanes(ab[u][k] >= r[u].p1.w);
                any |= pass[u][k];
            }
        }
        if (any == 0) continue;
        float t[U + 1][PPT];
        uint64_t stop = 0;
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            t[0][k] = T[k];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float a_raw = r[u].p1.z * __builtin_amdgcn_exp2f(ab[u][k]);
                ab[u][k] = in(pass[u][k]) ? fminf(amax, a_raw) : 0.0f;
                t[u + 1][k] = __builtin_fmaf(-t[u][k], ab[u][k], t[u][k]);
            }
            stop |= lanes(!(t[U][k] >= tmin));
        }
        const uint32_t pos1 = pos0 + (uint32_t)e + 1u;
        if (stop != 0) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int k = 0; k < PPT; ++k) {
                    // (a pixel that stops passes none of the later three)
                    const uint64_t now = pass[u][k] & lanes(dy[k] == dy[k]);
                    const float al = in(now) ? ab[u][k] : 0.0f;
                    const float Tn = __builtin_fmaf(-T[k], al, T[k]);
                    const uint64_t stops = lanes(Tn < tmin), blend = now & ~stops;
                    const float wgt = (in(stops) ? 0.0f : al) * T[k];
                    C0[k] = __builtin_fmaf(r[u].p2.x, wgt, C0[k]);
                    C1[k] = __builtin_fmaf(r[u].p2.y, wgt, C1[k]);
                    C2[k] = __builtin_fmaf(r[u].p2.z, wgt, C2[k]);
                    T[k] = in(stops) ? T[k] : Tn;
                    dy[k] = in(stops) ? __builtin_nanf("") : dy[k];
                    last[k] = in(blend) ? pos1 + (uint32_t)u : last[k];
                    if (COUNT) nb[k] += in(blend) ? 1u : 0u;
                }
            }
            continue;
        }
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float wgt = ab[u][k] * t[u][k];
                C0[k] = __builtin_fmaf(r[u].p2.x, wgt, C0[k]);
                C1[k] = __builtin_fmaf(r[u].p2.y, wgt, C1[k]);
                C2[k] = __builtin_fmaf(r[u].p2.z, wgt, C2[k]);
                last[k] = in(pass[u][k]) ? pos1 + (uint32_t)u : last[k];
                if (COUNT) nb[k] += in(pass[u][k]) ? 1u : 0u;
            }
            T[k] = t[U][k];
        }
    }
}

// A colour that is infinite or NaN belongs to the pixels that blend it alone,
// but the loops add 0 times an entry's colour to the wave's other pixels, and
// the four-at-a-time loop also that of an entry that no pixel takes.  Its odd
// components are therefore staged as 0, a batch with such a colour is walked
// entry by entry, and the pixels that have blended the entry (its position is
// their last) get the components then.
__device__ __forceinline__ void hide_odd(LdsRec& r)
{
    r.p2.x = __builtin_isfinite(r.p2.x) ? r.p2.x : 0.0f;
    r.p2.y = __builtin_isfinite(r.p2.y) ? r.p2.y : 0.0f;
    r.p2.z = __builtin_isfinite(r.p2.z) ? r.p2.z : 0.0f;
}

template <int PPT, bool MIXED>
__device__ __forceinline__ void add_odd(const RasterArgs& a, const LdsRec& r, uint32_t pos1, const uint32_t (&last)[PPT],
                                        float (&C0)[PPT], float (&C1)[PPT], float (&C2)[PPT])
{
    const Staged t = load_staged<MIXED>(a, __float_as_uint(r.p2.w));
    const float x = t.r - r.p2.x, y = t.g - r.p2.y, z = t.b - r.p2.z;
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        C0[k] += last[k] == pos1 ? x : 0.0f;
        C1[k] += last[k] == pos1 ? y : 0.0f;
        C2[k] += last[k] == pos1 ? z : 0.0f;
    }
}

// COUNT: also count the blended entries per pixel (into a.n_blend); a
// separate instantiation, so that the plain forward carries no counters.
// ALONE: the waves are too few to hide each other's latencies (fwd_batch4).
template <int PPT, int GSR_BATCH, bool COUNT, bool MIXED, bool ALONE>
__device__ __forceinline__ void fwd_tile(const RasterArgs& a, const TileCtx<PPT>& c, LdsRec* rec)
{
    const int lane = threadIdx.x;
    const bool overflow = uniform((int)a.counters->overflow) != 0;
    const uint2 range = overflow ? make_uint2(0u, 0u) : tile_range(a, c.tile);
    const float amax = a.cfg.alpha_max, tmin = a.cfg.T_min;
    float T[PPT], C0[PPT], C1[PPT], C2[PPT], dy[PPT];
    uint32_t last[PPT], nb[PPT];
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        T[k] = 1.0f;
        C0[k] = C1[k] = C2[k] = 0.0f;
        last[k] = nb[k] = 0u;
        dy[k] = c.inside(k) ? c.dy[k] : __builtin_nanf("");
    }
    for (uint32_t base = range.x; base < range.y; base += GSR_BATCH) {
        uint64_t live = 0;
#pragma unroll
        for (int k = 0; k < PPT; ++k) live |= __builtin_amdgcn_ballot_w64(dy[k] == dy[k]);
        if (live == 0) break;
        bool may = false, small = false, odd = false;
#pragma unroll
        for (int r = 0; r < GSR_BATCH / 64; ++r) {
            const uint32_t j = base + lane + 64 * r;
            if (j < range.y) {
                const Entry e = stage_record<MIXED>(a, a.vals[j], c.xc, c.yc, rec[lane + 64 * r]);
                may |= !(e.o < amax);
                odd |= e.odd;
                if (e.odd) hide_odd(rec[lane + 64 * r]);
                if (!ALONE && PPT == 4 && r == 0) small = few_rows(rec[lane], 0.375f * (float)a.cfg.tile_h);
            } else if (ALONE) {
                rec[lane + 64 * r].p0 = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                rec[lane + 64 * r].p1 = make_float4(0.0f, 0.0f, 0.0f, INFINITY);
                rec[lane + 64 * r].p2 = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            }
        }
        const uint64_t few = lanes(small);
        const bool clamps = lanes(may) != 0, odds = lanes(odd) != 0;
        __syncthreads();
        const int cnt = (int)min((uint32_t)GSR_BATCH, range.y - base);
        const uint32_t pos0 = base - range.x;
        // small entries: more than half of the batch's first 64 reach no more
        // than three quarters of the tile's rows (half of them measured 428 us
        // for 419 at the five views of 500k Gaussians); with fewer than four
        // rows a lane there is little to skip.  With 8 pixels per lane a
        // second copy of the loop costs registers that the waves need more
        // (96 and spills instead of 88)
        if (ALONE && !odds) {
            fwd_batch4<PPT, COUNT>(rec, cnt, pos0, amax, tmin, c.dx, dy, T, C0, C1, C2, last, nb);
            __syncthreads();
            continue;
        }
        const int step = odds ? 1 : cnt;
        for (int e = 0; e < cnt; e += step) {
            const LdsRec* at = rec + e;
            const uint32_t p = pos0 + (uint32_t)e;
            if (!ALONE && PPT == 4 && 2 * __popcll(few) > cnt / (GSR_BATCH / 64))
                fwd_batch<PPT, COUNT, true, PPT == 4>(at, step, p, amax, tmin, c.dx, dy, T, C0, C1, C2, last, nb);
            else if (ALONE || PPT > 4 || clamps)
                fwd_batch<PPT, COUNT, true, false>(at, step, p, amax, tmin, c.dx, dy, T, C0, C1, C2, last, nb);
            else
                fwd_batch<PPT, COUNT, false, false>(at, step, p, amax, tmin, c.dx, dy, T, C0, C1, C2, last, nb);
            if (odds) add_odd<PPT, MIXED>(a, *at, p + 1u, last, C0, C1, C2);
        }
        __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        if (!c.inside(k)) continue;
        if (overflow) {
            const float q = __builtin_nanf("");
            put_rgb<MIXED>(a.rgb, c.rgb0(k), q);
            put_rgb<MIXED>(a.rgb, c.rgb0(k) + c.plane, q);
            put_rgb<MIXED>(a.rgb, c.rgb0(k) + 2 * c.plane, q);
            a.T_final[c.pix(k)] = q;
            a.n_contrib[c.pix(k)] = 0;
            if (COUNT) a.n_blend[c.pix(k)] = 0;
            continue;
        }
        put_rgb<MIXED>(a.rgb, c.rgb0(k), __builtin_fmaf(T[k], a.cfg.bg0, C0[k]));
        put_rgb<MIXED>(a.rgb, c.rgb0(k) + c.plane, __builtin_fmaf(T[k], a.cfg.bg1, C1[k]));
        put_rgb<MIXED>(a.rgb, c.rgb0(k) + 2 * c.plane, __builtin_fmaf(T[k], a.cfg.bg2, C2[k]));
        a.T_final[c.pix(k)] = T[k];
        a.n_contrib[c.pix(k)] = (int32_t)last[k];
        if (COUNT) a.n_blend[c.pix(k)] = (int32_t)nb[k];
    }
}

// The longest tiles are split: a wave's time is its tile's list, and the
// few longest lists would otherwise run alone at the end of the launch
// (measured: emptying the longest 1 % of the tiles at window-1M-10views,
// 5 % of the pairs, shortened the forward by 16 %).  A tile is long when
// its list holds at least half the pairs a resident wave would composite
// with the step's pairs spread evenly (GSR_FWD_WAVES resident waves), and
// at least GSR_FWD_LONG, rounded up to a power of two.  The processing
// order puts such tiles first (it is bucketed by floor(log2 length)), so
// they are the order's first K tiles, found by binary search.  Each is
// composited as FWD_SPLIT(PPT) parts, every part a wave with PPT / split of
// the lane's pixels and the whole list; a pixel's arithmetic is the same
// either way.  Splitting costs each part the whole list's per-entry work,
// so it pays only for the tail: where most tiles' lists are long (the
// 3M-Gaussian mapping views) the threshold rises with the pair count.
#ifndef GSR_FWD_SPLIT_MAX
#define GSR_FWD_SPLIT_MAX 4   // parts of the longest tiles (twice the threshold or more)
#endif
#ifndef GSR_FWD_LONG_PRIO
#define GSR_FWD_LONG_PRIO 2   // issue priority of the long tiles' waves (s_setprio, 0..3)
#endif

template <int PPT>
struct FwdSplit {
    static constexpr int parts = PPT < GSR_FWD_SPLIT ? PPT : GSR_FWD_SPLIT;
    static constexpr int ppt = PPT / parts;
    // tiles of twice the threshold or more: more parts, fewer pixels each
    static constexpr int parts2 = PPT < GSR_FWD_SPLIT_MAX ? PPT : (GSR_FWD_SPLIT_MAX < parts ? parts : GSR_FWD_SPLIT_MAX);
    static constexpr int ppt2 = PPT / parts2;
};

__device__ __forceinline__ uint32_t long_threshold(const RasterArgs& a)
{
    const unsigned long long even = a.counters->pairs / (2ull * GSR_FWD_WAVES);
    uint32_t t = GSR_FWD_LONG;
    while ((unsigned long long)t < even && t < (1u << 30)) t <<= 1;
    return t;
}

__device__ __forceinline__ int long_tiles(const RasterArgs& a, int total_tiles, uint32_t thr)
{
    int lo = 0, hi = total_tiles;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        const uint2 r = a.ranges[a.order[mid]];
        if (r.y - r.x < thr) hi = mid;
        else lo = mid + 1;
    }
    return lo;
}

template <int PPT, int GSR_BATCH, bool COUNT, bool MIXED>
__global__ __launch_bounds__(64, 5) void k_raster_fwd(RasterArgs a)
{
    __shared__ LdsRec rec[GSR_BATCH];
    const TileCtx<PPT> c = tile_ctx<PPT>(a);
    if (FwdSplit<PPT>::parts > 1) {
        const uint2 r = tile_range(a, c.tile);
        if (r.y - r.x >= long_threshold(a)) return;  // composited in parts by k_raster_fwd_long
    }
    fwd_tile<PPT, GSR_BATCH, COUNT, MIXED, false>(a, c, rec);
}

// Few tiles: every tile in PARTS parts, each a wave with PPT / PARTS of the
// lane's pixels and the whole list.  A lone wave's entry takes 650 cycles,
// two and a half times its issue (the chain of LDS read, alpha, T and the
// branches): 12 tiles of 716 entries 196 us, 1200 tiles of 162 (up to 332)
// entries 92 us, 825 of 104 77 us.  In four parts of one pixel a lane, four
// entries at a time, these take 67, 46 and 32 us; 3225 tiles of 318 entries,
// in two parts, 197 -> 155 us (in four 182: the parts' record reads fill the
// LDS; two entries at a time 162; records read ahead into registers 174).
template <int PPT, int PARTS, int GSR_BATCH, bool COUNT, bool MIXED>
__global__ __launch_bounds__(64, PPT / PARTS <= 2 ? 6 : 4) void k_raster_fwd_few(RasterArgs a)
{
    constexpr int Q = PPT / PARTS;
    __shared__ LdsRec rec[GSR_BATCH];
    const int tile = uniform((int)a.order[blockIdx.x / PARTS]);
    const TileCtx<Q> c = tile_ctx_at<Q>(a, tile, (int)(blockIdx.x % PARTS) * Q);
    fwd_tile<Q, GSR_BATCH, COUNT, MIXED, true>(a, c, rec);
}

// Persistent waves that take (long tile, part) items from a queue (zeroed
// before the launch) until the long tiles' parts are done.  The K2 tiles of
// twice the threshold or more (the order's first) come in parts2 parts, the
// others in parts; items go longest tile first.  The waves raise their issue
// priority: each carries a whole list and ends the forward, while the short
// tiles' waves beside them on the same SIMDs can wait a little.
template <int PPT, int GSR_BATCH, bool COUNT, bool MIXED>
__global__ __launch_bounds__(64, 5) void k_raster_fwd_long(RasterArgs a, int total_tiles)
{
    using F = FwdSplit<PPT>;
    constexpr int S = F::parts, Q = F::ppt, S2 = F::parts2, Q2 = F::ppt2;
    __shared__ LdsRec rec[GSR_BATCH];
    if (GSR_FWD_LONG_PRIO) __builtin_amdgcn_s_setprio(GSR_FWD_LONG_PRIO);
    const uint32_t thr = long_threshold(a);
    const int k2 = S2 > S ? long_tiles(a, total_tiles, 2u * thr) : 0;
    const int items2 = k2 * S2;
    const int items = items2 + (long_tiles(a, total_tiles, thr) - k2) * S;
    for (;;) {
        uint32_t item = 0u;
        if (threadIdx.x == 0) item = atomicAdd(a.fwd_queue, 1u);
        item = (uint32_t)__builtin_amdgcn_readfirstlane((int)item);
        if ((int)item >= items) break;
        if ((int)item < items2) {
            const int tile = (int)a.order[item / S2];
            const TileCtx<Q2> c = tile_ctx_at<Q2>(a, tile, (int)(item % S2) * Q2);
            fwd_tile<Q2, GSR_BATCH, COUNT, MIXED, false>(a, c, rec);
        } else {
            const uint32_t j = item - (uint32_t)items2;
            const int tile = (int)a.order[k2 + (int)(j / S)];
            const TileCtx<Q> c = tile_ctx_at<Q>(a, tile, (int)(j % S) * Q);
            fwd_tile<Q, GSR_BATCH, COUNT, MIXED, false>(a, c, rec);
        }
    }
}

__global__ void k_zero_queue(uint32_t* q)
{
    *q = 0u;
}

// scale of field f (du, dv, dA, dB, dC, -, dr, dg, db) from the reduced
// power2-space partials to the screen-space gradient (the opacity field is
// scaled by the record's 1/o)
__device__ __forceinline__ float field_scale(int f)
{
    return f < 2 ? -GSR_LN2 : (f == 3 ? -1.0f : (f < 5 ? -0.5f : 1.0f));
}

// Deterministic mode: the tile totals are added exactly, as fixed-point
// numbers, so that the sums do not depend on the order in which tiles run.
// A field is held in GSR_FIX_LIMBS signed 64-bit limbs; limb k collects the
// bits [32 k, 32 k + 32) of every addend (the lowest bit weighing
// 2^-GSR_FIX_UNIT) with its sign, without carries, which leaves 31 bits of
// headroom for the count of addends.  A float addend M 2^(E - 150) (M its
// 24-bit significand) spans at most two limbs: two integer atomics, no
// return value.  A slot's limbs are stored limb-major ([limb][field], 72
// bytes per limb), so that the 9 lanes of an entry's first atomic mostly
// hit one 72-byte block, as the FP64 path's do.  Bits below 2^-96 are
// dropped (truncation toward zero); magnitudes of 2^32 and beyond,
// infinities and NaN saturate to just below 2^32.
__device__ __forceinline__ void fixed_add(unsigned long long* limbs, int stride, float v)
{
    const uint32_t bits = __float_as_uint(v);
    const int E = (int)((bits >> 23) & 0xffu);
    if (E == 0) return;  // zero or subnormal: below the lowest bit
    uint32_t M = (bits & 0x7fffffu) | 0x800000u;
    int p = E - 150 + GSR_FIX_UNIT;  // weight 2^(p - 96) of M's lowest bit
    if (p > 32 * (GSR_FIX_LIMBS - 1) + 8) {
        M = 0xffffffu;
        p = 32 * (GSR_FIX_LIMBS - 1) + 8;
    }
    if (p < 0) {
        if (p <= -24) return;
        M >>= -p;
        p = 0;
    }
    const int k = p >> 5;
    const unsigned long long wide = (unsigned long long)M << (p & 31);
    const unsigned long long c0 = wide & 0xffffffffull, c1 = wide >> 32;
    const bool neg = (bits >> 31) != 0u;
    atomicAdd(&limbs[k * stride], neg ? 0ull - c0 : c0);
    if (c1 != 0ull && k + 1 < GSR_FIX_LIMBS) atomicAdd(&limbs[(k + 1) * stride], neg ? 0ull - c1 : c1);
}

// the value of a fixed-point field: carries propagated upwards (limbs 0..2
// end in [0, 2^32), the top limb keeps the sign); a negative total is
// negated and normalised again, so that the magnitude is summed from the
// top without cancellation
__device__ __forceinline__ double fixed_value(const unsigned long long* limbs, int stride)
{
    long long c[GSR_FIX_LIMBS];
#pragma unroll
    for (int k = 0; k < GSR_FIX_LIMBS; ++k) c[k] = (long long)limbs[k * stride];
#pragma unroll
    for (int k = 0; k + 1 < GSR_FIX_LIMBS; ++k) {
        c[k + 1] += c[k] >> 32;
        c[k] &= 0xffffffffll;
    }
    const bool neg = c[GSR_FIX_LIMBS - 1] < 0;
    if (neg) {
#pragma unroll
        for (int k = 0; k < GSR_FIX_LIMBS; ++k) c[k] = -c[k];
#pragma unroll
        for (int k = 0; k + 1 < GSR_FIX_LIMBS; ++k) {
            c[k + 1] += c[k] >> 32;
            c[k] &= 0xffffffffll;
        }
    }
    // the top limb's lowest bit weighs 2^(32 (limbs - 1) - unit) = 1
    static_assert(32 * (GSR_FIX_LIMBS - 1) == GSR_FIX_UNIT, "the top limb counts units of 1");
    double v = (double)c[0];
#pragma unroll
    for (int k = 1; k < GSR_FIX_LIMBS; ++k) v = (double)c[k] + v * 0x1p-32;
    return neg ? -v : v;
}

// Counts the tile as done for its view; the tile completing a whole
// backward of the view (the view's count reaching a multiple of its tiles:
// the count runs on across backward calls, so it needs no reset) stamps the
// view's completion time.
__device__ __forceinline__ void view_done(const RasterArgs& a, int tile, int lane)
{
    if (lane != 0) return;
    const int v = view_of_tile(a.views, tile);
    const unsigned long long tiles = (unsigned long long)(a.views->v[v].tiles_x * a.views->v[v].tiles_y);
    const unsigned long long old = atomicAdd(&a.tiles_done[v], 1ull);
    if ((old + 1ull) % tiles == 0ull) a.stamps[v] = (unsigned long long)wall_clock64();
}

// Adds a tile's total of screen-space field f to slot's accumulator: an FP64
// atomic, or (deterministic mode) the exact fixed-point limbs.
template <bool DET>
__device__ __forceinline__ void add_field(const RasterArgs& a, uint32_t slot, int f, float value)
{
    if (DET) fixed_add(a.acc + GSR_G2 * GSR_FIX_LIMBS * (int64_t)slot + f, GSR_G2, value);
    else atomic_add_f64(a.grad2d + GSR_G2 * (uint64_t)slot + (uint32_t)f, (double)value);
}

// The ninth field (the blue colour partial) of a reduced entry waits for the
// next reduced entry's, and the two are summed over the wave in one chain
// (wave_sum_pair); slot is wave-uniform.
struct PendingField {
    int have;
    int slot;
    float w;
};

// The sums of an entry's terms over a lane's pixels.
struct PixelSums {
    float D = 0.0f, Dy = 0.0f, Dyy = 0.0f, c0 = 0.0f, c1 = 0.0f, c2 = 0.0f;
    // a pixel's dd = alpha dL/dalpha and weight, its upstream gradient and
    // its row offset (and that squared)
    __device__ __forceinline__ void add(float dd, float wgt, float g0, float g1, float g2, float dy, float dyy)
    {
        c0 = __builtin_fmaf(g0, wgt, c0);
        c1 = __builtin_fmaf(g1, wgt, c1);
        c2 = __builtin_fmaf(g2, wgt, c2);
        D += dd;
        Dy = __builtin_fmaf(dd, dy, Dy);
        Dyy = __builtin_fmaf(dd, dyy, Dyy);
    }
    // the same with the upstream gradient left out where the weight is 0
    __device__ __forceinline__ void add_own(float2 t, float g0, float g1, float g2, float dy, float dyy)
    {
        const bool own = t.y != 0.0f;
        add(t.x, t.y, own ? g0 : 0.0f, own ? g1 : 0.0f, own ? g2 : 0.0f, dy, dyy);
    }
};

// The lane's nine screen-space partials of an entry.  power2 partials per
// pixel: d/du = -(2 a2 dx + b2 dy + gx), d/dv = -(b2 dx + 2 c2 dy + gy) (d =
// pixel - tile centre), and d/d(A, B, C) = k (fx^2, 2 fx fy, fy^2) with (fx,
// fy) = d + o the offset from the projected centre; d alpha / d o = alpha / o.
__device__ __forceinline__ void bwd_partials(const LdsRec& r, const ColTerms& ct, float dx, const PixelSums& p,
                                             float (&v)[9])
{
    const float fx = dx + r.p3.x;
    const float Fy = __builtin_fmaf(r.p3.y, p.D, p.Dy);  // sum dd fy
    // (2 a2 dx as a2 (2 dx): the same product, with 2 dx a constant of the lane)
    v[0] = __builtin_fmaf(__builtin_fmaf(r.p0.w, 2.0f * dx, r.p0.y), p.D, r.p1.x * p.Dy);
    v[1] = __builtin_fmaf(ct.s1, p.D, r.p3.w * p.Dy);
    v[2] = fx * (fx * p.D);
    v[3] = fx * Fy;
    v[4] = __builtin_fmaf(r.p3.y, Fy + p.Dy, p.Dyy);
    v[5] = p.D;
    v[6] = p.c0;
    v[7] = p.c1;
    v[8] = p.c2;
}

// Adds an entry's first eight reduced fields (lane 8 f holds field f's).
template <bool DET>
__device__ __forceinline__ void bwd_add8(const RasterArgs& a, uint32_t slot, float s, float inv_o, int lane)
{
    if ((lane & 7) != 0) return;
    const int f = lane >> 3;
    const float value = s * (f == 5 ? inv_o : field_scale(f));
    if (DET) {
        add_field<DET>(a, slot, f, value);
    } else {
        // the slot's address stays scalar (left to itself the compiler folds
        // it into a 64-bit multiply-add per lane)
        uint64_t base = (uint64_t)a.grad2d + sizeof(double) * GSR_G2 * (uint64_t)slot;
        asm("" : "+s"(base));
        typedef __attribute__((address_space(1))) double global_double;
        __builtin_amdgcn_global_atomic_fadd_f64(reinterpret_cast<global_double*>(base) + (uint32_t)f, (double)value);
    }
}

// The wave's reduction of an entry's partials and their addition to the
// slot's accumulators.
template <bool DET>
__device__ __forceinline__ void bwd_reduce(const RasterArgs& a, const LdsRec& r, const ColTerms& ct, float dx,
                                           const PixelSums& p, int lane, PendingField& pend)
{
    float v[9];
    bwd_partials(r, ct, dx, p, v);
    const float s = wave_sum8_transposed(v, lane);
    const uint32_t slot = (uint32_t)uniform(__float_as_int(r.p2.w));
    bwd_add8<DET>(a, slot, s, r.p3.z, lane);
    if (uniform(pend.have)) {
        // lane 1 holds the waiting entry's total, lane 33 this one's
        const float w = wave_sum_pair(pend.w, v[8]);
        if ((lane & 31) == 1) add_field<DET>(a, lane < 32 ? (uint32_t)pend.slot : slot, 8, w);
        pend.have = 0;
    } else {
        pend.w = v[8];
        pend.slot = (int)slot;
        pend.have = 1;
    }
}

// One entry of the backward replay for the lane's pixels, then the wave's
// reduction (bwd_reduce).  Per pixel, with rcp = 1 / (1 - alpha), T_j = T
// rcp the transmittance before the entry, gcol = g . c and gsk the running
// g . (colour behind) + dL/dT_final T_final:
//   dL/dalpha = T_j gcol - gsk rcp,
//   gsk'      = gsk + alpha T_j gcol,
//   dd        = alpha dL/dalpha = gsk' - gsk rcp   (one FMA);
// a pixel the entry does not reach takes alpha = 0, for which rcp(1) = 1
// exactly, so T, gsk and every partial stay unchanged without selects.
// CLAMP: the entry may clamp at alpha_max (o >= alpha_max), where alpha has
// no gradient (dd = 0) but still attenuates.  ODD: an upstream gradient or a
// colour of the tile is infinite or NaN; it reaches the entries that its
// pixels blend (0 times it would reach the others as well), so the pixels
// that the entry does not reach are left out by selects.
template <int PPT, bool CLAMP, bool DET, bool ODD>
__device__ __forceinline__ void bwd_entry(const RasterArgs& a, const LdsRec& r, const ColTerms& ct,
                                          const float (&p2)[PPT], const uint64_t (&on)[PPT], float amax,
                                          const TileCtx<PPT>& c, const float (&g0)[PPT], const float (&g1)[PPT],
                                          const float (&g2)[PPT], const float (&dy2)[PPT], float (&T)[PPT],
                                          float (&gsk)[PPT], int lane, PendingField& pend)
{
    PixelSums p;
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        if (on[k] == 0) continue;
        const float a_raw = r.p1.z * __builtin_amdgcn_exp2f(p2[k]);
        const float alpha = in(on[k]) ? (CLAMP ? fminf(a_raw, amax) : a_raw) : 0.0f;
        const float rcp = __builtin_amdgcn_rcpf(1.0f - alpha);
        const float Tb = T[k] * rcp;
        float gcol = __builtin_fmaf(g0[k], r.p2.x, __builtin_fmaf(g1[k], r.p2.y, g2[k] * r.p2.z));
        if (ODD) gcol = in(on[k]) ? gcol : 0.0f;
        const float wgt = alpha * Tb;
        const float gsk_new = __builtin_fmaf(wgt, gcol, gsk[k]);
        float dd = __builtin_fmaf(-gsk[k], rcp, gsk_new);
        if (CLAMP) dd = a_raw < amax ? dd : 0.0f;
        if (ODD) dd = in(on[k]) ? dd : 0.0f;
        gsk[k] = gsk_new;
        T[k] = Tb;
        if (ODD)
            p.add(dd, wgt, in(on[k]) ? g0[k] : 0.0f, in(on[k]) ? g1[k] : 0.0f, in(on[k]) ? g2[k] : 0.0f, c.dy[k], dy2[k]);
        else
            p.add(dd, wgt, g0[k], g1[k], g2[k], c.dy[k], dy2[k]);
    }
    bwd_reduce<DET>(a, r, ct, c.dx, p, lane, pend);
}

// The staged entries rec[0, cnt), from the list's position top down.
// CLAMPS: the batch holds an entry that may clamp, so every entry is asked
// (alpha = o G <= o: a test uniform over the wave); FULL: every pixel of the
// tile blended an entry at top or behind it, so no position is tested; ODD as
// for bwd_entry.
template <int PPT, bool CLAMPS, bool FULL, bool DET, bool ODD>
__device__ __forceinline__ void bwd_batch(const RasterArgs& a, const LdsRec* rec, int cnt, uint32_t top, float amax,
                                          const TileCtx<PPT>& c, const uint32_t (&my_n)[PPT], const float (&g0)[PPT],
                                          const float (&g1)[PPT], const float (&g2)[PPT], const float (&dy2)[PPT],
                                          float (&T)[PPT], float (&gsk)[PPT], int lane, PendingField& pend)
{
    for (int e = 0; e < cnt; ++e) {
        const uint32_t pos = top - (uint32_t)e;
        const LdsRec r = rec[e];
        const ColTerms ct = col_terms(r, c.dx);
        float p2[PPT];
        uint64_t on[PPT], any = 0;
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            p2[k] = power2(ct, r.p1.y, c.dy[k]);
            on[k] = lanes(p2[k] >= r.p1.w);
            if (!FULL) on[k] &= lanes(pos < my_n[k]);
            any |= on[k];
        }
        if (any == 0) continue;
        if (CLAMPS && may_clamp(r.p1.z, amax))
            bwd_entry<PPT, true, DET, ODD>(a, r, ct, p2, on, amax, c, g0, g1, g2, dy2, T, gsk, lane, pend);
        else
            bwd_entry<PPT, false, DET, ODD>(a, r, ct, p2, on, amax, c, g0, g1, g2, dy2, T, gsk, lane, pend);
    }
}

template <int PPT, int GSR_BATCH, bool DET, bool MIXED>
__global__ __launch_bounds__(64, PPT <= 4 ? 5 : 3) void k_raster_bwd(RasterArgs a)
{
    __shared__ LdsRec rec[GSR_BATCH];
    const TileCtx<PPT> c = tile_ctx<PPT>(a);
    // the accumulators are in use from here on (the clearing kernel, which
    // reads the flag, has completed before this kernel starts)
    if (blockIdx.x == 0 && threadIdx.x == 0) a.counters->grad_dirty = 1u;
    const int lane = threadIdx.x;
    if (uniform((int)a.counters->overflow)) {
        view_done(a, c.tile, lane);
        return;
    }
    const uint2 range = tile_range(a, c.tile);
    const float amax = a.cfg.alpha_max;

    float T[PPT], Tf[PPT], gsk[PPT], g0[PPT], g1[PPT], g2[PPT], dy2[PPT];
    uint32_t my_n[PPT];
    uint32_t lane_max = 0, lane_min = 0xffffffffu;
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        Tf[k] = 1.0f;
        g0[k] = g1[k] = g2[k] = 0.0f;
        float gT = 0.0f;
        my_n[k] = 0u;
        if (c.inside(k)) {
            Tf[k] = a.T_final_in[c.pix(k)];
            my_n[k] = (uint32_t)a.n_contrib_in[c.pix(k)];
            g0[k] = a.dL_drgb[c.rgb0(k)];
            g1[k] = a.dL_drgb[c.rgb0(k) + c.plane];
            g2[k] = a.dL_drgb[c.rgb0(k) + 2 * c.plane];
            if (a.dL_dT) gT = a.dL_dT[c.pix(k)];
        }
        T[k] = Tf[k];
        dy2[k] = c.dy[k] * c.dy[k];
        // g . (colour behind) + dL/dT_final T_final, maintained incrementally
        gsk[k] = __builtin_fmaf(gT, Tf[k], Tf[k] * (g0[k] * a.cfg.bg0 + g1[k] * a.cfg.bg1 + g2[k] * a.cfg.bg2));
        lane_max = max(lane_max, my_n[k]);
        lane_min = min(lane_min, my_n[k]);
    }
    for (int off = 32; off > 0; off >>= 1) {
        lane_max = max(lane_max, (uint32_t)__shfl_xor((int)lane_max, off, 64));
        lane_min = min(lane_min, (uint32_t)__shfl_xor((int)lane_min, off, 64));
    }
    bool upstream = false;
#pragma unroll
    for (int k = 0; k < PPT; ++k)
        upstream |= !(__builtin_isfinite(g0[k]) && __builtin_isfinite(g1[k]) && __builtin_isfinite(g2[k]) &&
                      __builtin_isfinite(gsk[k]));
    bool odd = lanes(upstream) != 0;
    // positions below this are blended by every pixel (0 where the tile
    // reaches outside the view)
    const uint32_t full = (uint32_t)uniform((int)lane_min);
    const uint32_t end = range.x + min((uint32_t)uniform((int)lane_max), range.y - range.x);

    PendingField pend{0, 0, 0.0f};
    for (uint32_t hi_ = end; hi_ > range.x;) {
        const uint32_t lo_ = hi_ - range.x > (uint32_t)GSR_BATCH ? hi_ - GSR_BATCH : range.x;
        const int cnt = (int)(hi_ - lo_);
        bool may = false, colour = false;
#pragma unroll
        for (int r = 0; r < GSR_BATCH / 64; ++r) {
            const int t = lane + 64 * r;
            if (t < cnt) {
                const Entry e = stage_record<MIXED>(a, a.vals[hi_ - 1 - t], c.xc, c.yc, rec[t]);
                may |= !(e.o < amax);
                colour |= e.odd;
            }
        }
        const bool clamps = lanes(may) != 0;
        odd |= lanes(colour) != 0;  // (and the entries before it, through gsk)
        __syncthreads();
        const uint32_t top = hi_ - 1 - range.x;
        if (odd)
            bwd_batch<PPT, true, false, DET, true>(a, rec, cnt, top, amax, c, my_n, g0, g1, g2, dy2, T, gsk, lane, pend);
        else if (clamps)
            bwd_batch<PPT, true, false, DET, false>(a, rec, cnt, top, amax, c, my_n, g0, g1, g2, dy2, T, gsk, lane, pend);
        else if (top < full)
            bwd_batch<PPT, false, true, DET, false>(a, rec, cnt, top, amax, c, my_n, g0, g1, g2, dy2, T, gsk, lane, pend);
        else
            bwd_batch<PPT, false, false, DET, false>(a, rec, cnt, top, amax, c, my_n, g0, g1, g2, dy2, T, gsk, lane, pend);
        __syncthreads();
        hi_ = lo_;
    }
    if (uniform(pend.have)) {  // the last reduced entry's ninth field, alone
        const float w = wave_sum_pair(pend.w, 0.0f);
        if (lane == 1) add_field<DET>(a, (uint32_t)pend.slot, 8, w);
    }
    view_done(a, c.tile, lane);
}

// Few tiles: 2 W waves to a tile.  Entries are replayed GSR_BWD_GROUP at a
// time.  The lane's pixels are dealt to the first W waves, which run a group
// through them (four entries' alphas in flight, only T and gsk passing from
// one to the next) and leave each pixel's two terms, alpha dL/dalpha and the
// weight, in LDS; meanwhile the other W waves take whole entries of the group
// before, add all of the lane's pixels up in the single wave's order and
// reduce them, two entries at a time.  The arithmetic and its order are those
// of k_raster_bwd, the sums equal bit for bit.  Terms and staged records are
// double-buffered, so a group costs one barrier, and a batch is staged while
// the one before is replayed.  A lone wave's entry takes 1000 cycles, twice
// its issue; here a group of 8 takes as long as its replay or its reduction,
// about 2700.  12 tiles of 716 entries 297 -> 104 us (the same waves doing
// both in turn 156), 1200 tiles of 162 137 -> 100, 825 of 104 in deterministic
// mode 150 -> 78, 1200 tiles of 512 pixels 743 -> 550 us; but 2400 tiles of 256
// pixels 684 -> 796 us: the passes through LDS are issue that a full chip
// lacks, hence GSR_BWD_FEW_TILES (1.5 tiles to a SIMD).
template <int PPT>
struct BwdFew {
    static constexpr int waves = PPT < 4 ? PPT : 4;  // W
    static constexpr int ppt = PPT / waves;          // pixels a lane of one wave
};

template <int PPT, bool DET, bool MIXED>
__global__ __launch_bounds__(128 * BwdFew<PPT>::waves, 4) void k_raster_bwd_few(RasterArgs a)
{
    constexpr int W = BwdFew<PPT>::waves, Q = BwdFew<PPT>::ppt, G = GSR_BWD_GROUP, U = 4, B = 64;
    static_assert(G % U == 0 && B % G == 0 && B / G >= 4 && W <= 4 && G % (2 * W) == 0, "");
    __shared__ LdsRec rec[2][B];
    __shared__ float2 term[2][G][PPT][64];
    __shared__ uint32_t reached[2][4];  // entries that reach wave w's pixels, a bit each
    __shared__ uint32_t rec_odd[2];     // whether a colour of rec[.] is infinite or NaN
    const int lane = threadIdx.x & 63, wave = uniform((int)(threadIdx.x >> 6));
    const bool replays = wave < W;
    const int w = replays ? wave : wave - W;
    const int tile = uniform((int)a.order[blockIdx.x]);
    if (blockIdx.x == 0 && threadIdx.x == 0) a.counters->grad_dirty = 1u;
    if (uniform((int)a.counters->overflow)) {
        view_done(a, tile, (int)threadIdx.x);
        return;
    }
    const TileCtx<PPT> c = tile_ctx_at<PPT>(a, tile, 0);
    const uint2 range = tile_range(a, tile);
    uint32_t lane_max = 0;
#pragma unroll
    for (int k = 0; k < PPT; ++k)
        if (c.inside(k)) lane_max = max(lane_max, (uint32_t)a.n_contrib_in[c.pix(k)]);
    for (int off = 32; off > 0; off >>= 1) lane_max = max(lane_max, (uint32_t)__shfl_xor((int)lane_max, off, 64));
    // entries to replay, from position count - 1 down
    const int count = (int)min((uint32_t)uniform((int)lane_max), range.y - range.x);
    const int groups = (count + G - 1) / G;
    // records i .. i + B - 1 of the replay, null past its end
    auto stage = [&](int i) {
        LdsRec& r = rec[(i / B) & 1][lane];
        bool odd = false;
        if (i + lane < count) {
            odd = stage_record<MIXED>(a, a.vals[range.x + (uint32_t)(count - 1 - i - lane)], c.xc, c.yc, r).odd;
        } else {
            r.p0 = r.p2 = r.p3 = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            r.p1 = make_float4(0.0f, 0.0f, 0.0f, INFINITY);
        }
        const uint64_t any = lanes(odd);
        if (lane == 0) rec_odd[(i / B) & 1] = any != 0;
    };
    if (wave == W) stage(0);

    if (replays) {
        const float amax = a.cfg.alpha_max;
        const TileCtx<Q> o = tile_ctx_at<Q>(a, tile, w * Q);
        float T[Q], gsk[Q], h0[Q], h1[Q], h2[Q];
        uint32_t my_n[Q];
        bool upstream = false;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            float Tf = 1.0f, gT = 0.0f;
            h0[q] = h1[q] = h2[q] = 0.0f;
            my_n[q] = 0u;
            if (o.inside(q)) {
                Tf = a.T_final_in[o.pix(q)];
                my_n[q] = (uint32_t)a.n_contrib_in[o.pix(q)];
                h0[q] = a.dL_drgb[o.rgb0(q)];
                h1[q] = a.dL_drgb[o.rgb0(q) + o.plane];
                h2[q] = a.dL_drgb[o.rgb0(q) + 2 * o.plane];
                if (a.dL_dT) gT = a.dL_dT[o.pix(q)];
            }
            T[q] = Tf;
            gsk[q] = __builtin_fmaf(gT, Tf, Tf * (h0[q] * a.cfg.bg0 + h1[q] * a.cfg.bg1 + h2[q] * a.cfg.bg2));
            upstream |= !(__builtin_isfinite(h0[q]) && __builtin_isfinite(h1[q]) && __builtin_isfinite(h2[q]) &&
                          __builtin_isfinite(gsk[q]));
        }
        bool odd = lanes(upstream) != 0;
        __syncthreads();
        // group gr; ODD as for bwd_entry
        auto replay = [&](auto odd_variant, int gr) {
            constexpr bool ODD = decltype(odd_variant)::value;
            const LdsRec* rg = &rec[(gr * G / B) & 1][gr * G % B];
            const int buf = gr & 1;
            const uint32_t top = (uint32_t)(count - 1 - gr * G);  // (below 0 only at null records)
            uint32_t reach = 0;
#pragma unroll
            for (int e = 0; e < G; e += U) {
                LdsRec r[U];
#pragma unroll
                for (int u = 0; u < U; ++u) r[u] = rg[e + u];
                float p2[U][Q], alpha[U][Q], rcp[U][Q], gcol[U][Q];
                uint64_t on[U][Q], any = 0;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const ColTerms ct = col_terms(r[u], o.dx);
                    uint64_t any_u = 0;
#pragma unroll
                    for (int q = 0; q < Q; ++q) {
                        p2[u][q] = power2(ct, r[u].p1.y, o.dy[q]);
                        on[u][q] = lanes(p2[u][q] >= r[u].p1.w) & lanes(top - (uint32_t)(e + u) < my_n[q]);
                        any_u |= on[u][q];
                    }
                    reach |= any_u != 0 ? 1u << (e + u) : 0u;
                    any |= any_u;
                }
                if (any == 0) continue;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const float lim = may_clamp(r[u].p1.z, amax) ? amax : INFINITY;
#pragma unroll
                    for (int q = 0; q < Q; ++q) {
                        p2[u][q] = r[u].p1.z * __builtin_amdgcn_exp2f(p2[u][q]);
                        alpha[u][q] = in(on[u][q]) ? fminf(p2[u][q], lim) : 0.0f;
                        rcp[u][q] = __builtin_amdgcn_rcpf(1.0f - alpha[u][q]);
                        gcol[u][q] = __builtin_fmaf(h0[q], r[u].p2.x, __builtin_fmaf(h1[q], r[u].p2.y, h2[q] * r[u].p2.z));
                        if (ODD) gcol[u][q] = in(on[u][q]) ? gcol[u][q] : 0.0f;
                        on[u][q] = (ODD ? on[u][q] : ~0ull) & lanes(p2[u][q] < lim);
                    }
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
#pragma unroll
                    for (int q = 0; q < Q; ++q) {
                        const float Tb = T[q] * rcp[u][q];
                        const float wgt = alpha[u][q] * Tb;
                        const float gsk_new = __builtin_fmaf(wgt, gcol[u][q], gsk[q]);
                        const float dd = __builtin_fmaf(-gsk[q], rcp[u][q], gsk_new);
                        gsk[q] = gsk_new;
                        T[q] = Tb;
                        term[buf][e + u][w * Q + q][lane] = make_float2(in(on[u][q]) ? dd : 0.0f, wgt);
                    }
                }
            }
            if (lane == 0) reached[buf][w] = reach;
        };
        // (an odd colour stays in gsk: two loops, so that the first keeps the
        // registers and the schedule that it has without the second)
        int gr = 0;
        for (; gr < groups; ++gr) {
            if (gr * G % B == 0) odd |= uniform((int)rec_odd[(gr * G / B) & 1]) != 0;
            if (odd) break;
            replay(std::false_type{}, gr);
            __syncthreads();
        }
        for (; gr < groups; ++gr) {
            replay(std::true_type{}, gr);
            __syncthreads();
        }
    } else {
        float g0[PPT], g1[PPT], g2[PPT], dy2[PPT];
        bool upstream = false;
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            g0[k] = g1[k] = g2[k] = 0.0f;
            if (c.inside(k)) {
                g0[k] = a.dL_drgb[c.rgb0(k)];
                g1[k] = a.dL_drgb[c.rgb0(k) + c.plane];
                g2[k] = a.dL_drgb[c.rgb0(k) + 2 * c.plane];
            }
            dy2[k] = c.dy[k] * c.dy[k];
            upstream |= !(__builtin_isfinite(g0[k]) && __builtin_isfinite(g1[k]) && __builtin_isfinite(g2[k]));
        }
        const bool odd = lanes(upstream) != 0;
        PendingField pend{0, 0, 0.0f};
        __syncthreads();
        // step gr reduces group gr - 1 (after the last barrier, the last)
        for (int gr = 0; gr <= groups; ++gr) {
            // the batch after this one, once the one before it is reduced
            if (w == 0 && gr % (B / G) == 2 && (gr / (B / G) + 1) * B < count) stage((gr / (B / G) + 1) * B);
            if (gr > 0) {
                const LdsRec* rg = &rec[((gr - 1) * G / B) & 1][(gr - 1) * G % B];
                const int buf = (gr - 1) & 1;
                uint32_t hit[W], hits = 0;
#pragma unroll
                for (int k = 0; k < W; ++k) {
                    hit[k] = (uint32_t)uniform((int)reached[buf][k]);
                    hits |= hit[k];
                }
                // this wave's entries, two at a time (their reductions overlap)
#pragma unroll
                for (int e = 0; e < G; e += 2 * W) {
                    const int e0 = e + w, e1 = e + w + W;
                    const bool has0 = (hits >> e0) & 1u, has1 = (hits >> e1) & 1u;
                    if (!has0 && !has1) continue;
                    const LdsRec r0 = rg[e0], r1 = rg[e1];
                    float2 t0[PPT], t1[PPT];
#pragma unroll
                    for (int k = 0; k < PPT; ++k) {
                        t0[k] = term[buf][e0][k][lane];
                        t1[k] = term[buf][e1][k][lane];
                    }
                    PixelSums p0, p1;
                    if (odd) {  // (a pixel that the entry does not reach has weight 0)
#pragma unroll
                        for (int k = 0; k < PPT; ++k) {
                            if ((hit[k / Q] >> e0) & 1u) p0.add_own(t0[k], g0[k], g1[k], g2[k], c.dy[k], dy2[k]);
                            if ((hit[k / Q] >> e1) & 1u) p1.add_own(t1[k], g0[k], g1[k], g2[k], c.dy[k], dy2[k]);
                        }
                    } else {
#pragma unroll
                        for (int k = 0; k < PPT; ++k) {
                            if ((hit[k / Q] >> e0) & 1u) p0.add(t0[k].x, t0[k].y, g0[k], g1[k], g2[k], c.dy[k], dy2[k]);
                            if ((hit[k / Q] >> e1) & 1u) p1.add(t1[k].x, t1[k].y, g0[k], g1[k], g2[k], c.dy[k], dy2[k]);
                        }
                    }
                    if (has0 && has1) {
                        float v0[9], v1[9];
                        bwd_partials(r0, col_terms(r0, c.dx), c.dx, p0, v0);
                        bwd_partials(r1, col_terms(r1, c.dx), c.dx, p1, v1);
                        const float s0 = wave_sum8_transposed(v0, lane), s1 = wave_sum8_transposed(v1, lane);
                        const float x = wave_sum_pair(v0[8], v1[8]);
                        const uint32_t slot0 = (uint32_t)uniform(__float_as_int(r0.p2.w));
                        const uint32_t slot1 = (uint32_t)uniform(__float_as_int(r1.p2.w));
                        bwd_add8<DET>(a, slot0, s0, r0.p3.z, lane);
                        bwd_add8<DET>(a, slot1, s1, r1.p3.z, lane);
                        if ((lane & 31) == 1) add_field<DET>(a, lane < 32 ? slot0 : slot1, 8, x);
                    } else if (has0) {
                        bwd_reduce<DET>(a, r0, col_terms(r0, c.dx), c.dx, p0, lane, pend);
                    } else {
                        bwd_reduce<DET>(a, r1, col_terms(r1, c.dx), c.dx, p1, lane, pend);
                    }
                }
            }
            if (gr < groups) __syncthreads();
        }
        if (uniform(pend.have)) {  // the last reduced entry's ninth field, alone
            const float x = wave_sum_pair(pend.w, 0.0f);
            if (lane == 1) add_field<DET>(a, (uint32_t)pend.slot, 8, x);
        }
    }
    __syncthreads();
    view_done(a, tile, (int)threadIdx.x);
}

// Parts of every tile: as many (up to the lane's pixels) as keep the waves at
// GSR_FWD_FEW_WAVES (8 to a SIMD, what is resident at once) or less; with
// more tiles the chip is full and the parts' repeated work per entry costs
// what they gain (16125 tiles: 419 us whole).  The parts stage 64 records at
// a time whatever the plan's batch, which changes no result: 4 KB of LDS
// leave room for the 8 waves.
static int fwd_parts(int tiles, int ppt)
{
    int parts = ppt;
    while (parts > 1 && (int64_t)tiles * parts > GSR_FWD_FEW_WAVES) parts /= 2;
    return parts;
}

template <int PPT, int PARTS, int B, bool COUNT, bool MIXED>
static void launch_fwd_few(const RasterArgs& a, int tiles, int parts, hipStream_t s)
{
    if constexpr (PARTS > 1) {
        if (parts == PARTS)
            hipLaunchKernelGGL((k_raster_fwd_few<PPT, PARTS, B, COUNT, MIXED>), dim3((unsigned)tiles * PARTS), dim3(64),
                               0, s, a);
        else
            launch_fwd_few<PPT, PARTS / 2, B, COUNT, MIXED>(a, tiles, parts, s);
    }
}

template <int PPT, int B, bool COUNT, bool MIXED>
static hipError_t launch_fwd_b(const RasterArgs& a, int tiles, hipStream_t s, hipStream_t side, hipEvent_t fork,
                               hipEvent_t join)
{
    const int parts = fwd_parts(tiles, PPT);
    if (parts > 1) {
        launch_fwd_few<PPT, PPT, 64, COUNT, MIXED>(a, tiles, parts, s);
        return hipGetLastError();
    }
    // the long tiles' parts run on `side`, forked from `s` and joined back
    // (the fork and join are graph edges when `s` is being captured)
    hipError_t e = hipSuccess;
    if (FwdSplit<PPT>::parts > 1) {
        e = hipEventRecord(fork, s);
        if (e == hipSuccess) e = hipStreamWaitEvent(side, fork, 0);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_zero_queue, dim3(1), dim3(1), 0, side, a.fwd_queue);
        hipLaunchKernelGGL((k_raster_fwd_long<PPT, B, COUNT, MIXED>), dim3(GSR_FWD_LONG_WAVES), dim3(64), 0, side,
                           a, tiles);
    }
    hipLaunchKernelGGL((k_raster_fwd<PPT, B, COUNT, MIXED>), dim3(tiles), dim3(64), 0, s, a);
    e = hipGetLastError();
    if (FwdSplit<PPT>::parts > 1) {
        if (e == hipSuccess) e = hipEventRecord(join, side);
        if (e == hipSuccess) e = hipStreamWaitEvent(s, join, 0);
    }
    return e;
}

template <int PPT, bool COUNT, bool MIXED>
static hipError_t launch_fwd_c(const RasterArgs& a, int tiles, int batch, hipStream_t s, hipStream_t side,
                               hipEvent_t fork, hipEvent_t join)
{
    switch (batch) {
    case 64: return launch_fwd_b<PPT, 64, COUNT, MIXED>(a, tiles, s, side, fork, join);
    case 128: return launch_fwd_b<PPT, 128, COUNT, MIXED>(a, tiles, s, side, fork, join);
    case 256: return launch_fwd_b<PPT, 256, COUNT, MIXED>(a, tiles, s, side, fork, join);
    default: return hipErrorInvalidValue;
    }
}

template <int PPT>
static hipError_t launch_fwd_t(const RasterArgs& a, int tiles, int batch, hipStream_t s, hipStream_t side,
                               hipEvent_t fork, hipEvent_t join)
{
    if (a.cfg.mixed)
        return a.n_blend ? launch_fwd_c<PPT, true, true>(a, tiles, batch, s, side, fork, join)
                         : launch_fwd_c<PPT, false, true>(a, tiles, batch, s, side, fork, join);
    return a.n_blend ? launch_fwd_c<PPT, true, false>(a, tiles, batch, s, side, fork, join)
                     : launch_fwd_c<PPT, false, false>(a, tiles, batch, s, side, fork, join);
}

template <int PPT, bool DET, bool MIXED>
static hipError_t launch_bwd_d(const RasterArgs& a, int tiles, int batch, hipStream_t s)
{
    if constexpr (PPT > 1) {
        if (tiles <= GSR_BWD_FEW_TILES) {  // (64 records at a time whatever the batch, which changes no result)
            hipLaunchKernelGGL((k_raster_bwd_few<PPT, DET, MIXED>), dim3(tiles), dim3(128 * BwdFew<PPT>::waves), 0, s, a);
            return hipSuccess;
        }
    }
    switch (batch) {
    case 64: hipLaunchKernelGGL((k_raster_bwd<PPT, 64, DET, MIXED>), dim3(tiles), dim3(64), 0, s, a); break;
    case 128: hipLaunchKernelGGL((k_raster_bwd<PPT, 128, DET, MIXED>), dim3(tiles), dim3(64), 0, s, a); break;
    case 256: hipLaunchKernelGGL((k_raster_bwd<PPT, 256, DET, MIXED>), dim3(tiles), dim3(64), 0, s, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipSuccess;
}

template <int PPT>
static hipError_t launch_bwd_t(const RasterArgs& a, int tiles, int batch, hipStream_t s)
{
    if (a.cfg.mixed)
        return a.acc ? launch_bwd_d<PPT, true, true>(a, tiles, batch, s)
                     : launch_bwd_d<PPT, false, true>(a, tiles, batch, s);
    return a.acc ? launch_bwd_d<PPT, true, false>(a, tiles, batch, s)
                 : launch_bwd_d<PPT, false, false>(a, tiles, batch, s);
}

hipError_t launch_raster_fwd(const RasterArgs& a, int total_tiles, int tile_px, int batch, hipStream_t s,
                             hipStream_t side, hipEvent_t fork, hipEvent_t join)
{
    if (total_tiles == 0) return hipSuccess;
    switch (tile_px) {
    case 64: return launch_fwd_t<1>(a, total_tiles, batch, s, side, fork, join);
    case 128: return launch_fwd_t<2>(a, total_tiles, batch, s, side, fork, join);
    case 256: return launch_fwd_t<4>(a, total_tiles, batch, s, side, fork, join);
    case 512: return launch_fwd_t<8>(a, total_tiles, batch, s, side, fork, join);
    default: return hipErrorInvalidValue;
    }
}

// zero the screen-space accumulators of every projected slot (rx >= 0) when
// a backward has added to them since the projection zeroed them; the
// backward only ever adds to and reads such slots, so each backward starts
// from zero however often it is called
__global__ void k_clear_grad2d(const Counters* counters, const float4* geom, double* grad2d, int64_t slots)
{
    if (!counters->grad_dirty) return;
    for (int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; s < slots;
         s += (int64_t)gridDim.x * blockDim.x) {
        if (geom[s].z >= 0.0f) {
#pragma unroll
            for (int f = 0; f < GSR_G2; ++f) grad2d[GSR_G2 * s + f] = 0.0;
        }
    }
}

// deterministic mode: the same for the fixed-point accumulators
__global__ void k_clear_acc(const Counters* counters, const float4* geom, unsigned long long* acc, int64_t slots)
{
    if (!counters->grad_dirty) return;
    for (int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; s < slots;
         s += (int64_t)gridDim.x * blockDim.x) {
        if (geom[s].z >= 0.0f) {
            ulonglong2* p = reinterpret_cast<ulonglong2*>(acc + GSR_G2 * GSR_FIX_LIMBS * s);
#pragma unroll
            for (int k = 0; k < GSR_G2 * GSR_FIX_LIMBS / 2; ++k) p[k] = make_ulonglong2(0ull, 0ull);
        }
    }
}

// deterministic mode: the accumulators of every projected slot into grad2d
__global__ void k_fix_to_grad2d(const float4* geom, const unsigned long long* acc, double* grad2d, int64_t slots)
{
    for (int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; s < slots;
         s += (int64_t)gridDim.x * blockDim.x) {
        if (geom[s].z >= 0.0f) {
#pragma unroll
            for (int f = 0; f < GSR_G2; ++f)
                grad2d[GSR_G2 * s + f] = fixed_value(acc + GSR_G2 * GSR_FIX_LIMBS * s + f, GSR_G2);
        }
    }
}

hipError_t launch_clear_grad2d(const RasterArgs& a, hipStream_t s)
{
    if (a.slots <= 0) return hipSuccess;
    int64_t blocks = (a.slots + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    if (a.acc)
        hipLaunchKernelGGL(k_clear_acc, dim3((unsigned)blocks), dim3(256), 0, s, a.counters, a.geom, a.acc,
                           a.slots);
    else
        hipLaunchKernelGGL(k_clear_grad2d, dim3((unsigned)blocks), dim3(256), 0, s, a.counters, a.geom, a.grad2d,
                           a.slots);
    return hipGetLastError();
}

hipError_t launch_raster_bwd(const RasterArgs& a, int total_tiles, int tile_px, int batch, hipStream_t s)
{
    if (total_tiles == 0) return hipSuccess;
    hipError_t e;
    switch (tile_px) {
    case 64: e = launch_bwd_t<1>(a, total_tiles, batch, s); break;
    case 128: e = launch_bwd_t<2>(a, total_tiles, batch, s); break;
    case 256: e = launch_bwd_t<4>(a, total_tiles, batch, s); break;
    case 512: e = launch_bwd_t<8>(a, total_tiles, batch, s); break;
    default: return hipErrorInvalidValue;
    }
    if (e == hipSuccess && a.acc && a.slots > 0) {
        int64_t blocks = (a.slots + 255) / 256;
        if (blocks > 8192) blocks = 8192;
        hipLaunchKernelGGL(k_fix_to_grad2d, dim3((unsigned)blocks), dim3(256), 0, s, a.geom, a.acc, a.grad2d,
                           a.slots);
    }
    return e != hipSuccess ? e : hipGetLastError();
}

// ---------------------------------------------------------------------------
// L1 photometric loss seed, Eq. (photometric): dL/dC = sign(C - target) / count

__device__ __forceinline__ float l1_sign(float x, float t, float scale)
{
    const float d = x - t;
    return d > 0.0f ? scale : (d < 0.0f ? -scale : 0.0f);
}

template <bool HALF>
__global__ void k_loss_l1(LossArgs a)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.count;
         i += (int64_t)gridDim.x * blockDim.x) {
        const float x = HALF ? __half2float(static_cast<const __half*>(a.rgb)[i]) : static_cast<const float*>(a.rgb)[i];
        a.dL_drgb[i] = l1_sign(x, a.target[i], a.scale);
    }
}

// the float32 image four values at a time (count a multiple of 4, the three
// buffers 16-byte aligned)
__global__ void k_loss_l1_vec(LossArgs a)
{
    const float4* rgb = static_cast<const float4*>(a.rgb);
    const float4* tgt = reinterpret_cast<const float4*>(a.target);
    float4* out = reinterpret_cast<float4*>(a.dL_drgb);
    const int64_t n4 = a.count / 4;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += (int64_t)gridDim.x * blockDim.x) {
        const float4 x = rgb[i], t = tgt[i];
        out[i] = make_float4(l1_sign(x.x, t.x, a.scale), l1_sign(x.y, t.y, a.scale), l1_sign(x.z, t.z, a.scale),
                             l1_sign(x.w, t.w, a.scale));
    }
}

hipError_t launch_loss_l1(const LossArgs& a, hipStream_t s)
{
    if (a.count == 0) return hipSuccess;
    int64_t blocks = (a.count + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    const bool vec = !a.half_image && a.count % 4 == 0 && (((uintptr_t)a.rgb | (uintptr_t)a.target |
                                                            (uintptr_t)a.dL_drgb) & 15) == 0;
    if (vec) {
        int64_t vb = (a.count / 4 + 255) / 256;
        if (vb > 65536) vb = 65536;
        hipLaunchKernelGGL(k_loss_l1_vec, dim3((unsigned)vb), dim3(256), 0, s, a);
    } else if (a.half_image) {
        hipLaunchKernelGGL(k_loss_l1<true>, dim3((unsigned)blocks), dim3(256), 0, s, a);
    } else {
        hipLaunchKernelGGL(k_loss_l1<false>, dim3((unsigned)blocks), dim3(256), 0, s, a);
    }
    return hipGetLastError();
}

}  // namespace gsr
