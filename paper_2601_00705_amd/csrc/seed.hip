// seed.hip -- the one-shot Gaussian seeding from dense correspondences (Sec.
// "Dense Feature Matching" and the appendix's initialisation), one to four
// lanes per reference pixel.
//
// k_seed_triangulate: for every neighbour n of the reference keyframe, the
//   two-view linear system A X = 0 (rows x P^3 - P^1, y P^3 - P^2 of both
//   views) is solved in double by a one-sided Jacobi SVD of the 4x4 A: plane
//   rotations orthogonalise A's columns and accumulate V; the column of V
//   whose rotated column of A has the smallest norm is the right singular
//   vector of the smallest singular value.  Among the neighbours the
//   hypothesis with the smallest reprojection error (RMS of the two
//   reprojection distances, in front of both cameras) is kept, ties going to
//   the larger baseline angle; it is rejected when its error reaches
//   max_reproj or its angle is below min_parallax.  Eq. (conf) gives
//   kappa_bar, Eq. (app-alpha-init) the opacity; the colour is the median of
//   the exposure-corrected bilinear samples over the supporting views (the
//   reference, and every neighbour whose match lies within max_reproj of the
//   kept point's projection).
// The neighbour searches behind the initial scales are in knn.hip.
#include "kernels.h"
#include "seed_lanes.h"

namespace gsr {

#define GSR_SEED_THREADS 256

// ---------------------------------------------------------------------------
// triangulation

// right singular vector of the smallest singular value of the 4x4 A (rows)
__device__ void smallest_right_singular(double A[4][4], double out[4])
{
    double V[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) V[i][j] = i == j ? 1.0 : 0.0;
    for (int sweep = 0; sweep < 40; ++sweep) {
        bool rotated = false;
#pragma unroll
        for (int p = 0; p < 3; ++p) {
#pragma unroll
            for (int q = p + 1; q < 4; ++q) {
                double al = 0.0, be = 0.0, ga = 0.0;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    al += A[i][p] * A[i][p];
                    be += A[i][q] * A[i][q];
                    ga += A[i][p] * A[i][q];
                }
                // a pair counts as orthogonal at ~4.5 machine epsilons of
                // its norms: below that the rounding of the dot products
                // themselves dominates, and a stricter test never settles
                // (every system would run to the sweep cap)
                if (ga == 0.0 || ga * ga <= 1e-30 * (al * be)) continue;
                rotated = true;
                // t = sgn(zeta) / (|zeta| + sqrt(1 + zeta^2)), zeta = d / (2 ga),
                // with numerator and denominator times 2 |ga|: one root and
                // one quotient, then one reciprocal root, instead of three of
                // each (they are most of a rotation's instructions)
                const double d = be - al, g2 = 2.0 * ga;
                const double t = (d >= 0.0 ? g2 : -g2) / (fabs(d) + sqrt(d * d + g2 * g2));
                const double c = rsqrt(1.0 + t * t), s = c * t;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const double ap = A[i][p], aq = A[i][q];
                    A[i][p] = c * ap - s * aq;
                    A[i][q] = s * ap + c * aq;
                    const double vp = V[i][p], vq = V[i][q];
                    V[i][p] = c * vp - s * vq;
                    V[i][q] = s * vp + c * vq;
                }
            }
        }
        if (!rotated) break;
    }
    int best = 0;
    double bn = 0.0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        double nrm = 0.0;
#pragma unroll
        for (int i = 0; i < 4; ++i) nrm += A[i][j] * A[i][j];
        if (j == 0 || nrm < bn) {
            bn = nrm;
            best = j;
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) out[i] = V[i][best];
}

__device__ __forceinline__ void project_px(const double* P, const double X[3], double& u, double& v, double& z)
{
    const double y0 = P[0] * X[0] + P[1] * X[1] + P[2] * X[2] + P[3];
    const double y1 = P[4] * X[0] + P[5] * X[1] + P[6] * X[2] + P[7];
    z = P[8] * X[0] + P[9] * X[1] + P[10] * X[2] + P[11];
    u = y0 / z;
    v = y1 / z;
}

// bilinear sample of channel c, pixel centres at +1/2, clamped to the border
__device__ __forceinline__ double bilinear(const SeedView& vw, int c, double x, double y)
{
    const int W = vw.width, H = vw.height;
    const double fx = fmin(fmax(x - 0.5, 0.0), (double)(W - 1));
    const double fy = fmin(fmax(y - 0.5, 0.0), (double)(H - 1));
    const int x0 = (int)floor(fx), y0 = (int)floor(fy);
    const int x1 = min(x0 + 1, W - 1), y1 = min(y0 + 1, H - 1);
    const double ax = fx - x0, ay = fy - y0;
    const float* p = vw.image + (int64_t)c * W * H;
    return (double)p[y0 * W + x0] * (1.0 - ax) * (1.0 - ay) + (double)p[y0 * W + x1] * ax * (1.0 - ay) +
           (double)p[y1 * W + x0] * (1.0 - ax) * ay + (double)p[y1 * W + x1] * ax * ay;
}

// A hypothesis of one neighbour: the point, its error and angle, or none.
struct Hypothesis {
    bool ok;
    double err, ang, X[3];
};

__device__ __forceinline__ Hypothesis hypothesis(const SeedArgs& a, int64_t i, int k, const double (&xr)[2])
{
    Hypothesis hy;
    hy.ok = false;
    const SeedView& R = a.views[0];
    const SeedView& N = a.views[1 + k];
    const double xn[2] = {(double)a.x_nb[(int64_t)(2 * k) * a.n + i], (double)a.x_nb[(int64_t)(2 * k + 1) * a.n + i]};
    double A[4][4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        A[0][j] = xr[0] * R.P[8 + j] - R.P[j];
        A[1][j] = xr[1] * R.P[8 + j] - R.P[4 + j];
        A[2][j] = xn[0] * N.P[8 + j] - N.P[j];
        A[3][j] = xn[1] * N.P[8 + j] - N.P[4 + j];
    }
    double h[4];
    smallest_right_singular(A, h);
    hy.err = hy.ang = hy.X[0] = hy.X[1] = hy.X[2] = 0.0;
    if (h[3] == 0.0) return hy;
    const double X[3] = {h[0] / h[3], h[1] / h[3], h[2] / h[3]};
    double ur, vr, zr, un, vn, zn;
    project_px(R.P, X, ur, vr, zr);
    project_px(N.P, X, un, vn, zn);
    if (!(zr > 0.0 && zn > 0.0)) return hy;
    const double e0 = ur - xr[0], e1 = vr - xr[1], e2 = un - xn[0], e3 = vn - xn[1];
    hy.err = sqrt(0.5 * ((e0 * e0 + e1 * e1) + (e2 * e2 + e3 * e3)));
    const double ra[3] = {X[0] - R.centre[0], X[1] - R.centre[1], X[2] - R.centre[2]};
    const double rb[3] = {X[0] - N.centre[0], X[1] - N.centre[1], X[2] - N.centre[2]};
    const double dot = ra[0] * rb[0] + ra[1] * rb[1] + ra[2] * rb[2];
    const double na = sqrt(ra[0] * ra[0] + ra[1] * ra[1] + ra[2] * ra[2]);
    const double nb = sqrt(rb[0] * rb[0] + rb[1] * rb[1] + rb[2] * rb[2]);
    hy.ang = acos(fmin(fmax(dot / (na * nb), -1.0), 1.0));
    hy.X[0] = X[0];
    hy.X[1] = X[1];
    hy.X[2] = X[2];
    hy.ok = true;
    return hy;
}

// G lanes to a pixel (seed_lanes): each solves the systems of
// every G-th neighbour, the hypotheses are compared in the neighbours' order,
// and the supporting views and the colour's channels are dealt to the lanes.
// Bound by the FP64 rotations where pixels fill the chip (500k, four
// neighbours: 451 us at 1, 2 or 4 lanes a pixel alike), and by one pixel's
// chain of them where they do not: 1000 pixels took 69 us with a lane each, 41
// with two, 24 with four.  Half of a rotation was its three roots and three
// quotients; with one root, one quotient and one reciprocal root these are
// 370 and 20 us.
template <int G>
__global__ __launch_bounds__(GSR_SEED_THREADS) void k_seed_triangulate(SeedArgs a)
{
    const int64_t t = (int64_t)blockIdx.x * GSR_SEED_THREADS + threadIdx.x;
    const int64_t i = t / G;
    const int q = (int)(threadIdx.x & (G - 1));
    if (i >= a.n) return;  // (whole groups of lanes)
    const int K = a.K;
    const double xr[2] = {(double)a.x_ref[i], (double)a.x_ref[a.n + i]};

    double best_err = INFINITY, best_ang = -1.0, bX[3] = {0.0, 0.0, 0.0};
    int best = -1;
    for (int k0 = 0; k0 < K; k0 += G) {
        Hypothesis hy;
        hy.ok = false;
        hy.err = hy.ang = hy.X[0] = hy.X[1] = hy.X[2] = 0.0;
        if (k0 + q < K) hy = hypothesis(a, i, k0 + q, xr);
        int win = -1;
#pragma unroll
        for (int l = 0; l < G; ++l) {
            const bool ok = G == 1 ? hy.ok : __shfl(hy.ok ? 1 : 0, l, G) != 0;
            const double err = G == 1 ? hy.err : __shfl(hy.err, l, G);
            const double ang = G == 1 ? hy.ang : __shfl(hy.ang, l, G);
            if (ok && (best < 0 || err < best_err || (err == best_err && ang > best_ang))) {
                best_err = err;
                best_ang = ang;
                best = k0 + l;
                win = l;
            }
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double x = G == 1 ? hy.X[c] : __shfl(hy.X[c], max(win, 0), G);
            bX[c] = win >= 0 ? x : bX[c];
        }
    }
    // a point whose float32 position overflows is no usable Gaussian
    const bool finite = isfinite((float)bX[0]) && isfinite((float)bX[1]) && isfinite((float)bX[2]);
    const bool ok = best >= 0 && best_err < a.max_reproj && best_ang >= a.min_parallax && finite;
    if (q == 0) {
        // Eq. (conf) and Eq. (app-alpha-init)
        double ks = 0.0;
        for (int k = 0; k < K; ++k) ks += (double)a.kappa[(int64_t)k * a.n + i];
        const double kbar = ks / (double)K;
        const double alpha = a.alpha_lo + (a.alpha_hi - a.alpha_lo) * kbar;
        if (a.kappa_bar) a.kappa_bar[i] = (float)kbar;
        a.opacity_logit[i] = (float)log(alpha / (1.0 - alpha));
        a.valid[i] = ok ? 1 : 0;
        if (a.best) a.best[i] = best;
        if (a.err) a.err[i] = (float)best_err;
        if (a.angle) a.angle[i] = best >= 0 ? (float)best_ang : 0.0f;
#pragma unroll
        for (int c = 0; c < 3; ++c) a.mean[(int64_t)c * a.n + i] = (float)bX[c];
    }

    // colour: median of the corrected samples over the supporting views.
    // The supporting views form a bit mask; per channel the samples sit in a
    // fixed register array (absent views as +inf), sorted by an unrolled
    // odd-even transposition network, and the median is picked by index
    // compares, so that nothing is indexed dynamically (no scratch memory).
    uint32_t support = 0u;
    if (ok) {
        support = 1u;
        for (int v = 1 + q; v <= K; v += G) {
            const double xn0 = (double)a.x_nb[(int64_t)(2 * (v - 1)) * a.n + i];
            const double xn1 = (double)a.x_nb[(int64_t)(2 * (v - 1) + 1) * a.n + i];
            double u, w, z;
            project_px(a.views[v].P, bX, u, w, z);
            const double du = u - xn0, dv = w - xn1;
            if (sqrt(du * du + dv * dv) < a.max_reproj) support |= 1u << v;
        }
    }
#pragma unroll
    for (int o = 1; o < G; o <<= 1) support |= (uint32_t)__shfl_xor((int)support, o, G);
    const int m = __popc(support);
    constexpr int NS = GSR_SEED_MAX_NEIGHBOURS + 1;
    for (int c = q; c < 3; c += G) {
        double smp[NS];
#pragma unroll
        for (int v = 0; v < NS; ++v) {
            smp[v] = INFINITY;
            if ((support >> v) & 1u) {
                const double px = v == 0 ? xr[0] : (double)a.x_nb[(int64_t)(2 * (v - 1)) * a.n + i];
                const double py = v == 0 ? xr[1] : (double)a.x_nb[(int64_t)(2 * (v - 1) + 1) * a.n + i];
                const SeedView& vw = a.views[v];
                smp[v] = (bilinear(vw, c, px, py) - vw.bias) / vw.gain;
            }
        }
#pragma unroll
        for (int round = 0; round < NS; ++round) {
#pragma unroll
            for (int j = round & 1; j + 1 < NS; j += 2) {
                const double lo = fmin(smp[j], smp[j + 1]), hi = fmax(smp[j], smp[j + 1]);
                smp[j] = lo;
                smp[j + 1] = hi;
            }
        }
        double lo_mid = 0.0, hi_mid = 0.0;
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            if (j == (m - 1) / 2) lo_mid = smp[j];
            if (j == m / 2) hi_mid = smp[j];
        }
        const double med = m == 0 ? 0.0 : ((m & 1) ? hi_mid : (lo_mid + hi_mid) / 2.0);
        a.colour[(int64_t)c * a.n + i] = (float)med;
    }
}

hipError_t launch_seed_triangulate(const SeedArgs& a, hipStream_t s)
{
    if (a.n == 0) return hipSuccess;
    const int G = seed_lanes(a.n, a.K);
    const int64_t blocks = (a.n * G + GSR_SEED_THREADS - 1) / GSR_SEED_THREADS;
    const dim3 grid((unsigned)blocks), block(GSR_SEED_THREADS);
    if (G == 4) hipLaunchKernelGGL(k_seed_triangulate<4>, grid, block, 0, s, a);
    else if (G == 2) hipLaunchKernelGGL(k_seed_triangulate<2>, grid, block, 0, s, a);
    else hipLaunchKernelGGL(k_seed_triangulate<1>, grid, block, 0, s, a);
    return hipGetLastError();
}

}  // namespace gsr
