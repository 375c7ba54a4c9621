// fiberhit: ray/fiber intersection for AMD MI355X (gfx950).
//
// Method: Binder & Keller, "Fast, High Precision Ray/Fiber Intersection using
// Tight, Disjoint Bounding Volumes" (arXiv 1811.03374). One lane owns one
// (ray, fiber) pair. The fiber is moved into the frame of the ray once
// (Section 3.3), held in the {p, d, t0, t1} form of Section 3.1, and
// subdivided at the parametric centre inside bounding cylinders cropped by
// end-cap and split planes (Sections 3.2, 3.3). The recursion is iterated with
// one bit per level (Section 3.3); a backtrack rebuilds the pending sibling by
// replaying the split rules from the root along the integer path, which gives
// bit-for-bit the node that the descent produced (no cancellation from
// re-evaluating the curve at absolute parameters).
//
// Arithmetic notes for gfx950:
//  * everything is FP32 VALU work (no MFMA: nothing here is a contraction);
//  * the ray-frame projection runs once per pair in FP64 (full VALU rate on
//    CDNA4) from exact differences of the float32 inputs, so the root's
//    {p, d, t0, t1} components are each correctly rounded to float32 -- the
//    traversal never forms a difference of rounded absolute coordinates;
//  * the file is compiled with -ffp-contract=off: every FMA is written out, so
//    the descent and the replay round identically.
//
// Readings where the paper is silent or its listings disagree are the same as
// those of the FP64 CPU oracle (visibility needs a non-empty cropped
// interval, the leaf t is the entry into the capped leaf cylinder, planes
// parallel to the ray and axes parallel to the ray get explicit rules, zero
// tangents fall back to the next non-negligible control-polygon edge).

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdlib>
#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <tuple>
#include <vector>

#include "fiberhit.h"

namespace {

constexpr int kWave = 64;                     // gfx950 wavefront
#ifndef FIBERHIT_QUEUE
#define FIBERHIT_QUEUE 64                     // build knob: queue entries per wave
#endif
constexpr int kQueue = FIBERHIT_QUEUE;        // prepared roots per wave (LDS queue)

// Entry x of the queue ring, for 0 <= x < 3 kQueue.
__device__ __forceinline__ int qslot(int x)
{
    x = x >= kQueue ? x - kQueue : x;
    return x >= kQueue ? x - kQueue : x;
}
constexpr int kQWords = 21;                   // root node (16), lo, hi, tmax, pair, scene * 64 + stall * 32 + depth
constexpr uint32_t kRootSize = 1u << 23;      // parametric domain [0, 1) in units of 2^-23
constexpr uint32_t kStallBit = 1u << 31;       // flag bit kept in a lane's interval start
constexpr uint32_t kStartMask = kRootSize - 1u;
constexpr int kMaxTrips = 1 << 16;            // hang guard; the longest degenerate pairs seen need 850 trips
#ifndef FIBERHIT_PARENT_CACHE
#define FIBERHIT_PARENT_CACHE 1
#endif
constexpr bool kParentCache = FIBERHIT_PARENT_CACHE != 0;   // cache the latest both-hit parent in LDS
#ifndef FIBERHIT_FUSED_REFILL
#define FIBERHIT_FUSED_REFILL 1                    // free lanes that take queued roots (single calls)
#endif
#ifndef FIBERHIT_REFINE_REFILL
#define FIBERHIT_REFINE_REFILL 1                   // the same for refined calls
#endif

struct V4 { float x, y, z, w; };
struct Node { V4 p, d, t0, t1; };             // Section 3.1: p = p0, d = p3-p0, t0 = p1-p0, t1 = p3-p2

__device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float vsqrt(float x) { return __builtin_amdgcn_sqrtf(x); }

__device__ __forceinline__ float dot3(float ax, float ay, float az, float bx, float by, float bz)
{
    return fmaf(ax, bx, fmaf(ay, by, az * bz));
}

// A tangent whose squared length is at most 2^-40 of the squared chord (cc)
// has no reliable direction: at a cusp or a vanishing end tangent its
// components are rounding noise of the control points. The cap and split
// planes then take the next control-polygon edge or the chord instead. With
// a zero chord only the zero vector is negligible.
__device__ __forceinline__ bool negligible(float x, float y, float z, float cc)
{
    return fmaf(x, x, fmaf(y, y, z * z)) <= 0x1p-40f * cc;
}

// ---------------------------------------------------------------------------
// Ray frame (Section 3.3)
// ---------------------------------------------------------------------------

// 1/sqrt(x) and 1/x in double: hardware estimates refined by two Newton
// steps each (quadratic convergence from ~2^-22 to full double precision).
__device__ __forceinline__ double rsqrt64(double x)
{
    double y = __builtin_amdgcn_rsq(x);
    const double hx = 0.5 * x;
    y = y * fma(-hx * y, y, 1.5);
    y = y * fma(-hx * y, y, 1.5);
    return y;
}

__device__ __forceinline__ double rcp64(double x)
{
    double y = __builtin_amdgcn_rcp(x);
    y = fma(fma(-x, y, 1.0), y, y);
    y = fma(fma(-x, y, 1.0), y, y);
    return y;
}

// Orthonormal basis (u, v) completing the unit w: Duff et al. 2017, the
// revision of Frisvad's construction cited in Section 3.3.
__device__ __forceinline__ void make_onb(double wx, double wy, double wz,
                                         double u[3], double v[3])
{
    const double s = copysign(1.0, wz);
    const double a = -rcp64(s + wz);
    const double b = wx * wy * a;
    u[0] = fma(s * wx * wx, a, 1.0);
    u[1] = s * b;
    u[2] = -s * wx;
    v[0] = b;
    v[1] = fma(wy * wy, a, s);
    v[2] = -wy;
}


// ---------------------------------------------------------------------------
// Node geometry
// ---------------------------------------------------------------------------

// t interval between the node's two end-cap planes (Section 3.3, cropping),
// intersected with [0, tmax]. Start cap: plane through p, normal t0, curve on
// the positive side. End cap: plane through p + d, normal t1, curve on the
// negative side. A negligible end tangent falls back to the next
// control-polygon edge from that end (p2 - p0, resp. p3 - p1), then the chord.
__device__ __forceinline__ void cap_interval(const Node &c, float tmax, float &lo, float &hi)
{
    float n0x = c.t0.x, n0y = c.t0.y, n0z = c.t0.z;
    float n1x = c.t1.x, n1y = c.t1.y, n1z = c.t1.z;
    const float cc = dot3(c.d.x, c.d.y, c.d.z, c.d.x, c.d.y, c.d.z);
    if (negligible(n0x, n0y, n0z, cc) || negligible(n1x, n1y, n1z, cc)) {
        // rare (a vanishing end tangent): kept out of the common path
        if (negligible(n0x, n0y, n0z, cc)) { n0x = c.d.x - c.t1.x; n0y = c.d.y - c.t1.y; n0z = c.d.z - c.t1.z; }
        if (negligible(n0x, n0y, n0z, cc)) { n0x = c.d.x; n0y = c.d.y; n0z = c.d.z; }
        if (negligible(n1x, n1y, n1z, cc)) { n1x = c.d.x - c.t0.x; n1y = c.d.y - c.t0.y; n1z = c.d.z - c.t0.z; }
        if (negligible(n1x, n1y, n1z, cc)) { n1x = c.d.x; n1y = c.d.y; n1z = c.d.z; }
    }

    // both crossings are computed and selected by the signs of the normals'
    // z (no divergent branches); a plane parallel to the ray keeps the whole
    // ray or none of it
    const float c0 = dot3(c.p.x, c.p.y, c.p.z, n0x, n0y, n0z);
    const float q0 = c0 * rcp(n0z);
    const float ex = c.p.x + c.d.x, ey = c.p.y + c.d.y, ez = c.p.z + c.d.z;
    const float c1 = dot3(ex, ey, ez, n1x, n1y, n1z);
    const float q1 = c1 * rcp(n1z);
    float l = n0z > 0.0f ? fmaxf(0.0f, q0) : 0.0f;
    float h = n0z < 0.0f ? fminf(tmax, q0) : tmax;
    h = n1z > 0.0f ? fminf(h, q1) : h;
    l = n1z < 0.0f ? fmaxf(l, q1) : l;
    const bool empty = (n0z == 0.0f && c0 > 0.0f) || (n1z == 0.0f && c1 < 0.0f);
    lo = empty ? INFINITY : l;
    hi = empty ? -INFINITY : h;
}

// Conservative cylinder radius (Section 3.3): largest distance of the inner
// control points (t0 and -t1 relative to the chord ends) to the chord line,
// plus the largest radius control value (convex hull of the radius Bezier).
// QUAD: the node is the exact cubic elevation of a quadratic (Appendix B.1:
// q1 = (p0 + 2 p1) / 3, q2 = (2 p1 + p2) / 3): the same curve, halves and
// planes. Its bound is the quadratic's: the middle control point p1 lies at
// 3/2 of the elevated inner points' distance from the chord, and the middle
// radius value is r0 + 3/2 t0.w = r2 - 3/2 t1.w.
template <bool QUAD = false>
__device__ __forceinline__ float conservative_radius(const Node &c)
{
    const float cc = dot3(c.d.x, c.d.y, c.d.z, c.d.x, c.d.y, c.d.z);
    const float ic = cc > 0.0f ? rcp(cc) : 0.0f;
    const float b0 = dot3(c.t0.x, c.t0.y, c.t0.z, c.d.x, c.d.y, c.d.z) * ic;
    const float e0x = fmaf(-b0, c.d.x, c.t0.x), e0y = fmaf(-b0, c.d.y, c.t0.y), e0z = fmaf(-b0, c.d.z, c.t0.z);
    const float b1 = dot3(c.t1.x, c.t1.y, c.t1.z, c.d.x, c.d.y, c.d.z) * ic;
    const float e1x = fmaf(-b1, c.d.x, c.t1.x), e1y = fmaf(-b1, c.d.y, c.t1.y), e1z = fmaf(-b1, c.d.z, c.t1.z);
    const float l0 = dot3(e0x, e0y, e0z, e0x, e0y, e0z);
    const float l1 = dot3(e1x, e1y, e1z, e1x, e1y, e1z);
    if constexpr (QUAD) {
        const float r1 = fmaxf(fmaf(1.5f, c.t0.w, 0.0f), fmaf(-1.5f, c.t1.w, c.d.w));
        const float rmax = c.p.w + fmaxf(fmaxf(0.0f, c.d.w), r1);
        return 1.5f * vsqrt(fmaxf(l0, l1)) + rmax;
    }
    const float rmax = c.p.w + fmaxf(fmaxf(0.0f, c.t0.w), fmaxf(c.d.w, c.d.w - c.t1.w));
    return vsqrt(fmaxf(l0, l1)) + rmax;
}

// Unit ray (origin, +z) against the infinite cylinder of radius r about the
// line through o along a (Appendix A). False on a miss.
__device__ __forceinline__ bool unit_ray_cylinder(const V4 &o, const V4 &a, float r, float &te, float &tx)
{
    // both cases are evaluated and selected: no divergent branch. The axis
    // counts as parallel to the ray when its across-ray part is below 2^-50
    // of its along-ray part (or zero): beyond that the general formula's
    // terms (up to a.z^2 / g) would leave the float range, while the
    // cylinder it describes already spans the whole ray. The test is relative:
    // the chord of a node next to a cusp or a stalled end shrinks like 4^-level,
    // and an absolute threshold took such nodes for parallel ones.
    const float g = fmaf(a.x, a.x, a.y * a.y);
    const bool parallel = g <= 0x1p-100f * (a.z * a.z);
    const float dd = fmaf(a.x, o.y, -(a.y * o.x));
    const float h = rcp(g);
    const float e = fmaf(-(dd * dd), h, r * r);
    const float tc = fmaf(-a.z, fmaf(a.x, o.x, a.y * o.y) * h, o.z);
    const float s = vsqrt(e * fmaf(a.z, a.z, g) * h);
    const bool inside = fmaf(o.x, o.x, o.y * o.y) < r * r;
    te = parallel ? -INFINITY : tc - s;
    tx = parallel ? INFINITY : tc + s;
    return parallel ? inside : e >= 0.0f;
}

// Split quantities of Section 3.1: centre offset dp and split tangent tc
// (1/8 of -q0 - q1 + q2 + q3, the children's tangent at the split point).
// A negligible split tangent is rounding noise of the exact value zero: the
// split point is a cusp, and the children take a zero tangent there (xyz;
// the radius channel keeps its slope), as if the curve had been split at the
// cusp beforehand. Returns whether that happened.
__device__ __forceinline__ bool split_terms(const Node &c, V4 &dp, V4 &tc)
{
    dp.x = fmaf(0.375f, c.t0.x - c.t1.x, 0.5f * c.d.x);
    dp.y = fmaf(0.375f, c.t0.y - c.t1.y, 0.5f * c.d.y);
    dp.z = fmaf(0.375f, c.t0.z - c.t1.z, 0.5f * c.d.z);
    dp.w = fmaf(0.375f, c.t0.w - c.t1.w, 0.5f * c.d.w);
    tc.x = fmaf(-0.125f, c.t0.x + c.t1.x, 0.25f * c.d.x);
    tc.y = fmaf(-0.125f, c.t0.y + c.t1.y, 0.25f * c.d.y);
    tc.z = fmaf(-0.125f, c.t0.z + c.t1.z, 0.25f * c.d.z);
    tc.w = fmaf(-0.125f, c.t0.w + c.t1.w, 0.25f * c.d.w);
    const bool cusp = negligible(tc.x, tc.y, tc.z, dot3(c.d.x, c.d.y, c.d.z, c.d.x, c.d.y, c.d.z));
    tc.x = cusp ? 0.0f : tc.x;
    tc.y = cusp ? 0.0f : tc.y;
    tc.z = cusp ? 0.0f : tc.z;
    return cusp;
}

// Keep one half (Section 3.1): left (p, dp, t0/2, tc) or right (p+dp, d-dp, tc, t1/2).
__device__ __forceinline__ void take_child(Node &c, const V4 &dp, const V4 &tc, bool right)
{
#define FI_TAKE(k)                                                    \
    {                                                                 \
        const float pr = c.p.k + dp.k, dr = c.d.k - dp.k;             \
        const float h0 = 0.5f * c.t0.k, h1 = 0.5f * c.t1.k;           \
        c.p.k = right ? pr : c.p.k;                                   \
        c.d.k = right ? dr : dp.k;                                    \
        c.t0.k = right ? tc.k : h0;                                   \
        c.t1.k = right ? h1 : tc.k;                                   \
    }
    FI_TAKE(x) FI_TAKE(y) FI_TAKE(z) FI_TAKE(w)
#undef FI_TAKE
}

// ---------------------------------------------------------------------------
// Per-lane traversal state
// ---------------------------------------------------------------------------

struct Args {
    const float *rays; int64_t ray_stride; int64_t n_rays;
    const float *fibers; int64_t fiber_stride; int64_t n_fibers;
    const int32_t *pair_ray; const int32_t *pair_fiber; const uint8_t *pair_depth;
    int32_t depth; int64_t n_pairs;
    float *t_out; float *u_out; uint8_t *hit_out;
    int32_t *counts;                       // counting mode
    double *t64_out; double *u64_out;      // refinement
    float *normal_out;                     // normals (3 rows of n_pairs), or null
    // candidate lists: pair i is ray i against one candidate after another,
    // from number cand_first on (cand_fiber[cand_off[i] + cand_first]), each
    // tested against the ray shortened to the nearest hit so far; pair_depth
    // then indexes the candidates. Null cand_off: plain pairs.
    const int64_t *cand_off; const int32_t *cand_fiber; int32_t cand_first; int64_t n_cand;
    int32_t *fiber_out;                    // the fiber of each ray's nearest hit
};

// ---------------------------------------------------------------------------
// FP64 surface solve (FI_FP64_REFINE)
// ---------------------------------------------------------------------------
//
// The leaf cylinders converge to the solid swept by a disc of radius r(u)
// centred on C(u) in the plane normal to C'(u) (Sec. 3.2: the limit surface
// of the cylinders maps the intersection to the closest point on the curve),
// closed by the end discs. With refinement, a pair of depth > 16 runs the
// traversal with every pruning test enlarged by a bound on its FP32 rounding,
// so that no leaf holding part of that solid along the ray is pruned. A pair
// that reaches no leaf misses; one that does is decided in FP64 over the whole
// curve. In the ray frame (ray point P = (0, 0, t)):
//   the ray meets the disc plane of u at   t(u) = <C, C'> / C'_z
//   it lies in that disc when              phi(u) = |P(t(u)) - C(u)|^2 - r(u)^2 <= 0
//   boundary points solve                  f1 = <P - C, C'> = 0, f2 = |P - C|^2 - r^2 = 0
// narrow_curve cuts the curve to the part within its radius of the ray (most
// misses end there), simple_candidates decides short pieces with one closest
// point, and curve_candidates searches the rest: Newton's method on (f1, f2)
// from the FP32 leaf hit, roots of phi (sampled and bracketed), the end discs,
// t = 0 when the origin lies in a disc. The smallest candidate in [0, tmax) is
// the hit.

constexpr int kRefineAbove = 16;         // refine pairs of depth > 16
constexpr double kNewtonTol = 1e-9;      // relative residuals of an accepted Newton point
constexpr int kCurveSamples = 64;        // phi samples over the whole curve (local minima are searched)

struct Curve64 {
    double q[4][4];                      // control points in the FP64 ray frame (x, y, z, r)
    double scale;                        // largest control-point coordinate
    bool regular;                        // the edges of the control polygon agree in direction (C' keeps away from 0)
};

// quad: F is a quadratic table (12 rows), taken as its exact cubic elevation
__device__ __forceinline__ bool curve_in_ray_frame(const float *R, int64_t rs, const float *F,
                                                   int64_t fs, Curve64 &c, double *frame = nullptr,
                                                   bool quad = false)
{
    const double ox = R[0], oy = R[rs], oz = R[2 * rs];
    const double dx = R[3 * rs], dy = R[4 * rs], dz = R[5 * rs];
    const double n2 = fma(dx, dx, fma(dy, dy, dz * dz));
    if (!(n2 > 0.0) || !(n2 < INFINITY)) return false;
    const double il = 1.0 / sqrt(n2);
    const double w[3] = {dx * il, dy * il, dz * il};
    double u[3], v[3];
    make_onb(w[0], w[1], w[2], u, v);
    if (frame) {
#pragma unroll
        for (int k = 0; k < 3; ++k) { frame[k] = u[k]; frame[3 + k] = v[k]; frame[6 + k] = w[k]; }
    }
    double P[4][4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int row = quad ? 4 * (k == 3 ? 2 : k) + j : 4 * k + j;
            P[k][j] = (double)F[row * fs];
        }
    if (quad) {                      // P holds p0, p1, p2, p2: elevate
        double e1[4], e2[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            e1[j] = (P[0][j] + 2.0 * P[1][j]) / 3.0;
            e2[j] = (2.0 * P[1][j] + P[2][j]) / 3.0;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) { P[1][j] = e1[j]; P[2][j] = e2[j]; }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double ex = P[k][0] - ox;
        const double ey = P[k][1] - oy;
        const double ez = P[k][2] - oz;
        c.q[k][0] = fma(ex, u[0], fma(ey, u[1], ez * u[2]));
        c.q[k][1] = fma(ex, v[0], fma(ey, v[1], ez * v[2]));
        c.q[k][2] = fma(ex, w[0], fma(ey, w[1], ez * w[2]));
        c.q[k][3] = P[k][3];
    }
    c.scale = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        c.scale = fmax(c.scale, fmax(fabs(c.q[k][0]), fmax(fabs(c.q[k][1]), fabs(c.q[k][2]))));
    double e[3][3];
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int j = 0; j < 3; ++j) e[k][j] = c.q[k + 1][j] - c.q[k][j];
    c.regular = e[0][0] * e[1][0] + e[0][1] * e[1][1] + e[0][2] * e[1][2] > 0.0 &&
                e[1][0] * e[2][0] + e[1][1] * e[2][1] + e[1][2] * e[2][2] > 0.0 &&
                e[0][0] * e[2][0] + e[0][1] * e[2][1] + e[0][2] * e[2][2] > 0.0;
    return true;
}

// A boundary point needs a disc plane: where C'(u) vanishes (a zero end
// tangent, a cusp) <P - C, C'> = 0 holds for every P, and |P - C| = r(u)
// would describe a sphere, not the swept solid.
__device__ __forceinline__ bool has_disc(const Curve64 &c, const double D[4])
{
    return sqrt(D[0] * D[0] + D[1] * D[1] + D[2] * D[2]) > 1e-12 * c.scale;
}

// C(u) (with radius), D = C'(u)/3 (with r'/3) and E = C''(u)/6 (xyz)
__device__ __forceinline__ void eval_curve(const Curve64 &c, double u, double C[4], double D[4], double E[3])
{
    const double v = 1.0 - u;
    const double b0 = v * v * v, b1 = 3.0 * u * v * v, b2 = 3.0 * u * u * v, b3 = u * u * u;
    const double e0 = v * v, e1 = 2.0 * u * v, e2 = u * u;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        C[k] = fma(b0, c.q[0][k], fma(b1, c.q[1][k], fma(b2, c.q[2][k], b3 * c.q[3][k])));
        D[k] = fma(e0, c.q[1][k] - c.q[0][k], fma(e1, c.q[2][k] - c.q[1][k], e2 * (c.q[3][k] - c.q[2][k])));
    }
#pragma unroll
    for (int k = 0; k < 3; ++k)
        E[k] = fma(v, c.q[2][k] - 2.0 * c.q[1][k] + c.q[0][k], u * (c.q[3][k] - 2.0 * c.q[2][k] + c.q[1][k]));
}

// Normal of the disc at an end of the curve whose tangent vanishes (squared
// length at most 2^-40 of the squared chord; p1 = p0 or p2 = p3): the disc
// planes of the nearby u converge to the plane normal to the next
// control-polygon edge from that end (p2 - p0, resp. p3 - p1), or to the
// chord if that vanishes too. D (C'/3 at u) is replaced by that direction;
// elsewhere it is left alone.
__device__ __forceinline__ void end_disc_normal(const Curve64 &c, double u, double D[4])
{
    if (u != 0.0 && u != 1.0) return;
    const double ax = c.q[3][0] - c.q[0][0], ay = c.q[3][1] - c.q[0][1], az = c.q[3][2] - c.q[0][2];
    const double lim = 0x1p-40 * (ax * ax + ay * ay + az * az);
    if (D[0] * D[0] + D[1] * D[1] + D[2] * D[2] > lim) return;
    const int from = u == 0.0 ? 0 : 1, to = u == 0.0 ? 2 : 3;     // p2 - p0 or p3 - p1
    double nx = c.q[to][0] - c.q[from][0], ny = c.q[to][1] - c.q[from][1], nz = c.q[to][2] - c.q[from][2];
    if (nx * nx + ny * ny + nz * nz <= lim) { nx = ax; ny = ay; nz = az; }
    D[0] = nx;
    D[1] = ny;
    D[2] = nz;
}

// Ray point in the disc plane at u, and its signed excess |P-C|^2 - r^2.
__device__ __forceinline__ bool disc_point(const Curve64 &c, double u, double &t, double &phi)
{
    double C[4], D[4], E[3];
    eval_curve(c, u, C, D, E);
    end_disc_normal(c, u, D);
    if (D[2] == 0.0) return false;
    t = (C[0] * D[0] + C[1] * D[1] + C[2] * D[2]) / D[2];
    const double h = t - C[2];
    phi = C[0] * C[0] + C[1] * C[1] + h * h - C[3] * C[3];
    return true;
}

// phi(u) D_z^2 without the division: (C_x^2 + C_y^2 - r^2) D_z^2 +
// (C_x D_x + C_y D_y)^2 (the ray point's offset from the disc centre along
// the ray is (C_x D_x + C_y D_y) / D_z). Same sign as phi where the disc
// plane crosses the ray (D_z != 0); for the root search, which needs the
// sign and, within a narrow bracket where D_z barely changes, the shape.
__device__ __forceinline__ bool disc_excess_scaled(const Curve64 &c, double u, double &g)
{
    double C[4], D[4], E[3];
    eval_curve(c, u, C, D, E);
    end_disc_normal(c, u, D);
    if (D[2] == 0.0) return false;
    const double a = C[0] * D[0] + C[1] * D[1];
    g = (C[0] * C[0] + C[1] * C[1] - C[3] * C[3]) * (D[2] * D[2]) + a * a;
    return true;
}

// Does phi have a minimum inside the sample interval next to the end u (0 or
// 1), given that the end sample is the lower of the two? Only if phi turns
// there: it falls from u = 0, or rises into u = 1. From the slope of phi at
// the end (t = N / D_z with N = <C, D>, D = C'/3, D' = 2E):
//   phi' = 6 (C_x D_x + C_y D_y) + 2 (t - C_z)(t' - 3 D_z) - 6 r D_r,
//   t'   = ((3 |D|^2 + 2 <C, E>) D_z - 2 N E_z) / D_z^2.
// At a vanishing end tangent (no disc plane of its own; the limit plane
// serves) the slope is not formed and the interval is searched.
__device__ __forceinline__ bool end_turns(const Curve64 &c, double u)
{
    double C[4], D[4], E[3];
    eval_curve(c, u, C, D, E);
    const double ax = c.q[3][0] - c.q[0][0], ay = c.q[3][1] - c.q[0][1], az = c.q[3][2] - c.q[0][2];
    if (D[0] * D[0] + D[1] * D[1] + D[2] * D[2] <= 0x1p-40 * (ax * ax + ay * ay + az * az)) return true;
    if (D[2] == 0.0) return true;
    const double N = C[0] * D[0] + C[1] * D[1] + C[2] * D[2];
    const double t = N / D[2];
    const double dN = 3.0 * (D[0] * D[0] + D[1] * D[1] + D[2] * D[2]) + 2.0 * (C[0] * E[0] + C[1] * E[1] + C[2] * E[2]);
    const double dt = (dN * D[2] - 2.0 * N * E[2]) / (D[2] * D[2]);
    const double dphi = 6.0 * (C[0] * D[0] + C[1] * D[1]) + 2.0 * (t - C[2]) * (dt - 3.0 * D[2]) - 6.0 * C[3] * D[3];
    return u == 0.0 ? !(dphi >= 0.0) : !(dphi <= 0.0);       // NaN: searched
}

// t of a boundary point known to lie on the circle of the disc at u (C, D
// from eval_curve) whose plane crossing is t_plane = <C, D> / D_z. On the
// circle the same point is also C_z +- sqrt(r^2 - C_x^2 - C_y^2). The plane
// form loses about |C| |D| / |D_z| units of rounding as the disc plane turns
// towards the ray (D_z -> 0, near-collinear curves seen along their normal);
// the circle form loses about r^2 / sqrt(r^2 - C_x^2 - C_y^2) as the ray
// grazes the circle. The better conditioned form is returned, its sign
// taken from the plane form.
__device__ __forceinline__ double circle_t(const double C[4], const double D[4], double t_plane)
{
    const double rest = C[3] * C[3] - C[0] * C[0] - C[1] * C[1];
    if (!(rest > 0.0)) return t_plane;
    const double sr = sqrt(rest);
    const double e_plane = sqrt((C[0] * C[0] + C[1] * C[1] + C[2] * C[2]) * (D[0] * D[0] + D[1] * D[1] + D[2] * D[2])) /
                           fabs(D[2]);
    const double e_circle = C[3] * C[3] / sr;
    if (!(e_circle < e_plane)) return t_plane;
    return t_plane >= C[2] ? C[2] + sr : C[2] - sr;
}

// Newton's method on (f1, f2) from (t, u): true when it converges to a
// boundary point of the swept solid (entry or exit).
__device__ __forceinline__ bool newton_surface(const Curve64 &c, double &t, double &u)
{
    for (int it = 0; it < 10; ++it) {
        double C[4], D[4], E[3];
        eval_curve(c, u, C, D, E);
        const double h = t - C[2];
        const double f1 = h * D[2] - C[0] * D[0] - C[1] * D[1];
        const double f2 = C[0] * C[0] + C[1] * C[1] + h * h - C[3] * C[3];
        const double dd = D[0] * D[0] + D[1] * D[1] + D[2] * D[2];
        const double a11 = D[2];
        const double a12 = -3.0 * dd + 2.0 * (-C[0] * E[0] - C[1] * E[1] + h * E[2]);
        const double a21 = 2.0 * h;
        const double a22 = -6.0 * f1 - 6.0 * C[3] * D[3];
        const double det = a11 * a22 - a12 * a21;
        if (!(fabs(det) > 0.0)) return false;
        const double dt = (-f1 * a22 + f2 * a12) / det;
        const double du = (-f2 * a11 + f1 * a21) / det;
        t += dt;
        u += du;
        if (!(fabs(u) < 4.0) || !isfinite(t)) return false;
        if (fabs(du) <= 4e-16 && fabs(dt) <= 4e-16 * fabs(t)) break;
    }
    double C[4], D[4], E[3];
    eval_curve(c, u, C, D, E);
    const double h = t - C[2];
    const double scale = fmax(C[3] * C[3], 1e-300);
    const double f1 = h * D[2] - C[0] * D[0] - C[1] * D[1];
    const double f2 = C[0] * C[0] + C[1] * C[1] + h * h - C[3] * C[3];
    const double dn = sqrt(D[0] * D[0] + D[1] * D[1] + D[2] * D[2]);
    // the residual floor is set by cancellation in C (control points far
    // from the ray), so the test is loose; near a tangent ray a point that
    // passes it can still lie measurably off the surface (see bracket_polish)
    return has_disc(c, D) && fabs(f2) <= kNewtonTol * scale && fabs(f1) <= kNewtonTol * C[3] * dn;
}

// The root of g = s z^2 + a^2 (s = C_x^2 + C_y^2 - r^2, a = C_x D_x + C_y D_y,
// z = D_z: phi z^2, without a division) in a sign change [lo, hi] on which z
// keeps its sign (lo_in: g(lo) <= 0), from the estimate x: Newton's method kept
// inside the bracket, which every point narrows; a step that leaves it, or that
// hardly shrinks, bisects. Ends at steps below 2^-53. Returns the
// boundary point in (t, u).
__device__ __forceinline__ void side_root(const Curve64 &c, double lo, double hi, bool lo_in, double x, double &t,
                                          double &u)
{
    double last = hi - lo;
    if (!(x > lo && x < hi)) x = 0.5 * (lo + hi);
    for (int j = 0; j < 100; ++j) {
        double C[4], D[4], E[3];
        eval_curve(c, x, C, D, E);
        const double a = C[0] * D[0] + C[1] * D[1];
        const double s = C[0] * C[0] + C[1] * C[1] - C[3] * C[3];
        const double da = 3.0 * (D[0] * D[0] + D[1] * D[1]) + 2.0 * (C[0] * E[0] + C[1] * E[1]);
        const double z2 = D[2] * D[2];
        const double g = fma(s, z2, a * a);
        const double dg = fma(6.0 * (a - C[3] * D[3]), z2, fma(4.0 * s * D[2], E[2], 2.0 * a * da));
        if ((g <= 0.0) == lo_in) lo = x;
        else hi = x;
        const double step = g / dg;
        double y = x - step;
        if (!(y > lo && y < hi) || !(fabs(step) <= 0.8 * last)) {
            if (fabs(step) <= 0x1p-54) break;
            y = 0.5 * (lo + hi);
            if (!(y > lo && y < hi)) break;
        }
        last = fabs(y - x);
        x = y;
        if (last <= 0x1p-53) break;
    }
    u = x;
    double C[4], D[4], E[3];
    eval_curve(c, u, C, D, E);
    t = circle_t(C, D, (C[0] * D[0] + C[1] * D[1] + C[2] * D[2]) / D[2]);
}

// The boundary point in a sign change of phi on [lo, hi] (lo_in:
// phi(lo) <= 0): by side_root where the curve turns and slows down little on
// the bracket and D_z keeps its size (to a factor of 4, by the Bernstein
// coefficients of D), so that there is one. Otherwise (next to a cusp above
// all) phi may have poles and more roots than one there, and the bracket is
// narrowed step by step to
// at most 2^-53, then the root polished by Newton's method, kept
// only if it stays within a few final brackets (a polish that wanders
// further follows the residual's rounding, not the root); returns the
// boundary point in (t, u).
// The bracket is narrowed by the ITP method (interpolate, truncate, project;
// Oliveira and Takahashi, ACM Trans. Math. Softw. 47(1), 2020): each step
// takes the false-position estimate from the end values, moves it towards
// the midpoint by 0.2 (width)^2 / (initial width) (at least the final
// bracket), and keeps it within a distance of the midpoint that shrinks as
// the step budget is used up. It never takes more than one step beyond
// bisection, and on the simple roots that phi has where the ray crosses the
// boundary it takes about ten (a wave runs the steps of its slowest lane;
// bisection took 44).
__device__ __forceinline__ bool boundary_root(const Curve64 &c, double lo, double hi, bool lo_in, double &t,
                                              double &u)
{
    if (c.regular) {
        double C[4], D[4], E[3], F[4], G[3];
        eval_curve(c, lo, C, D, E);
        const double al = C[0] * D[0] + C[1] * D[1], sl = C[0] * C[0] + C[1] * C[1] - C[3] * C[3];
        eval_curve(c, hi, C, F, G);
        const double ah = C[0] * F[0] + C[1] * F[1], sh = C[0] * C[0] + C[1] * C[1] - C[3] * C[3];
        const double mx = fma(hi - lo, E[0], D[0]), my = fma(hi - lo, E[1], D[1]), mz = fma(hi - lo, E[2], D[2]);
        const double zs = copysign(1.0, D[2]) * fmin(fabs(D[2]), fmin(fabs(mz), fabs(F[2])));
        const double zl = fmax(fabs(D[2]), fmax(fabs(mz), fabs(F[2])));
        // of the three coefficients of D: least product with any other
        const double dm = fmin(D[0] * mx + D[1] * my + D[2] * mz,
                               fmin(F[0] * mx + F[1] * my + F[2] * mz, F[0] * D[0] + F[1] * D[1] + F[2] * D[2]));
        const double dl = fmax(D[0] * D[0] + D[1] * D[1] + D[2] * D[2],
                               fmax(mx * mx + my * my + mz * mz, F[0] * F[0] + F[1] * F[1] + F[2] * F[2]));
        if (D[2] * F[2] > 0.0 && D[2] * mz > 0.0 && fabs(zs) >= 0.25 * zl && dm >= 0.25 * dl) {
            const double gl = fma(sl, D[2] * D[2], al * al), gh = fma(sh, F[2] * F[2], ah * ah);
            if ((gl <= 0.0) == lo_in && (gh <= 0.0) != lo_in) {
                // the root of the parabola with its minimum at the inner end
                const double gi = lo_in ? gl : gh, go = lo_in ? gh : gl, w = (hi - lo) * sqrt(gi / (gi - go));
                side_root(c, lo, hi, lo_in, lo_in ? lo + w : hi - w, t, u);
                eval_curve(c, u, C, D, E);
                return has_disc(c, D);
            }
        }
    }
    constexpr double kEps = 0x1p-54;                // half the final bracket
    // g = phi with the sign that makes g(lo) <= 0 <= g(hi). It only places
    // the estimate (the bracket follows the sign of phi, as in bisection),
    // so it is kept in FP32, which saves registers: the estimate's relative
    // error of about 2^-24 still shrinks the bracket by about that factor a
    // step near the root.
    const float sg = lo_in ? 1.0f : -1.0f;
    float gl = 0.0f, gh = 0.0f;
    {
        double pl, ph;
        if (disc_excess_scaled(c, lo, pl) && disc_excess_scaled(c, hi, ph)) {
            gl = sg * (float)pl;
            gh = sg * (float)ph;
        }
    }
    const float k1 = 0.2f / (float)(hi - lo);
    const int nmax = ilogb((hi - lo) / (2.0 * kEps)) + 2;       // bisection's steps, rounded up, plus one
    for (int j = 0; j <= nmax && hi - lo > 2.0 * kEps; ++j) {
        const double w = hi - lo, mid = 0.5 * (lo + hi);
        double xf = mid;
        if (gl <= 0.0f && gh >= 0.0f && gh > gl) xf = lo + w * (double)(gl / (gl - gh));
        const double s = mid >= xf ? 1.0 : -1.0;
        // at least the final bracket: an estimate that lands on the root
        // then still steps past it, and the far end moves as well
        const double delta = fmax((double)k1 * w * w, 2.0 * kEps);
        const double xt = delta <= fabs(mid - xf) ? xf + s * delta : mid;
        const double r = ldexp(kEps, nmax - j) - 0.5 * w;
        double x = fabs(xt - mid) <= r ? xt : mid - s * r;
        if (!(x > lo && x < hi)) x = mid;
        if (!(x > lo && x < hi)) break;
        double xphi;
        if (!disc_excess_scaled(c, x, xphi)) return false;
        if ((xphi <= 0.0) == lo_in) {
            lo = x;
            gl = sg * (float)xphi;
        } else {
            hi = x;
            gh = sg * (float)xphi;
        }
    }
    u = 0.5 * (lo + hi);
    double phi;
    if (!disc_point(c, u, t, phi)) return false;
    {
        double C[4], D[4], E[3];
        eval_curve(c, u, C, D, E);
        if (!has_disc(c, D)) return false;
        t = circle_t(C, D, t);
    }
    double tn = t, un = u;
    if (newton_surface(c, tn, un) && fabs(un - u) <= 4.0 * (hi - lo) + 0x1p-50) {
        t = tn;
        u = un;
    }
    return true;
}

// A Newton point re-derived from a sign change of phi around it. Near a
// tangent ray the boundary point is ill-conditioned: a residual small enough
// to pass Newton's test still moves t by far more than rounding (a residual
// e * r^2 moves t by about e * r / sqrt(2 * penetration / r)). Brackets of
// growing width around u are tried; the first with a sign change is
// narrowed to its root. Without one the point is kept.
__device__ __forceinline__ void bracket_polish(const Curve64 &c, double &t, double &u)
{
    double w = 0x1p-32;
    for (int it = 0; it < 8; ++it, w *= 8.0) {
        double ta, pa, tb, pb;
        if (!disc_point(c, u - w, ta, pa) || !disc_point(c, u + w, tb, pb)) return;
        if ((pa <= 0.0) != (pb <= 0.0)) {
            double tt, uu;
            if (boundary_root(c, u - w, u + w, pa <= 0.0, tt, uu)) {
                t = tt;
                u = uu;
            }
            return;
        }
    }
}

// The part [a, b] of the curve outside which it stays further than its
// radius from the ray: every boundary point, end disc and disc that holds the
// origin lies at |C_xy(u)| <= r(u). The piece on [a, b] stays within
// 3/4 max |e_k| of its chord at the same parameter (e_k: what the inner
// control points are off the chord's third points), so only parameters whose
// chord point lies within that plus the largest radius of the ray remain: an
// interval. Each round narrows the piece to it; what the piece bends off its
// chord falls with the square of its length, so two to four rounds leave
// little more than the part within the radius. False when nothing remains:
// the ray misses. The hardware reciprocal and root (2^-22) are covered by the
// 1e-5 added to the distance and the 1e-6 added to the interval.
struct Part {
    double a, b;
    double reach;                        // the piece's distance bound from its chord, radius included
};

// One round on the piece [p.a, p.b]: 0 nothing remains, 1 narrowed to a piece
// of at least 0.7 of it (or not at all), 2 narrowed further.
__device__ __forceinline__ int narrow_piece(const Curve64 &c, Part &p)
{
    const double w = p.b - p.a;
    double p0[3], p3[3], d0[3], d3[3];              // x, y, r of the piece: ends and end edges
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const double u = e ? p.b : p.a, v = 1.0 - u;
        const double b0 = v * v * v, b1 = 3.0 * u * v * v, b2 = 3.0 * u * u * v, b3 = u * u * u;
        const double e0 = v * v, e1 = 2.0 * u * v, e2 = u * u;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int j = k < 2 ? k : 3;
            const double C = fma(b0, c.q[0][j], fma(b1, c.q[1][j], fma(b2, c.q[2][j], b3 * c.q[3][j])));
            const double D = fma(e0, c.q[1][j] - c.q[0][j],
                                 fma(e1, c.q[2][j] - c.q[1][j], e2 * (c.q[3][j] - c.q[2][j]))) * w;
            (e ? p3 : p0)[k] = C;
            (e ? d3 : d0)[k] = D;
        }
    }
    const double dx = p3[0] - p0[0], dy = p3[1] - p0[1];
    constexpr double third = 1.0 / 3.0;
    const double ax = fma(-third, dx, d0[0]), ay = fma(-third, dy, d0[1]);
    const double bx = fma(-third, dx, d3[0]), by = fma(-third, dy, d3[1]);
    const double bend = fmax(fma(ax, ax, ay * ay), fma(bx, bx, by * by));
    const double rad = fmax(fmax(fabs(p0[2]), fabs(p3[2])), fmax(fabs(p0[2] + d0[2]), fabs(p3[2] - d3[2])));
    p.reach = fma(0.75 * 1.00001, bend > 0.0 ? bend * __builtin_amdgcn_rsq(bend) : 0.0,
                  fma(1.00001, rad, 1e-14 * c.scale));
    const double dd = fma(dx, dx, dy * dy);
    const double inv = __builtin_amdgcn_rcp(dd);
    const double cr = p0[0] * dy - p0[1] * dx;
    const double rest = fma(p.reach, p.reach, -(cr * cr) * inv * (1.0 - 1e-6));
    if (rest < 0.0) return 0;
    const double half = rest * inv;
    if (!(half > 0.0 && half < 1e30)) return 1;     // no chord across the ray: nothing to narrow by
    const double h = half * __builtin_amdgcn_rsq(half) * (1.0 + 1e-6);
    const double mid = -fma(p0[0], dx, p0[1] * dy) * inv;
    const double pad = fma(1e-6, fabs(mid) + h, 1e-6);
    const double lo = mid - h - pad, hi = mid + h + pad;
    if (hi < 0.0 || lo > 1.0) return 0;
    p.b = hi < 1.0 ? fma(w, hi, p.a) : p.b;
    p.a = lo > 0.0 ? fma(w, lo, p.a) : p.a;
    return p.b - p.a < 0.7 * w ? 2 : 1;
}

__device__ __forceinline__ bool narrow_curve(const Curve64 &c, Part &p)
{
    p.a = 0.0;
    p.b = 1.0;
    int r = 2;
    for (int it = 0; it < 5 && r == 2; ++it) r = narrow_piece(c, p);
    return r != 0;
}

// Boundary points of a piece on which the curve is nearly straight, the part
// that can lie within its radius of the ray being short (on hair a few
// thousandths of the curve). With s = C_x^2 + C_y^2 - r^2,
// a = C_x D_x + C_y D_y and z = D_z, phi = s + (a / z)^2: where the curve is
// closest to the ray (a = 0, at xn) phi is s, and phi is close to the
// parabola s - 6 r D_r (u - xn) + K (u - xn)^2, K = (a' / z)^2 + 3 a'. So one
// evaluation decides whether the ray meets the side, and Newton's method on
// g = s z^2 + a^2 finds both boundary points from the parabola's roots in two
// or three steps, for grazing rays too. False where the piece is not that
// simple -- it bends, the discs are nearly parallel to the ray, the taper is
// steep, the ray touches within the taper's or the residual test's reach, the
// origin lies between the boundary points -- and the search below decides.
__device__ __forceinline__ bool simple_candidates(const Curve64 &c, const Part &part, double tmax, double &t_best,
                                                  double &u_best)
{
    const double lo = part.a, hi = part.b, v = hi - lo;
    if (!(v <= 0.5)) return false;
    double al, ah;
    {
        // phi has one minimum on the piece: a grows (a' = 3 D_xy^2 + 2 <C, E>_xy,
        // |C_xy| within the reach), z keeps its sign, and a / z grows with a
        // (|a z'| < a' |z|, z' = 2 E_z), so that s and (a / z)^2 both fall
        // before the closest point and rise after it; a mild taper moves the
        // minimum a little. Bounds from the Bernstein coefficients of D
        // (three) and E (its ends).
        double C[4], D[4], E[3], F[4], G[3];
        eval_curve(c, lo, C, D, E);
        al = C[0] * D[0] + C[1] * D[1];
        eval_curve(c, hi, C, F, G);
        ah = C[0] * F[0] + C[1] * F[1];
        const double ex = fmax(fabs(E[0]), fabs(G[0])), ey = fmax(fabs(E[1]), fabs(G[1]));
        const double ez = fmax(fabs(E[2]), fabs(G[2])), e2 = fma(ex, ex, ey * ey);
        const double mx = fma(v, E[0], D[0]), my = fma(v, E[1], D[1]), mz = fma(v, E[2], D[2]);
        const double sx = D[0] + F[0], sy = D[1] + F[1];
        const double low = fmin(fma(D[0], sx, D[1] * sy), fmin(fma(mx, sx, my * sy), fma(F[0], sx, F[1] * sy)));
        if (!(low > 0.0)) return false;
        const double dmin = low * low * __builtin_amdgcn_rcp(fma(sx, sx, sy * sy)) * 0.999999;
        const double dmax = fmax(fma(D[0], D[0], D[1] * D[1]),
                                 fmax(fma(mx, mx, my * my), fma(F[0], F[0], F[1] * F[1])));
        const double sg = copysign(1.0, D[2]), z = fmin(sg * D[2], fmin(sg * mz, sg * F[2]));
        const double R = part.reach;
        if (!(z > 0.0) || !(z * z >= 0x1p-20 * (dmax + z * z)) || !(4.0 * R * R * e2 <= dmin * dmin) ||
            !(16.0 * R * R * dmax * ez * ez <= dmin * dmin * z * z))
            return false;
        const double er = fmax(fabs(c.q[2][3] - 2.0 * c.q[1][3] + c.q[0][3]),
                               fabs(c.q[3][3] - 2.0 * c.q[2][3] + c.q[1][3]));
        const double dr = fma(v, er, fmax(fabs(D[3]), fabs(F[3])));
        if (!(16.0 * dr * dr <= dmin) || !(8.0 * R * er <= dmin)) return false;
    }
    // ends of the piece: outside but where the curve itself ends
    double t, phi = 1.0, ts = INFINITY, us = 0.0;
    const bool lo_in = lo <= 0.0 && disc_point(c, 0.0, t, phi) && phi <= 0.0;
    if (lo_in) { ts = t; us = 0.0; }
    const bool hi_in = hi >= 1.0 && disc_point(c, 1.0, t, phi) && phi <= 0.0;
    if (hi_in && t < ts) { ts = t; us = 1.0; }
    if (ts <= 0.0) return false;
    // closest point: Newton's method inside the bracket
    double xn = al >= 0.0 ? lo : hi, C[4], D[4], E[3];
    if (al < 0.0 && ah > 0.0) {
        double l = lo, h = hi, last = v;
        xn = fma(v, al / (al - ah), lo);
        for (int j = 0; j < 60; ++j) {
            eval_curve(c, xn, C, D, E);
            const double a = C[0] * D[0] + C[1] * D[1];
            const double da = 3.0 * (D[0] * D[0] + D[1] * D[1]) + 2.0 * (C[0] * E[0] + C[1] * E[1]);
            if (a > 0.0) h = xn;
            else l = xn;
            const double step = a / da;
            double y = xn - step;
            if (!(y > l && y < h) || !(fabs(step) <= 0.8 * last)) {
                if (fabs(step) <= 0x1p-54) break;
                y = 0.5 * (l + h);
                if (!(y > l && y < h)) break;
            }
            last = fabs(y - xn);
            xn = y;
            if (last <= 0x1p-40) break;          // phi is flat there: enough to decide by
        }
    }
    eval_curve(c, xn, C, D, E);
    const double r2 = C[3] * C[3], s = C[0] * C[0] + C[1] * C[1] - r2;
    const double da = 3.0 * (D[0] * D[0] + D[1] * D[1]) + 2.0 * (C[0] * E[0] + C[1] * E[1]);
    const double K = fma(da / D[2], da / D[2], 3.0 * da), rd = 3.0 * C[3] * D[3];
    const bool inner = xn > lo && xn < hi;
    const double room = 4.0 * (rd * rd / K) + 4.0 * kNewtonTol * r2;
    if (fabs(s) <= room) return false;                          // touches
    if (!inner && !(lo_in || hi_in)) {
        // the closest point is an end of the curve: outside its disc, the
        // side is not met unless the taper or the discs' tilt reaches back
        const double a = C[0] * D[0] + C[1] * D[1];
        const double f = s + (a / D[2]) * (a / D[2]);
        if (!(f > 0.0) || !(s > 0.0)) return false;
        const double f1 = 6.0 * (a - C[3] * D[3]) + 2.0 * (a / D[2]) * (da / D[2]);
        if ((xn == lo) != (f1 > 0.0)) return false;             // phi falls into the piece
    }
    if (ts < tmax && ts < t_best) { t_best = ts; u_best = us; }
    const bool n_in = inner ? s < 0.0 : xn == lo ? lo_in : hi_in;
    const double w = sqrt(fmax(-s, 0.0) / K);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const double l = j ? xn : lo, h = j ? hi : xn;
        const bool li = j ? n_in : lo_in, hin = j ? hi_in : n_in;
        if (li == hin || !(h > l)) continue;
        if (!inner && s > 0.0) return false;
        double tr, ur;
        side_root(c, l, h, li, j ? xn + w : xn - w, tr, ur);
        if (!(tr > 0.0)) return false;                          // the origin may be inside
        if (tr < tmax && tr < t_best) { t_best = tr; u_best = ur; }
    }
    return true;
}

// Boundary points of the swept solid along the ray; the earliest with t in
// [0, tmax) is kept in (t_best, u_best). (t0, u0) is the FP32 leaf hit. Also the
// end discs, and t = 0 when the origin lies in one of the discs. The earliest
// boundary point of the solid is its entry (or the origin, when inside), so
// no entry/exit classification is needed.
// For the pairs that narrow_curve and simple_candidates leave open. phi is
// sampled at the parameters k / kCurveSamples about the part of the curve that
// can lie within its radius of the ray (elsewhere phi is above zero and
// nothing can be found) in two passes, so that the lanes of a wave stay
// together: the first records, per sample interval, the events that need a
// search (a sign change of phi, a local minimum of phi above zero, a crossing
// of the disc plane through the origin) as bit masks; the second searches the
// recorded events one after another. A wave then runs one search per event of
// its busiest lane, not the union of every lane's searches at every sample.
__device__ __forceinline__ void curve_candidates(const Curve64 &c, const Part &part, double tmax, double t0, double u0,
                                                 double &t_best, double &u_best)
{
    constexpr int NS = kCurveSamples;
    auto take = [&](double t, double u) {
        if (t >= 0.0 && t < tmax && t < t_best) { t_best = t; u_best = u; }
    };
    {
        double t = t0, u = u0;
        if (newton_surface(c, t, u)) {
            bracket_polish(c, t, u);
            if (u >= 0.0 && u <= 1.0) take(t, u);
        }
    }
    auto at = [](int k) { return (double)k * (1.0 / NS); };
    // every event whose search could find a point has its bracket, up to two
    // sample intervals, about the part: samples k0..k1
    const int k0 = max(0, (int)floor(part.a * NS) - 2), k1 = min(NS, (int)ceil(part.b * NS) + 2);
    // sample k (k < 64): inside (phi <= 0) and t <= 0 flags in bit k; events
    // on (k-1, k] in bit k-1
    uint64_t in_m = 0, tneg_m = 0, sign_m = 0, min_m = 0, org_m = 0;
    // the first sample counts as a minimum (event 1) only where phi turns
    // inside the first interval
    double pt = 0.0, pphi = 0.0, ppphi = k0 > 0 || !end_turns(c, 0.0) ? -INFINITY : INFINITY;
    bool pok = disc_point(c, at(k0), pt, pphi);
    if (pok && pphi <= 0.0) in_m |= (uint64_t)1 << k0;
    if (pok && pt <= 0.0) tneg_m |= (uint64_t)1 << k0;
    for (int k = k0 + 1; k <= k1; ++k) {
        double ct = 0.0, cphi = 0.0;
        const bool cok = disc_point(c, at(k), ct, cphi);
        const uint64_t bit = (uint64_t)1 << (k - 1);
        if (cok && cphi <= 0.0 && k < NS) in_m |= bit << 1;
        if (cok && ct <= 0.0 && k < NS) tneg_m |= bit << 1;
        if (pok && cok) {
            if ((pphi <= 0.0) != (cphi <= 0.0)) sign_m |= bit;
            else if (pphi > 0.0 && cphi > pphi && ppphi > pphi) min_m |= bit;
            if ((pt <= 0.0) != (ct <= 0.0) && (pphi <= 0.0 || cphi <= 0.0)) org_m |= bit;
        }
        ppphi = pok ? pphi : INFINITY;
        pt = ct; pphi = cphi; pok = cok;
    }
    // phi still falling at the last sample: a dip can sit between the last
    // two samples (as at a stalled end, where the disc planes turn fast as
    // u -> 1), where phi turns before the end; recorded as the event of a
    // minimum at sample NS - 1 (searched on (u[NS-2], u[NS]), which holds it)
    if (k1 == NS && pok && pphi > 0.0 && ppphi > pphi && end_turns(c, 1.0)) min_m |= (uint64_t)1 << (NS - 1);
    auto flag = [](uint64_t m, int k) { return ((m >> k) & 1u) != 0u; };
    auto next_event = [](uint64_t &m) {        // lowest recorded event (1..NS; -1: none), removed from the mask
        const int k = m ? __builtin_ctzll(m) + 1 : -1;
        m &= m - 1u;
        return k;
    };
    // sign changes: one boundary point between the samples
    for (int k; (k = next_event(sign_m)) >= 0;) {
        {
            double t, u;
            if (boundary_root(c, at(k - 1), at(k), flag(in_m, k - 1), t, u)) take(t, u);
        }
    }
    // a local minimum of phi above zero at sample k-1: a dip below zero
    // narrower than the sampling has two boundary points in (u[k-2], u[k]).
    // The dip is searched by Brent's minimisation (Brent, Algorithms for
    // Minimization without Derivatives, 1973, ch. 5): a parabola through
    // the three best points so far, replaced by a golden-section step
    // whenever its step is not acceptable, from the lowest sample. It stops
    // at the first point with phi <= 0, or once the bracket around the best
    // point is 2^-33 of the initial one (where 48 golden-section steps end,
    // 0.618^48), in about a third of their evaluations.
    for (int k; (k = next_event(min_m)) >= 0;) {
        {
            constexpr double g = 0.38196601125010515;         // golden-section step
            double a = at(k >= 2 ? k - 2 : 0), b = at(k), tt;
            // phi stays above zero where the curve stays off the ray
            Part dip{a, b, 0.0};
            if (narrow_piece(c, dip) == 0) continue;
            const double tol = (b - a) * 0x1p-35;
            double x = at(k - 1), fx = 0.0;
            bool ok = disc_point(c, x, tt, fx);
            double xw = x, xv = x, fw = fx, fv = fx, d = 0.0, e = 0.0;
            for (int it = 0; ok && it < 64 && fx > 0.0; ++it) {
                const double m = 0.5 * (a + b);
                if (fabs(x - m) <= 2.0 * tol - 0.5 * (b - a)) break;
                bool gold = true;
                if (fabs(e) > tol) {
                    const double r = (x - xw) * (fx - fv);
                    double q = (x - xv) * (fx - fw);
                    double p = (x - xv) * q - (x - xw) * r;
                    q = 2.0 * (q - r);
                    if (q > 0.0) p = -p;
                    else q = -q;
                    const double e_old = e;
                    e = d;
                    if (fabs(p) < fabs(0.5 * q * e_old) && p > q * (a - x) && p < q * (b - x)) {
                        d = p / q;                               // the parabola's step
                        const double un = x + d;
                        if (un - a < 2.0 * tol || b - un < 2.0 * tol) d = m >= x ? tol : -tol;
                        gold = false;
                    }
                }
                if (gold) {
                    e = (x >= m ? a : b) - x;
                    d = g * e;
                }
                const double un = fabs(d) >= tol ? x + d : x + (d > 0.0 ? tol : -tol);
                double fu;
                ok = disc_point(c, un, tt, fu);
                if (!ok) break;
                if (fu <= fx) {
                    if (un >= x) a = x;
                    else b = x;
                    xv = xw; fv = fw;
                    xw = x; fw = fx;
                    x = un; fx = fu;
                } else {
                    if (un < x) a = un;
                    else b = un;
                    if (fu <= fw || xw == x) {
                        xv = xw; fv = fw;
                        xw = un; fw = fu;
                    } else if (fu <= fv || xv == x || xv == xw) {
                        xv = un; fv = fu;
                    }
                }
            }
            if (ok && fx <= 0.0) {
                // the minimisation's bracket ends lie above zero (samples,
                // or points it evaluated before the first one at or below
                // zero), so they bracket the two boundary points more
                // tightly than the samples
                const double um = x;
                double t, u;
                if (boundary_root(c, a, um, false, t, u)) take(t, u);
                if (boundary_root(c, um, b, true, t, u)) take(t, u);
            }
        }
    }
    // the disc plane sweeps through the origin: is the origin in that disc?
    for (int k; (k = next_event(org_m)) >= 0;) {
        {
            double lo = at(k - 1), hi = at(k);
            const bool lo_neg = flag(tneg_m, k - 1);
            for (int it = 0; it < 64; ++it) {
                const double mid = 0.5 * (lo + hi);
                double mt, mphi;
                if (!disc_point(c, mid, mt, mphi)) break;
                if ((mt <= 0.0) == lo_neg) lo = mid; else hi = mid;
            }
            const double uz = 0.5 * (lo + hi);
            double C[4], D[4], E[3];
            eval_curve(c, uz, C, D, E);
            if (C[0] * C[0] + C[1] * C[1] + C[2] * C[2] <= C[3] * C[3]) take(0.0, uz);
        }
    }
    // end discs
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        if ((e == 0 && part.a > 0.0) || (e == 1 && part.b < 1.0)) continue;
        double C[4], D[4], E[3];
        eval_curve(c, (double)e, C, D, E);
        end_disc_normal(c, (double)e, D);      // a vanishing end tangent: the limit plane
        if (D[2] == 0.0) continue;
        const double tc = (C[0] * D[0] + C[1] * D[1] + C[2] * D[2]) / D[2];
        const double hz = tc - C[2];
        if (C[0] * C[0] + C[1] * C[1] + hz * hz <= C[3] * C[3]) take(tc, (double)e);
    }
}

struct Lane {
    Node c;                       // current node, {p, d, t0, t1} in the ray frame
    Node root;                    // the pair's root (replays of the split rules start here)
    float lo, hi;                 // cropped t interval of the current node
    float tmax, t;                // ray tmax; hit distance once found
    uint32_t bits, start, size;   // Section 3.3: pending-sibling bits, integer interval (start:
                                  // bits 0..22; bit 31 set when the pair's end nodes may stall,
                                  // see stall_possible)
    uint32_t min_size;            // leaf size 2^(23 - depth)
    uint32_t cached;              // size of the pending children whose parent is cached (0: none)
    int32_t waiting;              // refined candidate lists: parked at its first leaf until the wave
                                  //   decides it
    float ru;                     //   the FP32 u of the leaf hit (Newton's start)
    int32_t scene;                // batched: the problem this pair belongs to
    int32_t pair;                 // index of the pair within its problem
    float slack;                  // conservative mode: bound on across-ray rounding of any node
                                  // (negative: a pair of depth <= 16, searched by the plain rules)
    int32_t trips, splits, backtracks;
    float u;                      // u of a leaf hit
    int32_t level;                // level of a leaf hit
};

enum { kGoOn = 0, kHit = 1, kMiss = 2 };

// Traversal variants: plain, counting, and conservative (for FP64 refinement:
// every pruning test is enlarged by a bound on its FP32 rounding error, so no
// surface point within that error is pruned; FP64 then decides).
enum { kPlain = 0, kCount = 1, kConservative = 2 };

// Per-lane LDS column (conflict-free: lane-contiguous rows of 64 floats) that
// caches the parent of the most recent split that left a sibling pending, so
// that the usual backtrack (to that sibling) rebuilds it with one split. Other
// backtracks replay the split rules from the root, re-read from the lane's
// root slot.
__device__ __forceinline__ void lds_put(float *col, const Node &r)
{
    const float *f = &r.p.x;
#pragma unroll
    for (int k = 0; k < 16; ++k) col[k * kWave] = f[k];
}

__device__ __forceinline__ void lds_get(const float *col, Node &r)
{
    float *f = &r.p.x;
#pragma unroll
    for (int k = 0; k < 16; ++k) f[k] = col[k * kWave];
}


// Each split rounds a node's position at the magnitude of its partial sum,
// which starts at the root's across-ray extent, so deep nodes inherit errors
// of a few ulp of that extent; 2^-18 of it is a generous bound.
__device__ __forceinline__ float root_slack(const Node &r)
{
    return (fabsf(r.p.x) + fabsf(r.p.y) + fabsf(r.d.x) + fabsf(r.d.y) +
            fabsf(r.t0.x) + fabsf(r.t0.y) + fabsf(r.t1.x) + fabsf(r.t1.y)) * 0x1p-18f;
}

// Pruning test of a node (Section 3.2): does the ray meet the conservative
// cylinder inside the node's cropped interval? `lo_used` / `hi_used` are the
// interval the test used (enlarged in conservative mode); a leaf's t is taken
// from its start.
template <int MODE, bool QUAD = false>
__device__ __forceinline__ bool node_visible(const Node &c, float lo, float hi, float slack, float &te,
                                             float &tx, float &lo_used, float &hi_used)
{
    float rad = conservative_radius<QUAD>(c);
    if (MODE == kConservative && slack >= 0.0f) {
        rad += slack + rad * 0x1p-18f;
        // an interval emptied on purpose (a parked lane, a cap plane parallel
        // to the ray that excludes it) must stay empty: no slack, since
        // infinite bounds would turn it into NaN, which fmaxf/fminf ignore
        const bool open = lo < INFINITY && hi > -INFINITY;
        const float tslack = open ? (fabsf(lo) + fabsf(hi < INFINITY ? hi : lo)) * 0x1p-17f : 0.0f;
        lo -= tslack;
        hi += tslack;
    }
    lo_used = lo;
    hi_used = hi;
    return unit_ray_cylinder(c.p, c.d, rad, te, tx) && fmaxf(te, lo) <= fminf(tx, hi);
}

// Bound on the rounding of a ray-plane distance c / n_z with c = <point, n>:
// the products' magnitudes over |n_z| (obliquity amplifies), plus the size
// of the result, at 2^-18 (64 ulp).
__device__ __forceinline__ float plane_slack(float px, float py, float pz, float nx, float ny, float nz, float t)
{
    return (fabsf(px * nx) + fabsf(py * ny) + fabsf(pz * nz)) * rcp(fabsf(nz)) * 0x1p-18f +
           fabsf(t) * 0x1p-18f;
}

// u of a leaf hit (Section 3.3): the hit point projected onto the leaf chord.
__device__ __forceinline__ float leaf_u(const Lane &L)
{
    const float cc = dot3(L.c.d.x, L.c.d.y, L.c.d.z, L.c.d.x, L.c.d.y, L.c.d.z);
    float ul = 0.0f;
    if (cc > 0.0f) {
        ul = dot3(-L.c.p.x, -L.c.p.y, L.t - L.c.p.z, L.c.d.x, L.c.d.y, L.c.d.z) * rcp(cc);
        ul = fminf(1.0f, fmaxf(0.0f, ul));
    }
    return fmaf(ul, (float)L.size * 0x1p-23f, (float)(L.start & kStartMask) * 0x1p-23f);
}

// FP64 decision of a pair of depth > 16 whose conservative search reached a
// leaf: the earliest boundary point of the swept solid along the ray over the
// whole curve, t in [0, tmax).
struct Refined {
    double t = INFINITY, u = __builtin_nan("");
    bool hit = false;
    float nx = __builtin_nanf(""), ny = __builtin_nanf(""), nz = __builtin_nanf("");   // world space
};

// Outward unit normal of the swept solid at a refined hit (ray frame):
// at an end disc (u = 0 or 1) minus the start tangent or the end tangent
// (their limits where they vanish); on the side, where the surface is
// C(u) + r(u) e with e a unit vector normal to C'(u), the unit direction e
// from C(u) to the hit, tilted against the tangent T by the taper:
// e - r' / (|C'| - r <e, C''> / |C'|) T (the disc's normal plane turns with
// the curve, hence the curvature term). In the units of eval_curve (D = C'/3
// with r'/3, E = C''/6) the tilt is 3 D_r / (3 |D| - 2 r <e, E> / |D|). The
// origin inside the solid (t = 0) has no surface crossing: NaN.
__device__ __forceinline__ void solid_normal(const Curve64 &c, double t, double u, double n[3])
{
    double C[4], D[4], E[3];
    eval_curve(c, u, C, D, E);
    if (t == 0.0) {
        n[0] = n[1] = n[2] = __builtin_nan("");
        return;
    }
    if (u == 0.0 || u == 1.0) {
        end_disc_normal(c, u, D);
        const double s = (u == 0.0 ? -1.0 : 1.0) * rsqrt64(D[0] * D[0] + D[1] * D[1] + D[2] * D[2]);
        n[0] = s * D[0];
        n[1] = s * D[1];
        n[2] = s * D[2];
        return;
    }
    double ex = -C[0], ey = -C[1], ez = t - C[2];
    const double ie = rsqrt64(ex * ex + ey * ey + ez * ez);
    ex *= ie; ey *= ie; ez *= ie;
    const double dl = sqrt(D[0] * D[0] + D[1] * D[1] + D[2] * D[2]);
    const double tilt = -3.0 * D[3] / (3.0 * dl - 2.0 * C[3] * (ex * E[0] + ey * E[1] + ez * E[2]) / dl);
    n[0] = ex + tilt * D[0] / dl;
    n[1] = ey + tilt * D[1] / dl;
    n[2] = ez + tilt * D[2] / dl;
}

// The result of a search that ended at (t, u), with the normal turned back
// into world space.
__device__ __forceinline__ Refined refined_at(const Curve64 &cv, const double frame[9], double t, double u, bool normal)
{
    Refined r;
    if (t < INFINITY) {
        r.t = t;
        r.u = u;
        r.hit = true;
        if (normal) {
            double n[3];
            solid_normal(cv, t, u, n);
            // back to world space: n.x u + n.y v + n.z w, unit length
            const double wx = n[0] * frame[0] + n[1] * frame[3] + n[2] * frame[6];
            const double wy = n[0] * frame[1] + n[1] * frame[4] + n[2] * frame[7];
            const double wz = n[0] * frame[2] + n[1] * frame[5] + n[2] * frame[8];
            const double il = rsqrt64(wx * wx + wy * wy + wz * wz);
            r.nx = (float)(wx * il);
            r.ny = (float)(wy * il);
            r.nz = (float)(wz * il);
        }
    }
    return r;
}

// Candidate lists: the decision inside the traversal kernel, for fiber `fi`
// within `tmax`, the ray shortened to its FP64 nearest hit so far. Arguments
// and result go by value: a reference to the caller's lane state or to the
// kernel's arguments would keep them in scratch memory for the whole kernel
// (the call is not inlined), every trip included.
__device__ __noinline__ Refined refine_whole_curve(const float *rays, int64_t ray_stride, const float *fibers,
                                                   int64_t fiber_stride, int64_t ri, int64_t fi, double tmax, float t0,
                                                   float u0, bool normal)
{
    Curve64 cv;
    double frame[9];
    if (!curve_in_ray_frame(rays + ri, ray_stride, fibers + fi, fiber_stride, cv, frame, false)) return Refined{};
    double t = INFINITY, u = __builtin_nan("");
    Part part;
    if (narrow_curve(cv, part) && !simple_candidates(cv, part, tmax, t, u)) {
        t = INFINITY;
        u = __builtin_nan("");
        curve_candidates(cv, part, tmax, (double)t0, (double)u0, t, u);
    }
    return refined_at(cv, frame, t, u, normal);
}

// One loop trip of the paper's iteration (Appendix C, final listing): a
// pruning test of the current node, then a descent, a leaf hit, a miss, or a
// jump to the deepest pending sibling.
// The descent (split, ordering, child) is straight-line code computed for
// every continuing lane; a lane that backtracks then overwrites its result
// with the rebuilt sibling. The new node thus has a single definition point,
// which spares the copies of the whole lane state that a merge of separately
// computed nodes costs, and a backtracking lane only adds the rebuild.
// The split of the current node (Section 3.1 / 3.2): centre offset and split
// tangent, the split plane's crossing tp with the ray, whether the ray meets
// both halves inside [te, tx], which half it meets first, and the interval
// of that half (narrowed at tp).
struct Split {
    V4 dp, tc;
    float nlo, nhi;
    bool both, near_right, oblique;
};

template <int MODE>
__device__ __forceinline__ void split_plane(const Lane &L, float te, float tx, Split &sp)
{
    // at a cusp (no split tangent) the split plane is normal to the chord
    const bool cusp = split_terms(L.c, sp.dp, sp.tc);
    const float nx = cusp ? L.c.d.x : sp.tc.x;
    const float ny = cusp ? L.c.d.y : sp.tc.y;
    const float nz = cusp ? L.c.d.z : sp.tc.z;
    const float qx = L.c.p.x + sp.dp.x, qy = L.c.p.y + sp.dp.y, qz = L.c.p.z + sp.dp.z;
    const float cs = dot3(qx, qy, qz, nx, ny, nz);
    const float tp = cs * rcp(nz);
    sp.oblique = nz != 0.0f;
    sp.nlo = L.lo;
    sp.nhi = L.hi;
    if (MODE == kConservative && L.slack >= 0.0f) {
        // visit both halves unless the crossing is clearly outside [te, tx];
        // narrow by the far side of tp's rounding bound
        const float ep = plane_slack(qx, qy, qz, nx, ny, nz, tp);
        sp.both = sp.oblique ? (te - ep < tp && tp < tx + ep)
                             : (cs == 0.0f || fabsf(cs) <= L.slack * (fabsf(nx) + fabsf(ny)));
        if (tp > te) sp.nhi = fminf(sp.nhi, tp + ep);
        else         sp.nlo = fmaxf(sp.nlo, tp - ep);
    } else {
        sp.both = sp.oblique ? (te < tp && tp < tx) : cs == 0.0f;
        if (tp > te) sp.nhi = fminf(sp.nhi, tp);
        else         sp.nlo = fmaxf(sp.nlo, tp);
    }
    // a plane parallel to the ray leaves the whole ray on the side of sign(-cs)
    sp.near_right = sp.oblique ? ((tp > te) != (nz > 0.0f)) : cs < 0.0f;
}

// Bookkeeping of a descent into the near half (Section 3.3: one level down,
// the far half pending when the ray meets both).
template <bool PC>
__device__ __forceinline__ void descend_state(Lane &L, const Split &sp)
{
    if (sp.oblique) { L.lo = sp.nlo; L.hi = sp.nhi; }
    L.size >>= 1;
    if (sp.both) {
        L.bits ^= L.size;
        if (PC) L.cached = L.size;
    }
    if (sp.near_right) L.start ^= L.size;
}

// Where a backtrack that misses the parent cache finds its pair's root: in
// the lane's registers (16 more VGPRs per lane, which the occupancy that
// the LDS queue allows can hold), so a replay starts without a memory
// access.
struct RegRoot {
    __device__ __forceinline__ void get(const Lane &L, Node &n) const { n = L.root; }
};

// What the normal of a leaf hit needs from the leaf, taken before the trip
// moves on to a child: the ray-frame vector from the leaf chord's point at
// the hit's projection to the hit point, and whether the hit entered the
// leaf through a plane (the interval's start) rather than the cylinder's
// side.
struct HitGeo {
    float vx, vy, vz;
    bool plane;
};

__device__ __forceinline__ HitGeo hit_geo(const Node &c, float t, bool plane)
{
    const float cc = dot3(c.d.x, c.d.y, c.d.z, c.d.x, c.d.y, c.d.z);
    float ul = 0.0f;
    if (cc > 0.0f) {
        ul = dot3(-c.p.x, -c.p.y, t - c.p.z, c.d.x, c.d.y, c.d.z) * rcp(cc);
        ul = fminf(1.0f, fmaxf(0.0f, ul));
    }
    return HitGeo{-fmaf(ul, c.d.x, c.p.x), -fmaf(ul, c.d.y, c.p.y), t - fmaf(ul, c.d.z, c.p.z), plane};
}

// Stalled end nodes. Where an end tangent vanishes the curve leaves that end
// with vanishing speed, and the end nodes' chords shrink like 4^-level: from
// some level on, all their control points coincide to FP32 precision, every
// test on them is rounding noise, and a search through them can visit
// thousands of nodes. A node that holds an end of the curve (u = 0 or u = 1)
// and whose extent -- the largest squared length of its chord and end
// tangents -- is at most (2^-20 X)^2 (X: the largest ray-frame coordinate of
// the root's control points) and at most 2^-16 of the root's extent times
// 4^-level, is therefore a leaf. Near a vanishing end tangent the curve keeps
// a fixed direction, so such a node's end planes stay perpendicular to its
// chord and its cylinder stays closed. Cusps (interior stalls, where the
// direction reverses) are not cut short.
__device__ __forceinline__ float node_extent(const Node &c)
{
    const float cc = dot3(c.d.x, c.d.y, c.d.z, c.d.x, c.d.y, c.d.z);
    const float a0 = dot3(c.t0.x, c.t0.y, c.t0.z, c.t0.x, c.t0.y, c.t0.z);
    const float a1 = dot3(c.t1.x, c.t1.y, c.t1.z, c.t1.x, c.t1.y, c.t1.z);
    return fmaxf(cc, fmaxf(a0, a1));
}

// The end nodes' outer tangents shrink exactly like 2^-level (halving is
// exact), so their extents stay at least |t0|^2 4^-level (start) and
// |t1|^2 4^-level (end): a pair whose root end tangents both exceed 2^-15 of
// the root's extent (a factor 2 above the bound, against rounding) can never
// stall, and its lanes skip the test. Decided in the setup round, with the
// root's other tests.
__device__ __forceinline__ bool stall_possible(const Node &r)
{
    const float a0 = dot3(r.t0.x, r.t0.y, r.t0.z, r.t0.x, r.t0.y, r.t0.z);
    const float a1 = dot3(r.t1.x, r.t1.y, r.t1.z, r.t1.x, r.t1.y, r.t1.z);
    const float ext = node_extent(r);
    return a0 <= 0x1p-15f * ext || a1 <= 0x1p-15f * ext;
}

// (2^-20 X)^2 of the pair's root (X: its largest ray-frame coordinate)
__device__ __forceinline__ float stall_abs(const Node &r)
{
    const float ex = r.p.x + r.d.x, ey = r.p.y + r.d.y, ez = r.p.z + r.d.z;     // p3
    float X = fmaxf(fabsf(r.p.x), fmaxf(fabsf(r.p.y), fabsf(r.p.z)));
    X = fmaxf(X, fmaxf(fabsf(r.p.x + r.t0.x), fmaxf(fabsf(r.p.y + r.t0.y), fabsf(r.p.z + r.t0.z))));
    X = fmaxf(X, fmaxf(fabsf(ex - r.t1.x), fmaxf(fabsf(ey - r.t1.y), fabsf(ez - r.t1.z))));
    X = fmaxf(X, fmaxf(fabsf(ex), fmaxf(fabsf(ey), fabsf(ez))));
    return 0x1p-40f * X * X;
}

__device__ __forceinline__ bool stalled_end(const Lane &L)
{
    if (!(L.start & kStallBit)) return false;
    const float s = (float)L.size * 0x1p-23f;                 // 2^-level
    const float rel = 0x1p-16f * node_extent(L.root) * s * s;
    // the chord alone fails the relative bound at every regular node: the
    // extent (at least the chord) is only formed where it passes
    const float cc = dot3(L.c.d.x, L.c.d.y, L.c.d.z, L.c.d.x, L.c.d.y, L.c.d.z);
    if (!(cc <= rel)) return false;
    const float e = node_extent(L.c);
    const uint32_t start = L.start & kStartMask;
    const bool end = start == 0u || start + L.size == kRootSize;
    return end && e <= rel && e <= stall_abs(L.root);
}

// PC: the parent cache in LDS (else every backtrack replays from the root).
// PARK: a refined pair's lane parks at its first leaf (candidate lists).
template <int MODE, bool QUAD, bool PC, bool PARK, class Root>
__device__ __forceinline__ int trip(Lane &L, const Root &root, float *col, HitGeo &hg)
{
    float te, tx, lo, hi;
    bool vis = node_visible<MODE, QUAD>(L.c, L.lo, L.hi, L.slack, te, tx, lo, hi);
    const bool leaf = L.size <= L.min_size || stalled_end(L);
    if (MODE == kConservative && PARK && vis && leaf && L.slack >= 0.0f) {
        // refinement: the first leaf reached means the solid may be hit; park
        // the lane (empty interval, no pending sibling) until the wave decides
        // its parked pairs in FP64, keeping the leaf hit as Newton's start
        L.t = fmaxf(te, lo);
        L.ru = leaf_u(L);
        L.bits = 0;
        L.lo = INFINITY;
        L.hi = -INFINITY;
        L.waiting = 1;
        vis = false;
    }
    // A lane that stops here still runs the rest of the trip (its state is
    // not used again): without early returns the lane state keeps one set of
    // registers across the loop instead of being copied at every exit.
    int st = kGoOn;
    if (vis && leaf) {
        L.t = fmaxf(te, lo);
        hg = hit_geo(L.c, L.t, te < lo);
        L.u = leaf_u(L);
        L.level = 23 - (31 - __builtin_clz(L.size));
        st = kHit;
    }
    const bool over = ++L.trips > kMaxTrips;          // hang guard (each trip is a test)
    if ((!vis && L.bits == 0) || over) st = kMiss;
    // A backtracking lane first rebuilds the parent of its pending sibling
    // (Section 3.3: the deepest level with a pending sibling) -- the cached
    // parent, or a replay of the split rules from the root along the integer
    // path -- and then takes the same split as a descending lane: one split
    // per trip for every continuing lane.
    const bool back = !vis && st == kGoOn;
    if (back) {
        L.size = L.bits & (0u - L.bits);
        L.start ^= L.size;
        L.bits ^= L.size;
        L.start &= ~(L.size - 1u);
        if (PC && L.cached == L.size) {
            lds_get(col, L.c);
        } else {
            root.get(L, L.c);
            for (uint32_t b = kRootSize >> 1; b > L.size; b >>= 1) {
                V4 rdp, rtc;
                split_terms(L.c, rdp, rtc);
                take_child(L.c, rdp, rtc, (L.start & b) != 0u);
            }
        }
        L.cached = 0;
    }
    // Section 3.1 / 3.2: split plane through the centre, normal to the split
    // tangent; a descending lane goes to the half the ray meets first
    Split sp;
    split_plane<MODE>(L, te, tx, sp);
    const bool descend = vis && st == kGoOn;
    if (PC && descend && sp.both) lds_put(col, L.c);
    const bool right = back ? (L.start & L.size) != 0u : sp.near_right;
    take_child(L.c, sp.dp, sp.tc, right);
    if (back) {
        cap_interval(L.c, L.tmax, L.lo, L.hi);
    } else if (descend) {
        descend_state<PC>(L, sp);
    }
    // work counters (counting variant only), branch-free
    if (MODE == kCount) {
        L.splits += descend ? 1 : 0;
        L.backtracks += back ? 1 : 0;
    }
    return st;
}

// Normal at a leaf hit (Appendix C, the final computation of an
// intersection). A hit through the leaf cylinder's side gets the direction
// from the leaf chord's point at the hit's projection to the hit point. A hit
// through a plane (the start of the leaf's interval) whose point lies on the
// curve's start or end cap plane -- within (8 + 2 level) 2^-24 X, the node
// error bound of the leaf's level plus this test's own rounding, X the
// largest ray-frame coordinate of the control points -- gets that cap's
// outward normal: minus the start tangent, the end tangent, with the cap
// planes' fallbacks where a tangent vanishes (the nearer plane when both
// qualify). Other plane entries keep the radial direction. At depth 22 a
// leaf is shorter than FP32 resolves along the ray, so the first leaf can
// look empty and hand its hit to the next one through their common split
// plane: the tolerance keeps such hits on the cap. The vector is formed in
// the ray frame and turned back into world space with the frame of the
// pair's ray (rebuilt in FP64, as for the projection).
template <bool CAND>
__device__ __forceinline__ void leaf_normal(const Args &a, int64_t i, const Lane &L, const HitGeo &hg, float &nx,
                                            float &ny, float &nz)
{
    float vx = hg.vx, vy = hg.vy, vz = hg.vz;
    if (hg.plane) {
        const Node &r = L.root;
        const float cc = dot3(r.d.x, r.d.y, r.d.z, r.d.x, r.d.y, r.d.z);
        // cap normals: p1 - p0, else p2 - p0, else p3 - p0; p3 - p2, else p3 - p1, else p3 - p0
        float ax = r.t0.x, ay = r.t0.y, az = r.t0.z;
        if (negligible(ax, ay, az, cc)) { ax = r.d.x - r.t1.x; ay = r.d.y - r.t1.y; az = r.d.z - r.t1.z; }
        if (negligible(ax, ay, az, cc)) { ax = r.d.x; ay = r.d.y; az = r.d.z; }
        float bx = r.t1.x, by = r.t1.y, bz = r.t1.z;
        if (negligible(bx, by, bz, cc)) { bx = r.d.x - r.t0.x; by = r.d.y - r.t0.y; bz = r.d.z - r.t0.z; }
        if (negligible(bx, by, bz, cc)) { bx = r.d.x; by = r.d.y; bz = r.d.z; }
        const float ex = r.p.x + r.d.x, ey = r.p.y + r.d.y, ez = r.p.z + r.d.z;     // p3
        const float d0 = fabsf(L.t * az - dot3(r.p.x, r.p.y, r.p.z, ax, ay, az)) * rcp(vsqrt(dot3(ax, ay, az, ax, ay, az)));
        const float d1 = fabsf(L.t * bz - dot3(ex, ey, ez, bx, by, bz)) * rcp(vsqrt(dot3(bx, by, bz, bx, by, bz)));
        float X = 0.0f;
        X = fmaxf(X, fmaxf(fabsf(r.p.x), fmaxf(fabsf(r.p.y), fabsf(r.p.z))));
        X = fmaxf(X, fmaxf(fabsf(r.p.x + r.t0.x), fmaxf(fabsf(r.p.y + r.t0.y), fabsf(r.p.z + r.t0.z))));
        X = fmaxf(X, fmaxf(fabsf(ex - r.t1.x), fmaxf(fabsf(ey - r.t1.y), fabsf(ez - r.t1.z))));
        X = fmaxf(X, fmaxf(fabsf(ex), fmaxf(fabsf(ey), fabsf(ez))));
        const float tol = (float)(8 + 2 * L.level) * 0x1p-24f * X;
        const bool near1 = d1 < d0;
        if (fminf(d0, d1) <= tol) {
            vx = near1 ? bx : -ax;
            vy = near1 ? by : -ay;
            vz = near1 ? bz : -az;
        }
    }
    const int64_t ri = a.pair_ray && !CAND ? (int64_t)a.pair_ray[i] : i;
    const float *R = a.rays + ri;
    const int64_t rs = a.ray_stride;
    const double dx = R[3 * rs], dy = R[4 * rs], dz = R[5 * rs];
    const double il = rsqrt64(fma(dx, dx, fma(dy, dy, dz * dz)));
    const double w[3] = {dx * il, dy * il, dz * il};
    double u[3], v[3];
    make_onb(w[0], w[1], w[2], u, v);
    const double wx = fma((double)vx, u[0], fma((double)vy, v[0], (double)vz * w[0]));
    const double wy = fma((double)vx, u[1], fma((double)vy, v[1], (double)vz * w[1]));
    const double wz = fma((double)vx, u[2], fma((double)vy, v[2], (double)vz * w[2]));
    const double in = rsqrt64(fma(wx, wx, fma(wy, wy, wz * wz)));
    nx = (float)(wx * in);
    ny = (float)(wy * in);
    nz = (float)(wz * in);
}

// Candidate lists start as misses (each position then writes the hits).
template <int MODE>
__device__ __forceinline__ void cand_init(const Args &a, int64_t i)
{
    a.t_out[i] = INFINITY;
    a.u_out[i] = __builtin_nanf("");
    a.hit_out[i] = 0;
    a.fiber_out[i] = -1;
    if (MODE == kConservative) {
        a.t64_out[i] = INFINITY;
        a.u64_out[i] = __builtin_nan("");
    }
    if (a.normal_out) {
        a.normal_out[i] = __builtin_nanf("");
        a.normal_out[a.n_pairs + i] = __builtin_nanf("");
        a.normal_out[2 * a.n_pairs + i] = __builtin_nanf("");
    }
}

// Write the result of pair i (Section 3.3: u from projecting the hit point
// onto the leaf chord; hit when t < tmax). A refined pair (depth > 16 under
// FI_FP64_REFINE) reports its FP64 surface hit, decided in FP64.
// `hg` is the leaf geometry of a plain hit; `ref` the FP64 result of a
// refined candidate (used when `reached`). A refined pair that reached a leaf
// is marked for refine_range instead, its FP32 leaf hit in t and u. CAND:
// candidate lists (see Args).
constexpr uint8_t kToRefine = 2;               // hit_out of a pair that refine_range decides
template <int MODE, bool CAND = false>
__device__ __forceinline__ void finish(const Args &a, int64_t i, const Lane &L, bool reached,
                                       HitGeo hg = HitGeo{}, Refined ref = Refined{}, int round = 0)
{
    float t = INFINITY, u = __builtin_nanf("");
    double t64 = INFINITY, u64 = __builtin_nan("");
    bool hit = false;
    if (MODE == kConservative && !CAND && L.slack >= 0.0f && reached) {
        a.t_out[i] = L.t;
        a.u_out[i] = L.u;
        a.hit_out[i] = kToRefine;
        return;
    }
    if (MODE == kConservative && L.slack >= 0.0f) {
        if (CAND && reached) {
            t64 = ref.t;
            u64 = ref.u;
            t = (float)t64;
            u = (float)u64;
            hit = true;
        }
    } else if (reached && L.t < L.tmax) {
        t = L.t;
        u = L.u;
        t64 = t;
        u64 = u;
        hit = true;
    }
    if constexpr (CAND) {
        // candidate lists: a miss leaves the ray's nearest hit so far; a
        // hit (nearer by construction: tmax was shortened to it) replaces it
        if (!hit) return;
        a.fiber_out[i] = a.cand_fiber[a.cand_off[i] + a.cand_first + round];
    }
    a.t_out[i] = t;
    a.u_out[i] = u;
    a.hit_out[i] = hit ? 1 : 0;
    if (MODE == kConservative) {
        a.t64_out[i] = t64;
        a.u64_out[i] = u64;
    }
    if (MODE != kCount && a.normal_out) {
        float nx = __builtin_nanf(""), ny = nx, nz = nx;
        if (MODE == kConservative && L.slack >= 0.0f) {
            if (hit) { nx = ref.nx; ny = ref.ny; nz = ref.nz; }
        } else if (hit) {
            leaf_normal<CAND>(a, i, L, hg, nx, ny, nz);
        }
        a.normal_out[i] = nx;
        a.normal_out[a.n_pairs + i] = ny;
        a.normal_out[2 * a.n_pairs + i] = nz;
    }
    if (MODE == kCount) {
        int32_t *cn = a.counts + 4 * i;
        cn[0] = L.trips;
        cn[1] = L.splits;
        cn[2] = L.backtracks;
        cn[3] = hit ? L.level : -1;
    }
}

template <int MODE>
__device__ __forceinline__ void finish_invalid(const Args &a, int64_t i)
{
    a.t_out[i] = INFINITY;
    a.u_out[i] = __builtin_nanf("");
    a.hit_out[i] = 0;
    if (MODE == kConservative) {
        a.t64_out[i] = INFINITY;
        a.u64_out[i] = __builtin_nan("");
    }
    if (MODE != kCount && a.normal_out) {
        a.normal_out[i] = __builtin_nanf("");
        a.normal_out[a.n_pairs + i] = __builtin_nanf("");
        a.normal_out[2 * a.n_pairs + i] = __builtin_nanf("");
    }
    if (MODE == kCount) {
        int32_t *cn = a.counts + 4 * i;
        cn[0] = 0; cn[1] = 0; cn[2] = 0; cn[3] = -1;
    }
}

__device__ __forceinline__ uint32_t lanes_below(uint64_t mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Scene of global pair g: offsets[s] <= g < offsets[s + 1] (empty scenes skipped).
__device__ __forceinline__ int find_scene(const int64_t *offsets, int n_scenes, int64_t g)
{
    int lo = 0, hi = n_scenes;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (offsets[mid] <= g) lo = mid;
        else hi = mid;
    }
    return lo;
}

// N rows of a table at one column, row pointer by row pointer. With the row
// offsets k * stride computed ahead, in 40 scalar registers, other arguments
// were read again in every setup round; this and fiber records read 16 bytes
// at a time (instead of 4, at one cache line per lane each): 2^24 hair pairs
// 1910 -> 1862 us, 2^18 candidate lists 778 -> 675, 256 scenes 1468 -> 1360.
template <int N>
__device__ __forceinline__ void load_rows(const float *p, int64_t stride, float (&x)[N])
{
#pragma unroll
    for (int k = 0; k < N; ++k) {
        x[k] = *p;
        if (k + 1 < N) {
            p += stride;
            asm("" : "+v"(p));
        }
    }
}

// Load pair i and move it into the ray frame: the root node in the
// {p, d, t0, t1} form (Section 3.1), written to q[k * kQueue] (k = 0..15: p,
// d, t0, t1, each x, y, z, w) as each part is computed, so that the FP64
// frame and the finished root never take registers at the same time. False
// when the pair is a definite miss (bad index, depth, direction, tmax or a
// non-finite root).
// The projection runs once per pair in FP64 (full rate on this chip): the
// differences of the float32 control points and of the origin are exact in
// double, so p is the rounded frame position of p0 and d, t0, t1 are the
// rounded frame images of p3-p0, p1-p0, p3-p2 -- each component accurate to
// its own float32 ulp, including the tiny across-ray or along-ray parts of
// nearly parallel or nearly perpendicular tangents.
// `aos`, when given, holds the fibers as 16 consecutive floats each (see
// k_fibers_aos): a gathered fiber is then one or two cache lines instead of
// one line per coordinate row.
// In candidate mode (cand_off given) pair i is ray i against its candidate
// number cand_first + round; a ray without that candidate, or with an invalid one,
// is a definite miss too (its callers then leave the ray's nearest hit so far
// as it is), and tmax is the ray's tmax shortened to that hit.
// QUAD: the fiber table holds quadratics (12 rows: p0, p1, p2), loaded as
// their exact cubic elevation (t0 = 2/3 (p1 - p0), t1 = 2/3 (p2 - p1)).
template <bool CAND, bool QUAD = false>
__device__ __forceinline__ bool load_pair(const Args &a, int64_t i, float *q, float &tmax, uint32_t &depth,
                                          const float *aos, int round = 0)
{
    int64_t ri, fi;
    if constexpr (CAND) {
        const int64_t o = a.cand_off[i] + a.cand_first + round;
        if (o >= a.cand_off[i + 1] || o < 0 || o >= a.n_cand) return false;
        ri = i;
        fi = a.cand_fiber[o];
        depth = a.pair_depth ? (uint32_t)a.pair_depth[o] : (uint32_t)a.depth;
    } else {
        ri = a.pair_ray ? (int64_t)a.pair_ray[i] : i;
        fi = a.pair_fiber ? (int64_t)a.pair_fiber[i] : i;
        depth = a.pair_depth ? (uint32_t)a.pair_depth[i] : (uint32_t)a.depth;
    }
    if (ri < 0 || ri >= a.n_rays || fi < 0 || fi >= a.n_fibers || depth > FI_MAX_DEPTH) return false;
    float R[7], F[QUAD ? 12 : 16];
    load_rows(a.rays + ri, a.ray_stride, R);
    if (aos) {
        const float4 *f = (const float4 *)aos + 4 * fi;
#pragma unroll
        for (int k = 0; k < (QUAD ? 3 : 4); ++k) {
            const float4 x = f[k];
            F[4 * k] = x.x;
            F[4 * k + 1] = x.y;
            F[4 * k + 2] = x.z;
            F[4 * k + 3] = x.w;
        }
    } else {
        load_rows(a.fibers + fi, a.fiber_stride, F);
    }
    tmax = R[6];
    if (!(tmax == tmax)) return false;
    if constexpr (CAND) {
        if (a.t64_out) {
            // refined candidates: the FP64 nearest hit so far, rounded up
            // (the FP32 search prunes conservatively; FP64 decides)
            const double b = a.t64_out[i];
            float f = (float)b;
            if ((double)f < b) f = __uint_as_float(__float_as_uint(f) + 1u);     // b >= 0: one ulp up
            tmax = fminf(tmax, f);
        } else {
            tmax = fminf(tmax, a.t_out[i]);
        }
    }
    const double dx = R[3], dy = R[4], dz = R[5];
    const double n2 = fma(dx, dx, fma(dy, dy, dz * dz));
    if (!(n2 > 0.0) || !(n2 < INFINITY)) return false;
    const double il = rsqrt64(n2);
    const double w[3] = {dx * il, dy * il, dz * il};
    double u[3], v[3];
    make_onb(w[0], w[1], w[2], u, v);
    bool finite = true;
    auto proj = [&](double ex, double ey, double ez, double ew, int k, bool check) {
        const float x = (float)fma(ex, u[0], fma(ey, u[1], ez * u[2]));
        const float y = (float)fma(ex, v[0], fma(ey, v[1], ez * v[2]));
        const float z = (float)fma(ex, w[0], fma(ey, w[1], ez * w[2]));
        if (check) finite = finite && isfinite(x) && isfinite(y) && isfinite(z);
        q[(4 * k) * kQueue] = x;
        q[(4 * k + 1) * kQueue] = y;
        q[(4 * k + 2) * kQueue] = z;
        q[(4 * k + 3) * kQueue] = (float)ew;
    };
    const float p0x = F[0], p0y = F[1], p0z = F[2], p0w = F[3];
    proj((double)p0x - (double)R[0], (double)p0y - (double)R[1], (double)p0z - (double)R[2], (double)p0w, 0,
         true);
    if constexpr (QUAD) {
        const float p2x = F[8], p2y = F[9], p2z = F[10], p2w = F[11];
        const float p1x = F[4], p1y = F[5], p1z = F[6], p1w = F[7];
        constexpr double k23 = 2.0 / 3.0;
        proj((double)p2x - p0x, (double)p2y - p0y, (double)p2z - p0z, (double)p2w - p0w, 1, true);
        proj(((double)p1x - p0x) * k23, ((double)p1y - p0y) * k23, ((double)p1z - p0z) * k23,
             ((double)p1w - p0w) * k23, 2, false);
        proj(((double)p2x - p1x) * k23, ((double)p2y - p1y) * k23, ((double)p2z - p1z) * k23,
             ((double)p2w - p1w) * k23, 3, false);
        return finite;
    }
    const float p3x = F[12], p3y = F[13], p3z = F[14], p3w = F[15];
    proj((double)p3x - p0x, (double)p3y - p0y, (double)p3z - p0z, (double)p3w - p0w, 1, true);
    proj((double)F[4] - p0x, (double)F[5] - p0y, (double)F[6] - p0z, (double)F[7] - p0w, 2,
         false);
    proj((double)p3x - F[8], (double)p3y - F[9], (double)p3z - F[10], (double)p3w - F[11], 3,
         false);
    return finite;
}

// The kernel of every call: each persistent 64-lane wave takes an even share
// of the call's pairs (of the whole scene table for a batch), contiguous so
// that its loads are coalesced. Pairs reach the lanes through a queue of
// prepared roots in LDS:
//  * a setup round, run by the whole wave when the queue cannot serve its
//    free lanes, loads up to 64 pairs (one per lane), moves them into the
//    ray frame in FP64 and tests their roots; pairs decided there (a miss, a
//    root that is the leaf, a bad pair) are written out at once, the others
//    are appended to the queue (root node, its cap interval, tmax, pair);
//  * at every trip, each free lane takes the next queued root (copying it to
//    its root slot for the backtracks that miss the parent cache), and its
//    first trip tests the root and takes the first split.
// Setup rounds thus run with every lane busy and pay their load latency
// once per up to 64 pairs, while a lane that finishes a pair waits no more
// than one trip for the next (a round of loads, the FP64 frame and the root
// test costs about three trips' time). The attribute sets the register
// budget; the LDS (queue and parent cache, 9.5 KiB) allows 16 waves per CU.

// A scene descriptor's fields that pair loading and finishing read, as
// wave-uniform values.
template <class T>
__device__ __forceinline__ T *uniform_ptr(T *p)
{
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (T *)(((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ int64_t uniform_i64(int64_t x)
{
    return (int64_t)(((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)x >> 32)) << 32) |
                     __builtin_amdgcn_readfirstlane((uint32_t)x));
}

__device__ __forceinline__ void uniform_scene(const Args &s, Args &o)
{
    o.rays = uniform_ptr(s.rays);
    o.ray_stride = uniform_i64(s.ray_stride);
    o.n_rays = uniform_i64(s.n_rays);
    o.fibers = uniform_ptr(s.fibers);
    o.fiber_stride = uniform_i64(s.fiber_stride);
    o.n_fibers = uniform_i64(s.n_fibers);
    o.pair_ray = uniform_ptr(s.pair_ray);
    o.pair_fiber = uniform_ptr(s.pair_fiber);
    o.pair_depth = uniform_ptr(s.pair_depth);
    o.depth = __builtin_amdgcn_readfirstlane(s.depth);
    o.t_out = uniform_ptr(s.t_out);
    o.u_out = uniform_ptr(s.u_out);
    o.hit_out = uniform_ptr(s.hit_out);
    o.counts = uniform_ptr(s.counts);
    o.t64_out = uniform_ptr(s.t64_out);
    o.u64_out = uniform_ptr(s.u64_out);
    o.normal_out = uniform_ptr(s.normal_out);
    o.n_pairs = uniform_i64(s.n_pairs);
}

// The wave's contiguous range of the call's pairs (an even share).
__device__ __forceinline__ void wave_range(int64_t w, int64_t waves, int64_t count, int64_t &begin, int64_t &end)
{
    const int64_t share = (count + waves - 1) / waves;
    begin = w * share < count ? w * share : count;
    end = (w + 1) * share < count ? (w + 1) * share : count;
}

// The FP64 decisions of a wave's pairs begin .. end - 1 that reached a leaf
// (hit_out == kToRefine), once its traversal is done. The wave lists those
// marked, up to kList pairs at a time, decides each with a lane of its own as
// far as narrow_curve and simple_candidates go, lists what they leave open (over
// the part of the list that has been read) and searches that, so that both
// passes run with full waves and no lane waits, parked, for the last of its
// wave. Bound by FP64 arithmetic and, beside it, by the longest pairs of the
// traversal, which the other waves' decisions hide: a
// kernel of its own for the decisions was as fast on hair (409 against 399 us
// per 10^6 pairs) but waited for them (500,009 degenerate pairs 1.57 against
// 1.14 ms). Before, with the lanes parked at their leaves and every pair
// running 65 samples and two long bracketed searches: 1.14 and 1.41 ms.
constexpr int kList = 16 * kWave;              // pairs listed at a time

template <bool BATCHED, bool QUAD>
__device__ __forceinline__ void refine_range(const Args &a0, const Args *scenes, const int64_t *offsets, int n_scenes,
                                             int64_t begin, int64_t end, const float *aos, int *list)
{
    const int lane = (int)threadIdx.x;
    // batched: the scenes of the share, among which a pair's is searched by
    // halves (2^20 hair pairs in 2^20 scenes: 626 us, one after another 927; in
    // one scene 362)
    int scene0 = 0, scenes_here = 1;
    if constexpr (BATCHED) {
        scene0 = find_scene(offsets, n_scenes, begin);
        scenes_here = find_scene(offsets + scene0, n_scenes - scene0, end - 1) + 1;
    }
    for (int64_t first = begin; first < end; first += kList) {
        const int size = end - first < kList ? (int)(end - first) : kList;
        // pair k of this part: its index in its scene, and the scene
        auto place = [&](int k, int &sc) {
            int64_t i = first + k;
            if constexpr (BATCHED) {
                sc = scene0 + find_scene(offsets + scene0, scenes_here, i);
                i -= offsets[sc];
            }
            return i;
        };
        int n = 0, n_open = 0;
        for (int k0 = 0; k0 < size; k0 += kWave) {
            bool marked = false;
            if (k0 + lane < size) {
                int sc = 0;
                const int64_t i = place(k0 + lane, sc);
                marked = (BATCHED ? scenes[sc].hit_out : a0.hit_out)[i] == kToRefine;
            }
            const uint64_t m = __ballot(marked);
            if (marked) list[n + (int)lanes_below(m)] = k0 + lane;
            n += __popcll(m);
        }
        __syncthreads();
        for (int pass = 0; pass < 2; ++pass) {
            const int todo = pass ? n_open : n;
            for (int e0 = 0; e0 < todo; e0 += kWave) {
                bool left = false;
                int k = 0;
                if (e0 + lane < todo) {
                    k = list[e0 + lane];
                    int sc = 0;
                    const int64_t i = place(k, sc);
                    const Args &a = BATCHED ? scenes[sc] : a0;
                    const int64_t ri = a.pair_ray ? (int64_t)a.pair_ray[i] : i;
                    const int64_t fi = a.pair_fiber ? (int64_t)a.pair_fiber[i] : i;
                    Curve64 cv;
                    double frame[9];
                    double t = INFINITY, u = __builtin_nan("");
                    // (a marked pair has a finite, non-zero direction)
                    curve_in_ray_frame(a.rays + ri, a.ray_stride, aos ? aos + 16 * fi : a.fibers + fi,
                                       aos ? 1 : a.fiber_stride, cv, frame, QUAD);
                    const double tmax = a.rays[6 * a.ray_stride + ri];
                    Part part;
                    if (narrow_curve(cv, part)) {
                        if (pass) curve_candidates(cv, part, tmax, (double)a.t_out[i], (double)a.u_out[i], t, u);
                        else left = !simple_candidates(cv, part, tmax, t, u);
                    }
                    if (!left) {
                        const Refined r = refined_at(cv, frame, t, u, a.normal_out != nullptr);
                        a.t_out[i] = (float)r.t;
                        a.u_out[i] = (float)r.u;
                        a.hit_out[i] = r.hit ? 1 : 0;
                        a.t64_out[i] = r.t;
                        a.u64_out[i] = r.u;
                        if (a.normal_out) {
                            a.normal_out[i] = r.nx;
                            a.normal_out[a.n_pairs + i] = r.ny;
                            a.normal_out[2 * a.n_pairs + i] = r.nz;
                        }
                    }
                }
                const uint64_t m = __ballot(left);
                if (left) list[n_open + (int)lanes_below(m)] = k;
                n_open += __popcll(m);
            }
            __syncthreads();
        }
    }
}

// Shared searches. Once a wave has no more pairs to start, its free lanes take
// pending siblings off its busy lanes: a lane hands over the shallowest one
// (which it would visit last), and the helper rebuilds that node as a backtrack
// would. The nodes of a pair are then visited at the same time instead of one
// after another, with the same arithmetic; the result is that of the first leaf
// in the order of the search. `order` is a lane's place in it: a helper's is
// its donor's and the bit of the level handed over, since it comes after all
// that is left of its donor and before the donor's earlier helpers (what a lane
// hands over lies ever deeper). `group` labels the pair (the lane that had it
// first), and `stop` is the first leaf's place so far. A leaf before it writes
// its result over the later one's, and the lanes behind it end; every pair
// starts as a miss, so that a lane that misses just ends.
// What bounds the end of a call is its longest pair: a trip of a wave alone on
// its SIMD takes 0.7 to 1 us, and a few pairs in a million need a hundred and
// more (degenerate ones up to 850). A trip with a rebuild takes two to three
// times as long, and most searches end within a hundred trips: a wave starts to
// share once it has run 96 since its last pair, at every second trip. Mean of 6
// inputs of mixed pairs at depth 22, not shared, from 32 trips on, from 96 on:
// 13,039 pairs 61.1, 74.3, 61.3 us; 40,000 72.2, 88.1, 72.6; 299,993 110, 126,
// 110; 524,289 238, 171, 201; 2^20 266, 227, 238; 299,993 quadratic pairs 178,
// 138, 163; 60,000 refined degenerate pairs 695, 344, 377. An input whose longest
// search ends soon after sharing starts loses by it: of 16 inputs of 299,993
// pairs the times against not sharing are 0.56 to 1.24 (five above 1.05), of 2^20
// 0.33 to 1.09, of 40,000 1.00 to 1.15 (one above 1.03); from 32 trips on 40,000
// pairs took 1.20 times as long on the whole: 5 % for the start, next to nothing
// for one hand-over, the rest for one at every second trip. Hand-overs 8, 16 or
// 32 trips apart from 32, 48 or 64 on and at every second trip from 96 or 128 on
// gained nothing against 96 (51 calls, 6 inputs, against not sharing at all:
// 0.964 of the time with 96, 0.964 to 0.993 with those), nor did waiting longer
// after helpers that ended at once (all calls 1 to 3 % slower).
// The count of a call's pairs says nothing about its longest search: rules by
// it (48 trips up to 2^16 pairs, 64 above 2^19) made 13,039 and 40,000 pairs 17 %
// slower than not sharing. Nor do a wave's busy lanes: they are few by then (a
// limit of 2, 4 or 8 changed nothing). The trips are those of the loop for pairs
// of their own: a second loop behind it cost every call 1 to 2 %.
#ifndef FIBERHIT_LONG_SEARCH
#define FIBERHIT_LONG_SEARCH 96                // build knob: trips without a new pair after which searches are shared
#endif
constexpr int kLongSearch = FIBERHIT_LONG_SEARCH;

// A search of more than kMaxTrips trips is a miss, shared or not. The trips of a
// group's lanes (`total`, added up as they end; those behind a leaf left out)
// are at least what the search takes alone up to its leaf: a hit with no more
// than the limit stands. With more it may or may not, and the wave runs its
// share a second time, sharing nothing. (Counted by each lane for itself, the
// limit let shared searches find leaves behind it: fibers so small that FP32
// products underflow, arcs of an extent of 1e-6, need so many trips.) Until a wave
// has spent kSharedTrips on shared searches no pair of it can have taken too
// many, and nothing is looked at: calls take the same time as without the look
// (a lane that starts its pair again by itself cost them 2 %, marked pairs
// picked out of the share 1 %). The longest searches of 1.7 M degenerate pairs
// (44,133 trips; 79.4 ms not shared) take 3.6 ms.
constexpr int kSharedTrips = kMaxTrips / 2;
constexpr uint32_t kMostShared = 16 * kMaxTrips;   // trips of a group's lanes after which it is given up

struct Shared {                                // in LDS, where the queue was
    uint32_t order[kWave], group[kWave], stop[kWave], donor[kWave], total[kWave];
    float root[16 * kWave];                    // the groups' roots, in columns
};

__device__ __forceinline__ void start_sharing(const Lane &L, Shared &sh)
{
    const uint32_t lane = threadIdx.x;
    sh.order[lane] = 0;
    sh.group[lane] = lane;
    sh.stop[lane] = 0xffffffffu;
    sh.total[lane] = 0;
    lds_put(sh.root + lane, L.root);
    __syncthreads();
}

// Free lanes take pending siblings, one per donor. A sibling close to the
// leaves is not worth the rebuild.
__device__ __forceinline__ void share_work(Lane &L, bool &active, Shared &sh)
{
    const uint32_t top = L.bits ? 0x80000000u >> __builtin_clz(L.bits) : 0u;
    const bool donor = active && top > 4u * L.min_size;
    const uint64_t dm = __ballot(donor), fm = __ballot(!active);
    if (dm == 0 || fm == 0) return;
    const int lane = (int)threadIdx.x;
    const int rd = (int)lanes_below(dm), rf = (int)lanes_below(fm);
    const int k = min(__popcll(dm), __popcll(fm));
    if (donor && rd < k) sh.donor[rd] = (uint32_t)lane;
    __syncthreads();
    const bool taker = !active && rf < k;
    const int from = taker ? (int)sh.donor[rf] : lane;
    const uint32_t bits = __shfl(top, from), start = __shfl(L.start, from), min_size = __shfl(L.min_size, from);
    const int pair = __shfl(L.pair, from), scene = __shfl(L.scene, from);
    const float tmax = __shfl(L.tmax, from), slack = __shfl(L.slack, from);
    if (donor && rd < k) L.bits ^= top;
    if (taker) {
        L.bits = bits;
        L.start = start;
        L.min_size = min_size;
        L.pair = pair;
        L.scene = scene;
        L.tmax = tmax;
        L.slack = slack;
        L.size = kRootSize;
        L.cached = 0;
        L.waiting = 0;
        L.trips = 0;
        sh.order[lane] = sh.order[from] | bits;
        const uint32_t group = sh.group[from];
        sh.group[lane] = group;
        lds_get(sh.root + group, L.root);
        active = true;                         // its interval is empty: the next trip backtracks to the sibling
    }
    __syncthreads();
}

// End of a trip of shared searches: does this lane, at a leaf, come before all
// leaves reached so far? The lanes behind a leaf end.
__device__ __forceinline__ bool first_leaf(bool &active, bool leaf, Shared &sh)
{
    if (__ballot(leaf) == 0) return false;
    const int lane = (int)threadIdx.x;
    const uint32_t order = sh.order[lane];
    uint32_t *stop = &sh.stop[sh.group[lane]];
    if (leaf) __hip_atomic_fetch_min(stop, order, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __syncthreads();
    const uint32_t first = *stop;
    __syncthreads();
    if (order > first) active = false;
    return leaf && order == first;
}

// Once a wave has spent kSharedTrips on shared searches: may this lane's search
// have met the trip limit before its leaf? `done`: it has ended in this trip. A
// group ends with such a lane, or is given up and its lanes end.
__device__ __forceinline__ bool unsure_search(bool &active, bool done, Shared &sh)
{
    const int lane = (int)threadIdx.x;
    sh.donor[lane] = 0;
    __syncthreads();
    const uint32_t group = sh.group[lane], total = sh.total[group];
    const bool cut = active && total > kMostShared;
    if (active && !done && !cut) sh.donor[group] = 1;         // the group goes on
    __syncthreads();
    const bool over = done && sh.stop[group] != 0xffffffffu && total > (uint32_t)kMaxTrips && sh.donor[group] == 0;
    __syncthreads();
    if (cut) active = false;
    return cut || over;
}

// Candidate lists. A ray's candidates are tested one after another, each against
// the ray shortened to its nearest hit so far; a wave keeps its rays from the
// first candidate to the last. A ray whose search has ended waits, if its list
// goes on, in a ring in LDS until a setup round prepares its next candidate
// beside others (and beside the first ones of new rays). Up to 128 rays of a
// wave are under way (64 searched, 64 in the queue), so that the ring has room
// for all of them. Bound by the same trips as single calls, and by the longest
// list of a small call. A setup round waits for 8 rays, or for the wave's last
// search (16: 304 instead of 285 us for 2^18 hair lists, 126 instead of 131 for
// 65,537 mixed ones; 32: 319 and 176).
// One launch for each position of the lists, with the lanes that were done idle
// until the longest search of the position had ended, took 642 and 429 us, and
// 1333 instead of 242 for 65,536 refined lists.
#ifndef FIBERHIT_READY
#define FIBERHIT_READY 8                      // build knob: rays a setup round waits for
#endif
constexpr int kReady = FIBERHIT_READY;
#ifndef FIBERHIT_MAX_ROUNDS
#define FIBERHIT_MAX_ROUNDS (1 << 24)         // build knob: candidates of a list a launch tests
#endif
constexpr int32_t kMaxRounds = FIBERHIT_MAX_ROUNDS;
static_assert(kMaxRounds <= 1 << 24, "a queue entry holds twice a candidate's number above 6 other bits");

struct Waiting {                               // a ring
    int ray[2 * kWave], round[2 * kWave];
};

__device__ __forceinline__ int wslot(int k) { return k & (2 * kWave - 1); }

#ifndef FIBERHIT_WAVES
#define FIBERHIT_WAVES 4                      // build knob: register budget (waves per SIMD)
#endif
template <int MODE, bool BATCHED, bool CAND = false, bool QUAD = false, bool PC = kParentCache>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(MODE == kConservative ? 4 : FIBERHIT_WAVES, 8)))
void k_fused(Args a0, const Args *scenes, const int64_t *offsets, int n_scenes, int64_t count, int refill,
             const float *aos)
{
    __shared__ float s_cache[16 * kWave];
    __shared__ float s_queue[kQWords * kQueue];
    static_assert(sizeof(Shared) <= sizeof(s_queue) && kQWords * kQueue >= kList,
                  "shared searches and refine_range's list take the queue's place");
    const int lane = (int)threadIdx.x;
    float *col = s_cache + lane;
    const int64_t w = blockIdx.x, waves = gridDim.x;
    __shared__ int s_waiting[CAND ? 4 * kWave : 1];
    static_assert(!CAND || sizeof(Waiting) == sizeof(s_waiting), "rays between two candidates");
    Waiting &waiting = *(Waiting *)s_waiting;
    int64_t next, end;                                                  // wave-uniform range
    wave_range(w, waves, count, next, end);
    // what of it is not prepared yet: 32 bits, so that the test of every trip
    // takes scalar instructions (64-bit ones compare in vector registers; 2^24
    // hair pairs 1888 -> 1848 us)
    int left = end > next ? (int)(end - next) : 0;
    const RegRoot root{};
    // batched: pairs are numbered across the scene table; the wave's share
    // is contiguous, so the scene of its next pair only moves forward
    int scene0 = 0;                      // scene of the wave's next pair (wave-uniform)
    Args cur = a0;                       // batched: scene0's descriptor, read once per change
    int64_t base0 = 0, bound0 = count;   // batched: scene0's first pair, and the next scene's
    if constexpr (BATCHED) {
        scene0 = __builtin_amdgcn_readfirstlane(next < count ? find_scene(offsets, n_scenes, next) : 0);
        uniform_scene(scenes[scene0], cur);
        base0 = uniform_i64(offsets[scene0]);
        bound0 = uniform_i64(offsets[scene0 + 1]);
    }
    const int rounds = CAND ? n_scenes : 0;                             // candidates tested of a list
    int w_head = 0, w_count = 0;         // the rays that wait for their next candidate
    int q_head = 0, q_count = 0;         // the queue: entries q_head .. q_head + q_count - 1 (mod kQueue)
    Lane L = {};
    L.lo = INFINITY;                                                   // an empty interval: no work
    L.hi = -INFINITY;
    bool active = false;
    // counted searches stay as they are, and so do candidate lists (a list's
    // hit counts if it is nearer than the one before)
    constexpr bool kShared = MODE != kCount && !CAND;
    Shared &sh = *(Shared *)s_queue;
    int tail = 0;                        // trips since the wave's last pair was started
    int spent = 0;                       // trips of its lanes while they share searches,
    uint64_t unsure = 0;                 //   and whether one may have met the trip limit
    constexpr int kNeverShare = -(1 << 30);                            // what `tail` becomes then
    for (;;) {
        const uint64_t free_mask = __ballot(!active);
        const int n_free = __popcll(free_mask);
        int take = 0, from = 0, round = 0;
        bool setup = false;
        if constexpr (CAND) {
            if ((left | q_count | w_count) == 0 && n_free == kWave) break;
            // new rays as far as the ring has room for all that are under way
            const int room = 2 * kWave - w_count - q_count - (kWave - n_free);
            const int n_ready = w_count + (left < room ? left : room);
            setup = n_ready >= kReady ? q_count < n_free : n_ready > 0 && q_count == 0 && n_free == kWave;
            from = w_count < kQueue - q_count ? w_count : kQueue - q_count;
            take = kQueue - q_count - from;
            take = take < room ? take : room;
            take = take < left ? take : left;
        } else {
            if ((left | q_count) == 0) {
                if (n_free == kWave) break;
                if (kShared && ++tail >= kLongSearch) {
                    if (tail == kLongSearch) {
                        start_sharing(L, sh);
                        if (active) {
                            if constexpr (BATCHED) finish<MODE>(scenes[L.scene], L.pair, L, false);
                            else finish<MODE>(a0, L.pair, L, false);
                        }
                        // a search near the limit already
                        if (__ballot(active && L.trips > kMaxTrips - kSharedTrips) != 0) spent = kSharedTrips;
                    }
                    if (((tail - kLongSearch) & 1) == 0) share_work(L, active, sh);
                }
            }
        }
        if (CAND ? setup : left != 0 && q_count < n_free) {
            // setup round: lane k prepares pair next + k, or (candidate lists)
            // the next candidate of a ray that waits or the first of a new one
            bool prepares = false, more = false;
            int64_t idx = next + lane;
            if constexpr (CAND) {
                __threadfence_block();             // the hits of other lanes (t_out)
                prepares = lane < from + take;
                idx = 0;
                if (prepares) {
                    if (lane < from) {
                        idx = waiting.ray[wslot(w_head + lane)];
                        round = waiting.round[wslot(w_head + lane)];
                    } else {
                        idx = next + (lane - from);
                        if (a0.cand_first == 0) cand_init<MODE>(a0, idx);
                    }
                    const int64_t len = a0.cand_off[idx + 1] - a0.cand_off[idx] - a0.cand_first;
                    prepares = round < rounds && round < len;
                    more = round + 1 < rounds && round + 1 < len;
                }
                w_head = wslot(w_head + from);
                w_count -= from;
            } else {
                take = left < kQueue - q_count ? left : kQueue - q_count;
            }
            bool queued = false;
            Node r = {};
            float rlo = 0.0f, rhi = 0.0f, rtmax = 0.0f;
            uint32_t depth = 0;
            int sc = CAND ? 2 * round + (more ? 1 : 0) : scene0;
            // each preparing lane stages its root in the queue entry after the
            // current tail plus its lane number; survivors then move to
            // consecutive entries (every lane has read its own entry back
            // before any lane writes)
            float *stage = s_queue + qslot(q_head + q_count + lane);
            if (CAND ? prepares : lane < take) {
                Args a = a0;
                if constexpr (BATCHED) {
                    if (idx < bound0) {
                        idx -= base0;
                        a = cur;
                    } else {
                        while (sc + 1 < n_scenes && offsets[sc + 1] <= idx) ++sc;
                        idx -= offsets[sc];
                        a = scenes[sc];
                    }
                }
                const bool ok = load_pair<CAND, QUAD>(a, idx, stage, rtmax, depth, aos, round);
                asm volatile("" ::: "memory");
                float *f = &r.p.x;
#pragma unroll
                for (int k = 0; k < 16; ++k) f[k] = stage[k * kQueue];
                // batched: the descriptor of the outputs is read again; held
                // across the load of the pair it cost 3 spilled registers (128
                // against 124 now; batches of 8 to 256 scenes 0 to 1.5 % faster)
                const Args &o = BATCHED ? scenes[sc] : a0;
                if (!ok) {
                    if (!CAND) finish_invalid<MODE>(o, idx);
                } else {
                    cap_interval(r, rtmax, rlo, rhi);
                    float te, tx, lu, hu;
                    const float slack = MODE == kConservative && depth > kRefineAbove ? root_slack(r) : -1.0f;
                    const bool vis = node_visible<MODE, QUAD>(r, rlo, rhi, slack, te, tx, lu, hu);
                    if (vis && depth > 0) {
                        queued = true;
                    } else {
                        // decided at the root: a miss, or the root is the leaf
                        Lane D = {};
                        D.c = r;
                        D.root = r;
                        D.tmax = rtmax;
                        D.t = fmaxf(te, lu);

                        D.start = 0;
                        D.size = kRootSize;
                        D.u = leaf_u(D);
                        D.level = 0;
                        D.trips = 1;
                        D.slack = slack;
                        finish<MODE, CAND>(o, idx, D, vis, hit_geo(r, D.t, te < lu), Refined{}, round);
                    }
                }
            }
            asm volatile("" ::: "memory");
            const uint64_t qm = __ballot(queued);
            if (queued) {
                const int e = qslot(q_head + q_count + (int)lanes_below(qm));
                float *q = s_queue + e;
                if (q != stage) {
                    const float *f = &r.p.x;
#pragma unroll
                    for (int k = 0; k < 16; ++k) q[k * kQueue] = f[k];
                }
                q[16 * kQueue] = rlo;
                q[17 * kQueue] = rhi;
                q[18 * kQueue] = rtmax;
                q[19 * kQueue] = __int_as_float((int)idx);
                q[20 * kQueue] = __int_as_float((sc << 6) | (stall_possible(r) ? 32 : 0) | (int)depth);
            }
            q_count += __popcll(qm);
            next += take;
            left -= take;
            if constexpr (CAND) {
                const bool again = prepares && !queued && more;
                const uint64_t am = __ballot(again);
                if (again) {
                    const int e = wslot(w_head + w_count + (int)lanes_below(am));
                    waiting.ray[e] = (int)idx;
                    waiting.round[e] = round + 1;
                }
                w_count += __popcll(am);
            }
            if constexpr (BATCHED) {
                if (next < count && next >= bound0) {
                    while (scene0 + 1 < n_scenes && offsets[scene0 + 1] <= next) ++scene0;
                    scene0 = __builtin_amdgcn_readfirstlane(scene0);
                    uniform_scene(scenes[scene0], cur);
                    base0 = uniform_i64(offsets[scene0]);
                    bound0 = uniform_i64(offsets[scene0 + 1]);
                }
            }
        }
        if (q_count > 0 && n_free >= (refill < q_count ? refill : q_count)) {
            // free lanes take the next queued roots
            const int k = n_free < q_count ? n_free : q_count;
            if (!active) {
                const int rank = (int)lanes_below(free_mask);
                if (rank < k) {
                    const float *q = s_queue + qslot(q_head + rank);
                    float *f = &L.c.p.x;
#pragma unroll
                    for (int j = 0; j < 16; ++j) f[j] = q[j * kQueue];
                    L.lo = q[16 * kQueue];
                    L.hi = q[17 * kQueue];
                    L.tmax = q[18 * kQueue];
                    L.pair = __float_as_int(q[19 * kQueue]);
                    const int ds = __float_as_int(q[20 * kQueue]);
                    const uint32_t depth = (uint32_t)ds & 31u;
                    L.scene = ds >> 6;
                    L.root = L.c;
                    L.min_size = kRootSize >> depth;
                    L.slack = MODE == kConservative && depth > kRefineAbove ? root_slack(L.c) : -1.0f;
                    L.start = (ds & 32) ? kStallBit : 0u;
                    L.size = kRootSize;
                    L.bits = 0;
                    L.cached = 0;
                    L.waiting = 0;
                    L.trips = 0;
                    L.splits = L.backtracks = 0;
                    active = true;
                }
            }
            q_head = qslot(q_head + k);
            q_count -= k;
        }
        // No edge back to the setup that bypasses the trip: a wave whose
        // fresh pairs were all decided at the root runs one idle trip instead.
        // With a single path around the loop the lane state keeps one set of
        // registers; a bypass edge had made the compiler copy the node and
        // the traversal state at every trip (about 45 moves, measured 12-14 %
        // of the call).
        HitGeo hg;
        const int st = trip<MODE, QUAD, PC, CAND>(L, root, col, hg);
        const bool done = active && st != kGoOn && !(MODE == kConservative && L.waiting);
        bool decides = done;
        // (out of the common path: without the hints calls took 1 % longer)
        if (kShared && __builtin_expect(tail >= kLongSearch, 0)) {
            decides = first_leaf(active, done && st == kHit, sh);
            if (done && (active || decides))
                __hip_atomic_fetch_add(&sh.total[sh.group[lane]], (uint32_t)L.trips, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
            spent += kWave - n_free;
            if (__builtin_expect(spent > kSharedTrips - kWave, 0)) {
                unsure |= __ballot(unsure_search(active, done, sh));
                if (unsure != 0 && __ballot(active && !done) == 0) {
                    // the wave's share again
                    wave_range(w, waves, count, next, end);
                    left = (int)(end - next);
                    q_head = 0;
                    tail = kNeverShare;
                    spent = 0;
                    if constexpr (BATCHED) {
                        scene0 = __builtin_amdgcn_readfirstlane(find_scene(offsets, n_scenes, next));
                        uniform_scene(scenes[scene0], cur);
                        base0 = uniform_i64(offsets[scene0]);
                        bound0 = uniform_i64(offsets[scene0 + 1]);
                    }
                }
            }
        }
        if (decides) {
            if constexpr (BATCHED) {
                // lanes of the wave's current scene read its output
                // pointers with uniform loads; others (a scene boundary
                // inside the wave) load their scene's
                if (L.scene == scene0) finish<MODE>(cur, L.pair, L, st == kHit, hg);
                else finish<MODE>(scenes[L.scene], L.pair, L, st == kHit, hg);
            } else {
                finish<MODE, CAND>(a0, L.pair, L, st == kHit, hg, Refined{}, L.scene >> 1);
            }
        }
        if (done) active = false;
        bool again = CAND && done && (L.scene & 1);       // candidate lists: the ray has another candidate
        const int ray = L.pair, at = L.scene >> 1;
        if constexpr (MODE == kConservative && CAND) {
            // the FP64 searches run for all parked lanes at once (SIMD lanes
            // of one call) when no busy lane is left: every lane of the wave
            // then shares the search's passes (measured: 2x faster on hair
            // than batches of 16 parked lanes)
            const uint64_t parked = __ballot(L.waiting != 0);
            if (parked != 0 && __ballot(active && !L.waiting) == 0) {
                if (L.waiting) {
                    L.waiting = 0;
                    // plain values, not references (see refine_whole_curve)
                    const float *rays = a0.rays, *fibers = a0.fibers;
                    const int64_t rs = a0.ray_stride, fs = a0.fiber_stride;
                    // the ray's tmax shortened to its FP64 nearest hit so far
                    const int64_t fi = a0.cand_fiber[a0.cand_off[L.pair] + a0.cand_first + at];
                    const double tlim = fmin((double)rays[6 * rs + L.pair], a0.t64_out[L.pair]);
                    const int32_t pair = L.pair;
                    const Refined r = refine_whole_curve(rays, rs, fibers, fs, pair, fi, tlim, L.t, L.ru,
                                                         a0.normal_out != nullptr);
                    // the output pointers are read after the call (not kept
                    // live across it); a refined pair's finish reads only the
                    // search's result from the lane (slack >= 0)
                    Lane R = {};
                    finish<MODE, CAND>(a0, pair, R, r.hit, HitGeo{}, r, at);
                    active = false;
                    again = (L.scene & 1) != 0;
                }
                // every lane is free now. Its traversal state is reset, so
                // that none of it is live across the searches (kept, it
                // had to be saved and restored around the call)
                L = Lane{};
            }
        }
        if constexpr (CAND) {
            const uint64_t am = __ballot(again);
            if (again) {
                const int e = wslot(w_head + w_count + (int)lanes_below(am));
                waiting.ray[e] = ray;
                waiting.round[e] = at + 1;
            }
            w_count += __popcll(am);
        }
        if (!active) {
            L.lo = INFINITY;
            L.hi = -INFINITY;
            L.bits = 0;
        }
    }
    if constexpr (MODE == kConservative && !CAND) {
        // the arguments are read again from where the launch put them: kept
        // for after the loop they had pushed others out of the scalar registers
        const Args *args = (const Args *)__builtin_amdgcn_kernarg_segment_ptr();
        // the wave's own marks, written above by other lanes
        __threadfence_block();
        __syncthreads();
        wave_range(w, waves, count, next, end);
        refine_range<BATCHED, QUAD>(*args, scenes, offsets, n_scenes, next, end, aos, (int *)s_queue);
    }
}

// Fibers transposed to 16 consecutive floats each, for calls that gather them
// through pair indices (one lane per fiber: coalesced row reads, 64-byte
// records written as four 16-byte stores).
__global__ __launch_bounds__(256) void k_fibers_aos(const float *F, int64_t fs, int64_t nf, float4 *out)
{
    const int64_t f = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (f >= nf) return;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        out[4 * f + k] = make_float4(F[(4 * k) * fs + f], F[(4 * k + 1) * fs + f], F[(4 * k + 2) * fs + f],
                                     F[(4 * k + 3) * fs + f]);
}

int check_common(const float *rays, int64_t ray_stride, int64_t n_rays,
                 const float *fibers, int64_t fiber_stride, int64_t n_fibers,
                 const int32_t *pair_ray, const int32_t *pair_fiber,
                 int32_t depth, int64_t n_pairs, uint32_t flags,
                 const void *t_out, const void *u_out, const void *hit_out)
{
    if (n_pairs < 0 || n_rays < 0 || n_fibers < 0) return FI_ERR_RANGE;
    if (depth < 0 || depth > FI_MAX_DEPTH) return FI_ERR_RANGE;
    if ((flags & ~(uint32_t)(FI_FP64_REFINE | FI_COMPENSATED_PROJ | FI_QUADRATIC)) != 0u) return FI_ERR_RANGE;
    if (n_pairs == 0) return FI_OK;
    if (!rays || !fibers || !t_out || !u_out || !hit_out) return FI_ERR_NULL;
    if (ray_stride < n_rays || fiber_stride < n_fibers) return FI_ERR_RANGE;
    if (!pair_ray && n_pairs > n_rays) return FI_ERR_RANGE;
    if (!pair_fiber && n_pairs > n_fibers) return FI_ERR_RANGE;
    if (n_pairs > (int64_t)0x7fffffff - 64) return FI_ERR_RANGE;   // int32 pair indices in the lanes
    return FI_OK;
}

// ---------------------------------------------------------------------------
// Kernel variants and per-device state
// ---------------------------------------------------------------------------

using FusedFn = void (*)(Args, const Args *, const int64_t *, int, int64_t, int, const float *);
// [0] plain, [1] counting, [2] conservative (single calls), [3] plain and
// [4] conservative over a scene table, [5] plain and [6] conservative over
// candidate lists, [7..9] plain, counting and conservative on quadratic
// fibers, [10] plain and [11] conservative over a scene table without the
// parent cache (a tuning choice: every backtrack replays from the root)
constexpr int kVariants = 12;
const FusedFn kFused[kVariants] = {k_fused<kPlain, false>, k_fused<kCount, false>, k_fused<kConservative, false>,
                                   k_fused<kPlain, true>, k_fused<kConservative, true>,
                                   k_fused<kPlain, false, true>, k_fused<kConservative, false, true>,
                                   k_fused<kPlain, false, false, true>, k_fused<kCount, false, false, true>,
                                   k_fused<kConservative, false, false, true>,
                                   k_fused<kPlain, true, false, false, false>,
                                   k_fused<kConservative, true, false, false, false>};
constexpr int kBatchedVariant = 3;
constexpr int kBatchedRefineVariant = 4;
constexpr int kCandVariant = 5;              // + 1: refined
constexpr int kQuadVariant = 7;              // + kPlain, kCount, kConservative: quadratic fibers
constexpr int kBatchedReplayVariant = 10;    // + 1: refined

constexpr size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }
constexpr size_t kMaxRecordBytes = (size_t)1 << 30;                 // fiber records, largest table

constexpr int kMaxDevices = 64;
constexpr int kStageSlots = 4;                 // pinned staging for batched scene tables
constexpr size_t kStageBytes = 1u << 20;

// Fiber records of fiber_intersect_pairs_noalloc, for callers that cannot
// allocate: a fixed array in the code object, one copy per device, of
// kScratchBytes (32 MiB: the records of 524,288 fibers). Host code never
// passes the array's name to a kernel: each device's copy is reached through
// the address hipGetSymbolAddress gives for it (DeviceInfo::scratch).
constexpr size_t kScratchBytes = (size_t)32 << 20;
static __device__ __align__(256) float scratch[kScratchBytes / sizeof(float)];

struct DeviceInfo {
    std::atomic<bool> ready;
    int cus;
    char arch[64];                             // architecture name (gfx950...), without feature flags
    int fused_resident[kVariants];             // resident waves per CU, per variant (as kFused)
    float *scratch;                            // this device's copy of `scratch`
    std::mutex stage_mutex;
    void *stage[kStageSlots];                  // pinned host buffers for scene tables
    hipEvent_t stage_done[kStageSlots];
    int stage_next;
};
DeviceInfo g_dev[kMaxDevices];
std::mutex g_dev_mutex;

int current_device(int &dev)
{
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return FI_ERR_HIP;
    return FI_OK;
}

// Set-up of the current device, once: unit counts, occupancy of every kernel
// variant, the address of this device's scratch array and the pinned staging
// buffers of batched calls. Every entry point runs it on its first call on a
// device (fi_init_device runs it ahead).
int device_info(DeviceInfo *&out)
{
    int dev = 0;
    if (current_device(dev) != FI_OK) return FI_ERR_HIP;
    DeviceInfo &d = g_dev[dev];
    if (!d.ready.load(std::memory_order_acquire)) {
        std::lock_guard<std::mutex> lock(g_dev_mutex);
        if (!d.ready.load(std::memory_order_relaxed)) {
            if (hipDeviceGetAttribute(&d.cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
                return FI_ERR_HIP;
            hipDeviceProp_t prop;
            if (hipGetDeviceProperties(&prop, dev) != hipSuccess) return FI_ERR_HIP;
            size_t n = 0;
            while (n + 1 < sizeof d.arch && prop.gcnArchName[n] && prop.gcnArchName[n] != ':') {
                d.arch[n] = prop.gcnArchName[n];
                ++n;
            }
            d.arch[n] = '\0';
            for (int m = 0; m < kVariants; ++m) {
                int nb = 0;
                if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, (const void *)kFused[m], kWave, 0) != hipSuccess)
                    return FI_ERR_HIP;
                d.fused_resident[m] = nb > 0 ? nb : 1;
            }
            // the device address of this device's copy of the static
            // scratch array (taken with the device current)
            d.scratch = nullptr;
            if (hipGetSymbolAddress((void **)&d.scratch, HIP_SYMBOL(scratch)) != hipSuccess || !d.scratch)
                return FI_ERR_HIP;
            for (int k = 0; k < kStageSlots; ++k) {
                if (hipHostMalloc(&d.stage[k], kStageBytes, hipHostMallocDefault) != hipSuccess) return FI_ERR_HIP;
                if (hipEventCreateWithFlags(&d.stage_done[k], hipEventDisableTiming) != hipSuccess) return FI_ERR_HIP;
            }
            d.stage_next = 0;
            d.ready.store(true, std::memory_order_release);
        }
    }
    out = &d;
    return FI_OK;
}

// Fiber records of a single call: when it gathers fibers through pair_fiber
// and reads each fiber about once or more, the fibers are first copied to
// 16-float records (one pass over the table): a gathered fiber is then one
// or two cache lines instead of one line per coordinate row. What the size
// queries and the no-allocation entry point answer; a call of few pairs
// (kRowPairs, see launch) leaves the room for them unused.
size_t record_bytes(int64_t n_pairs, int64_t n_fibers, bool gathered)
{
    const size_t need = (size_t)(n_fibers > 0 ? n_fibers : 0) * 16 * sizeof(float);
    return gathered && n_fibers > 0 && n_pairs >= n_fibers && need <= kMaxRecordBytes ? align256(need) : 0;
}

// Launch defaults of single-problem calls (and of batches without a tuned
// entry); measured choices, overridable when building.
#ifndef FIBERHIT_DEFAULT_REFILL
#define FIBERHIT_DEFAULT_REFILL 1
#endif
#ifndef FIBERHIT_DEFAULT_WAVES_PER_SIMD
#define FIBERHIT_DEFAULT_WAVES_PER_SIMD 0
#endif
fi_tuning default_tuning(bool refine)
{
    return fi_tuning{refine ? FIBERHIT_REFINE_REFILL : FIBERHIT_DEFAULT_REFILL, FIBERHIT_DEFAULT_WAVES_PER_SIMD, 0};
}

// Autotune results: keyed by the GPU architecture, the refinement flag and
// the batch's class -- log2 of its total pairs, log2 of its problem count and
// a depth bucket of its largest depth (<= 9, <= 16, deeper). A batch launched
// without an explicit tuning uses the entry of its class if one exists. The
// table lives for the process; fiber_tuning_save / fiber_tuning_load keep it
// in a text file across processes.
using TuneKey = std::tuple<std::string, int, int, int, int>;
std::mutex g_tune_mutex;
std::map<TuneKey, fi_tuning> g_tune_cache;

int log2_floor(int64_t x)
{
    int l = 0;
    while (l < 62 && ((int64_t)1 << (l + 1)) <= x) ++l;
    return l;
}

int depth_bucket(int max_depth) { return max_depth <= 9 ? 0 : max_depth <= 16 ? 1 : 2; }

TuneKey tune_key(const std::string &arch, int64_t total, int n_scenes, int max_depth, bool refine)
{
    return TuneKey{arch, refine ? 1 : 0, log2_floor(total), log2_floor(n_scenes), depth_bucket(max_depth)};
}

int check_tuning(const fi_tuning &t)
{
    if (t.refill < 1 || t.refill > kWave || t.waves_per_simd < 0 || t.waves_per_simd > 16 || t.stack < 0 ||
        t.stack > 1)
        return FI_ERR_RANGE;
    return FI_OK;
}

int max_scene_depth(const fi_scene *sc, int32_t n)
{
    int d = 0;
    for (int k = 0; k < n; ++k) d = sc[k].depth > d ? sc[k].depth : d;
    return d;
}

int64_t total_pairs(const fi_scene *sc, int32_t n)
{
    int64_t t = 0;
    for (int k = 0; k < n; ++k) t += sc[k].n_pairs > 0 ? sc[k].n_pairs : 0;
    return t;
}

// The remembered tuning of this batch's class on the current device, else
// the defaults.
fi_tuning tuned_or_default(const fi_scene *sc, int32_t n, bool refine)
{
    DeviceInfo *d = nullptr;
    if (device_info(d) != FI_OK) return default_tuning(refine);
    std::lock_guard<std::mutex> lock(g_tune_mutex);
    const auto it = g_tune_cache.find(tune_key(d->arch, total_pairs(sc, n), n, max_scene_depth(sc, n), refine));
    return it == g_tune_cache.end() ? default_tuning(refine) : it->second;
}

void remember_tuning(const fi_scene *sc, int32_t n, bool refine, const fi_tuning &t)
{
    DeviceInfo *d = nullptr;
    if (device_info(d) != FI_OK) return;
    std::lock_guard<std::mutex> lock(g_tune_mutex);
    g_tune_cache[tune_key(d->arch, total_pairs(sc, n), n, max_scene_depth(sc, n), refine)] = t;
}


// Persistent waves of a single call: twice the resident waves, each with
// half the share. The second half starts as waves of the first finish, so
// waves whose pairs happened to need few trips take more of the work and
// the call's tail shrinks. Measured against the resident waves alone (A/B
// on one box, 2^20 pairs): depth 22 198 against 232 us, depth 9 123
// against 115 us, the two calls overlapped on two streams 228.5 against
// 230 us; hair (2^24 pairs) 1.23 / 1.90 against 1.26 / 1.96 ms; refined
// hair 3.93 against 4.13 ms per 2^22 pairs. Four times the resident waves
// was slower (overlapped 283 us), and so were twice the waves for deep
// calls only (overlapped 250 us: the shallow call's waves then wait behind
// the deep call's), a grid skewed towards the waves that start first on
// each SIMD, and issue priority by progress through the share. Candidate
// lists keep the resident waves: twice as many changed six calls (3001 to
// 524,288 lists, two of them refined) by -3 to +1 %. Refined calls keep them
// too: a wave lists its share's pairs for the FP64 decisions, and longer lists
// fill its lanes better (hair 399 against 438 us per 10^6 pairs, 500,009
// degenerate pairs 1.14 against 1.34 ms).
int64_t single_call_waves(const DeviceInfo &d, int mode, const Args &)
{
    const bool cand = mode == kCandVariant || mode == kCandVariant + 1;
    const bool refine = mode == kConservative || mode == kQuadVariant + kConservative;
    return (cand || refine ? 1 : 2) * (int64_t)d.fused_resident[mode] * d.cus;
}

constexpr int64_t kRowPairs = 1 << 16;

// Enqueue one single call on `s`: the fiber records (when `aos` is given and the
// pairs are many), then one persistent launch of about one wave per 64 pairs,
// at most `max_waves`. `rounds`: how many candidates of each list it tests
// (candidate lists).
int launch(const DeviceInfo &d, int mode, const Args &a, float *aos, hipStream_t s, int rounds = 0)
{
    const int64_t max_waves = single_call_waves(d, mode, a);
    // Few pairs read the rows: the records' pass takes 2 to 3 us of the call
    // before its first pair. 4096 pairs of 64 fibers 23.0 -> 20.8 us, 65,536
    // hair pairs over 4000 segments 27.7 -> 26.4 and over 65,536 the same
    // (37.3); at 2^18 pairs the records are the faster way (45.7 against 49.7
    // over 1000 segments), and at 65,537 candidate lists (97 against 106).
    if (!a.cand_off && a.n_pairs <= kRowPairs) aos = nullptr;
    if (aos && a.cand_first == 0)
        hipLaunchKernelGGL(k_fibers_aos, dim3((unsigned)((a.n_fibers + 255) / 256)), dim3(256), 0, s,
                           a.fibers, a.fiber_stride, a.n_fibers, (float4 *)aos);
    int64_t g = (a.n_pairs + kWave - 1) / kWave;
    if (g > max_waves) g = max_waves;
    if (g > 0)
        hipLaunchKernelGGL(kFused[mode], dim3((unsigned)g), dim3(kWave), 0, s, a, nullptr, nullptr, rounds,
                           a.n_pairs,
                           mode == kConservative || mode == kCandVariant + 1 ||
                                   mode == kQuadVariant + kConservative
                               ? FIBERHIT_REFINE_REFILL
                               : FIBERHIT_FUSED_REFILL,
                           aos);
    return hipGetLastError() == hipSuccess ? FI_OK : FI_ERR_HIP;
}

// A single call with the fiber records (if it gathers fibers) in the
// caller's workspace, room permitting.
int launch_with_workspace(int mode, const Args &a, void *workspace, size_t workspace_bytes, void *stream,
                          bool quad = false)
{
    if (workspace && ((uintptr_t)workspace & 255u) != 0u) return FI_ERR_WORKSPACE;
    (void)hipGetLastError();
    DeviceInfo *d = nullptr;
    const int st = device_info(d);
    if (st != FI_OK) return st;
    // quadratic tables are read in place (the records hold cubic rows)
    const size_t rec = quad ? 0 : record_bytes(a.n_pairs, a.n_fibers, a.pair_fiber != nullptr);
    float *aos = rec && workspace && workspace_bytes >= rec ? (float *)workspace : nullptr;
    return launch(*d, mode, a, aos, (hipStream_t)stream);
}

// ---------------------------------------------------------------------------
// Batched problems
// ---------------------------------------------------------------------------

size_t scene_table_bytes(int n) { return align256((size_t)n * sizeof(Args)) + align256((size_t)(n + 1) * sizeof(int64_t)); }

int scenes_to_table(const fi_scene *sc, int32_t n, uint32_t flags, Args *tab, int64_t *off)
{
    const bool refine = (flags & FI_FP64_REFINE) != 0u;
    off[0] = 0;
    for (int k = 0; k < n; ++k) {
        const fi_scene &x = sc[k];
        const int st = check_common(x.rays, x.ray_stride, x.n_rays, x.fibers, x.fiber_stride, x.n_fibers,
                                    x.pair_ray, x.pair_fiber, x.depth, x.n_pairs, flags, x.t_out, x.u_out, x.hit_out);
        if (st != FI_OK) return st;
        if (refine && x.n_pairs > 0 && (!x.t64_out || !x.u64_out)) return FI_ERR_NULL;
        tab[k] = Args{x.rays, x.ray_stride, x.n_rays, x.fibers, x.fiber_stride, x.n_fibers,
                      x.pair_ray, x.pair_fiber, x.pair_depth, x.depth, x.n_pairs,
                      x.t_out, x.u_out, x.hit_out, nullptr,
                      refine ? x.t64_out : nullptr, refine ? x.u64_out : nullptr, x.normal_out};
        off[k + 1] = off[k] + x.n_pairs;
    }
    if (off[n] > (int64_t)0x7fffffff - 64) return FI_ERR_RANGE;
    return FI_OK;
}

// Layout of a batched workspace: scene table, pair offsets.
struct BatchLayout {
    Args *scenes;
    int64_t *offsets;
};

BatchLayout layout_of(void *ws, int n)
{
    char *p = (char *)ws;
    BatchLayout L;
    L.scenes = (Args *)p;
    L.offsets = (int64_t *)(p + align256((size_t)n * sizeof(Args)));
    return L;
}

// One persistent launch over all scenes of a batch: about one wave per 64
// pairs, at most the resident waves, or the tuning's waves per SIMD (fewer
// or more than fit).
void launch_batched(const DeviceInfo &d, const fi_tuning &t, const BatchLayout &L, int n_scenes, int64_t total,
                    bool refine, hipStream_t s)
{
    const int variant = t.stack == 1 ? kBatchedReplayVariant + (refine ? 1 : 0)
                                     : (refine ? kBatchedRefineVariant : kBatchedVariant);
    int per_cu = d.fused_resident[variant];
    // below the resident waves per SIMD: fewer waves; above: the grid holds
    // more waves than fit, and the dispatcher starts them as others end
    if (t.waves_per_simd > 0) per_cu = 4 * t.waves_per_simd;
    int64_t g = (total + kWave - 1) / kWave;
    if (g > (int64_t)per_cu * d.cus) g = (int64_t)per_cu * d.cus;
    if (g > 0)
        hipLaunchKernelGGL(kFused[variant], dim3((unsigned)g), dim3(kWave), 0, s, Args{}, L.scenes, L.offsets,
                           n_scenes, total, t.refill, nullptr);
}

int batched_enqueue(const fi_scene *scenes, int32_t n_scenes, uint32_t flags, const fi_tuning &t, void *workspace,
                    size_t workspace_bytes, hipStream_t s)
{
    DeviceInfo *d = nullptr;
    int st = device_info(d);
    if (st != FI_OK) return st;
    const size_t tb = scene_table_bytes(n_scenes);
    if (tb > kStageBytes) return FI_ERR_RANGE;
    if (!workspace || ((uintptr_t)workspace & 255u) != 0u || workspace_bytes < tb) return FI_ERR_WORKSPACE;
    std::lock_guard<std::mutex> lock(d->stage_mutex);
    const int k = d->stage_next;
    // the staging buffer's previous upload must have left it (rarely waits:
    // four buffers in turn)
    if (hipEventSynchronize(d->stage_done[k]) != hipSuccess) return FI_ERR_HIP;
    char *host = (char *)d->stage[k];
    int64_t *off = (int64_t *)(host + align256((size_t)n_scenes * sizeof(Args)));
    st = scenes_to_table(scenes, n_scenes, flags, (Args *)host, off);
    if (st != FI_OK) return st;
    const int64_t total = off[n_scenes];
    const BatchLayout L = layout_of(workspace, n_scenes);
    if (hipMemcpyAsync(workspace, host, tb, hipMemcpyHostToDevice, s) != hipSuccess) return FI_ERR_HIP;
    if (hipEventRecord(d->stage_done[k], s) != hipSuccess) return FI_ERR_HIP;
    d->stage_next = (k + 1) % kStageSlots;
    launch_batched(*d, t, L, n_scenes, total, (flags & FI_FP64_REFINE) != 0u, s);
    return hipGetLastError() == hipSuccess ? FI_OK : FI_ERR_HIP;
}

}  // namespace

struct fi_batch_plan {
    int device;
    void *mem;                 // device copy of the scene table and offsets
    int n_scenes;
    int64_t total;
    uint32_t flags;
    fi_tuning tuning;
    hipGraph_t graph;
    hipGraphExec_t exec;
};

extern "C" {
int fi_version(void) { return (0 << 16) | (9 << 8) | 0; }

const char *fi_strerror(int status)
{
    switch (status) {
    case FI_OK: return "ok";
    case FI_ERR_NULL: return "a required pointer is NULL";
    case FI_ERR_RANGE: return "a count, stride, depth or flag is out of range";
    case FI_ERR_HIP: return "the HIP runtime reported an error";
    case FI_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case FI_ERR_SCRATCH: return "the call needs more scratch than the no-allocation entry point holds";
    case FI_ERR_IO: return "a tuning table file could not be opened or written";
    default: return "unknown status";
    }
}

int fi_init_device(void)
{
    (void)hipGetLastError();
    DeviceInfo *d = nullptr;
    return device_info(d);
}

size_t fiber_pairs_workspace_bytes(int64_t n_pairs, int64_t n_fibers, int32_t gathered, uint32_t flags)
{
    if (n_pairs < 0 || n_fibers < 0 || (flags & FI_QUADRATIC) != 0u) return 0;
    return record_bytes(n_pairs, n_fibers, gathered != 0);
}

int fiber_intersect_pairs(const float *rays, int64_t ray_stride, int64_t n_rays,
                          const float *fibers, int64_t fiber_stride, int64_t n_fibers,
                          const int32_t *pair_ray, const int32_t *pair_fiber,
                          const uint8_t *pair_depth, int32_t depth, int64_t n_pairs,
                          uint32_t flags,
                          float *t_out, float *u_out, uint8_t *hit_out,
                          double *t64_out, double *u64_out, float *normal_out,
                          void *workspace, size_t workspace_bytes, void *stream)
{
    const int st = check_common(rays, ray_stride, n_rays, fibers, fiber_stride, n_fibers,
                                pair_ray, pair_fiber, depth, n_pairs, flags, t_out, u_out, hit_out);
    if (st != FI_OK || n_pairs == 0) return st;
    const bool refine = (flags & FI_FP64_REFINE) != 0u;
    if (refine && (!t64_out || !u64_out)) return FI_ERR_NULL;
    Args a{rays, ray_stride, n_rays, fibers, fiber_stride, n_fibers,
           pair_ray, pair_fiber, pair_depth, depth, n_pairs, t_out, u_out, hit_out, nullptr,
           refine ? t64_out : nullptr, refine ? u64_out : nullptr, normal_out};
    const bool quad = (flags & FI_QUADRATIC) != 0u;
    return launch_with_workspace((refine ? kConservative : kPlain) + (quad ? kQuadVariant : 0), a, workspace,
                                 workspace_bytes, stream, quad);
}

int fiber_intersect_pairs_noalloc(const float *rays, int64_t ray_stride, int64_t n_rays,
                                  const float *fibers, int64_t fiber_stride, int64_t n_fibers,
                                  const int32_t *pair_ray, const int32_t *pair_fiber,
                                  const uint8_t *pair_depth, int32_t depth, int64_t n_pairs,
                                  uint32_t flags,
                                  float *t_out, float *u_out, uint8_t *hit_out,
                                  double *t64_out, double *u64_out, float *normal_out,
                                  void *stream)
{
    const int st = check_common(rays, ray_stride, n_rays, fibers, fiber_stride, n_fibers,
                                pair_ray, pair_fiber, depth, n_pairs, flags, t_out, u_out, hit_out);
    if (st != FI_OK || n_pairs == 0) return st;
    const bool refine = (flags & FI_FP64_REFINE) != 0u;
    if (refine && (!t64_out || !u64_out)) return FI_ERR_NULL;
    const bool quad = (flags & FI_QUADRATIC) != 0u;
    const size_t rec = quad ? 0 : record_bytes(n_pairs, n_fibers, pair_fiber != nullptr);
    if (rec > kScratchBytes) return FI_ERR_SCRATCH;
    (void)hipGetLastError();
    DeviceInfo *d = nullptr;
    const int ds = device_info(d);
    if (ds != FI_OK) return ds;
    const int mode = (refine ? kConservative : kPlain) + (quad ? kQuadVariant : 0);
    Args a{rays, ray_stride, n_rays, fibers, fiber_stride, n_fibers,
           pair_ray, pair_fiber, pair_depth, depth, n_pairs, t_out, u_out, hit_out, nullptr,
           refine ? t64_out : nullptr, refine ? u64_out : nullptr, normal_out};
    // the fiber records of a gathered call go to this device's copy of the
    // scratch array (through its device address, never the array's name)
    return launch(*d, mode, a, rec ? d->scratch : nullptr, (hipStream_t)stream);
}

int fiber_intersect_counts(const float *rays, int64_t ray_stride, int64_t n_rays,
                           const float *fibers, int64_t fiber_stride, int64_t n_fibers,
                           const int32_t *pair_ray, const int32_t *pair_fiber,
                           const uint8_t *pair_depth, int32_t depth, int64_t n_pairs,
                           uint32_t flags,
                           float *t_out, float *u_out, uint8_t *hit_out,
                           int32_t *counts_out, void *workspace, size_t workspace_bytes, void *stream)
{
    const int st = check_common(rays, ray_stride, n_rays, fibers, fiber_stride, n_fibers,
                                pair_ray, pair_fiber, depth, n_pairs, flags, t_out, u_out, hit_out);
    if (st != FI_OK || n_pairs == 0) return st;
    if (!counts_out) return FI_ERR_NULL;
    if ((flags & FI_FP64_REFINE) != 0u) return FI_ERR_RANGE;
    Args a{rays, ray_stride, n_rays, fibers, fiber_stride, n_fibers,
           pair_ray, pair_fiber, pair_depth, depth, n_pairs, t_out, u_out, hit_out, counts_out, nullptr, nullptr,
           nullptr};
    const bool quad = (flags & FI_QUADRATIC) != 0u;
    return launch_with_workspace(kCount + (quad ? kQuadVariant : 0), a, workspace, workspace_bytes, stream, quad);
}

size_t fiber_candidates_workspace_bytes(int64_t n_candidates, int64_t n_fibers, uint32_t flags)
{
    (void)flags;
    if (n_candidates < 0 || n_fibers < 0) return 0;
    return record_bytes(n_candidates, n_fibers, true);
}

int fiber_intersect_candidates(const float *rays, int64_t ray_stride, int64_t n_rays,
                               const float *fibers, int64_t fiber_stride, int64_t n_fibers,
                               const int64_t *cand_offsets, const int32_t *cand_fiber,
                               const uint8_t *cand_depth, int32_t depth, int32_t max_candidates,
                               int64_t n_candidates, uint32_t flags,
                               float *t_out, float *u_out, uint8_t *hit_out, int32_t *fiber_out,
                               double *t64_out, double *u64_out, float *normal_out,
                               void *workspace, size_t workspace_bytes, void *stream)
{
    if (n_rays < 0 || n_fibers < 0 || n_candidates < 0 || max_candidates < 0) return FI_ERR_RANGE;
    if (depth < 0 || depth > FI_MAX_DEPTH) return FI_ERR_RANGE;
    if ((flags & ~(uint32_t)(FI_FP64_REFINE | FI_COMPENSATED_PROJ)) != 0u) return FI_ERR_RANGE;
    if (n_rays == 0) return FI_OK;
    if (!rays || !fibers || !cand_offsets || !t_out || !u_out || !hit_out || !fiber_out) return FI_ERR_NULL;
    if (n_candidates > 0 && !cand_fiber) return FI_ERR_NULL;
    if (ray_stride < n_rays || fiber_stride < n_fibers) return FI_ERR_RANGE;
    if (n_rays > (int64_t)0x7fffffff - 64) return FI_ERR_RANGE;
    const bool refine = (flags & FI_FP64_REFINE) != 0u;
    if (refine && (!t64_out || !u64_out)) return FI_ERR_NULL;
    if (workspace && ((uintptr_t)workspace & 255u) != 0u) return FI_ERR_WORKSPACE;
    (void)hipGetLastError();
    DeviceInfo *d = nullptr;
    const int ds = device_info(d);
    if (ds != FI_OK) return ds;
    const hipStream_t s = (hipStream_t)stream;
    const int mode = refine ? kCandVariant + 1 : kCandVariant;
    Args a{rays, ray_stride, n_rays, fibers, fiber_stride, n_fibers,
           nullptr, nullptr, cand_depth, depth, n_rays, t_out, u_out, hit_out, nullptr,
           refine ? t64_out : nullptr, refine ? u64_out : nullptr, normal_out,
           cand_offsets, cand_fiber, 0, n_candidates, fiber_out};
    const size_t rec = record_bytes(n_candidates, n_fibers, true);
    float *aos = rec && workspace && workspace_bytes >= rec ? (float *)workspace : nullptr;
    // one launch (a lane holds a candidate's place in its list in 24 bits)
    do {
        const int32_t rounds = std::min(max_candidates - a.cand_first, kMaxRounds);
        const int st = launch(*d, mode, a, aos, s, rounds);
        if (st != FI_OK) return st;
        a.cand_first += rounds;
    } while (a.cand_first < max_candidates);
    return FI_OK;
}

size_t fiber_batched_workspace_bytes(int32_t n_scenes, int64_t total_pairs)
{
    if (n_scenes < 0 || total_pairs < 0) return 0;
    return scene_table_bytes(n_scenes);
}

int fiber_intersect_batched(const fi_scene *scenes, int32_t n_scenes, const fi_tuning *tuning,
                            uint32_t flags, void *workspace, size_t workspace_bytes, void *stream)
{
    if (n_scenes < 0 || (flags & ~(uint32_t)(FI_FP64_REFINE | FI_COMPENSATED_PROJ)) != 0u) return FI_ERR_RANGE;
    if (n_scenes == 0) return FI_OK;
    if (!scenes) return FI_ERR_NULL;
    const bool refine = (flags & FI_FP64_REFINE) != 0u;
    const fi_tuning t = tuning ? *tuning : tuned_or_default(scenes, n_scenes, refine);
    if (check_tuning(t) != FI_OK) return FI_ERR_RANGE;
    (void)hipGetLastError();
    return batched_enqueue(scenes, n_scenes, flags, t, workspace, workspace_bytes, (hipStream_t)stream);
}

int fiber_batch_plan_create(const fi_scene *scenes, int32_t n_scenes, const fi_tuning *tuning,
                            uint32_t flags, fi_batch_plan **plan_out)
{
    if (!plan_out) return FI_ERR_NULL;
    *plan_out = nullptr;
    if (n_scenes <= 0 || (flags & ~(uint32_t)(FI_FP64_REFINE | FI_COMPENSATED_PROJ)) != 0u) return FI_ERR_RANGE;
    if (!scenes) return FI_ERR_NULL;
    const bool refine = (flags & FI_FP64_REFINE) != 0u;
    const fi_tuning t = tuning ? *tuning : tuned_or_default(scenes, n_scenes, refine);
    if (check_tuning(t) != FI_OK) return FI_ERR_RANGE;
    (void)hipGetLastError();
    DeviceInfo *d = nullptr;
    int st = device_info(d);
    if (st != FI_OK) return st;
    const size_t tb = scene_table_bytes(n_scenes);
    char *host = (char *)malloc(tb);
    if (!host) return FI_ERR_RANGE;
    int64_t *off = (int64_t *)(host + align256((size_t)n_scenes * sizeof(Args)));
    st = scenes_to_table(scenes, n_scenes, flags, (Args *)host, off);
    if (st != FI_OK) { free(host); return st; }
    fi_batch_plan *p = new fi_batch_plan();
    p->n_scenes = n_scenes;
    p->total = off[n_scenes];
    p->flags = flags;
    p->tuning = t;
    current_device(p->device);
    hipStream_t cs = nullptr;
    const size_t bytes = tb;
    bool ok = hipMalloc(&p->mem, bytes) == hipSuccess &&
              hipMemcpy(p->mem, host, tb, hipMemcpyHostToDevice) == hipSuccess &&
              hipStreamCreate(&cs) == hipSuccess;
    free(host);
    if (ok) {
        const BatchLayout L = layout_of(p->mem, n_scenes);
        ok = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal) == hipSuccess;
        if (ok) {
            launch_batched(*d, t, L, n_scenes, p->total, refine, cs);
            ok = hipStreamEndCapture(cs, &p->graph) == hipSuccess &&
                 hipGraphInstantiate(&p->exec, p->graph, nullptr, nullptr, 0) == hipSuccess;
        }
    }
    if (cs) (void)hipStreamDestroy(cs);
    if (!ok) {
        (void)hipGetLastError();
        if (p->exec) (void)hipGraphExecDestroy(p->exec);
        if (p->graph) (void)hipGraphDestroy(p->graph);
        if (p->mem) (void)hipFree(p->mem);
        delete p;
        return FI_ERR_HIP;
    }
    *plan_out = p;
    return FI_OK;
}

int fiber_batch_plan_launch(fi_batch_plan *plan, void *stream)
{
    if (!plan) return FI_ERR_NULL;
    (void)hipGetLastError();
    return hipGraphLaunch(plan->exec, (hipStream_t)stream) == hipSuccess ? FI_OK : FI_ERR_HIP;
}

int fiber_batch_plan_destroy(fi_batch_plan *plan)
{
    if (!plan) return FI_OK;
    int st = FI_OK;
    if (plan->exec && hipGraphExecDestroy(plan->exec) != hipSuccess) st = FI_ERR_HIP;
    if (plan->graph && hipGraphDestroy(plan->graph) != hipSuccess) st = FI_ERR_HIP;
    if (plan->mem && hipFree(plan->mem) != hipSuccess) st = FI_ERR_HIP;
    delete plan;
    return st;
}

int fiber_batch_plan_tuning(const fi_batch_plan *plan, fi_tuning *tuning_out)
{
    if (!plan || !tuning_out) return FI_ERR_NULL;
    *tuning_out = plan->tuning;
    return FI_OK;
}

int fiber_batch_autotune(const fi_scene *scenes, int32_t n_scenes, uint32_t flags, void *workspace,
                         size_t workspace_bytes, void *stream, int32_t repeats,
                         fi_tuning *best, float *best_ms)
{
    if (!best) return FI_ERR_NULL;
    if (n_scenes <= 0 || (flags & ~(uint32_t)(FI_FP64_REFINE | FI_COMPENSATED_PROJ)) != 0u || repeats < 1)
        return FI_ERR_RANGE;
    const bool refine = (flags & FI_FP64_REFINE) != 0u;
    hipStream_t s = (hipStream_t)stream;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) return FI_ERR_HIP;
    // plain waves refill late; refining ones (which decide their pairs after
    // their traversal) take the same time within 1 % with any of 1 to 56
    const int plain_refills[] = {32, 48, 56};
    const int refine_refills[] = {4, 8, 16};
    const int *refills = refine ? refine_refills : plain_refills;
    const int occ[] = {0, 8, 16};         // as many as fit (4), twice, four times
    float best_t = INFINITY;
    fi_tuning bt = default_tuning(refine);
    int st = FI_OK;
    for (int sk = 0; sk < 2 && st == FI_OK; ++sk)
    for (int oi = 0; oi < 3 && st == FI_OK; ++oi)
        for (int ri = 0; ri < 3 && st == FI_OK; ++ri) {
            const fi_tuning t{refills[ri], occ[oi], sk};
            float tmin = INFINITY;
            for (int r = 0; r <= repeats && st == FI_OK; ++r) {       // first run warms up
                if (hipEventRecord(e0, s) != hipSuccess) { st = FI_ERR_HIP; break; }
                st = fiber_intersect_batched(scenes, n_scenes, &t, flags, workspace, workspace_bytes, stream);
                if (st == FI_OK && hipEventRecord(e1, s) != hipSuccess) st = FI_ERR_HIP;
                if (st == FI_OK && hipEventSynchronize(e1) != hipSuccess) st = FI_ERR_HIP;
                float ms = 0.0f;
                if (st == FI_OK && r > 0 && hipEventElapsedTime(&ms, e0, e1) == hipSuccess && ms < tmin)
                    tmin = ms;
            }
            if (tmin < best_t) { best_t = tmin; bt = t; }
        }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (st != FI_OK) return st;
    *best = bt;
    if (best_ms) *best_ms = best_t;
    remember_tuning(scenes, n_scenes, refine, bt);
    return FI_OK;
}

// Tuning table files: a header line, then one entry per line --
// arch refine log2_pairs log2_scenes depth_bucket refill waves_per_simd stack
int fiber_tuning_save(const char *path)
{
    if (!path) return FI_ERR_NULL;
    std::vector<std::pair<TuneKey, fi_tuning>> rows;
    {
        std::lock_guard<std::mutex> lock(g_tune_mutex);
        rows.assign(g_tune_cache.begin(), g_tune_cache.end());
    }
    FILE *f = fopen(path, "w");
    if (!f) return FI_ERR_IO;
    bool ok = fprintf(f, "fiberhit-tuning 1\n") > 0;
    for (const auto &r : rows)
        ok = ok && fprintf(f, "%s %d %d %d %d %d %d %d\n", std::get<0>(r.first).c_str(), std::get<1>(r.first),
                           std::get<2>(r.first), std::get<3>(r.first), std::get<4>(r.first), r.second.refill,
                           r.second.waves_per_simd, r.second.stack) > 0;
    ok = (fclose(f) == 0) && ok;
    return ok ? FI_OK : FI_ERR_IO;
}

int fiber_tuning_load(const char *path)
{
    if (!path) return FI_ERR_NULL;
    FILE *f = fopen(path, "r");
    if (!f) return FI_ERR_IO;
    std::vector<std::pair<TuneKey, fi_tuning>> rows;
    char line[256];
    bool ok = fgets(line, sizeof line, f) && strcmp(line, "fiberhit-tuning 1\n") == 0;
    while (ok && fgets(line, sizeof line, f)) {
        char arch[64];
        int rf, lt, ls, db;
        fi_tuning t;
        char tail;
        if (sscanf(line, "%63s %d %d %d %d %d %d %d %c", arch, &rf, &lt, &ls, &db, &t.refill, &t.waves_per_simd,
                   &t.stack, &tail) != 8 ||
            rf < 0 || rf > 1 || lt < 0 || lt > 62 || ls < 0 || ls > 31 || db < 0 || db > 2 ||
            check_tuning(t) != FI_OK) {
            ok = false;
            break;
        }
        rows.push_back({TuneKey{arch, rf, lt, ls, db}, t});
    }
    fclose(f);
    if (!ok) return FI_ERR_RANGE;
    std::lock_guard<std::mutex> lock(g_tune_mutex);
    for (const auto &r : rows) g_tune_cache[r.first] = r.second;
    return FI_OK;
}

int fiber_tuning_lookup(const char *arch, uint32_t flags, int64_t total_pairs, int32_t n_scenes, int32_t max_depth,
                        fi_tuning *out)
{
    if (!arch || !out) return FI_ERR_NULL;
    if (total_pairs < 0 || n_scenes < 1 || max_depth < 0 || max_depth > FI_MAX_DEPTH ||
        (flags & ~(uint32_t)(FI_FP64_REFINE | FI_COMPENSATED_PROJ)) != 0u)
        return FI_ERR_RANGE;
    std::lock_guard<std::mutex> lock(g_tune_mutex);
    const auto it =
        g_tune_cache.find(tune_key(arch, total_pairs, n_scenes, max_depth, (flags & FI_FP64_REFINE) != 0u));
    if (it == g_tune_cache.end()) return FI_ERR_RANGE;
    *out = it->second;
    return FI_OK;
}

int fiber_tuning_clear(void)
{
    std::lock_guard<std::mutex> lock(g_tune_mutex);
    g_tune_cache.clear();
    return FI_OK;
}

}  // extern "C"
