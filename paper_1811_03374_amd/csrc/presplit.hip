// Fiber validation and pre-subdivision (Section 3.4) for gfx950.
//
// The paper's method needs curves whose recursive halves are separated by
// their split planes (the five inequalities of Section 3.4, proved in
// Appendix B.2) and whose swept solid does not reach across a cap plane
// (Section 3.4, the thick-fiber configuration of Fig. "EvilConfiguration").
// Curves that fail must be split beforehand. These kernels run before the
// per-pair test, all arithmetic in FP64 (passes over the fiber table, far from
// any hot loop).
//
// Cap-plane excess (reading R17): the disc at u (centre C(u), radius r(u),
// normal C'(u)) reaches furthest along a cap normal n at C(u) + r(u) m(u),
// m the unit component of n normal to C'(u) (Gram-Schmidt), i.e. r(u) sin
// of the angle between C'(u) and n beyond its centre. The excess over the
// start plane is r sin - <C(u) - p0, n0>, over the end plane r sin -
// <p3 - C(u), n1>; n0, n1 are the cap normals (the end tangents, or the
// next control-polygon edge, then the chord, where a tangent is negligible).
// A fiber is thick at an end when its largest excess exceeds 1e-9 of its
// extent (|p3 - p0| plus the largest radius value). The largest excess is
// searched on 105 parameters -- 63 evenly spaced, 20 packed geometrically
// towards each end (u = 2^-j and 1 - 2^-j, j = 7, 9, .., 45, where the excess
// shrinks with the distance to the end) and the two ends -- followed by a
// golden-section search in the bracket of the best sample.
//
// Most ends need no search: a bound on the excess (ends_clear) shows that
// their discs stay behind the cap plane. The rest are collected in LDS and
// searched by full waves, which stop at the first sample over the threshold
// where only the mask is wanted.
//
// Pre-subdivision: a fiber is halved by de Casteljau's construction at
// u = 1/2 (4-D, radius included), depth first and left half first, until a
// piece is valid or max_level halvings deep. Each node is rebuilt from the
// fiber by replaying the halvings along its path (at most max_level of
// them); the halving is exact in FP64 for the levels allowed here, so every
// piece is the exact sub-curve rounded once to float32.

#include <hip/hip_runtime.h>
#include <hipcub/hipcub.hpp>
#include <stdint.h>

#include "fiberhit.h"

namespace {

constexpr int kMaxSplitLevel = 10;

struct Q16 {
    double v[16];                       // p0..p3, each x, y, z, r
};

__device__ __forceinline__ void load_fiber(const float *F, int64_t fs, int64_t i, Q16 &q)
{
#pragma unroll
    for (int k = 0; k < 16; ++k) q.v[k] = (double)F[k * fs + i];
}

__device__ __forceinline__ double d3(double ax, double ay, double az, double bx, double by, double bz)
{
    return ax * bx + ay * by + az * bz;
}

// the five inequalities of Section 3.4: bit k set when inequality k fails
__device__ __forceinline__ int constraint_bits(const Q16 &q)
{
    const double *p = q.v;
    auto dd = [&](int a, int b, int c, int e) {        // <p_a - p_b, p_c - p_e>
        return d3(p[4 * a] - p[4 * b], p[4 * a + 1] - p[4 * b + 1], p[4 * a + 2] - p[4 * b + 2],
                  p[4 * c] - p[4 * e], p[4 * c + 1] - p[4 * e + 1], p[4 * c + 2] - p[4 * e + 2]);
    };
    int m = 0;
    if (!(dd(2, 0, 1, 0) >= 0.0)) m |= 1;
    if (!(dd(3, 1, 1, 0) >= 0.0)) m |= 2;
    if (!(dd(3, 1, 3, 2) >= 0.0)) m |= 4;
    if (!(dd(2, 0, 3, 2) >= 0.0)) m |= 8;
    if (!(dd(2, 0, 3, 1) >= 0.0)) m |= 16;
    return m;
}

// unit cap normal at the start (end = false) or end
__device__ __forceinline__ void cap_normal(const Q16 &q, bool end, double n[3])
{
    const double *p = q.v;
    const double ax = p[12] - p[0], ay = p[13] - p[1], az = p[14] - p[2];
    const double lim = 0x1p-40 * d3(ax, ay, az, ax, ay, az);
    // first non-negligible of (p1 - p0, p2 - p0, p3 - p0) / (p3 - p2, p3 - p1, p3 - p0)
    const int a0 = end ? 3 : 1, b0 = end ? 2 : 0;
    const int a1 = end ? 3 : 2, b1 = end ? 1 : 0;
    double x = p[4 * a0] - p[4 * b0], y = p[4 * a0 + 1] - p[4 * b0 + 1], z = p[4 * a0 + 2] - p[4 * b0 + 2];
    if (d3(x, y, z, x, y, z) <= lim) {
        x = p[4 * a1] - p[4 * b1]; y = p[4 * a1 + 1] - p[4 * b1 + 1]; z = p[4 * a1 + 2] - p[4 * b1 + 2];
    }
    if (d3(x, y, z, x, y, z) <= lim) { x = ax; y = ay; z = az; }
    const double il = 1.0 / sqrt(d3(x, y, z, x, y, z));
    n[0] = x * il; n[1] = y * il; n[2] = z * il;
}

// excess of the disc at u over a cap plane (-inf where C'(u) vanishes)
__device__ __forceinline__ double disc_excess(const Q16 &q, bool end, const double n[3], double u)
{
    const double *p = q.v;
    const double v = 1.0 - u;
    const double b0 = v * v * v, b1 = 3.0 * u * v * v, b2 = 3.0 * u * u * v, b3 = u * u * u;
    const double e0 = v * v, e1 = 2.0 * u * v, e2 = u * u;
    double C[4], D[3];
#pragma unroll
    for (int k = 0; k < 4; ++k) C[k] = b0 * p[k] + b1 * p[4 + k] + b2 * p[8 + k] + b3 * p[12 + k];
#pragma unroll
    for (int k = 0; k < 3; ++k)
        D[k] = e0 * (p[4 + k] - p[k]) + e1 * (p[8 + k] - p[4 + k]) + e2 * (p[12 + k] - p[8 + k]);
    const double dl2 = d3(D[0], D[1], D[2], D[0], D[1], D[2]);
    if (!(dl2 > 0.0)) return -INFINITY;
    const double cx = D[1] * n[2] - D[2] * n[1], cy = D[2] * n[0] - D[0] * n[2], cz = D[0] * n[1] - D[1] * n[0];
    const double s = sqrt(d3(cx, cy, cz, cx, cy, cz) / dl2);
    const double along = end ? d3(p[12] - C[0], p[13] - C[1], p[14] - C[2], n[0], n[1], n[2])
                             : d3(C[0] - p[0], C[1] - p[1], C[2] - p[2], n[0], n[1], n[2]);
    return C[3] * s - along;
}

constexpr int kSamples = 105;

// the k-th search parameter, increasing in k (see the file comment)
__device__ __forceinline__ double sample_u(int k)
{
    if (k <= 0) return 0.0;
    if (k <= 20) return ldexp(1.0, -45 + 2 * (k - 1));            // 2^-45 .. 2^-7
    if (k <= 83) return (double)(k - 20) / 64.0;                  // 1/64 .. 63/64
    if (k <= 103) return 1.0 - ldexp(1.0, -7 - 2 * (k - 84));      // 1 - 2^-7 .. 1 - 2^-45
    return 1.0;
}

// golden-section search in the bracket of the best sample (number kb)
__device__ double golden_excess(const Q16 &q, bool end, const double n[3], int kb, double best)
{
    constexpr double g = 0.38196601125010515;
    double a = sample_u(kb - 1), b = sample_u(kb + 1 < kSamples ? kb + 1 : kSamples - 1);
    double x1 = a + g * (b - a), x2 = b - g * (b - a);
    double f1 = disc_excess(q, end, n, x1), f2 = disc_excess(q, end, n, x2);
    for (int it = 0; it < 60; ++it) {
        if (f1 > f2) { b = x2; x2 = x1; f2 = f1; x1 = a + g * (b - a); f1 = disc_excess(q, end, n, x1); }
        else         { a = x1; x1 = x2; f1 = f2; x2 = b - g * (b - a); f2 = disc_excess(q, end, n, x2); }
    }
    return fmax(best, fmax(f1, f2));
}

__device__ double largest_excess(const Q16 &q, bool end)
{
    double n[3];
    cap_normal(q, end, n);
    double best = -INFINITY;
    int kb = 0;
    for (int k = 0; k < kSamples; ++k) {
        const double h = disc_excess(q, end, n, sample_u(k));
        if (h > best) { best = h; kb = k; }
    }
    return golden_excess(q, end, n, kb, best);
}

__device__ __forceinline__ double extent_of(const Q16 &q)
{
    const double *p = q.v;
    const double rmax = fmax(fmax(fabs(p[3]), fabs(p[7])), fmax(fabs(p[11]), fabs(p[15])));
    const double ax = p[12] - p[0], ay = p[13] - p[1], az = p[14] - p[2];
    return sqrt(d3(ax, ay, az, ax, ay, az)) + rmax;
}

__device__ __forceinline__ bool finite_fiber(const Q16 &q)
{
    bool ok = true;
#pragma unroll
    for (int k = 0; k < 16; ++k) ok = ok && isfinite(q.v[k]);
    return ok;
}

constexpr int kThickBits = 3 << 5;              // mask bits of the two ends

__device__ __forceinline__ void halve(Q16 &q, bool right)
{
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const double a = q.v[c], b = q.v[4 + c], d = q.v[8 + c], e = q.v[12 + c];
        const double m01 = (a + b) * 0.5, m12 = (b + d) * 0.5, m23 = (d + e) * 0.5;
        const double m012 = (m01 + m12) * 0.5, m123 = (m12 + m23) * 0.5;
        const double s = (m012 + m123) * 0.5;
        q.v[c] = right ? s : a;
        q.v[4 + c] = right ? m123 : m01;
        q.v[8 + c] = right ? m23 : m012;
        q.v[12 + c] = right ? e : s;
    }
}

// The fiber run backwards: its end becomes the start.
__device__ __forceinline__ void turn(Q16 &q)
{
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const double a = q.v[c], b = q.v[4 + c];
        q.v[c] = q.v[12 + c];
        q.v[4 + c] = q.v[8 + c];
        q.v[8 + c] = b;
        q.v[12 + c] = a;
    }
}

// Bounds on the excess that need no search. With d_k the edges of the
// control polygon, c the chord, N the start tangent d_1 (not normalised),
// a_k = <p_k - p0, N>, x_k = |d_k x N|, m = min <d_k, c> and r the largest
// radius value:
//   <C(u) - p0, N> = u A(u),  A >= A0 = min(3 a_1, 3/2 a_2, a_3)
//   |C'(u)/3 x N|  <= u max(2 x_2, x_3)        (x_1 = 0)
//   |C'(u)/3|      >= m / |c|
// so the excess r |C' x N| / |C'| - <C - p0, N> over the start plane is at
// most 0 for every u when r max(2 x_2, x_3) |c| <= m A0, with A0 and m
// positive (squared here, so that no root is taken; 1e-6 covers the
// rounding). Where the start tangent is negligible (the normal is then
// another edge, and x_1 does not vanish) nothing is claimed; a comparison
// with NaN claims nothing.
// The products are of eighth degree in the coordinates: bounds_hold keeps them
// from overflowing, and where the right side's factors are so small that its
// square may lose bits to underflow (and the left side may be 0) nothing is
// claimed.
constexpr double kLeast = 0x1p-500;

__device__ __forceinline__ bool behind_start(const Q16 &q)
{
    const double *p = q.v;
    double d[3][3], c[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
#pragma unroll
        for (int j = 0; j < 3; ++j) d[j][k] = p[4 * (j + 1) + k] - p[4 * j + k];
        c[k] = p[12 + k] - p[k];
    }
    const double cc = d3(c[0], c[1], c[2], c[0], c[1], c[2]);
    const double m = fmin(d3(d[0][0], d[0][1], d[0][2], c[0], c[1], c[2]),
                          fmin(d3(d[1][0], d[1][1], d[1][2], c[0], c[1], c[2]),
                               d3(d[2][0], d[2][1], d[2][2], c[0], c[1], c[2])));
    const double r = fmax(fmax(p[3], p[7]), fmax(fmax(p[11], p[15]), 0.0));
    const double *n = d[0];
    const double nn = d3(n[0], n[1], n[2], n[0], n[1], n[2]);
    const double b2 = nn + d3(d[1][0], d[1][1], d[1][2], n[0], n[1], n[2]);
    const double b3 = d3(c[0], c[1], c[2], n[0], n[1], n[2]);
    const double A0 = fmin(3.0 * nn, fmin(1.5 * b2, b3));
    auto cross2 = [&](const double *v) {
        const double x = v[1] * n[2] - v[2] * n[1], y = v[2] * n[0] - v[0] * n[2], z = v[0] * n[1] - v[1] * n[0];
        return d3(x, y, z, x, y, z);
    };
    const double x2 = fmax(4.0 * cross2(d[1]), cross2(d[2]));
    const double rhs = m * A0;
    return nn > 0x1p-40 * cc && A0 > 0.0 && rhs >= kLeast && r * r * x2 * cc <= (rhs * rhs) * (1.0 - 1e-6);
}

// The same for a later part of the curve (control points q) and the plane
// through p0 normal to n (not normalised): the discs stay behind it when
// r min(1, max |d_k x n| |c| / (m |n|)) <= min <q_k - p0, n> / |n|.
__device__ __forceinline__ bool part_behind(const Q16 &q, const double *p0, const double *n)
{
    const double *p = q.v;
    double c[3], x2 = 0.0, m = INFINITY, a = INFINITY;
#pragma unroll
    for (int k = 0; k < 3; ++k) c[k] = p[12 + k] - p[k];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const double e0 = p[4 * j + 4] - p[4 * j], e1 = p[4 * j + 5] - p[4 * j + 1], e2 = p[4 * j + 6] - p[4 * j + 2];
        const double x = e1 * n[2] - e2 * n[1], y = e2 * n[0] - e0 * n[2], z = e0 * n[1] - e1 * n[0];
        x2 = fmax(x2, d3(x, y, z, x, y, z));
        m = fmin(m, d3(e0, e1, e2, c[0], c[1], c[2]));
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
        a = fmin(a, d3(p[4 * j] - p0[0], p[4 * j + 1] - p0[1], p[4 * j + 2] - p0[2], n[0], n[1], n[2]));
    const double r = fmax(fmax(p[3], p[7]), fmax(fmax(p[11], p[15]), 0.0));
    const double cc = d3(c[0], c[1], c[2], c[0], c[1], c[2]), nn = d3(n[0], n[1], n[2], n[0], n[1], n[2]);
    const double room = a * a * (1.0 - 1e-6);
    return a >= kLeast && (r * r * nn <= room || (a * m >= kLeast && r * r * x2 * cc <= room * (m * m)));
}

// The excess as the search computes it is off by its rounding, up to 2^-49
// of the coordinates: the bounds stand in for the search only where that is
// below half the threshold of 1e-9 of the extent, and only for chords between
// 2^-40 and 2^64, so that products of eighth degree are finite and (but for
// what cancels) far above the subnormals. Without that, both sides of a bound
// could be 0 (extents below 2e-41) or infinite (near the largest float32), and
// thick ends passed as clear.
__device__ __forceinline__ bool bounds_hold(const Q16 &q)
{
    const double *p = q.v;
    constexpr double k = 0x1p-48 * 1e9;
    double M = 0x1p-40 / k;
#pragma unroll
    for (int j = 0; j < 16; ++j)
        if ((j & 3) != 3) M = fmax(M, fabs(p[j]));
    const double ax = p[12] - p[0], ay = p[13] - p[1], az = p[14] - p[2];
    const double cc = d3(ax, ay, az, ax, ay, az);
    M *= k;
    return cc > M * M && cc <= 0x1p128;
}

// The ends (bit 5 start, bit 6 end) at which the bounds show that no disc
// reaches over the cap plane.
__device__ __forceinline__ int ends_clear(const Q16 &q)
{
    if (!bounds_hold(q)) return 0;
    Q16 b = q;
    turn(b);
    return (behind_start(q) ? 32 : 0) | (behind_start(b) ? 64 : 0);
}

// The start of a fiber that fails behind_start as a whole, looked at closer:
// its second half and second quarter by part_behind, the rest again. (One
// more step settles next to nothing: measured on the synthetic tables.)
__device__ __forceinline__ bool behind_start_in_parts(const Q16 &q)
{
    const double n[3] = {q.v[4] - q.v[0], q.v[5] - q.v[1], q.v[6] - q.v[2]};
    const double c[3] = {q.v[12] - q.v[0], q.v[13] - q.v[1], q.v[14] - q.v[2]};
    if (!(d3(n[0], n[1], n[2], n[0], n[1], n[2]) > 0x1p-40 * d3(c[0], c[1], c[2], c[0], c[1], c[2])))
        return false;                           // the cap plane is not normal to n
    Q16 near = q;
    for (int j = 0; j < 2; ++j) {
        Q16 far = near;
        halve(far, true);
        if (!part_behind(far, q.v, n)) return false;
        halve(near, false);
        if (behind_start(near)) return true;
    }
    return false;
}

// The ends among `want` (bits 5 and 6: ends that ends_clear leaves open) of a
// finite fiber, looked at by one lane: `found` are thick, `open` need the
// whole search. Besides the bounds, the samples that usually show a thick end
// are tried: parameters in geometric steps from that end. ANY: one thick end
// is enough.
struct Ends {
    int found, open;
};

template <bool ANY>
__device__ Ends quick_ends(const Q16 &q, int want)
{
    const double lim = 1e-9 * extent_of(q);
    Ends r{0, 0};
    const bool bounds = bounds_hold(q);
    Q16 b = q;
    for (int e = 0; e < 2; ++e) {
        if ((want & (32 << e)) && !(ANY && r.found) && !(bounds && behind_start_in_parts(b))) {
            double n[3];
            cap_normal(q, e != 0, n);
            bool over = false;
            for (int j = 0; j < 12 && !over; ++j) {
                // 1/2, 1/4, .., 1/64, then 2^-7, 2^-9, .., 2^-17 from the end
                const double w = j < 6 ? ldexp(1.0, -1 - j) : ldexp(1.0, -7 - 2 * (j - 6));
                over = disc_excess(q, e != 0, n, e ? 1.0 - w : w) > lim;
            }
            if (over) r.found |= 32 << e;
            else r.open |= 32 << e;
        }
        turn(b);
    }
    if (ANY && r.found) r.open = 0;
    return r;
}

// Whether the search bracket at the start itself, [0, 2^-45], is settled
// without the golden-section search: there the excess is at most
// r u max(2 x_2, x_3) / (|N| |C'/3|) with |C'/3| >= |d_1| / 2.
__device__ __forceinline__ bool start_bracket_flat(const Q16 &q, double lim)
{
    const double *p = q.v;
    const double n[3] = {p[4] - p[0], p[5] - p[1], p[6] - p[2]};
    const double nn = d3(n[0], n[1], n[2], n[0], n[1], n[2]);
    double x2 = 0.0, dd = nn;
#pragma unroll
    for (int j = 1; j < 3; ++j) {
        const double e0 = p[4 * j + 4] - p[4 * j], e1 = p[4 * j + 5] - p[4 * j + 1], e2 = p[4 * j + 6] - p[4 * j + 2];
        const double x = e1 * n[2] - e2 * n[1], y = e2 * n[0] - e0 * n[2], z = e0 * n[1] - e1 * n[0];
        x2 = fmax(x2, 4.0 * d3(x, y, z, x, y, z));
        dd = fmax(dd, d3(e0, e1, e2, e0, e1, e2));
    }
    const double ax = p[12] - p[0], ay = p[13] - p[1], az = p[14] - p[2];
    const double r = fmax(fmax(fabs(p[3]), fabs(p[7])), fmax(fabs(p[11]), fabs(p[15])));
    const double rhs = 0.25 * lim * nn;
    return nn > 0x1p-40 * d3(ax, ay, az, ax, ay, az) && nn * 0x1p80 > dd && r * r * x2 * 0x1p-88 <= rhs * rhs;
}

// The thick ends among `open`, by the whole search of largest_excess shared
// by the kGroup lanes of a group, which hold the same fiber (`sub`: the lane's
// place in its group). The search stops once a sample is over the threshold
// (ANY: at the first thick end). A lane searching alone ran 105 samples and
// 62 golden-section points one after another, with most of its wave idle.
constexpr int kGroup = 8;

template <bool ANY>
__device__ int search_ends(const Q16 &q, int open, int sub)
{
    const double lim = 1e-9 * extent_of(q);
    const int base = (int)threadIdx.x & 63 & ~(kGroup - 1);
    int found = 0;
    for (int e = 0; e < 2; ++e) {
        if (!(open & (32 << e)) || (ANY && found)) continue;
        double n[3];
        cap_normal(q, e != 0, n);
        double best = -INFINITY;
        int kb = 0;
        bool over = false;
        for (int k = sub; k < kSamples + kGroup - 1 && !over; k += kGroup) {
            const double h = k < kSamples ? disc_excess(q, e != 0, n, sample_u(k)) : -INFINITY;
            if (h > best) { best = h; kb = k; }
            over = ((__ballot(h > lim) >> base) & ((1u << kGroup) - 1u)) != 0u;
        }
        if (!over) {
            // the group's best sample, the first of equal ones
            for (int m = kGroup / 2; m > 0; m >>= 1) {
                const double o = __shfl_xor(best, m);
                const int ok = __shfl_xor(kb, m);
                if (o > best || (o == best && ok < kb)) { best = o; kb = ok; }
            }
            bool flat = false;
            if (kb == (e ? kSamples - 1 : 0) && bounds_hold(q)) {
                Q16 b = q;
                if (e) turn(b);
                flat = start_bracket_flat(b, lim);
            }
            over = !flat && golden_excess(q, e != 0, n, kb, best) > lim;
        }
        if (over) found |= 32 << e;
    }
    return found;
}

// the node (level, index) of fiber i, replayed from the fiber
__device__ __forceinline__ void node_of(const float *F, int64_t fs, int64_t i, int level, uint32_t index, Q16 &q)
{
    load_fiber(F, fs, i, q);
    for (int l = level - 1; l >= 0; --l) halve(q, ((index >> l) & 1u) != 0u);
}

constexpr int kBlock = 256;                     // fibers per block of k_validate

// One lane per fiber decides the inequalities and the ends that the bounds
// settle; fibers with other ends go to a list in LDS, looked at by
// neighbouring lanes, and those that need it to a second one, searched by
// groups of lanes. Bound by memory where most ends are clear (68 bytes a
// fiber): 800,000 hair segments, 5 % of them hooked, take 24 us (2.3 TB/s)
// and took 1317 us with every end searched by its own lane. The excesses
// themselves (EXCESS) need every search, one lane per end.
template <bool EXCESS>
__global__ __launch_bounds__(kBlock) void k_validate(const float *F, int64_t fs, int64_t n, int32_t *mask,
                                                     float *excess)
{
    constexpr int kOwn = EXCESS ? kBlock / 2 : kBlock;       // fibers of a block
    __shared__ int s_mask[kOwn], s_queue[kBlock], s_full[kBlock], s_n[2];
    const int lane = (int)threadIdx.x;
    const int64_t first = (int64_t)blockIdx.x * kOwn, i = first + lane;
    const bool own = lane < kOwn && i < n;
    if (lane < 2) s_n[lane] = 0;
    __syncthreads();
    if (own) {
        Q16 q;
        load_fiber(F, fs, i, q);
        if (!finite_fiber(q)) {
            s_mask[lane] = 1 << 7;
            if (EXCESS) excess[2 * i] = excess[2 * i + 1] = __builtin_nanf("");
        } else {
            s_mask[lane] = constraint_bits(q);
            const int open = EXCESS ? kThickBits : kThickBits & ~ends_clear(q);
            if (EXCESS) {
                const int at = atomicAdd(&s_n[0], 2);
                s_queue[at] = 2 * lane;
                s_queue[at + 1] = 2 * lane + 1;
            } else if (open) {
                s_queue[atomicAdd(&s_n[0], 1)] = lane | (open << 8);
            }
        }
    }
    __syncthreads();
    for (int k = lane; k < s_n[0]; k += kBlock) {
        Q16 q;
        if (EXCESS) {
            const int l = s_queue[k] >> 1, e = s_queue[k] & 1;
            load_fiber(F, fs, first + l, q);
            const double x = largest_excess(q, e != 0) / extent_of(q);
            excess[2 * (first + l) + e] = (float)x;
            if (x > 1e-9) atomicOr(&s_mask[l], 32 << e);
        } else {
            const int l = s_queue[k] & 255;
            load_fiber(F, fs, first + l, q);
            const Ends r = quick_ends<false>(q, s_queue[k] >> 8);
            s_mask[l] |= r.found;
            if (r.open) s_full[atomicAdd(&s_n[1], 1)] = l | (r.open << 8);
        }
    }
    __syncthreads();
    if (!EXCESS) {
        for (int k = lane / kGroup; k < s_n[1]; k += kBlock / kGroup) {
            const int l = s_full[k] & 255;
            Q16 q;
            load_fiber(F, fs, first + l, q);
            const int found = search_ends<false>(q, s_full[k] >> 8, lane & (kGroup - 1));
            if ((lane & (kGroup - 1)) == 0) s_mask[l] |= found;
        }
        __syncthreads();
    }
    if (own) mask[i] = s_mask[lane];
}

// Pre-subdivision kernels: one wave per NF fibers. The nodes to decide sit on
// a stack in LDS (fiber, level, index), and the wave decides up to 64 of them
// at a time, so that a fiber with a deep tree is shared by all lanes instead
// of holding up 63 others; nodes whose decision needs a search of the
// cap-plane excess wait on a second list until they fill a wave, and those that
// need all of it on a third, where eight lanes share one. Each piece
// found sets the bit of its start (in units of 2^-max_level) in its fiber's
// bitmap, which orders the pieces whatever order they were found in.
// 131,072 degenerate curves to level 6 took 15.6 ms (count) and 27.8 ms
// (write) with one lane walking each fiber's tree by itself; now 0.8 and
// 1.3 ms.
// Bound by the latency of FP64 chains. Their registers are held to 256, for two
// waves a SIMD: without a limit the compiler took more, and 131,072 curves
// 2346 us instead of 2128 (for three waves 2181, for four 2203).
constexpr int kWave = 64;
#ifndef FIBERHIT_NODE_STACK
#define FIBERHIT_NODE_STACK 1024                // build knob: node stack entries of a wave
#endif
// The stack can fill: nodes that wait for a search come back as two halves
// whatever its height, and 64 trees ten levels deep have reached 2038 entries
// in a model of this order. What finds no room is walked by its own lane.
constexpr int kStack = FIBERHIT_NODE_STACK;
static_assert(kStack >= kWave, "the roots of a wave's fibers");
constexpr int kMapWords = (1 << kMaxSplitLevel) / 32;

template <int NF>                              // fibers a wave
struct WalkLds {
    uint32_t map[kMapWords * NF];              // word w of fiber f: map[w * NF + f]
    uint32_t stack[kStack], wait[2 * kWave], full[2 * kWave];
};

__device__ __forceinline__ uint32_t pack_node(int f, int level, uint32_t index)
{
    return (uint32_t)f | ((uint32_t)level << 6) | (index << 10);
}

__device__ __forceinline__ int lanes_below(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// What happens to a node of a finite fiber without a search: a piece (at the
// level limit), a halving (an inequality fails) or, with the inequalities
// met, a piece if both ends are clear and else a search.
enum { kPiece = 0, kHalve = 1, kSearch = 2 };

__device__ __forceinline__ int quick_decision(const Q16 &q, int level, int max_level)
{
    if (level >= max_level || !finite_fiber(q)) return kPiece;
    if (constraint_bits(q) != 0) return kHalve;
    return ends_clear(q) == kThickBits ? kPiece : kSearch;
}

template <int NF>
__device__ __forceinline__ void mark_piece(WalkLds<NF> &s, int f, int level, uint32_t index, int max_level)
{
    const uint32_t at = index << (max_level - level);
    atomicOr(&s.map[(at >> 5) * NF + f], 1u << (at & 31u));
}

// The pieces below one node, by its lane alone (where the stack is full).
template <int NF>
__device__ void walk_alone(WalkLds<NF> &s, const float *F, int64_t fs, int64_t i, int f, int level, uint32_t index,
                           int max_level)
{
    const int top = level;
    for (;;) {
        Q16 q;
        node_of(F, fs, i, level, index, q);
        int what = quick_decision(q, level, max_level);
        if (what == kSearch) {
            const int open = kThickBits & ~ends_clear(q);
            const double lim = 1e-9 * extent_of(q);
            const bool thick = (open & 32 && largest_excess(q, false) > lim) ||
                               (open & 64 && largest_excess(q, true) > lim);
            what = thick ? kHalve : kPiece;
        }
        if (what == kHalve) {
            ++level;                    // the left child
            index <<= 1;
            continue;
        }
        mark_piece(s, f, level, index, max_level);
        while (level > top && (index & 1u)) { index >>= 1; --level; }
        if (level == top) return;
        index += 1;                     // the right sibling
    }
}

// Marks the pieces of the wave's fibers first .. first + NF - 1 in the bitmaps.
// `root`: this lane's fiber is to be walked (otherwise its bitmap stays
// empty). Called by the whole wave.
template <int NF>
__device__ void walk_wave(WalkLds<NF> &s, const float *F, int64_t fs, int64_t first, int max_level, bool root)
{
    const int lane = (int)threadIdx.x;
    const int words = max_level >= 5 ? 1 << (max_level - 5) : 1;
    for (int w = lane; w < words * NF; w += kWave) s.map[w] = 0u;
    const uint64_t rm = __ballot(root);
    if (root) s.stack[lanes_below(rm)] = pack_node(lane, 0, 0u);
    int n_stack = __popcll(rm), n_wait = 0, n_full = 0;
    __syncthreads();
    while (n_stack > 0 || n_wait > 0 || n_full > 0) {
        // deepest list first once it fills a wave, so that every list stays
        // within its two waves of room
        const bool search = n_full > kWave || (n_stack == 0 && n_wait == 0);
        const bool quick = !search && (n_wait > kWave || n_stack == 0);
        int &from = search ? n_full : quick ? n_wait : n_stack;
        const int most = search ? kWave / kGroup : kWave;
        const int take = from < most ? from : most;
        from -= take;
        const int at = search ? lane / kGroup : lane;
        const bool on = at < take;
        const uint32_t node = on ? (search ? s.full : quick ? s.wait : s.stack)[from + at] : 0u;
        const int f = (int)(node & 63u), level = (int)((node >> 6) & 15u);
        const uint32_t index = (node >> 10) & ((1u << kMaxSplitLevel) - 1u);
        int what = -1, open = 0;
        if (on) {
            Q16 q;
            node_of(F, fs, first + f, level, index, q);
            if (search) {
                what = search_ends<true>(q, (int)(node >> 20) << 5, lane & (kGroup - 1)) ? kHalve : kPiece;
                if (lane & (kGroup - 1)) what = -1;
            } else if (quick) {
                const Ends r = quick_ends<true>(q, kThickBits & ~ends_clear(q));
                open = r.open;
                what = open ? kSearch : r.found ? kHalve : kPiece;
            } else {
                what = quick_decision(q, level, max_level);
            }
        }
        __syncthreads();
        if (what == kPiece) mark_piece(s, f, level, index, max_level);
        const uint64_t wm = __ballot(what == kSearch), hm = __ballot(what == kHalve);
        if (what == kSearch) {
            if (quick) s.full[n_full + lanes_below(wm)] = node | ((uint32_t)open >> 5 << 20);
            else s.wait[n_wait + lanes_below(wm)] = node;
        }
        (quick ? n_full : n_wait) += __popcll(wm);
        const int room = (kStack - n_stack) / 2, r = lanes_below(hm);
        if (what == kHalve) {
            if (r < room) {
                s.stack[n_stack + 2 * r] = pack_node(f, level + 1, 2u * index + 1u);
                s.stack[n_stack + 2 * r + 1] = pack_node(f, level + 1, 2u * index);
            } else {
                walk_alone(s, F, fs, first + f, f, level + 1, 2u * index, max_level);
                walk_alone(s, F, fs, first + f, f, level + 1, 2u * index + 1u, max_level);
            }
        }
        const int h = __popcll(hm);
        n_stack += 2 * (h < room ? h : room);
        __syncthreads();
    }
}

template <int NF>
__device__ __forceinline__ int map_count(const WalkLds<NF> &s, int f, int max_level)
{
    const int words = max_level >= 5 ? 1 << (max_level - 5) : 1;
    int c = 0;
    for (int w = 0; w < words; ++w) c += __popc(s.map[w * NF + f]);
    return c;
}

template <int NF>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(2, 8)))
void k_presplit_count(const float *F, int64_t fs, int64_t n, int max_level, int64_t *counts)
{
    __shared__ WalkLds<NF> s;
    const int lane = (int)threadIdx.x;
    const int64_t first = (int64_t)blockIdx.x * NF, i = first + lane;
    walk_wave(s, F, fs, first, max_level, lane < NF && i < n);
    if (lane >= NF) return;
    if (i < n) counts[i] = map_count(s, lane, max_level);
    else if (i == n) counts[n] = 0;     // the exclusive scan's total lands at index n
}

// The pieces are written in order, 64 at a time and one per lane, each lane
// finding its piece in the bitmaps: consecutive lanes write consecutive
// columns. A fiber with one piece is not walked again.
template <int NF>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(2, 8)))
void k_presplit_write(const float *F, int64_t fs, int64_t n, int max_level, const int64_t *offsets, int64_t n_pieces,
                      float *P, int64_t ps, int32_t *pfiber, float *pu0, float *pu1, int32_t *pmask)
{
    __shared__ WalkLds<NF> s;
    __shared__ int s_before[NF];     // pieces of the fibers before each one
    __shared__ uint16_t s_rank[4 * kWave];   // places of the waiting pieces in their fibers
    const int lane = (int)threadIdx.x;
    const int64_t first = (int64_t)blockIdx.x * NF, i = first + lane;
    const bool own = lane < NF && i < n;
    const bool single = own && offsets[i + 1] - offsets[i] == 1;
    walk_wave(s, F, fs, first, max_level, own && !single);
    if (single) s.map[lane] = 1u;
    __syncthreads();
    const int mine = own ? map_count(s, lane, max_level) : 0;
    int before = mine;                  // inclusive scan over the wave
    for (int d = 1; d < kWave; d <<= 1) {
        const int o = __shfl_up(before, d);
        if (lane >= d) before += o;
    }
    const int total = __shfl(before, kWave - 1);
    if (lane < NF) s_before[lane] = before - mine;
    __syncthreads();
    // pieces at the limit whose ends are not clear: once these fill a wave,
    // and at the end, their thick ends are looked at, the quick way first
    int n_wait = 0, n_full = 0;
    for (int at = 0; at < total || n_wait > 0 || n_full > 0;) {
        if (n_full > kWave || (at >= total && n_wait == 0)) {
            const int take = n_full < kWave / kGroup ? n_full : kWave / kGroup, g = lane / kGroup;
            n_full -= take;
            if (g < take) {
                const uint32_t node = s.full[n_full + g];
                const int f = (int)(node & 63u);
                Q16 q;
                node_of(F, fs, first + f, max_level, (node >> 10) & ((1u << kMaxSplitLevel) - 1u), q);
                const int found = search_ends<false>(q, (int)(node >> 20) << 5, lane & (kGroup - 1));
                if (found && (lane & (kGroup - 1)) == 0)
                    pmask[offsets[first + f] + s_rank[2 * kWave + n_full + g]] |= found;
            }
            __syncthreads();
            continue;
        }
        if (n_wait > kWave || at >= total) {
            const int take = n_wait < kWave ? n_wait : kWave;
            n_wait -= take;
            Ends r{0, 0};
            uint32_t node = 0u;
            int rank = 0;
            if (lane < take) {
                node = s.wait[n_wait + lane];
                rank = s_rank[n_wait + lane];
                const int f = (int)(node & 63u);
                Q16 q;
                node_of(F, fs, first + f, max_level, node >> 10, q);
                r = quick_ends<false>(q, kThickBits & ~ends_clear(q));
                if (r.found) pmask[offsets[first + f] + rank] |= r.found;
            }
            const uint64_t om = __ballot(r.open != 0);
            if (r.open) {
                const int e = n_full + lanes_below(om);
                s.full[e] = node | ((uint32_t)r.open >> 5 << 20);
                s_rank[2 * kWave + e] = (uint16_t)rank;
            }
            n_full += __popcll(om);
            __syncthreads();
            continue;
        }
        bool search = false;
        uint32_t index = 0u;
        int f = 0, r = 0;
        const int k = at + lane;
        if (k < total) {
            // the last fiber with at most k pieces before it, its piece r
            for (int d = NF / 2; d > 0; d >>= 1)
                if (s_before[f + d] <= k) f += d;
            r = k - s_before[f];
            int w = 0, c = r;
            while (c >= __popc(s.map[w * NF + f])) c -= __popc(s.map[w++ * NF + f]);
            uint32_t bits = s.map[w * NF + f];
            for (; c > 0; --c) bits &= bits - 1u;
            const int begin = 32 * w + __ffs((int)bits) - 1;
            bits &= bits - 1u;
            int end = 1 << max_level;          // the next piece's start
            if (bits) end = 32 * w + __ffs((int)bits) - 1;
            else
                for (int v = w + 1; 32 * v < end; ++v)
                    if (s.map[v * NF + f]) end = 32 * v + __ffs((int)s.map[v * NF + f]) - 1;
            const int level = max_level - (31 - __clz(end - begin));
            index = (uint32_t)begin >> (max_level - level);
            Q16 q;
            node_of(F, fs, first + f, level, index, q);
            const int64_t j = offsets[first + f] + r;
            if (j >= 0 && j < n_pieces) {
#pragma unroll
                for (int e = 0; e < 16; ++e) P[e * ps + j] = (float)q.v[e];
                const float width = ldexpf(1.0f, -level);
                pfiber[j] = (int32_t)(first + f);
                pu0[j] = (float)index * width;
                pu1[j] = (float)(index + 1u) * width;
                // a piece above the level limit is valid (or not finite)
                int m = 0;
                if (!finite_fiber(q)) {
                    m = 1 << 7;
                } else if (level >= max_level) {
                    m = constraint_bits(q);
                    search = ends_clear(q) != kThickBits;
                }
                pmask[j] = m;
            }
        }
        at += kWave;
        const uint64_t sm = __ballot(search);
        if (search) {
            const int e = n_wait + lanes_below(sm);
            s.wait[e] = pack_node(f, 0, index);
            s_rank[e] = (uint16_t)r;
        }
        n_wait += __popcll(sm);
        __syncthreads();
    }
}

// Fibers a wave: 64 fill its rounds best; up to 2^15 fibers, where that would
// leave half of the 1024 SIMDs without a wave, 16 (4,096 degenerate curves to
// level 4: 398 against 729 us; 131,072 to level 6: 3.7 against 2.7 ms).
int fibers_per_wave(int64_t n) { return n <= (1 << 15) ? 16 : 64; }

size_t scan_temp_bytes(int64_t n)
{
    size_t bytes = 0;
    if (hipcub::DeviceScan::ExclusiveSum(nullptr, bytes, (const int64_t *)nullptr, (int64_t *)nullptr,
                                         (int)(n + 1)) != hipSuccess)
        return 0;
    return bytes;
}

constexpr size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

extern "C" {

int fiber_validate(const float *fibers, int64_t fiber_stride, int64_t n_fibers, int32_t *mask_out,
                   float *excess_out, void *stream)
{
    if (n_fibers < 0 || fiber_stride < n_fibers) return FI_ERR_RANGE;
    if (n_fibers == 0) return FI_OK;
    if (!fibers || !mask_out) return FI_ERR_NULL;
    (void)hipGetLastError();
    // the excesses themselves need every search, the mask alone few
    const int own = excess_out ? kBlock / 2 : kBlock;
    hipLaunchKernelGGL(excess_out ? k_validate<true> : k_validate<false>,
                       dim3((unsigned)((n_fibers + own - 1) / own)), dim3(kBlock), 0, (hipStream_t)stream, fibers,
                       fiber_stride, n_fibers, mask_out, excess_out);
    return hipGetLastError() == hipSuccess ? FI_OK : FI_ERR_HIP;
}

size_t fiber_presplit_workspace_bytes(int64_t n_fibers)
{
    if (n_fibers < 0 || n_fibers > (int64_t)0x7ffffffe) return 0;
    return align256((size_t)(n_fibers + 1) * sizeof(int64_t)) + align256(scan_temp_bytes(n_fibers));
}

int fiber_presplit_count(const float *fibers, int64_t fiber_stride, int64_t n_fibers, int32_t max_level,
                         int64_t *offsets_out, void *workspace, size_t workspace_bytes, void *stream)
{
    if (n_fibers < 0 || fiber_stride < n_fibers || n_fibers > (int64_t)0x7ffffffe) return FI_ERR_RANGE;
    if (max_level < 0 || max_level > kMaxSplitLevel) return FI_ERR_RANGE;
    if (!offsets_out) return FI_ERR_NULL;
    if (n_fibers > 0 && !fibers) return FI_ERR_NULL;
    const size_t need = fiber_presplit_workspace_bytes(n_fibers);
    if (!workspace || ((uintptr_t)workspace & 255u) != 0u || workspace_bytes < need) return FI_ERR_WORKSPACE;
    const hipStream_t s = (hipStream_t)stream;
    int64_t *counts = (int64_t *)workspace;
    void *temp = (char *)workspace + align256((size_t)(n_fibers + 1) * sizeof(int64_t));
    size_t temp_bytes = need - align256((size_t)(n_fibers + 1) * sizeof(int64_t));
    (void)hipGetLastError();
    const int nf = fibers_per_wave(n_fibers);
    hipLaunchKernelGGL(nf == 16 ? k_presplit_count<16> : k_presplit_count<64>,
                       dim3((unsigned)((n_fibers + nf) / nf)), dim3(kWave), 0, s, fibers, fiber_stride, n_fibers,
                       max_level, counts);
    if (hipGetLastError() != hipSuccess) return FI_ERR_HIP;
    if (hipcub::DeviceScan::ExclusiveSum(temp, temp_bytes, counts, offsets_out, (int)(n_fibers + 1), s) !=
        hipSuccess)
        return FI_ERR_HIP;
    return hipGetLastError() == hipSuccess ? FI_OK : FI_ERR_HIP;
}

int fiber_presplit(const float *fibers, int64_t fiber_stride, int64_t n_fibers, int32_t max_level,
                   const int64_t *offsets, int64_t n_pieces, float *pieces_out, int64_t piece_stride,
                   int32_t *piece_fiber, float *piece_u0, float *piece_u1, int32_t *piece_mask, void *stream)
{
    if (n_fibers < 0 || fiber_stride < n_fibers || n_pieces < 0 || piece_stride < n_pieces) return FI_ERR_RANGE;
    if (max_level < 0 || max_level > kMaxSplitLevel) return FI_ERR_RANGE;
    if (n_fibers == 0) return FI_OK;
    if (!fibers || !offsets || !pieces_out || !piece_fiber || !piece_u0 || !piece_u1 || !piece_mask)
        return FI_ERR_NULL;
    (void)hipGetLastError();
    const int nf = fibers_per_wave(n_fibers);
    hipLaunchKernelGGL(nf == 16 ? k_presplit_write<16> : k_presplit_write<64>,
                       dim3((unsigned)((n_fibers + nf - 1) / nf)), dim3(kWave), 0, (hipStream_t)stream, fibers,
                       fiber_stride, n_fibers, max_level, offsets, n_pieces, pieces_out, piece_stride, piece_fiber,
                       piece_u0, piece_u1, piece_mask);
    return hipGetLastError() == hipSuccess ? FI_OK : FI_ERR_HIP;
}

}  // extern "C"
