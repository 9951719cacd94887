// Projected area of the P-NDF on gfx950 (section "Shadow-masking", Eq. lambda,
// Eq. area-integral, Eq. line-integral and the supplement's derivations).
//
//   P(w) = integral of D(m) max(m~ . w, 0) over the solid angle of m~,
//
// with the footprint kernel constant over each triangle (its value at the uv
// centroid).  Per triangle, after rotating about z so that w = (w_l, 0, w_z),
// w_l >= 0, the contribution is k / J times the integral of (w_l m_x / m~_z + w_z)
// over the part of the normal triangle inside the visible region V = {|m| <= 1,
// m~ . w >= 0}: the unit disk cut on the left by the semi-ellipse
// m_x = -w_z sqrt(1 - m_y^2).  V is convex.  By Stokes' theorem the area integral
// is the counter-clockwise boundary integral of F dm_y, F = w_z m_x - w_l m~_z,
// over the triangle's edges clipped to V and the pieces of V's boundary between
// them, all in closed form with A(y) = (asin y + y sqrt(1 - y^2)) / 2:
//   segment P -> Q:  w_z (Q_y - P_y)(P_x + Q_x) / 2 - w_l d_y rho^2 [A(p / rho)],
//                    d the unit direction, p the abscissa along d, rho^2 = 1 - s^2
//                    with s the line's distance to the origin;
//   circle piece:    w_z [A(y)] (m~_z = 0, m_x = sqrt(1 - y^2), y increasing);
//   ellipse piece:   -[A(y)] (F = -sqrt(1 - y^2) there, y decreasing).
// A triangle with its three vertices in V lies in V (convexity): three segments.
//
// Brute force like the paper's implementation: one wavefront per query (several in
// small batches), lanes over the included cells (two triangles each), FP64 throughout;
// the lanes' partial sums are reduced in the wave.  V lies right of the line
// m_x = -w_z (the ellipse's leftmost point), so a triangle left of it adds nothing; a
// triangle with its three vertices in V takes three segment terms at once (a cell
// whose two triangles both lie in V five: the shared diagonal once), each the
// trapezoid of its ends and a small correction (segment_short).  The others (4 % of the
// triangles of a 2048^2 power-law map, 6 % of a scratched one) wait in a per-wave LDS
// queue until 21 of them fill a round with one edge per lane: a lane's clipping would
// otherwise stall its wave, and one edge's code instead of three in a row is a third
// of the instructions to fetch (11000 to 4000) and of the registers (no clipping state in scratch
// memory).  The pieces of V's boundary, which few edges leave, wait once more, 64 to a
// round.  The footprint weight at a cell's centroids is a product of two factors that
// depend on its column and its row alone, formed once per query in LDS.
// Bound by FP64 vector instructions (78 % of the issue slots): 65536 queries of sigma 1
// to 8 on the 2048^2 power-law map take 1070 us and 7400 instructions per wavefront,
// against 1312 us and 10090 with arcsines for every segment, weights per cell and a
// triangle per lane in the clipping.
#include <algorithm>

#include "pndf_internal.h"

namespace pndf {
namespace {

__device__ __forceinline__ bool visible(double x, double y, double wz)
{
    return x * x + y * y <= 1.0 && (x >= 0.0 || x * x + wz * wz * y * y <= wz * wz);
}

// 1 / sqrt(x), x > 0, in FP64: the hardware estimate refined by two Newton steps
// y <- y (3/2 - x y^2 / 2) (each step squares the relative error), so the segment
// terms need no FP64 square root or division (unit direction, 1/rho, sqrt(1 - y^2)).
__device__ __forceinline__ double rsqrt_f64(double x)
{
    double y = __builtin_amdgcn_rsq(x);
    const double h = 0.5 * x;
    y = y * fma(-h * y, y, 1.5);
    y = y * fma(-h * y, y, 1.5);
    return y;
}

// 1 / x in FP64, x a normal number: the estimate and two Newton steps
__device__ __forceinline__ double rcp_f64(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    return fma(fma(-x, r, 1.0), r, r);
}

// sqrt(z) for 0 <= z <= 1 as z / sqrt(z) (exactly 0 at 0)
__device__ __forceinline__ double sqrt_unit(double z)
{
    return z > 0.0 ? z * rsqrt_f64(z) : 0.0;
}

// A(b) - A(a) with one arcsine: asin b - asin a = asin(b sqrt(1 - a^2) - a sqrt(1 - b^2))
// while the difference of the angles is within [-pi/2, pi/2], i.e. while
// sqrt(1 - a^2) sqrt(1 - b^2) + a b >= 0; else two
__device__ __forceinline__ double arc_prim_diff(double a, double b)
{
    a = fmin(1.0, fmax(-1.0, a));
    b = fmin(1.0, fmax(-1.0, b));
    const double ca = sqrt_unit(1.0 - a * a), cb = sqrt_unit(1.0 - b * b);
    const double d = ca * cb + a * b >= 0.0 ? asin(fmin(1.0, fmax(-1.0, b * ca - a * cb))) : asin(b) - asin(a);
    return 0.5 * (d + b * cb - a * ca);
}

// F dm_y along the segment P -> Q between points inside the unit disk, p and q their
// m~_z = sqrt(1 - m_x^2 - m_y^2).  With d = Q - P, l = |d|, M = d . (P + Q) / 2 (so
// that p^2 - q^2 = 2 M), E = l^2 rho^2 = l^2 - (P x Q)^2 and
// Y = 2 M^2 / (p + q) + l^2 (p + q) / 2, the angle that the segment subtends on its
// circle of radius rho has the sine z = Y l / E, and the closed form above becomes
//   d_y / 2 [w_z (P_x + Q_x) - w_l (p + q + (asin(z) / z - 1) Y / l^2)]
//     = d_y / 2 [w_z (P_x + Q_x) - w_l (p + q + Y (Y / E)^2 C(z^2))],
// C(u) = (asin(z) / z - 1) / u at u = z^2: the trapezoid rule and its correction, all
// terms of one sign, without a square root, an arcsine or a cancellation.  C is the polynomial
// of degree 8 that interpolates it at the 9 Chebyshev nodes of [0, 0.1] (from the series of
// the arcsine, in 60 decimal digits), 1.1e-16 off at most.  *ok is false beyond it (jumps of a
// scratched map), where the segment is longer than rho (the angle may then pass pi / 2)
// and where it hugs the circle: the triangle is then left to far_round.
__device__ __forceinline__ double segment_short(double px, double py, double p, double qx, double qy, double q, double wl,
                                                double wz, bool* ok)
{
    const double dx = qx - px, dy = qy - py, sx = px + qx, sy = py + qy, sp = p + q;
    const double l2 = dx * dx + dy * dy, c = dy * px - dx * py, E = l2 - c * c;
    const double M = 0.5 * (dx * sx + dy * sy);
    const double r = rcp_f64(sp * E);
    const double Y = 2.0 * M * M * (E * r) + 0.5 * l2 * sp, g = Y * (sp * r), u = g * g * l2;
    const double C[9] = {0.16666666666666677,  0.074999999999844316, 0.04464285718425845,
                         0.030381940216166695, 0.022372374707386941, 0.01734661732276873,
                         0.014066980567147705, 0.010577825252300511, 0.014580819628997006};
    double f = C[8];
#pragma unroll
    for (int i = 7; i >= 0; --i) f = fma(f, u, C[i]);
    *ok = (sp > 1e-3 && E > 1e-4 * l2 && l2 * l2 <= E && u <= 0.1) || l2 == 0.0;
    const double v = 0.5 * dy * (wz * sx - wl * (sp + Y * (g * g) * f));
    return l2 == 0.0 ? 0.0 : v;
}

// F dm_y along the segment P -> Q
__device__ inline double segment_int(double px, double py, double qx, double qy, double wl, double wz)
{
    double dx = qx - px, dy = qy - py;
    const double l2 = dx * dx + dy * dy;
    if (l2 == 0.0) return 0.0;
    const double lin = 0.5 * wz * dy * (px + qx);
    const double il = rsqrt_f64(l2);
    dx *= il;
    dy *= il;
    const double s = dy * px - dx * py;
    const double rho2 = 1.0 - s * s;
    if (rho2 <= 0.0) return lin;
    const double ir = rsqrt_f64(rho2);
    return lin - wl * dy * rho2 * arc_prim_diff((dx * px + dy * py) * ir, (dx * qx + dy * qy) * ir);
}

// place of a point of V's boundary on its counter-clockwise loop from (0, -1):
// right semicircle -> [0, 2], left semi-ellipse -> [2, 4].  On the semicircle
// means x >= 0 and on the unit circle (at w_z = 0 the semi-ellipse degenerates to
// the segment x = 0 inside the disk).
__device__ __forceinline__ double loop_pos(double x, double y)
{
    y = fmin(1.0, fmax(-1.0, y));
    return (x >= 0.0 && x * x + y * y >= 1.0 - 1e-9) ? 1.0 + y : 3.0 - y;
}

// F dm_y along V's boundary from loop place a to b (a <= b < a + 4)
__device__ inline double boundary_int(double a, double b, double wz)
{
    double sum = 0.0;
    for (int guard = 0; guard < 5 && a < b; ++guard) {
        const double half = floor(a * 0.5);
        const double stop = fmin(b, 2.0 * half + 2.0);
        const double ya = a - 2.0 * half, yb = stop - 2.0 * half;  // in [0, 2]
        const bool circ = ((int)half & 1) == 0;  // circle: y = place - 1, ellipse: y = 1 - place
        sum += (circ ? wz : 1.0) * arc_prim_diff(circ ? ya - 1.0 : 1.0 - yb, circ ? yb - 1.0 : 1.0 - ya);
        a = stop;
    }
    return sum;
}

__device__ __forceinline__ void cswap(double& a, double& b)
{
    const double lo = fmin(a, b), hi = fmax(a, b);
    a = lo;
    b = hi;
}

// parameter interval [t0, t1] of the segment P + t D (t in [0, 1]) inside V;
// false if empty.  The candidates: the ends, every meeting with the whole ellipse
// x^2 + wz^2 y^2 = wz^2 and, with CIRCLE (some end lies outside the unit disk), with
// the unit circle (V's boundary crossings are among them, the others only split the
// segment), and the line x = 0, the ellipse's limit as wz -> 0 (its discriminant is
// then a difference of equal products and may round below 0).  Unused slots repeat
// t = 1.  Sorted by a fixed network (registers only); V convex: the visible pieces
// between consecutive candidates form one interval.
template <bool CIRCLE>
__device__ __forceinline__ bool clip_edge(double px, double py, double dx, double dy, double wz, double* t0, double* t1)
{
    constexpr int N = CIRCLE ? 7 : 5;
    double ts[N];
    ts[0] = 0.0;
#pragma unroll
    for (int i = 1; i < N; ++i) ts[i] = 1.0;
#pragma unroll
    for (int curve = 0; curve < (CIRCLE ? 2 : 1); ++curve) {
        const double ey = curve == 1 ? 1.0 : wz * wz, rhs = curve == 1 ? 1.0 : wz * wz;
        const double qa = dx * dx + ey * dy * dy;
        const double qb = 2.0 * (px * dx + ey * py * dy);
        const double qc = px * px + ey * py * py - rhs;
        const double disc = qb * qb - 4.0 * qa * qc;
        if (qa > 0.0 && disc >= 0.0) {
            const double sq = disc > 1e-200 ? disc * rsqrt_f64(disc) : 0.0, inv = 0.5 * rcp_f64(qa);
            const double ra = (-qb - sq) * inv, rb = (-qb + sq) * inv;
            ts[2 + 2 * curve] = (ra > 0.0 && ra < 1.0) ? ra : 1.0;
            ts[3 + 2 * curve] = (rb > 0.0 && rb < 1.0) ? rb : 1.0;
        }
    }
    if (dx != 0.0) {
        const double t = -px * rcp_f64(dx);
        ts[N - 1] = (t > 0.0 && t < 1.0) ? t : 1.0;
    }
    if constexpr (CIRCLE) {
        // sorting network for 7 values
        cswap(ts[0], ts[6]); cswap(ts[2], ts[3]); cswap(ts[4], ts[5]);
        cswap(ts[0], ts[2]); cswap(ts[1], ts[4]); cswap(ts[3], ts[6]);
        cswap(ts[0], ts[1]); cswap(ts[2], ts[5]); cswap(ts[3], ts[4]);
        cswap(ts[1], ts[2]); cswap(ts[4], ts[6]);
        cswap(ts[2], ts[3]); cswap(ts[4], ts[5]);
        cswap(ts[1], ts[2]); cswap(ts[3], ts[4]); cswap(ts[5], ts[6]);
    } else {
        // 0 is the least and 1 the greatest already: the three between them
        cswap(ts[2], ts[3]);
        cswap(ts[3], ts[4]);
        cswap(ts[2], ts[3]);
        ts[1] = ts[2]; ts[2] = ts[3]; ts[3] = ts[4]; ts[4] = 1.0;
    }
    double lo = 2.0, hi = -1.0;
#pragma unroll
    for (int i = 0; i + 1 < N; ++i) {
        if (!(ts[i + 1] > ts[i])) continue;
        const double tm = 0.5 * (ts[i] + ts[i + 1]);
        if (visible(px + tm * dx, py + tm * dy, wz)) {
            lo = fmin(lo, ts[i]);
            hi = fmax(hi, ts[i + 1]);
        }
    }
    *t0 = lo;
    *t1 = hi;
    return hi > lo;
}

// counter-clockwise vertex order
__device__ __forceinline__ void orient_ccw(double v[6])
{
    const double a2 = (v[2] - v[0]) * (v[5] - v[1]) - (v[3] - v[1]) * (v[4] - v[0]);
    if (a2 < 0.0) {
        double t = v[2]; v[2] = v[4]; v[4] = t;
        t = v[3]; v[3] = v[5]; v[5] = t;
    }
}

// A triangle of cell (i, j) and its weight k / J: normals in the canonical frame.
__device__ __forceinline__ void cell_triangle(const HierDev& H, int i, int j, int half, double c, double sn,
                                              double r[6])
{
    const int wdt = H.n + 1;
    const float2* p = H.nrm + (int64_t)j * wdt + i;
    const float2 n1 = p[1], n2 = p[wdt];
    const float2 nc = half ? p[wdt + 1] : p[0];
    double v[6];
    if ((H.deg[(int64_t)j * H.n + i] >> half) & 1u) {
        eqtri_f64(0.5 * ((double)n1.x + (double)n2.x), 0.5 * ((double)n1.y + (double)n2.y), (double)H.rho, v);
    } else if (half == 0) {
        v[0] = nc.x; v[1] = nc.y; v[2] = n1.x; v[3] = n1.y; v[4] = n2.x; v[5] = n2.y;
    } else {
        v[0] = nc.x; v[1] = nc.y; v[2] = n2.x; v[3] = n2.y; v[4] = n1.x; v[5] = n1.y;
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        r[2 * k] = c * v[2 * k] + sn * v[2 * k + 1];
        r[2 * k + 1] = -sn * v[2 * k] + c * v[2 * k + 1];
    }
    orient_ccw(r);
}

constexpr int kClipRound = 21;  // triangles of a round: three lanes each
constexpr int kClipCap = 168;    // queued triangles per wave (a step adds at most 128 to two rests)
constexpr int kArcCap = 128;     // queued boundary pieces per wave (a round adds at most 63)

// Triangles that need clipping from the front, those within V with an edge beyond
// segment_short's range from the back; pieces of V's boundary.
struct ClipQueue {
    uint32_t cell[kClipCap];
    double w[kClipCap];
    double arc_a[kArcCap], arc_b[kArcCap], arc_w[kArcCap];
};

// corner `e` of a triangle, its successor at e = 1 .. 3
__device__ __forceinline__ void edge_of(const double v[6], int e, double* px, double* py, double* qx, double* qy)
{
    *px = e == 0 ? v[0] : (e == 1 ? v[2] : v[4]);
    *py = e == 0 ? v[1] : (e == 1 ? v[3] : v[5]);
    *qx = e == 0 ? v[2] : (e == 1 ? v[4] : v[0]);
    *qy = e == 0 ? v[3] : (e == 1 ? v[5] : v[1]);
}

// The queued triangles [at, at + cnt), all within V, an edge per lane.
__device__ __forceinline__ double far_round(const HierDev& H, const ClipQueue& Q, int at, int cnt, int lane, double c, double sn,
                                            double wl, double wz)
{
    const int t = (lane * 43) >> 7, e = lane - 3 * t;  // lane / 3 up to 63
    if (t >= cnt) return 0.0;
    const uint32_t id = Q.cell[at + t];
    double v[6], px, py, qx, qy;
    cell_triangle(H, (int)(id & 0x1fffu), (int)((id >> 13) & 0x1fffu), (int)(id >> 26), c, sn, v);
    edge_of(v, e, &px, &py, &qx, &qy);
    return Q.w[at + t] * segment_int(px, py, qx, qy, wl, wz);
}

// Integral of (w_l m_x / m~_z + w_z) over V within the queued triangles [at, at + cnt),
// an edge per lane: the edge clipped to V adds its segment, and where it does not end
// on the next edge's start the piece of V's boundary between them is queued (at *na), as
// few edges have one.  Returns this lane's share.
__device__ __forceinline__ double clip_round(const HierDev& H, ClipQueue& Q, int at, int cnt, int lane, double c, double sn,
                                             double wl, double wz, int* na)
{
    const int t = (lane * 43) >> 7, e = lane - 3 * t;  // lane / 3 up to 63
    const bool on = t < cnt;
    const uint32_t id = Q.cell[at + (on ? t : 0)];
    const double w = Q.w[at + (on ? t : 0)];
    double v[6], px, py, qx, qy;
    cell_triangle(H, (int)(id & 0x1fffu), (int)((id >> 13) & 0x1fffu), (int)(id >> 26), c, sn, v);
    edge_of(v, e, &px, &py, &qx, &qy);
    double t0 = 0.0, t1 = 0.0;
    // (the same for the wave: normal maps seldom reach the unit circle)
    const bool circle = __ballot(px * px + py * py > 1.0) != 0ull;
    const bool in = on && (circle ? clip_edge<true>(px, py, qx - px, qy - py, wz, &t0, &t1)
                                  : clip_edge<false>(px, py, qx - px, qy - py, wz, &t0, &t1));
    const double ex = t0 == 0.0 ? px : px + t0 * (qx - px), ey = t0 == 0.0 ? py : py + t0 * (qy - py);
    const double xx = t1 == 1.0 ? qx : px + t1 * (qx - px), xy = t1 == 1.0 ? qy : py + t1 * (qy - py);
    const uint32_t ins = (uint32_t)(__ballot(in) >> (3 * t)) & 7u;
    // the next edge in V
    int f = e == 2 ? 0 : e + 1;
    if (!((ins >> f) & 1u)) f = f == 2 ? 0 : f + 1;
    if (!((ins >> f) & 1u)) f = e;
    const double fx = __shfl(ex, 3 * t + f), fy = __shfl(ey, 3 * t + f);
    double sum = 0.0, a = 0.0, b = 0.0;
    bool arc = false;
    if (in) {
        sum = w * segment_int(ex, ey, xx, xy, wl, wz);
        arc = !(xx == fx && xy == fy);  // else it meets the next edge at a vertex
        a = loop_pos(xx, xy);
        b = loop_pos(fx, fy);
        if (b < a) b += 4.0;
    } else if (on && ins == 0u && e == 0) {
        // V inside the triangle (it holds the origin, a point of V) or disjoint
        arc = v[2] * v[5] - v[3] * v[4] >= 0.0 && v[4] * v[1] - v[5] * v[0] >= 0.0 && v[0] * v[3] - v[1] * v[2] >= 0.0;
        b = 4.0;
    }
    const uint64_t m = __ballot(arc);
    if (arc) {
        const int k = *na + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        Q.arc_a[k] = a;
        Q.arc_b[k] = b;
        Q.arc_w[k] = w;
    }
    *na += (int)__popcll(m);
    return sum;
}

constexpr int kAxisCells = 320;  // columns plus rows whose footprint factors fit the LDS table

// Footprint factor of one axis at the centroid of a cell's lower (h = 0) or upper
// triangle, summed over the included images (the product of both axes' factors and
// norm is the weight of hit_weight).
template <int KER>
__device__ inline double axis_weight(const QuerySetup& q, int axis, int start, int h, int logn)
{
    const double uoff = h ? 1.0 - 1.0 / 3.0 : 1.0 / 3.0;
    const float x = axis ? q.y : q.x;
    const int clo = axis ? q.cylo : q.cxlo, chi = axis ? q.cyhi : q.cxhi;
    if constexpr (KER == PNDF_KERNEL_BOX) {
        return box_axis(x, axis ? q.ry : q.rx, start, 1, uoff, clo, chi, logn);
    } else {
        const double k = axis ? q.ky : q.kx, base = (double)start + uoff - (double)x;
        const int p0 = ceil_div_pow2(clo - start, logn), p1 = floor_div_pow2(chi - start, logn);
        double g = 0.0;
        for (int p = p0; p <= p1; ++p) {
            const double d = base + (double)p * (double)(1 << logn);
            g += exp2(-(d * d * k));
        }
        return g;
    }
}

// One wavefront per workgroup in large batches: queries differ in cost by up to 64x
// (the support grows with sigma^2), and a workgroup of four queries held its slot until
// its slowest one ended (one per workgroup: -18 %).  In small batches W wavefronts share
// a query's cells.  Three wavefronts per SIMD: at four (128 registers) the segments
// spill and the same work takes 1316 us, at two 1350 us.
template <int KER, int W>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(3, 8))) void k_projected_area(HierDev H, ProjArgs a)
{
    __shared__ ClipQueue queues[W];
    __shared__ double axis[KER == PNDF_KERNEL_DISK ? 1 : 2 * kAxisCells];
    __shared__ double sums[W];
    if ((int64_t)blockIdx.x >= a.nq) return;
    const int64_t qi = a.order ? (int64_t)a.order[blockIdx.x] : (int64_t)blockIdx.x;
    const int lane = threadIdx.x & 63, wave = W == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    ClipQueue& Q = queues[wave];
    const pndf_query qr = a.q[qi];
    const QuerySetup q = setup_wave<KER>(qr, a.s2r, 0.f, H);
    const double wx = qr.hx, wy = qr.hy;
    const double wl2 = wx * wx + wy * wy;
    if (!q.valid || !(wl2 <= 1.0)) {
        if (threadIdx.x == 0) {
            a.P[qi] = __int_as_float(0x7fc00000);
            if (a.lambda) a.lambda[qi] = __int_as_float(0x7fc00000);
        }
        return;
    }
    const double wz = sqrt(1.0 - wl2), wl = sqrt(wl2);
    const double c = wl > 0.0 ? wx / wl : 1.0, sn = wl > 0.0 ? wy / wl : 0.0;
    const int n = H.n, msk = n - 1;
    const int spanx = q.cxhi - q.cxlo + 1, spany = q.cyhi - q.cylo + 1;
    const int nx = spanx >= n ? n : spanx, ny = spany >= n ? n : spany;
    const int total = nx * ny;
    const bool table = KER != PNDF_KERNEL_DISK && nx + ny <= kAxisCells;
    if (table) {
        // x factors (times the norm) of the lower and the upper centroids, then y's
        for (int i = threadIdx.x; i < 2 * (nx + ny); i += 64 * W) {
            const int ax = i >= 2 * nx, k = ax ? i - 2 * nx : i, m = ax ? ny : nx, h = k >= m, cell = h ? k - m : k;
            const int at = ax ? (spany >= n ? cell : ((q.cylo + cell) & msk)) : (spanx >= n ? cell : ((q.cxlo + cell) & msk));
            axis[i] = axis_weight<KER>(q, ax, at, h, H.logn) * (ax ? 1.0 : q.norm);
        }
        if (W == 1) wave_sync();
        else __syncthreads();
    }
    double acc = 0.0;
    int qn = 0, nf = 0, na = 0;  // queued triangles (front, back) and boundary pieces (wave-uniform)
    // this lane's cell, column ca and row cb of the included ones, and its stride
    constexpr int step = 64 * W;
    int ca = (wave * 64 + lane) % nx, cb = (wave * 64 + lane) / nx;
    const int da = step % nx, db = step / nx;
    for (int base = wave * 64; base < total; base += step) {
        uint32_t clip = 0, far = 0;  // bit h: this lane's triangle h needs clipping, the long form
        double kw[2] = {0.0, 0.0};
        uint32_t cell = 0;
        const int idx = base + lane;
        if (idx < total) {
            const int i = spanx >= n ? ca : ((q.cxlo + ca) & msk);
            const int j = spany >= n ? cb : ((q.cylo + cb) & msk);
            cell = (uint32_t)i | ((uint32_t)j << 13);
            const float2 dd = H.det[(int64_t)j * n + i];
            const uint32_t deg = H.deg[(int64_t)j * n + i] & 3u;
            // kernel at the uv centroid over the included images, divided by J
            double kh[2];
            if (table) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const double J = (double)(h ? dd.y : dd.x);
                    kh[h] = axis[h * nx + ca] * axis[2 * nx + h * ny + cb] * rcp_f64(J);
                }
            } else {
                kh[0] = hit_term<KER>(q, i, j, 0, 0, 1.0 / 3.0, 1.0 / 3.0, dd.x, H.logn);
                kh[1] = hit_term<KER>(q, i, j, 0, 1, 1.0 / 3.0, 1.0 / 3.0, dd.y, H.logn);
            }
            // lower (n0, n1, n2) and upper (n3, n2, n1) share the diagonal n1 -> n2, which the
            // upper runs backwards.  The corners are rotated once; a triangle's CCW boundary
            // integral is its orientation sign times the integral in vertex order, so with
            // both triangles inside V the diagonal's term is computed once with weight
            // s_l k_l - s_u k_u.  Both halves of a cell have the same replacement triangle: where
            // both are clamped it takes the lower one's place with both weights (1024^2,
            // patches of 16 x 16, 65536 queries of sigma 1 to 4: 375 us, 1271 when they were clipped); a
            // clamped half beside a regular one is left to clip_round.
            const int wdt = n + 1;
            const float2* p = H.nrm + (int64_t)j * wdt + i;
            const float2 nn[4] = {p[0], p[1], p[wdt], p[wdt + 1]};
            double x[4], y[4], mz[4];
            bool vis[4], left[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                x[k] = (double)nn[k].x;
                y[k] = (double)nn[k].y;
            }
            if (deg == 3u) {
                double v[6];
                eqtri_f64(0.5 * (x[1] + x[2]), 0.5 * (y[1] + y[2]), (double)H.rho, v);
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    x[k] = v[2 * k];
                    y[k] = v[2 * k + 1];
                }
                kh[0] += kh[1];
                kh[1] = 0.0;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const double u = x[k], w = y[k];
                x[k] = c * u + sn * w;
                y[k] = -sn * u + c * w;
                const double r2 = x[k] * x[k] + y[k] * y[k];
                vis[k] = visible(x[k], y[k], wz);
                left[k] = x[k] < -wz;
                mz[k] = sqrt_unit(fmax(0.0, 1.0 - r2));
            }
            const double sl = (x[1] - x[0]) * (y[2] - y[0]) - (y[1] - y[0]) * (x[2] - x[0]) < 0.0 ? -1.0 : 1.0;
            const double su = (x[2] - x[3]) * (y[1] - y[3]) - (y[2] - y[3]) * (x[1] - x[3]) < 0.0 ? -1.0 : 1.0;
            const bool lo_live = deg != 1u && kh[0] != 0.0 && !(left[0] && left[1] && left[2]);
            const bool up_live = deg != 2u && kh[1] != 0.0 && !(left[3] && left[2] && left[1]);
            const bool lo_full = lo_live && vis[0] && vis[1] && vis[2];
            const bool up_full = up_live && vis[3] && vis[2] && vis[1];
            bool lo_ok = lo_full, up_ok = up_full;
            if (lo_full || up_full) {
                // edges 0 -> 1, 2 -> 0 (lower), 3 -> 2, 1 -> 3 (upper), 1 -> 2 (both)
                constexpr int from[5] = {0, 2, 3, 1, 1}, to[5] = {1, 0, 2, 3, 2};
                double v[5];
                bool ok[5];
#pragma unroll
                for (int e = 0; e < 5; ++e) {
                    const int f = from[e], t = to[e];
                    v[e] = segment_short(x[f], y[f], mz[f], x[t], y[t], mz[t], wl, wz, &ok[e]);
                }
                lo_ok = lo_full && ok[0] && ok[1] && ok[4];
                up_ok = up_full && ok[2] && ok[3] && ok[4];
                if (lo_ok) acc += kh[0] * sl * (v[0] + v[4] + v[1]);
                if (up_ok) acc += kh[1] * su * (v[2] - v[4] + v[3]);
            }
            clip = (lo_live && !lo_full ? 1u : 0u) | (up_live && !up_full ? 2u : 0u);
            if (deg == 1u || deg == 2u) clip |= (deg == 1u ? kh[0] : kh[1]) != 0.0 ? deg : 0u;
            far = (lo_full && !lo_ok ? 1u : 0u) | (up_full && !up_ok ? 2u : 0u);
            kw[0] = kh[0];
            kw[1] = kh[1];
        }
        ca += da;
        cb += db;
        if (ca >= nx) {
            ca -= nx;
            ++cb;
        }
        // queue the triangles that need clipping (lane order)
        int tot;
        const int pos = wave_prefix_small(__popc(clip), &tot);
        int at = qn + pos;
#pragma unroll
        for (int half = 0; half < 2; ++half)
            if (clip & (1u << half)) {
                Q.cell[at] = cell | ((uint32_t)half << 26);
                Q.w[at] = kw[half];
                ++at;
            }
        qn += tot;
        if (__ballot(far != 0u) != 0ull) {
            at = kClipCap - 1 - nf - wave_prefix_small(__popc(far), &tot);
#pragma unroll
            for (int half = 0; half < 2; ++half)
                if (far & (1u << half)) {
                    Q.cell[at] = cell | ((uint32_t)half << 26);
                    Q.w[at] = kw[half];
                    --at;
                }
            nf += tot;
        }
        wave_sync();
        // full rounds, and at the end whatever is left
        const bool last = base + step >= total;
        const int least = last ? 1 : kClipRound;
        while (nf >= least) {
            const int cnt = min(nf, kClipRound);
            acc += far_round(H, Q, kClipCap - nf, cnt, lane, c, sn, wl, wz);
            nf -= cnt;
        }
        while (qn >= least || (last && na > 0)) {
            if (qn >= least) {
                const int cnt = min(qn, kClipRound);
                qn -= cnt;
                acc += clip_round(H, Q, qn, cnt, lane, c, sn, wl, wz, &na);
                wave_sync();
            }
            if (na >= 64 || (last && qn == 0)) {
                const int cnt = min(na, 64);
                na -= cnt;
                if (lane < cnt) acc += Q.arc_w[na + lane] * boundary_int(Q.arc_a[na + lane], Q.arc_b[na + lane], wz);
                wave_sync();
            }
        }
    }
    double P = wave_sum_f64(acc);
    if (W > 1) {
        if (lane == 0) sums[wave] = P;
        __syncthreads();
        P = sums[0];
        for (int w = 1; w < W; ++w) P += sums[w];
    }
    if (threadIdx.x == 0) {
        a.P[qi] = (float)P;
        if (a.lambda) a.lambda[qi] = (float)(P / wz - 1.0);
    }
}

// ---- heaviest-first order.  A query's cost grows with its number of included
// cells; the launch takes queries in decreasing cost class, so the longest ones
// start first and the batch does not end on a few long queries with the GPU
// otherwise idle.  Counting sort on 64 classes of log2 of the cell count (half
// octaves: up to 2^32 cells), in LDS per workgroup like the evaluation's spatial
// order.
constexpr int kCostBins = 64;

__device__ __forceinline__ uint32_t cost_class(const pndf_query& qr, float s2r, int n, int kernel, float eps, int L)
{
    const QuerySetup q = setup_query(qr, s2r, 0.f, L, eps, kernel);
    if (!q.valid) return 0u;
    const double cx = fmin((double)(q.cxhi - q.cxlo + 1), (double)n), cy = fmin((double)(q.cyhi - q.cylo + 1), (double)n);
    const int c = (int)floor(2.0 * log2(cx * cy));
    return (uint32_t)min(max(c, 0), kCostBins - 1);
}

__global__ void k_cost_hist(const pndf_query* __restrict__ q, int64_t nq, float s2r, int kernel, HierDev H,
                            uint32_t* __restrict__ key, uint32_t* __restrict__ hist)
{
    __shared__ uint32_t loc[kCostBins];
    if (threadIdx.x < kCostBins) loc[threadIdx.x] = 0u;
    __syncthreads();
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nq; i += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t k = (kCostBins - 1) - cost_class(q[i], s2r, H.n, kernel, H.eps, H.L);  // heaviest first
        key[i] = k;
        atomicAdd(&loc[k], 1u);
    }
    __syncthreads();
    if (threadIdx.x < kCostBins && loc[threadIdx.x]) atomicAdd(&hist[threadIdx.x], loc[threadIdx.x]);
}

// hist: the counters, then the cursors within the classes
__global__ void k_cost_scatter(const uint32_t* __restrict__ key, int64_t nq, uint32_t* __restrict__ hist,
                               uint32_t* __restrict__ order)
{
    __shared__ uint32_t loc[kCostBins], first[kCostBins];
    uint32_t* cursor = hist + kCostBins;
    if (threadIdx.x < kCostBins) {
        // the classes' first places, an exclusive scan by one wavefront
        const uint32_t v = hist[threadIdx.x];
        uint32_t run = v;
        for (int o = 1; o < kCostBins; o <<= 1) {
            const uint32_t u = __shfl_up(run, o);
            if ((int)threadIdx.x >= o) run += u;
        }
        first[threadIdx.x] = run - v;
        loc[threadIdx.x] = 0u;
    }
    __syncthreads();
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = i0; i < nq; i += stride) atomicAdd(&loc[key[i]], 1u);
    __syncthreads();
    if (threadIdx.x < kCostBins && loc[threadIdx.x]) loc[threadIdx.x] = first[threadIdx.x] + atomicAdd(&cursor[threadIdx.x], loc[threadIdx.x]);
    __syncthreads();
    for (int64_t i = i0; i < nq; i += stride) order[atomicAdd(&loc[key[i]], 1u)] = (uint32_t)i;
}

__global__ void k_cost_zero(uint32_t* hist)
{
    if (threadIdx.x < 2 * kCostBins) hist[threadIdx.x] = 0u;
}

}  // namespace

// Wavefronts that share a query (see k_projected_area): a small batch leaves the chip
// idle otherwise, and its longest query decides.  Of sigma 1 to 8 on a scratched 1024^2
// map, 8, 4 or 1 wavefronts each: 256 queries 60, 88, 340 us; 1024: -, 118, 349; 4096:
// -, 288, 443 (ordered).  Beyond, the queries fill the chip and the setup that each
// wavefront repeats costs more than the sharing gives (narrow footprints, 65536 queries: 564
// against 234 us).
static int projarea_waves(int64_t nq) { return nq <= 512 ? 8 : (nq <= 4096 ? 4 : 1); }

template <int KER>
static void launch_queries(const HierDev& H, const ProjArgs& c, hipStream_t s)
{
    const dim3 grid((unsigned)c.nq);
    const int w = projarea_waves(c.nq);
    if (w == 8) hipLaunchKernelGGL((k_projected_area<KER, 8>), grid, dim3(512), 0, s, H, c);
    else if (w == 4) hipLaunchKernelGGL((k_projected_area<KER, 4>), grid, dim3(256), 0, s, H, c);
    else hipLaunchKernelGGL((k_projected_area<KER, 1>), grid, dim3(64), 0, s, H, c);
}

hipError_t launch_projected_area(const HierDev& H, const ProjArgs& a, hipStream_t s)
{
    // one workgroup per query, in launches of at most launch_chunk() (2^24 x 64 = 2^30
    // work-items), each in heaviest-first order (workspace: order, keys and counters of
    // one launch, stream-ordered).  Up to kAllResident queries all run at once, in any
    // order.
    constexpr int64_t kAllResident = 4096;
    const int64_t chunk = launch_chunk();
    const int64_t most = std::min(chunk, a.nq);
    uint32_t* buf = nullptr;
    if (most > kAllResident) {
        const hipError_t e = stream_alloc((void**)&buf, sizeof(uint32_t) * (2 * (size_t)most + 2 * kCostBins), s);
        if (e != hipSuccess) return e;
    }
    for (int64_t off = 0; off < a.nq; off += chunk) {
        ProjArgs c = a;
        c.q = a.q + off;
        c.P = a.P + off;
        if (a.lambda) c.lambda = a.lambda + off;
        c.nq = std::min(chunk, a.nq - off);
        if (c.nq > kAllResident) {
            uint32_t* key = buf + most;
            uint32_t* hist = key + most;
            const unsigned g = (unsigned)std::min<int64_t>(256, (c.nq + 1023) / 1024);
            hipLaunchKernelGGL(k_cost_zero, dim3(1), dim3(2 * kCostBins), 0, s, hist);
            hipLaunchKernelGGL(k_cost_hist, dim3(g), dim3(256), 0, s, c.q, c.nq, c.s2r, c.kernel, H, key, hist);
            hipLaunchKernelGGL(k_cost_scatter, dim3(g), dim3(256), 0, s, key, c.nq, hist, buf);
            c.order = buf;
        }
        if (a.kernel == PNDF_KERNEL_DISK) launch_queries<PNDF_KERNEL_DISK>(H, c, s);
        else if (a.kernel == PNDF_KERNEL_BOX) launch_queries<PNDF_KERNEL_BOX>(H, c, s);
        else launch_queries<PNDF_KERNEL_GAUSSIAN>(H, c, s);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) {
            stream_free(buf, s);
            return e;
        }
    }
    stream_free(buf, s);
    return hipSuccess;
}

}  // namespace pndf
