// Hierarchy build: min-max boxes and least-squares cluster normals per quad-tree
// node (section "Acceleration by mesh clustering"; supplement "Derivations of
// Cluster Normal Optimization").
//
// The cluster objective of a node (Eq. normal_optimization) is a quadratic form in
// its four corner normals N0..N3: E(N) = C + tr(N^T B) + tr(N^T A N) / 2 with
//   A = 2 int w lambda lambda^T,  B = -2 int w lambda n^T,  C = int w |n|^2,
// lambda the cluster triangles' barycentric basis and w = 1 / max(Jacobian, eps)
// of each fine triangle.  Both cluster halves (lower: corners 0, 1, 2; upper:
// corners 3, 2, 1) carry these integrals over their own area in their own
// barycentric basis mu: a 3 x 3 Gram matrix G = 2 int w mu mu^T, H = -2 int w mu n^T
// and C.  A child half-triangle lies wholly inside one half of its parent, and the
// parent's barycentrics restricted to it are the child's barycentrics times the
// matrix Lam[i][k] = mu^parent_i(child vertex k), whose entries are 0, 1/2 or 1.  So
//   G_parent += Lam G_child Lam^T,  H_parent += Lam H_child,  C_parent += C_child
// are exact products (powers of two) summed, and every entry of G is a sum of
// non-negative terms: the recurrence is as accurate as integrating each node
// directly, in O(N^2) total work.  Level 0 is the fine triangle itself (area 1/2,
// linear normal field): G = w (1 + delta_ij) / 12, H_i = -(w / 12) (n_i + sum n_k),
// C = (w / 24) (sum |n_k|^2 + |sum n_k|^2).
//
// N* = -A^-1 B by Cholesky.  The residual e^l = E(N*) is then integrated directly
// over the node's fine triangles (the residual is linear on each:
// int w |r|^2 = (w / 24) (sum |r_k|^2 + |sum r_k|^2) from its vertex values), a sum
// of non-negative terms, instead of the difference C + tr(N*^T B) / 2 of large
// numbers.
#include <algorithm>

#include "pndf_internal.h"

namespace pndf {

namespace {

// Statistics of one cluster half: G (00, 01, 02, 11, 12, 22), H (3 x 2, row-major), C.
constexpr int kStat = 13;
constexpr int kG = 0, kH = 6, kC = 12;

__device__ __forceinline__ double jac64(float2 a, float2 b, float2 c)
{
    double p = __dmul_rn((double)c.x - (double)a.x, (double)b.y - (double)a.y);
    double q = __dmul_rn((double)c.y - (double)a.y, (double)b.x - (double)a.x);
    return fabs(__dsub_rn(p, q));
}

__device__ __forceinline__ double fine_weight(double det, double eps) { return 1.0 / (det < eps ? eps : det); }

// Statistics of a fine triangle with vertex normals (a, b, c) and weight w, in its
// own barycentric basis.
__device__ __forceinline__ void fine_stats(double w, float2 a, float2 b, float2 c, double* S)
{
    const double d = w / 6.0, f = w / 12.0;
    S[kG + 0] = d; S[kG + 1] = f; S[kG + 2] = f;
    S[kG + 3] = d; S[kG + 4] = f; S[kG + 5] = d;
    const double ax = a.x, ay = a.y, bx = b.x, by = b.y, cx = c.x, cy = c.y;
    const double sx = ax + bx + cx, sy = ay + by + cy;
    S[kH + 0] = -f * (ax + sx); S[kH + 1] = -f * (ay + sy);
    S[kH + 2] = -f * (bx + sx); S[kH + 3] = -f * (by + sy);
    S[kH + 4] = -f * (cx + sx); S[kH + 5] = -f * (cy + sy);
    const double q = ax * ax + ay * ay + bx * bx + by * by + cx * cx + cy * cy + sx * sx + sy * sy;
    S[kC] = (w / 24.0) * q;
}

// Barycentric basis of a parent half at parent-normalised (U, V): lower half over
// corners (0, 1, 2) = (1 - U - V, U, V); upper half over corners (3, 2, 1) =
// (U + V - 1, 1 - U, 1 - V).
__device__ __forceinline__ void half_basis(int hp, double U, double V, double mu[3])
{
    if (hp == 0) { mu[0] = 1.0 - U - V; mu[1] = U; mu[2] = V; }
    else { mu[0] = U + V - 1.0; mu[1] = 1.0 - U; mu[2] = 1.0 - V; }
}

// Add the statistics S of half hc of child (di, dj) (side 1/2 of the parent) to
// half hp of the parent.  Child lower vertices (in parent-normalised coordinates):
// (di, dj)/2, (di + 1, dj)/2, (di, dj + 1)/2; upper: (di + 1, dj + 1)/2,
// (di, dj + 1)/2, (di + 1, dj)/2.  Called with literal arguments Lam folds into
// constants.
__device__ __forceinline__ void add_child(int di, int dj, int hc, int hp, const double* S, double* P)
{
    const double x0 = 0.5 * di, x1 = 0.5 * (di + 1), y0 = 0.5 * dj, y1 = 0.5 * (dj + 1);
    const double vu[3] = {hc ? x1 : x0, hc ? x0 : x1, hc ? x1 : x0};
    const double vv[3] = {hc ? y1 : y0, hc ? y1 : y0, hc ? y0 : y1};
    double Lm[3][3];  // Lm[i][k] = mu^parent_i(child vertex k)
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        double mu[3];
        half_basis(hp, vu[k], vv[k], mu);
#pragma unroll
        for (int i = 0; i < 3; ++i) Lm[i][k] = mu[i];
    }
    const double G[3][3] = {{S[kG + 0], S[kG + 1], S[kG + 2]},
                            {S[kG + 1], S[kG + 3], S[kG + 4]},
                            {S[kG + 2], S[kG + 4], S[kG + 5]}};
    double T[3][3];  // Lm G
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int m = 0; m < 3; ++m) T[i][m] = Lm[i][0] * G[0][m] + Lm[i][1] * G[1][m] + Lm[i][2] * G[2][m];
    const int gi[3][3] = {{0, 1, 2}, {1, 3, 4}, {2, 4, 5}};
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = i; j < 3; ++j)
            P[kG + gi[i][j]] += T[i][0] * Lm[j][0] + T[i][1] * Lm[j][1] + T[i][2] * Lm[j][2];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int c = 0; c < 2; ++c)
            P[kH + 2 * i + c] += Lm[i][0] * S[kH + c] + Lm[i][1] * S[kH + 2 + c] + Lm[i][2] * S[kH + 4 + c];
    P[kC] += S[kC];
}

// Add the eight child halves of a node to its two halves: the lower-left child
// (c4 = 0) lies in the lower half, the upper-right one (c4 = 3) in the upper half,
// and the off-diagonal children split along the parent's diagonal (their lower
// halves below it).  C(c4, h) gives half h of child c4 = di + 2 dj.
template <typename ChildFn>
__device__ __forceinline__ void gather_children(ChildFn C, double* lo, double* up)
{
#pragma unroll
    for (int c4 = 0; c4 < 4; ++c4)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int hp = c4 == 0 ? 0 : (c4 == 3 ? 1 : h);
            add_child(c4 & 1, c4 >> 1, h, hp, C(c4, h), hp ? up : lo);
        }
}

// N* = -A^-1 B for the node's 4 x 4 A and 4 x 2 B assembled from its halves (lower
// over corners 0, 1, 2, upper over corners 3, 2, 1), by Cholesky (A is positive
// definite: every fine triangle has a positive weight).
__device__ void solve_cluster(const double* lo, const double* up, double N[4][2])
{
    double A[4][4] = {{0}}, B[4][2] = {{0}};
    const int vi[2][3] = {{0, 1, 2}, {3, 2, 1}};
    const int gi[3][3] = {{0, 1, 2}, {1, 3, 4}, {2, 4, 5}};
    const double* hs[2] = {lo, up};
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < 3; ++i) {
#pragma unroll
            for (int j = 0; j < 3; ++j) A[vi[h][i]][vi[h][j]] += hs[h][kG + gi[i][j]];
            B[vi[h][i]][0] += hs[h][kH + 2 * i];
            B[vi[h][i]][1] += hs[h][kH + 2 * i + 1];
        }
    double Lm[4][4] = {{0}};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        double d = A[j][j];
#pragma unroll
        for (int k = 0; k < j; ++k) d -= Lm[j][k] * Lm[j][k];
        d = sqrt(fmax(d, 1e-300));
        Lm[j][j] = d;
#pragma unroll
        for (int i = j + 1; i < 4; ++i) {
            double v = A[i][j];
#pragma unroll
            for (int k = 0; k < j; ++k) v -= Lm[i][k] * Lm[j][k];
            Lm[i][j] = v / d;
        }
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        double y[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            double v = -B[i][c];
#pragma unroll
            for (int k = 0; k < i; ++k) v -= Lm[i][k] * y[k];
            y[i] = v / Lm[i][i];
        }
#pragma unroll
        for (int i = 3; i >= 0; --i) {
            double v = y[i];
#pragma unroll
            for (int k = i + 1; k < 4; ++k) v -= Lm[k][i] * N[k][c];
            N[i][c] = v / Lm[i][i];
        }
    }
}

__device__ __forceinline__ void box_add(float4& b, float x, float y)
{
    b.x = fminf(b.x, x); b.y = fminf(b.y, y); b.z = fmaxf(b.z, x); b.w = fmaxf(b.w, y);
}

__device__ __forceinline__ void box_union(float4& b, const float4& o)
{
    b.x = fminf(b.x, o.x); b.y = fminf(b.y, o.y); b.z = fmaxf(b.z, o.z); b.w = fmaxf(b.w, o.w);
}

// Box of a replacement triangle centred at (cx, cy) with circumradius rho, with a
// margin that covers both the float32 and the FP64 vertex evaluations.
__device__ __forceinline__ void box_add_eqtri(float4& b, float cx, float cy, float rho)
{
    const float r = rho * (1.0f + 1e-6f) + 1e-6f;
    box_add(b, cx - r, cy - r);
    box_add(b, cx + r, cy + r);
}

__device__ __forceinline__ float4 empty_box()
{
    return make_float4(INFINITY, INFINITY, -INFINITY, -INFINITY);
}

// ---- octagons (see HierDev): bounds of x, y, u = x + y, v = x - y.  u and v are
// taken in FP64 and every bound is rounded outward to half precision, so unions of
// octagons are exact on the keys.
struct Oct {
    float4 b;        // min x, min y, max x, max y
    double ul, vl, uh, vh;
};

__device__ __forceinline__ Oct empty_oct()
{
    return Oct{empty_box(), (double)INFINITY, (double)INFINITY, -(double)INFINITY, -(double)INFINITY};
}

__device__ __forceinline__ void oct_add_diag(Oct& o, double u, double v, double r)
{
    o.ul = fmin(o.ul, u - r); o.vl = fmin(o.vl, v - r);
    o.uh = fmax(o.uh, u + r); o.vh = fmax(o.vh, v + r);
}

__device__ __forceinline__ void oct_add(Oct& o, float x, float y)
{
    box_add(o.b, x, y);
    oct_add_diag(o, (double)x + (double)y, (double)x - (double)y, 0.0);
}

// A replacement triangle lies in the disk of its circumradius rho, sqrt(2) rho wide
// along a diagonal; the margin as in box_add_eqtri.
__device__ __forceinline__ void oct_add_eqtri(Oct& o, float cx, float cy, float rho)
{
    box_add_eqtri(o.b, cx, cy, rho);
    oct_add_diag(o, (double)cx + (double)cy, (double)cx - (double)cy, 1.4142136 * ((double)rho * (1.0 + 1e-6) + 1e-6));
}

// keys of a pair of minima (rounded down) or maxima (rounded up); the zeros: a
// minimum of +0 becomes -0, a maximum of -0 becomes +0
__device__ __forceinline__ uint32_t min_keys(float a, float b)
{
    uint32_t x = __half_as_ushort(__float2half_rd(a)), y = __half_as_ushort(__float2half_rd(b));
    if (x == 0u) x = 0x8000u;
    if (y == 0u) y = 0x8000u;
    return half_key(x) | (half_key(y) << 16);
}

__device__ __forceinline__ uint32_t max_keys(float a, float b)
{
    uint32_t x = __half_as_ushort(__float2half_ru(a)), y = __half_as_ushort(__float2half_ru(b));
    if (x == 0x8000u) x = 0u;
    if (y == 0x8000u) y = 0u;
    return half_key(x) | (half_key(y) << 16);
}

__device__ __forceinline__ uint4 oct_keys(const Oct& o)
{
    return make_uint4(min_keys(o.b.x, o.b.y), max_keys(o.b.z, o.b.w),
                      min_keys(__double2float_rd(o.ul), __double2float_rd(o.vl)),
                      max_keys(__double2float_ru(o.uh), __double2float_ru(o.vh)));
}

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint4 oct_union(uint4 a, uint4 b)
{
    auto lo = [](uint32_t p, uint32_t q) {
        return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, p), __builtin_bit_cast(u16x2, q)));
    };
    auto hi = [](uint32_t p, uint32_t q) {
        return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, p), __builtin_bit_cast(u16x2, q)));
    };
    return make_uint4(lo(a.x, b.x), hi(a.y, b.y), lo(a.z, b.z), hi(a.w, b.w));
}

__device__ __forceinline__ uint4 oct_union4(const uint4* c)
{
    return oct_union(oct_union(c[0], c[1]), oct_union(c[2], c[3]));
}

// The arrays that the build writes, all levels packed, and one level's part of them.
struct BuildDev {
    uint4* oct_k;
    uint4* oct_c;
    float4* bbox;
    float4* bbox_all;
    float4* bbox_clu;
    float4* clu_n;
    float4* clu_t;
    float* clu_e;
    float2* clu_det;
    double* nfit;      // FP64 fits of levels kFitLevel and above (workspace)
    double* stat[2];   // half statistics of even and odd levels from 2 up (workspace)
};
constexpr int kFitLevel = 3;

struct LevelOut {
    uint4* oct_k;
    uint4* oct_s;
    uint4* oct_o;
    uint4* oct_u;
    float4* bbox;
    float4* bbox_all;
    float4* bbox_clu;
    float4* clu_n;
    float4* clu_t;
    float* clu_e;
    float2* clu_det;
    double* nfit;      // nullptr below kFitLevel
    double* stat;
};

__device__ __forceinline__ LevelOut level_out(const HierDev& H, const BuildDev& B, int level)
{
    const int64_t off = level_offset(H.logn, level);
    LevelOut o;
    o.oct_k = B.oct_k + off;
    o.oct_s = B.oct_c + (int64_t)kOctSub * H.nodes + off;
    o.oct_o = B.oct_c + (int64_t)kOctOwn * H.nodes + off;
    o.oct_u = B.oct_c + (int64_t)kOctKids * H.nodes + off;
    o.bbox = B.bbox + off;
    o.bbox_all = B.bbox_all + off;
    o.bbox_clu = B.bbox_clu + off;
    o.clu_n = B.clu_n + 2 * off;
    o.clu_t = B.clu_t + 2 * off;
    o.clu_e = B.clu_e + off;
    o.clu_det = B.clu_det + off;
    o.nfit = level >= kFitLevel ? B.nfit + 8 * (off - level_offset(H.logn, kFitLevel)) : nullptr;
    o.stat = B.stat[level & 1];
    return o;
}

// Store the fitted normals of node idx (level side s): float32 normals, the cluster
// triangles' Jacobians and clamp decisions (FP64 from the stored float32 normals, as
// the evaluation uses them) with the test record that carries them; returns the
// octagon of the cluster triangles.
__device__ __forceinline__ Oct store_cluster(const HierDev& H, const LevelOut& o, int64_t idx, int s, const double N[4][2])
{
    float2 f[4];
    for (int k = 0; k < 4; ++k) f[k] = make_float2((float)N[k][0], (float)N[k][1]);
    o.clu_n[2 * idx] = make_float4(f[0].x, f[0].y, f[1].x, f[1].y);
    o.clu_n[2 * idx + 1] = make_float4(f[2].x, f[2].y, f[3].x, f[3].y);
    const double s2 = (double)s * (double)s;
    const double dl = jac64(f[0], f[1], f[2]) / s2;
    const double du = jac64(f[3], f[2], f[1]) / s2;
    const double eps = (double)H.eps;
    const bool cl = dl < eps, cu = du < eps;
    o.clu_det[idx] = make_float2(cl ? H.eps : (float)dl, cu ? H.eps : (float)du);
    const float qnan = __int_as_float(0x7fc00000);
    o.clu_t[2 * idx] = make_float4(cl ? qnan : f[0].x, f[0].y, f[1].x, f[1].y);
    o.clu_t[2 * idx + 1] = make_float4(f[2].x, f[2].y, cu ? qnan : f[3].x, f[3].y);
    Oct b = empty_oct();
    const float cx = 0.5f * (f[1].x + f[2].x), cy = 0.5f * (f[1].y + f[2].y);
    const float rho = H.rho * (float)s;
    if (cl) oct_add_eqtri(b, cx, cy, rho);
    else { oct_add(b, f[0].x, f[0].y); oct_add(b, f[1].x, f[1].y); oct_add(b, f[2].x, f[2].y); }
    if (cu) oct_add_eqtri(b, cx, cy, rho);
    else { oct_add(b, f[3].x, f[3].y); oct_add(b, f[2].x, f[2].y); oct_add(b, f[1].x, f[1].y); }
    return b;
}

// Weights of a record's 8 fine triangles (w / 24): cell c4, lower then upper.
__device__ __forceinline__ void record_weights(const float2 tx[9], double eps, double w[8])
{
#pragma unroll
    for (int c4 = 0; c4 < 4; ++c4) {
        const int k = 3 * (c4 >> 1) + (c4 & 1);
        w[2 * c4] = fine_weight(jac64(tx[k], tx[k + 1], tx[k + 3]), eps) / 24.0;
        w[2 * c4 + 1] = fine_weight(jac64(tx[k + 4], tx[k + 3], tx[k + 1]), eps) / 24.0;
    }
}

// Residual of a level-1 record (its 8 fine triangles) against the fit N of its
// ancestor of side `side`, the record's corner at cells (li, lj) of it.  The
// interpolant (lower triangle N0 (1 - U - V) + N1 U + N2 V, upper N3 (U + V - 1) +
// N2 (1 - U) + N1 (1 - V)) is linear but for its crease,
//   N0 + (N1 - N0) U + (N2 - N0) V + (N0 - N1 - N2 + N3) max(0, U + V - 1),
// so a corner takes two additions and a product per component.
__device__ __forceinline__ double record_residual(const float2 tx[9], const double w[8], const double* N, int side, int li,
                                                  int lj)
{
    const double inv = 1.0 / side;
    const double bx = (N[2] - N[0]) * inv, by = (N[3] - N[1]) * inv, cx = (N[4] - N[0]) * inv, cy = (N[5] - N[1]) * inv;
    const double dx = (N[0] - N[2] - N[4] + N[6]) * inv, dy = (N[1] - N[3] - N[5] + N[7]) * inv;
    const double ax = N[0] + bx * li + cx * lj, ay = N[1] + by * li + cy * lj;
    const int over = li + lj - side;
    // row by row, so that two rows of corner residuals are live at a time
    double rx[6], ry[6];
    auto row = [&](int y, int at) {
#pragma unroll
        for (int x = 0; x < 3; ++x) {
            const double m = (double)max(0, over + x + y);
            rx[at + x] = (double)tx[3 * y + x].x - (ax + bx * x + cx * y + dx * m);
            ry[at + x] = (double)tx[3 * y + x].y - (ay + by * x + cy * y + dy * m);
        }
    };
    row(0, 0);
    double r = 0.0;
#pragma unroll
    for (int dj = 0; dj < 2; ++dj) {
        row(dj + 1, 3);
#pragma unroll
        for (int di = 0; di < 2; ++di) {
            const int k = di;
            const int tri[2][3] = {{k, k + 1, k + 3}, {k + 4, k + 3, k + 1}};
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int p = tri[h][0], q = tri[h][1], s = tri[h][2];
                const double sx = rx[p] + rx[q] + rx[s], sy = ry[p] + ry[q] + ry[s];
                const double qq = rx[p] * rx[p] + ry[p] * ry[p] + rx[q] * rx[q] + ry[q] * ry[q] + rx[s] * rx[s] +
                                  ry[s] * ry[s] + sx * sx + sy * sy;
                r += w[2 * (2 * dj + di) + h] * qq;
            }
        }
#pragma unroll
        for (int x = 0; x < 3; ++x) {
            rx[x] = rx[3 + x];
            ry[x] = ry[3 + x];
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    return r;
}

// A level-1 node t (Morton code) from its 2 x 2 cells (8 fine triangles): leaf record,
// boxes and octagons; with clusters its half statistics (lo, up), fit and residual.
// Returns its corners in tx and its triangles' weights in wgt.
__device__ __forceinline__ void level1_node(const HierDev& H, const LevelOut& o, QuadRec* __restrict__ quad, int64_t t,
                                            int cluster, float2 tx[9], double wgt[8], double* lo, double* up)
{
    const int I = (int)morton_compact((uint32_t)t), J = (int)morton_compact((uint32_t)t >> 1);
    const int w = H.n + 1;
    uint8_t dg4[4];
    {
        QuadRec r;
        for (int y = 0; y < 3; ++y)
            for (int x = 0; x < 3; ++x) tx[3 * y + x] = r.t[3 * y + x] = H.nrm[(int64_t)(2 * J + y) * w + 2 * I + x];
        for (int dj = 0; dj < 2; ++dj)
            for (int di = 0; di < 2; ++di)
                dg4[2 * dj + di] = r.deg[2 * dj + di] = H.deg[(int64_t)(2 * J + dj) * H.n + 2 * I + di];
        r.pad = 0;
        quad[t] = r;
    }
    Oct box = empty_oct();
#pragma unroll
    for (int c4 = 0; c4 < 4; ++c4) {
        const int k = 3 * (c4 >> 1) + (c4 & 1);
        const float2 n0 = tx[k], n1 = tx[k + 1], n2 = tx[k + 3], n3 = tx[k + 4];
        const uint8_t dg = dg4[c4];
        const float cx = 0.5f * (n1.x + n2.x), cy = 0.5f * (n1.y + n2.y);
        if (dg & 1) oct_add_eqtri(box, cx, cy, H.rho);
        else { oct_add(box, n0.x, n0.y); oct_add(box, n1.x, n1.y); oct_add(box, n2.x, n2.y); }
        if (dg & 2) oct_add_eqtri(box, cx, cy, H.rho);
        else { oct_add(box, n3.x, n3.y); oct_add(box, n2.x, n2.y); oct_add(box, n1.x, n1.y); }
    }
    o.bbox[t] = box.b;
    const uint4 map_keys = oct_keys(box);
    o.oct_k[t] = map_keys;
    if (!cluster) return;
    const double eps = (double)H.eps;
    // the 8 fine triangles (cell c4 = di + 2 dj: lower (n0, n1, n2), upper (n3, n2, n1))
    // gathered into the node's halves
#pragma unroll
    for (int c4 = 0; c4 < 4; ++c4) {
        const int k = 3 * (c4 >> 1) + (c4 & 1);
        const float2 n0 = tx[k], n1 = tx[k + 1], n2 = tx[k + 3], n3 = tx[k + 4];
        double F[kStat];
        fine_stats(fine_weight(jac64(n0, n1, n2), eps), n0, n1, n2, F);
        add_child(c4 & 1, c4 >> 1, 0, c4 == 3 ? 1 : 0, F, c4 == 3 ? up : lo);
        fine_stats(fine_weight(jac64(n3, n2, n1), eps), n3, n2, n1, F);
        add_child(c4 & 1, c4 >> 1, 1, c4 == 0 ? 0 : 1, F, c4 == 0 ? lo : up);
    }
    double N[4][2];
    solve_cluster(lo, up, N);
    const Oct own = store_cluster(H, o, t, 2, N);
    const uint4 own_keys = oct_keys(own);
    float4 cb = own.b;
    o.bbox_clu[t] = cb;
    box_union(cb, box.b);
    o.bbox_all[t] = cb;
    o.oct_o[t] = own_keys;
    o.oct_s[t] = oct_union(own_keys, map_keys);
    // (a level-1 node's children are cells: never asked for, excludes nothing)
    o.oct_u[t] = make_uint4(0u, 0xffffffffu, 0u, 0xffffffffu);
    record_weights(tx, eps, wgt);
    o.clu_e[t] = (float)record_residual(tx, wgt, &N[0][0], 2, 0, 0);
}

// Level-1 nodes alone, one per thread (without clusters, or on the 2 x 2 map).
__global__ __launch_bounds__(128) void k_level1(HierDev H, BuildDev B, QuadRec* __restrict__ quad, int cluster)
{
    const int64_t m = H.n >> 1, t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= m * m) return;
    double lo[kStat] = {0}, up[kStat] = {0};
    float2 tx[9];
    double wgt[8];
    level1_node(H, level_out(H, B, 1), quad, t, cluster, tx, wgt, lo, up);
}

// Fit, boxes and octagons of node t of a level above 1 from its half statistics and
// its children's boxes (co: their level).
__device__ __forceinline__ void finish_node(const HierDev& H, const LevelOut& o, const LevelOut& co, int64_t t, int level,
                                            const double* lo, const double* up, double N[4][2])
{
    const int64_t c00 = 4 * t;
    solve_cluster(lo, up, N);
    const Oct own = store_cluster(H, o, t, 1 << level, N);
    const uint4 own_keys = oct_keys(own);
    o.oct_o[t] = own_keys;
    o.oct_s[t] = oct_union(own_keys, oct_union4(co.oct_s + c00));
    o.oct_u[t] = oct_union4(co.oct_o + c00);
    float4 cb = own.b;
    o.bbox_clu[t] = cb;
#pragma unroll
    for (int c = 0; c < 4; ++c) box_union(cb, co.bbox_all[c00 + c]);
    o.bbox_all[t] = cb;
}

__device__ __forceinline__ void union_boxes(const LevelOut& o, const LevelOut& co, int64_t t)
{
    const int64_t c00 = 4 * t;
    float4 box = co.bbox[c00];
#pragma unroll
    for (int c = 1; c < 4; ++c) box_union(box, co.bbox[c00 + c]);
    o.bbox[t] = box;
    o.oct_k[t] = oct_union4(co.oct_k + c00);
}

// Levels 1 and 2 with clusters, one level-1 node per thread and its parents by a
// quarter of the workgroup: the level-1 statistics pass through LDS (at 2048^2 they
// are 218 MB to write and to read again, and the fits 67 MB, of the 512 MB that a
// level-1 pass wrote), and both levels' residuals are integrated here, from corners
// that are still in registers.  (One level-2 node per thread, its children in turn,
// takes 308 registers: one wave per SIMD, 269 us at 2048^2; this way 183 us; the
// separate passes over both levels took 421.)
constexpr int kLow = 128;
__global__ __launch_bounds__(kLow) void k_levels12(HierDev H, BuildDev B, QuadRec* __restrict__ quad)
{
    __shared__ double st[kLow][2 * kStat + 1];  // (odd stride: no bank conflicts)
    __shared__ double fit[kLow / 4][8];
    const int64_t m1 = (int64_t)(H.n >> 1) * (H.n >> 1), t = (int64_t)blockIdx.x * kLow + threadIdx.x;
    const LevelOut o1 = level_out(H, B, 1), o2 = level_out(H, B, 2);
    float2 tx[9];
    double wgt[8];
    if (t < m1) {
        double lo[kStat] = {0}, up[kStat] = {0};
        level1_node(H, o1, quad, t, 1, tx, wgt, lo, up);
        for (int k = 0; k < kStat; ++k) {
            st[threadIdx.x][k] = lo[k];
            st[threadIdx.x][kStat + k] = up[k];
        }
    }
    __threadfence_block();
    __syncthreads();
    const int64_t p = (int64_t)blockIdx.x * (kLow / 4) + threadIdx.x;
    if (threadIdx.x < kLow / 4 && 4 * p < m1) {
        double lo[kStat] = {0}, up[kStat] = {0};
        gather_children([&](int c4, int h) { return &st[4 * threadIdx.x + c4][h * kStat]; }, lo, up);
        double* M = o2.stat + p * (2 * kStat);
        for (int k = 0; k < kStat; ++k) { M[k] = lo[k]; M[kStat + k] = up[k]; }
        union_boxes(o2, o1, p);
        double N[4][2];
        finish_node(H, o2, o1, p, 2, lo, up, N);
        for (int k = 0; k < 4; ++k) { fit[threadIdx.x][2 * k] = N[k][0]; fit[threadIdx.x][2 * k + 1] = N[k][1]; }
    }
    __syncthreads();
    double r = 0.0;
    const int c4 = threadIdx.x & 3;
    if (t < m1) r = record_residual(tx, wgt, fit[threadIdx.x >> 2], 4, 2 * (c4 & 1), 2 * (c4 >> 1));
    r += __shfl_xor(r, 1);
    r += __shfl_xor(r, 2);
    if (c4 == 0 && t < m1) o2.clu_e[t >> 2] = (float)r;
}

// Node t of level >= 2 from the level below: boxes and octagons are unions of the
// children's, half statistics gathered from theirs.
__device__ __forceinline__ void level_up_node(const HierDev& H, const BuildDev& B, int level, int64_t t, int cluster)
{
    const LevelOut o = level_out(H, B, level), co = level_out(H, B, level - 1);
    const int64_t c00 = 4 * t;
    union_boxes(o, co, t);
    if (!cluster) return;
    double lo[kStat] = {0}, up[kStat] = {0};
    gather_children([&](int c4, int h) { return co.stat + (c00 + c4) * (2 * kStat) + h * kStat; }, lo, up);
    double* M = o.stat + t * (2 * kStat);
    for (int k = 0; k < kStat; ++k) { M[k] = lo[k]; M[kStat + k] = up[k]; }
    double N[4][2];
    finish_node(H, o, co, t, level, lo, up, N);
    double* nf = o.nfit + 8 * t;
    for (int k = 0; k < 4; ++k) { nf[2 * k] = N[k][0]; nf[2 * k + 1] = N[k][1]; }
}

__global__ __launch_bounds__(64) void k_level_up(HierDev H, BuildDev B, int level, int cluster)
{
    const int64_t m = H.n >> level, t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < m * m) level_up_node(H, B, level, t, cluster);
}

// The levels of at most kTopNodes nodes, one after the other in one workgroup (a
// launch each took longer than their work).
constexpr int kTopNodes = 256;
__global__ __launch_bounds__(kTopNodes) void k_level_top(HierDev H, BuildDev B, int first, int cluster)
{
    for (int level = first; level <= H.L; ++level) {
        const int m = H.n >> level;
        if ((int)threadIdx.x < m * m) level_up_node(H, B, level, threadIdx.x, cluster);
        __threadfence_block();
        __syncthreads();
    }
}

constexpr int kResidBlock = 256;  // leaf records per block of the residual pass (a level-5 node)

// Residuals of levels kFitLevel and above, all in one pass: thread t (a level-1
// record, Morton order) integrates the residual of its 8 fine triangles against the
// FP64 fits of its ancestors t >> 2 (level - 1).  The 4^(level - 1) records of a node
// are consecutive: up to a whole block they are summed by a fixed tree and stored as
// e^l; above, each block leaves a partial sum per level for k_resid_sum.
// Deterministic.  (A pass per level read the records and formed the weights, eight
// divisions, anew each time: 56 us a level at 2048^2, 614 in all; now 106 us.)
__global__ __launch_bounds__(kResidBlock) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_resid(HierDev H, BuildDev B, double* __restrict__ part)
{
    __shared__ double red[kMaxLevels + 1][kResidBlock / 64];
    const int64_t m1 = (int64_t)(H.n >> 1) * (H.n >> 1);
    const int64_t t = (int64_t)blockIdx.x * kResidBlock + threadIdx.x;
    float2 tx[9];
    double wgt[8];
    if (t < m1) {
        const float4* rec = reinterpret_cast<const float4*>(H.quad + t);
        const float4 a = rec[0], b = rec[1], c = rec[2], d = rec[3], e = rec[4];
        tx[0] = make_float2(a.x, a.y); tx[1] = make_float2(a.z, a.w); tx[2] = make_float2(b.x, b.y);
        tx[3] = make_float2(b.z, b.w); tx[4] = make_float2(c.x, c.y); tx[5] = make_float2(c.z, c.w);
        tx[6] = make_float2(d.x, d.y); tx[7] = make_float2(d.z, d.w); tx[8] = make_float2(e.x, e.y);
        record_weights(tx, (double)H.eps, wgt);
    }
    const int ci = 2 * (int)morton_compact((uint32_t)t), cj = 2 * (int)morton_compact((uint32_t)t >> 1);
#pragma unroll 1
    for (int level = kFitLevel; level <= H.L; ++level) {
        const int sh = 2 * (level - 1), side = 1 << level;
        double r = 0.0;
        // (a block lies in one node from level 5 up: its fit through the scalar cache)
        const int64_t node = sh >= 8 ? ((int64_t)blockIdx.x * kResidBlock) >> sh : t >> sh;
        const double* N = B.nfit + 8 * (level_offset(H.logn, level) - level_offset(H.logn, kFitLevel) + node);
        if (t < m1) r = record_residual(tx, wgt, N, side, ci & (side - 1), cj & (side - 1));
        const int group = sh >= 6 ? 64 : 1 << sh;
#pragma unroll
        for (int st = 1; st < 64; st <<= 1)
            if (st < group) r += __shfl_xor(r, st);
        float* e = B.clu_e + level_offset(H.logn, level);
        if (sh <= 6) {
            if ((threadIdx.x & (group - 1)) == 0 && t < m1) e[t >> sh] = (float)r;
            continue;
        }
        if ((threadIdx.x & 63) == 0) red[level][threadIdx.x >> 6] = r;
    }
    __syncthreads();
    const int level = 5 + (int)threadIdx.x;
    if (level <= H.L) {
        const double s = (red[level][0] + red[level][1]) + (red[level][2] + red[level][3]);
        if (level == 5) B.clu_e[level_offset(H.logn, 5) + blockIdx.x] = (float)s;
        else part[(int64_t)(level - 6) * gridDim.x + blockIdx.x] = s;
    }
}

// The level and the node of entry i of the levels from `first` up, packed.
__device__ __forceinline__ int packed_level(const HierDev& H, int first, int64_t i, int64_t* node)
{
    int level = first;
    const int64_t off = level_offset(H.logn, first);
    while (level < H.L && i + off >= level_offset(H.logn, level + 1)) ++level;
    *node = i + off - level_offset(H.logn, level);
    return level;
}

// e^l of the nodes larger than a block of the residual pass (levels 6 and above), one
// workgroup per node: the sum of the node's consecutive block partials in a fixed
// order.
__global__ __launch_bounds__(256) void k_resid_sum(HierDev H, BuildDev B, const double* __restrict__ part, int64_t rblocks)
{
    __shared__ double red[256];
    int64_t k;
    const int level = packed_level(H, 6, blockIdx.x, &k);
    const int64_t per = (int64_t)1 << (2 * (level - 5));
    const double* p = part + (level - 6) * rblocks + k * per;
    double s = 0.0;
    for (int64_t i = threadIdx.x; i < per; i += 256) s += p[i];
    red[threadIdx.x] = s;
    for (int o = 128; o > 0; o >>= 1) {
        __syncthreads();
        if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    }
    if (threadIdx.x == 0) B.clu_e[level_offset(H.logn, level) + k] = (float)red[0];
}

// Row-major copies of up to kExports per-node arrays of one level in one launch.
__global__ void k_export_rowmajor(ExportArgs x, int m)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= (int64_t)m * m) return;
    const uint32_t I = (uint32_t)(k % m), J = (uint32_t)(k / m);
    const int64_t c = (int64_t)morton(I, J);
    for (int i = 0; i < x.count; ++i) {
        const int words = x.words[i];
        const uint32_t* a = x.src[i] + c * words;
        uint32_t* b = x.dst[i] + k * words;
        for (int w = 0; w < words; ++w) b[w] = a[w];
    }
}

}  // namespace

hipError_t export_rowmajor(const ExportArgs& x, int m, hipStream_t s)
{
    if (x.count == 0) return hipSuccess;
    const int64_t cnt = (int64_t)m * m;
    hipLaunchKernelGGL(k_export_rowmajor, dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0, s, x, m);
    return hipGetLastError();
}

// e^l and the largest e^l of the four children side by side (HierDev::clu_em): an
// expansion reads its four children's in one 32 B segment.
__global__ void k_residual_pairs(HierDev H, float2* __restrict__ em, float2* __restrict__ te)
{
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx < 2 * kMaxTiles) te[idx] = make_float2(0.f, 0.f);  // (for k_tile_residuals)
    if (idx >= (int64_t)H.nodes) return;
    int64_t t;
    const int level = packed_level(H, 1, idx, &t);
    float kids = INFINITY;
    if (level >= 2) {
        const float* ce = H.clu_e + level_offset(H.logn, level - 1) + 4 * t;
        kids = fmaxf(fmaxf(ce[0], ce[1]), fmaxf(ce[2], ce[3]));
    }
    em[idx] = make_float2(H.clu_e[idx], kids);
}

// A middle value of a level's residuals (HierDev::level_e): halfway between the mean of
// their logarithms and the logarithm of their mean, as few large ones (scratches) make
// many nodes above them; over at most 1024 nodes at even steps.
__device__ __forceinline__ void level_mean(const HierDev& H, int level, float (*red)[256], float* __restrict__ le)
{
    const int nodes = 1 << (2 * (H.logn - level)), count = min(nodes, 1024), t = (int)threadIdx.x;
    const float* e = H.clu_e + level_offset(H.logn, level);
    float v = 0.f, m = 0.f;
#pragma unroll 4
    for (int i = t; i < count; i += 256) {
        const float x = fmaxf(e[(int64_t)i * (nodes / count)], 1e-30f);
        v += log2f(x);
        m += x;
    }
    red[0][t] = v;
    red[1][t] = m;
    for (int o = 128; o > 0; o >>= 1) {
        __syncthreads();
        if (t < o) {
            red[0][t] += red[0][t + o];
            red[1][t] += red[1][t + o];
        }
    }
    if (t == 0) le[level] = 0.5f * (red[0][0] / (float)count + log2f(red[1][0] / (float)count));
}

// Largest residuals kTileDepth and kTileSpan levels beneath each node of the levels
// from kTileLevel up (HierDev::tile_e, cleared before): one workgroup per node and
// part of kTilePart values (the top nodes look over 4^9), the parts' maxima by atomic
// maximum (the values are not negative, so their bits compare like them).  The workgroups
// past the nodes take a level's middle residual each.
constexpr int kTilePart = 16384;
__global__ __launch_bounds__(256) void k_tile_residuals(HierDev H, float2* __restrict__ te, float* __restrict__ le)
{
    __shared__ float both[2][256];
    float* const red = both[0];
    const int tiles = (int)(H.nodes - level_offset(H.logn, kTileLevel));
    if ((int)blockIdx.x >= tiles) {
        if (blockIdx.y == 0) level_mean(H, (int)blockIdx.x - tiles + 1, both, le);
        return;
    }
    int64_t t;
    const int level = packed_level(H, kTileLevel, blockIdx.x, &t);
    for (int k = 0; k < 2; ++k) {
        const int down = min(k ? kTileSpan : kTileDepth, level - 1);  // (residuals start at level 1)
        const int per = 1 << (2 * down), first = blockIdx.y * kTilePart, last = min(per, first + kTilePart);
        if (first >= last) continue;
        const float* e = H.clu_e + level_offset(H.logn, level - down) + per * t;
        float v = 0.f;
#pragma unroll 8
        for (int i = first + (int)threadIdx.x; i < last; i += 256) v = fmaxf(v, e[i]);
        red[threadIdx.x] = v;
        for (int o = 128; o > 0; o >>= 1) {
            __syncthreads();
            if ((int)threadIdx.x < o) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + o]);
        }
        if (threadIdx.x == 0) atomicMax(reinterpret_cast<unsigned*>(te) + 2 * blockIdx.x + k, __float_as_uint(red[0]));
        __syncthreads();
    }
}

hipError_t build_hierarchy_levels(pndf_hier* h, hipStream_t s)
{
    const HierDev& H = h->dev;
    const int n = H.n, cluster = h->cluster;
    const int64_t m1 = (int64_t)(n >> 1) * (n >> 1), m2 = (int64_t)(n >> 2) * (n >> 2), m3 = (int64_t)(n >> 3) * (n >> 3);
    const int64_t rblocks = (m1 + kResidBlock - 1) / kResidBlock;
    const int64_t fits = H.L >= kFitLevel ? h->nodes - level_offset(H.logn, kFitLevel) : 0;
    BuildDev B{h->oct_k, h->oct_c, h->bbox, h->bbox_all, h->bbox_clu, h->clu_n, h->clu_t, h->clu_e, h->clu_det, nullptr, {}};
    // workspace (cluster fits only), one allocation: half statistics of even and odd
    // levels from 2 up, FP64 fits, block partials of the residual pass
    double* work = nullptr;
    double* part = nullptr;
    hipError_t err = hipSuccess;
    if (cluster && H.L >= 2) {
        const int upper = H.L > 5 ? H.L - 5 : 0;
        err = block_alloc(sizeof(double) * (size_t)(2 * kStat * (m2 + m3) + 8 * fits + upper * rblocks), (void**)&work);
        if (err != hipSuccess) return err;
        B.stat[0] = work;
        B.stat[1] = work + 2 * kStat * m2;
        B.nfit = B.stat[1] + 2 * kStat * m3;
        part = B.nfit + 8 * fits;
    }
    int level = 2;
    if (cluster && H.L >= 2) {
        hipLaunchKernelGGL(k_levels12, dim3((unsigned)((m1 + kLow - 1) / kLow)), dim3(kLow), 0, s, H, B, h->quad);
        level = 3;
    } else {
        hipLaunchKernelGGL(k_level1, dim3((unsigned)((m1 + 127) / 128)), dim3(128), 0, s, H, B, h->quad, cluster);
    }
    for (; level <= H.L && (int64_t)(n >> level) * (n >> level) > kTopNodes; ++level) {
        const int64_t m = (int64_t)(n >> level) * (n >> level);
        hipLaunchKernelGGL(k_level_up, dim3((unsigned)((m + 63) / 64)), dim3(64), 0, s, H, B, level, cluster);
    }
    if (level <= H.L) hipLaunchKernelGGL(k_level_top, dim3(1), dim3(kTopNodes), 0, s, H, B, level, cluster);
    if (cluster) {
        if (H.L >= kFitLevel)
            hipLaunchKernelGGL(k_resid, dim3((unsigned)rblocks), dim3(kResidBlock), 0, s, H, B, part);
        if (H.L >= 6)
            hipLaunchKernelGGL(k_resid_sum, dim3((unsigned)(h->nodes - level_offset(H.logn, 6))), dim3(256), 0, s, H, B, part,
                               rblocks);
        hipLaunchKernelGGL(k_residual_pairs, dim3((unsigned)((std::max<int64_t>(h->nodes, 2 * kMaxTiles) + 255) / 256)), dim3(256), 0, s, H, h->clu_em,
                           h->tile_e);
        if (has_tiles(H.logn)) {
            const unsigned parts = std::max(1u, (1u << (2 * kTileSpan)) / kTilePart);
            hipLaunchKernelGGL(k_tile_residuals, dim3((unsigned)(h->nodes - level_offset(H.logn, kTileLevel) + H.L), parts),
                               dim3(256), 0, s, H, h->tile_e, h->level_e);
        }
    }
    err = hipGetLastError();
    const hipError_t sync = hipStreamSynchronize(s);
    block_free(work);
    return err == hipSuccess ? sync : err;
}

}  // namespace pndf
