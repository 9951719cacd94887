// Sampling of the manifold P-NDF on gfx950: one thread per sample.
//
// A sample draws u from the footprint kernel over the support that the evaluation
// integrates and returns the normal m of the triangle containing u (section
// "Sampling and evaluation"): n(u) interpolated from the texel normals, the same
// barycentric point of the equilateral replacement for a clamped triangle
// (Eq. debias), and with the cut the cluster field n^l of the unit the evaluation
// uses at u (section "Acceleration by mesh clustering").  The density of m is then
// D(m) divided by D's total mass, for every footprint kernel and cut threshold.
//
// Support.  Without the cut, the included cells [cxlo, cxhi + 1] per axis; with
// it, the units of the cut (cells or cluster nodes) whose unrolled image meets the
// included cells.  The Gaussian is drawn per axis by inverse CDF on a range S
// (the included cells, or with the cut the entry-level nodes over them) and with
// the cut rejected when its unit misses the included cells; the caller supplies
// `attempts` uniform pairs per sample for that.  Disk and box supports lie inside
// the included cells and are drawn directly from the first pair.
//
// Work per sample: the query (24 B), one uniform pair (16 B), the cut levels'
// residuals (4 B each, from the entry level down to the cut), the unit's four corner
// normals and clamp bits (for a texel cell from its leaf record), and the outputs.
// The Gaussian draw (four normal distribution functions and two inverses per sample)
// is evaluated from one table in LDS: with the library's functions it took the
// vector ALU's whole time (2^22 samples at 2048^2, tau = 0: 168 -> 151 us, a third of
// the vector instructions; 10^6 at 4096^2 with the cut: 109 -> 93 us).  What bounds it
// now is the scattered reads: 167 B fetched per sample beside 72 B in and out.
#include <algorithm>

#include "pndf_internal.h"

namespace pndf {
namespace {

constexpr int kTailPieces = 68, kTailCoefs = 10;
__device__ const double kNormalTail[kTailPieces * kTailCoefs] = {
#include "normal_tail.inc"
};

// Phi(-t), t >= 0, from the table in LDS (0 from 8.5 on: below 1e-17), and with
// SLOPE its derivative.
template <bool SLOPE>
__device__ __forceinline__ double normal_tail(const double* tab, double t, double* slope)
{
    const double t8 = fmin(t, 8.5) * 8.0;
    const int k = min((int)t8, kTailPieces - 1);
    const double* c = tab + kTailCoefs * k;
    const double s = t8 - (double)k - 0.5;
    double v = c[9], d = 0.0;
#pragma unroll
    for (int i = 8; i >= 0; --i) {
        if (SLOPE) d = fma(d, s, v);
        v = fma(v, s, c[i]);
    }
    if (SLOPE) *slope = 8.0 * d;
    return t < 8.5 ? v : 0.0;
}

__device__ __forceinline__ double normal_cdf(const double* tab, double z)
{
    const double v = normal_tail<false>(tab, fabs(z), nullptr);
    return z < 0.0 ? v : 1.0 - v;
}

// The standard normal quantile at the tail probability r = Phi(-t) in [kLeastTail,
// 1/2]: t.  First in float32, t = (1 - 2 r) P(w) with w = -log(4 r (1 - r)) (the
// variable in which the quantile is nearly a polynomial: M. Giles, "Approximating the
// erfinv function", GPU Computing Gems, 2011), then one third-order step on
// Phi(-t) - r, which leaves less than 1e-16 of that.  P, of degree 10 in w - 5, is a
// weighted least-squares fit of t / (1 - 2 r) over 120001 values of t in [1e-4, 4.25],
// weights 1 - 2 r multiplied 200 times by (1/2 + error / largest error)^0.7 towards equal
// errors, the best of them: 1.6e-6 off at most.
constexpr double kLeastTail = 1.1e-5;  // t <= 4.24
__device__ __forceinline__ double normal_tail_quantile(const double* tab, double r)
{
    const float x = (float)(1.0 - 2.0 * r), rf = (float)r;
    const float w = -__logf(4.0f * rf * (1.0f - rf)) - 5.0f;
    const float P[11] = {2.941299200e+00f,  3.022185564e-01f,  -1.027329918e-02f, 1.867593091e-04f,
                         7.430269761e-05f,  -1.527700624e-05f, 1.442539087e-06f,  3.303221874e-08f,
                         -2.352648920e-08f, 1.219414680e-09f,  7.265217594e-11f};
    float f = P[10];
#pragma unroll
    for (int i = 9; i >= 0; --i) f = fmaf(f, w, P[i]);
    const double t = fmax(0.0, (double)(x * f));
    double slope;
    const double e = normal_tail<true>(tab, t, &slope) - r;
    double inv = __builtin_amdgcn_rcp(slope);
    inv = fma(fma(-slope, inv, 1.0), inv, inv);
    const double d = e * inv;
    return t - d + 0.5 * t * d * d;
}

// u on [a, b) from N(x, sig^2) truncated to [a, b), by inverse CDF: the library's
// functions (tails beyond the fit)
__device__ __noinline__ double trunc_gauss(double x, double sig, double a, double b, double xi)
{
    const double pa = normcdf((a - x) / sig), pb = normcdf((b - x) / sig);
    return x + sig * normcdfinv(pa + xi * (pb - pa));
}

// The same for both axes from the table; an axis whose draw falls into a tail (one in
// 45000 at a half-width of 3 sigma) takes the library's.
__device__ __forceinline__ double2 trunc_gauss2(const double* tab, const QuerySetup& q, float sx, float sy, double ax,
                                                double bx, double ay, double by, double2 xi)
{
    double u[2];
    const double c[2] = {(double)q.x, (double)q.y}, s[2] = {(double)sx, (double)sy};
    const double lo[2] = {ax, ay}, hi[2] = {bx, by}, x[2] = {xi.x, xi.y};
    bool tail[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const double inv = 1.0 / s[i];
        const double pa = normal_cdf(tab, (lo[i] - c[i]) * inv), pb = normal_cdf(tab, (hi[i] - c[i]) * inv);
        const double p = pa + x[i] * (pb - pa), r = fmin(p, 1.0 - p);
        tail[i] = !(r >= kLeastTail);
        const double t = normal_tail_quantile(tab, tail[i] ? 0.25 : r);
        u[i] = c[i] + s[i] * (p < 0.5 ? -t : t);
    }
    if (tail[0] | tail[1]) {
#pragma unroll 1
        for (int i = 0; i < 2; ++i)
            if (i ? tail[1] : tail[0]) {
                const double v = trunc_gauss(i ? c[1] : c[0], i ? s[1] : s[0], i ? lo[1] : lo[0], i ? hi[1] : hi[0],
                                             i ? x[1] : x[0]);
                if (i) u[1] = v; else u[0] = v;
            }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        if (u[i] < lo[i]) u[i] = lo[i];
        if (u[i] >= hi[i]) u[i] = nextafter(hi[i], lo[i]);
    }
    return make_double2(u[0], u[1]);
}

// does the unrolled image of the level-l unit that holds cell c meet the cells [clo, chi]
__device__ __forceinline__ bool unit_meets(int c, int l, int clo, int chi)
{
    const int start = (c >> l) << l;
    return start <= chi && start + (1 << l) - 1 >= clo;
}

template <int KER, bool CUT>
__global__ __launch_bounds__(256) void k_sample(HierDev H, SampleArgs a)
{
    constexpr bool kGauss = KER == PNDF_KERNEL_GAUSSIAN;
    __shared__ double tab[kGauss ? kTailPieces * kTailCoefs : 1];
    if (kGauss) {
        for (int i = threadIdx.x; i < kTailPieces * kTailCoefs; i += blockDim.x) tab[i] = kNormalTail[i];
        __syncthreads();
    }
    const int64_t k = a.first + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= a.end) return;
    const QuerySetup q = setup_query(a.q[k], a.s2r, CUT ? a.tau : 0.f, H.L, H.eps, KER);
    bool ok = q.valid;
    const double2* xi = reinterpret_cast<const double2*>(a.xi);
    double2 u = make_double2(__longlong_as_double(0x7ff8000000000000ll), __longlong_as_double(0x7ff8000000000000ll));
    float2 mo = make_float2(__int_as_float(0x7fc00000), __int_as_float(0x7fc00000));
    uint64_t id = ~0ull;
    // attempts that may be needed: only the Gaussian with the cut rejects
    const int tries = (KER == PNDF_KERNEL_GAUSSIAN && CUT) ? a.attempts : 1;
#pragma unroll 1
    for (int t = 0; ok && t < tries; ++t) {
        const double2 x = xi[(int64_t)t * a.nq + k];
        if (!(x.x >= 0.0 && x.x < 1.0 && x.y >= 0.0 && x.y < 1.0)) {
            ok = false;
            break;
        }
        if constexpr (KER == PNDF_KERNEL_DISK) {
            double sn, cs;
            sincospi(2.0 * x.y, &sn, &cs);
            const double rad = sqrt(x.x);
            u.x = (double)q.x + (double)q.rx * rad * cs;
            u.y = (double)q.y + (double)q.ry * rad * sn;
        } else if constexpr (KER == PNDF_KERNEL_BOX) {
            u.x = (double)q.x + (double)q.rx * (2.0 * x.x - 1.0);
            u.y = (double)q.y + (double)q.ry * (2.0 * x.y - 1.0);
        } else {
            const int l = CUT ? q.l0 : 0;
            const double ax = (double)(floor_div_pow2(q.cxlo, l) << l);
            const double bx = (double)((floor_div_pow2(q.cxhi, l) + 1) << l);
            const double ay = (double)(floor_div_pow2(q.cylo, l) << l);
            const double by = (double)((floor_div_pow2(q.cyhi, l) + 1) << l);
            u = trunc_gauss2(tab, q, a.q[k].sx, a.q[k].sy, ax, bx, ay, by, x);
        }
        // the unrolled cell that holds u, and the unit of the cut that holds it: the
        // first level from the entry level down whose residual is within the threshold,
        // else the cell (its ancestors' Morton codes are prefixes of its own)
        const int iu = (int)floor(u.x), ju = (int)floor(u.y);
        int lev = 0;
        if constexpr (CUT) {
            const uint32_t code = morton((uint32_t)(iu & (H.n - 1)), (uint32_t)(ju & (H.n - 1)));
            // (a short dependent chain per thread; the many threads in flight hide it.
            // Reading 2 or 4 levels at once changed nothing: it fetches lines of the
            // large low levels that the cut never asks for)
#pragma unroll 1
            for (int l = q.l0; l >= 1; --l)
                if (H.clu_e[level_offset(H.logn, l) + (code >> (2 * l))] <= q.t) {
                    lev = l;
                    break;
                }
            if (KER == PNDF_KERNEL_GAUSSIAN &&
                !(unit_meets(iu, lev, q.cxlo, q.cxhi) && unit_meets(ju, lev, q.cylo, q.cyhi)))
                continue;  // rejected: the unit lies outside the support
        }
        const int I = (iu >> lev) & ((H.n >> lev) - 1), J = (ju >> lev) & ((H.n >> lev) - 1);
        const double side = 1.0 / (double)(1 << lev);
        const double U = (u.x - (double)((iu >> lev) << lev)) * side, V = (u.y - (double)((ju >> lev) << lev)) * side;
        const int half = U + V < 1.0 ? 0 : 1;
        double w0, w1, w2;
        if (half == 0) {
            w0 = 1.0 - U - V; w1 = U; w2 = V;
        } else {
            w0 = U + V - 1.0; w1 = 1.0 - U; w2 = 1.0 - V;
        }
        float2 n0, n1, n2, n3;
        bool clamped;
        if (lev == 0) {
            // from the cell's 2 x 2 leaf record (its 3 x 3 corners and clamp bytes in
            // 80 B), not from two rows of the normal plane and the clamp array: one
            // scattered record instead of three scattered lines per sample
            const QuadRec* r = H.quad + morton((uint32_t)I >> 1, (uint32_t)J >> 1);
            const int di = I & 1, dj = J & 1, k = 3 * dj + di;
            n0 = r->t[k]; n1 = r->t[k + 1]; n2 = r->t[k + 3]; n3 = r->t[k + 4];
            clamped = (r->deg[2 * dj + di] >> half) & 1u;
        } else {
            const int64_t ix = level_offset(H.logn, lev) + morton((uint32_t)I, (uint32_t)J);
            const float4 ca = H.clu_t[2 * ix], cb = H.clu_t[2 * ix + 1];
            n0 = make_float2(ca.x, ca.y); n1 = make_float2(ca.z, ca.w);
            n2 = make_float2(cb.x, cb.y); n3 = make_float2(cb.z, cb.w);
            clamped = (clamp_bits(ca, cb) >> half) & 1u;
        }
        double v[6];
        if (clamped) {
            eqtri_f64(0.5 * ((double)n1.x + (double)n2.x), 0.5 * ((double)n1.y + (double)n2.y),
                      (double)(H.rho * (float)(1 << lev)), v);
        } else if (half == 0) {
            v[0] = n0.x; v[1] = n0.y; v[2] = n1.x; v[3] = n1.y; v[4] = n2.x; v[5] = n2.y;
        } else {
            v[0] = n3.x; v[1] = n3.y; v[2] = n2.x; v[3] = n2.y; v[4] = n1.x; v[5] = n1.y;
        }
        mo.x = (float)(w0 * v[0] + w1 * v[2] + w2 * v[4]);
        mo.y = (float)(w0 * v[1] + w1 * v[3] + w2 * v[5]);
        id = tri_id(lev, I, J, half);
        break;
    }
    if (!ok) u = make_double2(__longlong_as_double(0x7ff8000000000000ll), __longlong_as_double(0x7ff8000000000000ll));
    a.m[k] = mo;
    if (a.tri) a.tri[k] = id;
    if (a.u) a.u[k] = u;
}

// One thread per sample, in launches of at most launch_chunk() samples (the
// uniforms keep their stride nq: attempt t of sample k at t nq + k).
template <int KER>
void launch_kernel(const HierDev& H, const SampleArgs& a0, hipStream_t s)
{
    const int64_t chunk = launch_chunk();
    for (int64_t off = 0; off < a0.nq; off += chunk) {
        SampleArgs a = a0;
        a.first = off;
        a.end = std::min(a0.nq, off + chunk);
        const dim3 grid((unsigned)((a.end - a.first + 255) / 256)), block(256);
        if (a.tau > 0.f)
            hipLaunchKernelGGL((k_sample<KER, true>), grid, block, 0, s, H, a);
        else
            hipLaunchKernelGGL((k_sample<KER, false>), grid, block, 0, s, H, a);
        if (hipPeekAtLastError() != hipSuccess) return;
    }
}

}  // namespace

hipError_t launch_sample(const HierDev& H, const SampleArgs& a, hipStream_t s)
{
    if (a.nq == 0) return hipSuccess;
    if (a.kernel == PNDF_KERNEL_DISK)
        launch_kernel<PNDF_KERNEL_DISK>(H, a, s);
    else if (a.kernel == PNDF_KERNEL_BOX)
        launch_kernel<PNDF_KERNEL_BOX>(H, a, s);
    else
        launch_kernel<PNDF_KERNEL_GAUSSIAN>(H, a, s);
    return hipGetLastError();
}

}  // namespace pndf
