// P-NDF evaluation kernels (Eq. ndf_eval).
//
// A wavefront owns a query (or a subtree of one) at a time; its 64 lanes
// cooperate on the candidates:
//   - brute force: lanes stride over the included cells;
//   - hierarchical: a breadth-limited, depth-first quad-tree descent.  Each level
//     has a list in LDS; the wave pops up to 64 nodes of the lowest non-empty level
//     (one per lane), tests their children's octagons (and the cluster cut), and pushes
//     the surviving children with a ballot prefix.  A level-1 node tests the triangles
//     of its 2 x 2 cells from its leaf record.
//   - split: the wavefronts of a workgroup share a query of a small batch.
//   - tiles: queries wider than a 256-texel tile leave their surviving tiles as items,
//     which are sorted and evaluated tile by tile.
//   - persistent: a fixed grid of workers takes chunks of queries (each XCD from
//     its own share of the spatial order); once the queries run out, idle workers
//     ask the busy ones for part of their pending subtrees through a global task
//     queue.
// Triangle tests run in float32 and only queue the hits; a queued hit is confirmed
// and its barycentrics recomputed in FP64 from the float32 vertices 64 at a time
// (one per lane), so the recovered uv and the term are accurate even for sliver
// triangles while the traversal itself stays small.  The hit's Jacobian is formed there
// from the same corners, as the mesh build forms the stored one.  Terms are summed exactly (192-bit
// fixed point at a per-query binary point), so D does not depend on the order in
// which hits are found: all algorithms, batch compositions and work splits give
// the same bits.
#include <algorithm>
#include <mutex>

#include "pndf_internal.h"

namespace pndf {

namespace {

enum { kModeValue = 0, kModeCount = 1, kModeRecord = 2 };

struct Acc {
    Fix192 d{0, 0, 0};
    uint32_t nodes = 0, cells = 0, clusters = 0, hits = 0;
    bool donated = false;  // part of the work was handed to other waves (wave-uniform)
};

struct Rec {  // hit-record cursor (record mode)
    uint64_t* ids;
    float* terms;
    uint64_t pos, end;
};

// FP64 confirmation of a float32 hit, barycentrics and term; < 0 if rejected.  The
// offsets v - h of float32 values are exact in FP64 and the cyclic edge functions
// e_k (as in the float32 test) give the barycentrics l_k = e_k / S, S = e0 + e1 + e2
// (twice the signed area, never 0: clamped triangles are replaced).  One division,
// R = 1 / (S det), serves both quotients: 1 / S = det R and 1 / det = S R.
template <int KER>
__device__ __forceinline__ double confirm_and_term(const QuerySetup& q, const double v[6], int I,
                                                   int J, int lev, int half, float det_used,
                                                   int logn)
{
    const double hx = (double)q.hx, hy = (double)q.hy;
    const double ax = v[0] - hx, ay = v[1] - hy, bx = v[2] - hx, by = v[3] - hy;
    const double cx = v[4] - hx, cy = v[5] - hy;
    const double e0 = bx * cy - by * cx, e1 = cx * ay - cy * ax, e2 = ax * by - ay * bx;
    if (!((e0 >= 0.0 && e1 >= 0.0 && e2 >= 0.0) || (e0 <= 0.0 && e1 <= 0.0 && e2 <= 0.0))) return -1.0;
    const double S = e0 + e1 + e2, dj = (double)det_used;
    const double R = 1.0 / (S * dj);
    const double rs = dj * R;
    return hit_weight<KER>(q, I, J, lev, half, e1 * rs, e2 * rs, logn) * (S * R);
}

// Twice the area of a triangle (a, b, c) = v as the build evaluates it (products
// rounded before the difference).
__device__ __forceinline__ double hit_jacobian(const double v[6])
{
#pragma clang fp contract(off)
    const double p = (v[4] - v[0]) * (v[3] - v[1]), r = (v[5] - v[1]) * (v[2] - v[0]);
    return fabs(p - r);
}

// Per-lane hit sink of one hit-processing round: value/count modes add the term to
// the exact accumulator at once; record mode also keeps (id, term) until the wave
// writes its records in lane order.
template <int MODE>
struct HitSink {
    uint64_t id = 0;
    float term = 0.f;
    int n = 0;
    __device__ __forceinline__ void put(const QuerySetup& q, Acc& acc, uint64_t tid, double t)
    {
        fix_add_term(acc.d, t, q.fexp);
        acc.hits += 1;
        if (MODE == kModeRecord) {
            id = tid;
            term = (float)t;
        }
        n = 1;
    }
};

// Write the wave's records in lane order, never leaving the query's own CSR slot
// [pos, end).  Every lane must call it.
template <int MODE>
__device__ __forceinline__ void flush_records(HitSink<MODE>& hs, Rec& rec)
{
    if (MODE == kModeRecord) {
        const uint64_t b = __ballot(hs.n);
        const uint64_t at = rec.pos + __popcll(b & ((1ull << lane_id()) - 1ull));
        if (hs.n && at < rec.end) {
            rec.ids[at] = hs.id;
            rec.terms[at] = hs.term;
        }
        rec.pos += __popcll(b);
    }
    hs.n = 0;
}

// Exclusive prefix over the wave of a per-lane count in [0, 15], and the total.
__device__ __forceinline__ int wave_prefix16(int c, int* total)
{
    const uint64_t b0 = __ballot(c & 1), b1 = __ballot(c & 2), b2 = __ballot(c & 4), b3 = __ballot(c & 8);
    const uint64_t lt = (1ull << lane_id()) - 1ull;
    *total = __popcll(b0) + 2 * __popcll(b1) + 4 * __popcll(b2) + 8 * __popcll(b3);
    return __popcll(b0 & lt) + 2 * __popcll(b1 & lt) + 4 * __popcll(b2 & lt) + 8 * __popcll(b3 & lt);
}

// ---- float32 triangle tests.  They only decide which triangles are hit; every hit
// becomes a 32-bit entry of the wave's hit queue, and the FP64 confirmation,
// barycentrics and term run later with one hit per lane (hit_entry), so the
// traversal keeps few registers and the FP64 work runs with full waves.
//   leaf cell    (0 << 30) | m << 3 | c4 << 1 | half   cell c4 = 2 dj + di of level-1 record m
//   plane cell   (1 << 30) | j << 14 | i << 1 | half   texel cell (i, j), i, j < 8192
//   cluster      (2 << 30) | lev << 25 | m << 1 | half   node m (Morton) of level lev >= 1
// A lane's hits are a bit mask over the low bits of its entry code.
constexpr uint32_t kHitPlane = 1u << 30, kHitCluster = 2u << 30;

// Traversal list items are Morton codes (at most 24 bits); the top bit marks a node
// whose region lies wholly inside the query's box, so that its descendants skip the
// spatial tests.  (With the cluster cut, a node's residual is compared with the
// query's threshold when its parent expands -- the four children's residuals are
// read with their boxes -- and a node under the cut goes to the cluster queue
// instead of a list.  Bit 30 then marks a node whose four children are all under
// the cut: the largest of their residuals, read with the node's own, is within the
// threshold, so its expansion reads only the children's boxes.)
constexpr uint32_t kInside = 1u << 31;
constexpr uint32_t kAllCut = 1u << 30;
constexpr uint32_t kCodeMask = (1u << 30) - 1u;

// Inclusive same-sign test of a triangle's three edge values: h inside or on it.
__device__ __forceinline__ uint32_t same_sign3(float a, float b, float c)
{
    return (uint32_t)(fminf(fminf(a, b), c) >= 0.f) | (uint32_t)(fmaxf(fmaxf(a, b), c) <= 0.f);
}

// A clamped half is replaced by its equilateral triangle (Eq. debias), the same for
// both halves of a cell (centred on the shared diagonal's midpoint): set the bits
// of the clamped halves (dg) of a cell's 2-bit mask from that triangle's test.
__device__ __forceinline__ uint32_t patch_clamped(const QuerySetup& q, float rho, float2 n1, float2 n2,
                                                  uint32_t dg, uint32_t m2)
{
    float v[6];
    eqtri_f32(0.5f * (n1.x + n2.x), 0.5f * (n1.y + n2.y), rho, v);
    const uint32_t e = (uint32_t)tri_hit_f32(v, q.hx, q.hy);
    if (dg & 1u) m2 = (m2 & ~1u) | e;
    if (dg & 2u) m2 = (m2 & ~2u) | (e << 1);
    return m2;
}

// The two triangles of a cell from its four corner normals and clamp bits: bit 0
// lower (n0, n1, n2), bit 1 upper (n3, n2, n1).  Every edge value is computed in
// one canonical direction (bottom and top edges left to right, left and right
// edges upwards, the diagonal from n1 to n2) and only its sign is flipped where a
// triangle runs along it the other way, so a cell tested alone and the same cell
// tested within its 2 x 2 block (which shares edges between cells) decide alike.
__device__ __forceinline__ uint32_t cell_mask(const QuerySetup& q, float rho, float2 n0, float2 n1, float2 n2,
                                              float2 n3, uint32_t dg)
{
    const float q0x = n0.x - q.hx, q0y = n0.y - q.hy, q1x = n1.x - q.hx, q1y = n1.y - q.hy;
    const float q2x = n2.x - q.hx, q2y = n2.y - q.hy, q3x = n3.x - q.hx, q3y = n3.y - q.hy;
    const float h01 = cross2(q0x, q0y, q1x, q1y), h23 = cross2(q2x, q2y, q3x, q3y);
    const float v02 = cross2(q0x, q0y, q2x, q2y), v13 = cross2(q1x, q1y, q3x, q3y);
    const float d12 = cross2(q1x, q1y, q2x, q2y);
    // lower: (d12, -v02, h01); upper: (-d12, v13, -h23), negated as a whole
    uint32_t m = same_sign3(d12, -v02, h01) | (same_sign3(d12, -v13, h23) << 1);
    if (dg & 3u) m = patch_clamped(q, rho, n1, n2, dg, m);
    return m;
}

// A texel cell tested from the padded normal plane (brute force, tiny footprints).
__device__ __forceinline__ uint32_t plane_cell_mask(const HierDev& H, const QuerySetup& q, int i, int j,
                                                    Acc& acc)
{
    const int w = H.n + 1;
    const float2* p = H.nrm + (int64_t)j * w + i;
    acc.cells += 1;
    return cell_mask(q, H.rho, p[0], p[1], p[w], p[w + 1], H.deg[(int64_t)j * H.n + i]);
}

// Along one axis, the level-c node columns (side 2^c; M = N >> c of them on the
// torus) that meet the unrolled cell range [clo, chi] form one cyclic run of n
// columns starting at a, and those with an image wholly inside the range a run of
// ni starting at ai (n or ni = M: every column).  Column X belongs to a run iff
// ((X - a) mod M) < n.  The runs depend only on the query and the level
// (wave-uniform), so each node's spatial tests are a subtraction, a mask and a
// compare per axis and child.
struct AxisRuns {
    int a, n, ai, ni;
};

__device__ __forceinline__ AxisRuns axis_runs(int clo, int chi, int c, int M)
{
    AxisRuns r;
    r.a = clo >> c;
    r.n = min((chi >> c) - r.a + 1, M);
    r.ai = -((-clo) >> c);
    r.ni = max(0, min(((chi + 1) >> c) - r.ai, M));
    return r;
}

// Bits 0 / 1: the columns 2X and 2X + 1 of the level below X (mask mk = M - 1
// there) in the run (a, n).
__device__ __forceinline__ uint32_t pair_in_run(int X, int a, int n, int mk)
{
    const int d = 2 * X - a;
    return (uint32_t)((d & mk) < n) | ((uint32_t)(((d + 1) & mk) < n) << 1);
}

// Bits c = 2 dj + di of the 2 x 2 block from its column bits x and row bits y.
__device__ __forceinline__ uint32_t quad_bits(uint32_t x, uint32_t y)
{
    return (x & (y & 1u ? 3u : 0u)) | ((x & (y & 2u ? 3u : 0u)) << 2);
}

// The 2 x 2 cells of level-1 node m (its leaf record), those overlapping the box
// (all four when the node lies inside it): bit 2 c4 + half for cell c4 = 2 dj + di.
// The block's nine corners give 16 distinct edges (6 horizontal, 6 vertical and 4
// diagonals), each computed once in its canonical direction as in cell_mask, so
// the bits equal cell_mask's for each cell.  rx, ry: the level-0 runs.
__device__ __forceinline__ uint32_t leaf_quad_mask(const HierDev& H, const QuerySetup& q, uint32_t m, bool inside,
                                                   const AxisRuns& rx, const AxisRuns& ry, Acc& acc)
{
    const float4* r = reinterpret_cast<const float4*>(H.quad + m);
    const float4 a = r[0], b = r[1], c = r[2], d = r[3], e = r[4];
    const float tx[9] = {a.x, a.z, b.x, b.z, c.x, c.z, d.x, d.z, e.x};
    const float ty[9] = {a.y, a.w, b.y, b.w, c.y, c.w, d.y, d.w, e.y};
    const uint32_t dg4 = __float_as_uint(e.z);
    uint32_t ov = 0xfu;
    if (!inside) {
        const int mk = H.n - 1;
        ov = quad_bits(pair_in_run((int)morton_compact(m), rx.a, rx.n, mk),
                       pair_in_run((int)morton_compact(m >> 1), ry.a, ry.n, mk));
    }
    acc.cells += (uint32_t)__popc(ov);
    // row by row (rows of corners 0-2 bottom to top), so that only two rows of
    // offsets and their edges are live at a time
    uint32_t mask = 0;
    float bx[3], by[3], bh[2];  // the lower row's offsets and its horizontal edges
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        bx[c] = tx[c] - q.hx;
        by[c] = ty[c] - q.hy;
    }
    bh[0] = cross2(bx[0], by[0], bx[1], by[1]);
    bh[1] = cross2(bx[1], by[1], bx[2], by[2]);
#pragma unroll
    for (int dj = 0; dj < 2; ++dj) {
        float ux[3], uy[3], uh[2], vt[3];  // the upper row, its horizontal edges, the vertical edges
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            ux[c] = tx[3 * dj + 3 + c] - q.hx;
            uy[c] = ty[3 * dj + 3 + c] - q.hy;
            vt[c] = cross2(bx[c], by[c], ux[c], uy[c]);
        }
        uh[0] = cross2(ux[0], uy[0], ux[1], uy[1]);
        uh[1] = cross2(ux[1], uy[1], ux[2], uy[2]);
#pragma unroll
        for (int di = 0; di < 2; ++di) {
            const float d12 = cross2(bx[di + 1], by[di + 1], ux[di], uy[di]);
            mask |= (same_sign3(d12, -vt[di], bh[di]) | (same_sign3(d12, -vt[di + 1], uh[di]) << 1))
                    << (2 * (2 * dj + di));
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            bx[c] = ux[c];
            by[c] = uy[c];
        }
        bh[0] = uh[0];
        bh[1] = uh[1];
    }
    if (dg4 & 0x03030303u) {
        // rare: a clamped triangle (its cell's replacement) is tested on its own; the
        // corners are read again (cached) rather than kept live through the tests
        const QuadRec* rec = H.quad + m;
        for (int c4 = 0; c4 < 4; ++c4) {
            const uint32_t dg = (dg4 >> (8 * c4)) & 3u;
            if (dg) {
                const int k = 3 * (c4 >> 1) + (c4 & 1);
                const uint32_t m2 = patch_clamped(q, H.rho, rec->t[k + 1], rec->t[k + 3], dg, (mask >> (2 * c4)) & 3u);
                mask = (mask & ~(3u << (2 * c4))) | (m2 << (2 * c4));
            }
        }
    }
    const uint32_t ov2 = (ov & 1u) * 3u | ((ov >> 1) & 1u) * 12u | ((ov >> 2) & 1u) * 48u | ((ov >> 3) & 1u) * 192u;
    return mask & ov2;
}

// The two cluster triangles of node idx (level lev): bit half.
__device__ __forceinline__ uint32_t cluster_mask(const HierDev& H, const QuerySetup& q, int lev, int64_t idx,
                                                 Acc& acc)
{
    const float4 a = H.clu_t[2 * idx], b = H.clu_t[2 * idx + 1];
    const uint32_t dg = clamp_bits(a, b);
    const float rho = H.rho * (float)(1 << lev);
    const float cx = 0.5f * (a.z + b.x), cy = 0.5f * (a.w + b.y);
    float vl[6], vu[6];
    if (dg & 1) eqtri_f32(cx, cy, rho, vl);
    else { vl[0] = a.x; vl[1] = a.y; vl[2] = a.z; vl[3] = a.w; vl[4] = b.x; vl[5] = b.y; }
    if (dg & 2) eqtri_f32(cx, cy, rho, vu);
    else { vu[0] = b.z; vu[1] = b.w; vu[2] = b.x; vu[3] = b.y; vu[4] = a.z; vu[5] = a.w; }
    acc.clusters += 1;
    return (uint32_t)tri_hit_f32(vl, q.hx, q.hy) | ((uint32_t)tri_hit_f32(vu, q.hx, q.hy) << 1);
}

// ---- FP64 stage: one queued hit.
template <int MODE, int KER>
__device__ __forceinline__ void hit_entry(const HierDev& H, const QuerySetup& q, uint32_t e, Acc& acc,
                                          HitSink<MODE>& hs)
{
    const int half = (int)(e & 1u);
    const uint32_t kind = e >> 30;
    double v[6];
    bool clamped;
    int I, J, lev;
    if (kind == (kHitCluster >> 30)) {
        lev = (int)((e >> 25) & 0xfu);
        const uint32_t m = (e >> 1) & 0xffffffu;
        const int64_t idx = level_offset(H.logn, lev) + m;
        I = (int)morton_compact(m);
        J = (int)morton_compact(m >> 1);
        const float4 a = H.clu_t[2 * idx], b = H.clu_t[2 * idx + 1];
        clamped = (clamp_bits(a, b) & (1u << half)) != 0u;
        if (clamped) {
            eqtri_f64(0.5 * ((double)a.z + (double)b.x), 0.5 * ((double)a.w + (double)b.y),
                      (double)(H.rho * (float)(1 << lev)), v);
        } else if (half == 0) {
            v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y;
        } else {
            v[0] = b.z; v[1] = b.w; v[2] = b.x; v[3] = b.y; v[4] = a.z; v[5] = a.w;
        }
    } else {
        float2 n0, n1, n2, n3;
        uint32_t dg;
        lev = 0;
        if (kind == 0) {
            const uint32_t m = (e >> 3) & 0xffffffu;
            const int c4 = (int)((e >> 1) & 3u), di = c4 & 1, dj = c4 >> 1;
            const QuadRec* r = H.quad + m;
            const int k = 3 * dj + di;
            n0 = r->t[k]; n1 = r->t[k + 1]; n2 = r->t[k + 3]; n3 = r->t[k + 4];
            dg = r->deg[c4];
            I = 2 * (int)morton_compact(m) + di;
            J = 2 * (int)morton_compact(m >> 1) + dj;
        } else {
            I = (int)((e >> 1) & 0x1fffu);
            J = (int)((e >> 14) & 0x1fffu);
            const int w = H.n + 1;
            const float2* p = H.nrm + (int64_t)J * w + I;
            n0 = p[0]; n1 = p[1]; n2 = p[w]; n3 = p[w + 1];
            dg = H.deg[(int64_t)J * H.n + I];
        }
        clamped = (dg & (1u << half)) != 0u;
        if (clamped) {
            eqtri_f64(0.5 * ((double)n1.x + (double)n2.x), 0.5 * ((double)n1.y + (double)n2.y), (double)H.rho, v);
        } else if (half == 0) {
            v[0] = n0.x; v[1] = n0.y; v[2] = n1.x; v[3] = n1.y; v[4] = n2.x; v[5] = n2.y;
        } else {
            v[0] = n3.x; v[1] = n3.y; v[2] = n2.x; v[3] = n2.y; v[4] = n1.x; v[5] = n1.y;
        }
    }
    // the Jacobian is formed again from the corners just read, bit for bit the stored
    // one: each stored value is 8 scattered bytes, a whole line from memory per hit
    const float det_used = clamped ? H.eps : (float)(hit_jacobian(v) * (1.0 / (double)(1u << (2 * lev))));
    const double t = confirm_and_term<KER>(q, v, I, J, lev, half, det_used, H.logn);
    if (t >= 0.0) hs.put(q, acc, tri_id(lev, I, J, half), t);
}

// The wave's hit queue: hq (kHitCap entries in LDS), hn entries (wave-uniform).
// Each lane's float32 hits wait in a bit mask (entry ebase | bit) until they are
// queued; the traversal loops run a round of the FP64 stage (hit_round, one call
// site per kernel so it is inlined once) whenever 64 hits are queued and at the end.
template <int MODE, int KER>
__device__ __forceinline__ void hit_round(const HierDev& H, const QuerySetup& q, const uint32_t* src, int cnt,
                                          Acc& acc, Rec& rec)
{
    HitSink<MODE> hs;
    if (lane_id() < cnt) hit_entry<MODE, KER>(H, q, src[lane_id()], acc, hs);
    flush_records<MODE>(hs, rec);
    wave_sync();
}

// Move the lanes' pending hits into the queue (as many as fit, in lane order).
__device__ __forceinline__ void queue_hits(uint32_t* hq, int& hn, uint32_t& pend, uint32_t ebase)
{
    if (__ballot(pend != 0u) == 0ull) return;
    int total;
    const int pos = wave_prefix16(__popc(pend), &total);
    if (total == 0) return;
    int at = hn + pos;
    while (pend && at < kHitCap) {
        hq[at++] = ebase | (uint32_t)(__ffs(pend) - 1);
        pend &= pend - 1u;
    }
    hn = min(hn + total, kHitCap);
    wave_sync();
}

// Is the query normal inside an octagon (HierDev)?  The query's keys are those of its
// x, y, x + y and x - y rounded to the nearest half: rounding is monotone, so an
// octagon whose set holds h holds it.  Each packed saturating difference is zero
// where its two bounds hold, so one compare decides all eight.
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t sub_sat2(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_sub_sat(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}
__device__ __forceinline__ bool in_octagon(const QuerySetup& q, uint4 o)
{
    return ((sub_sat2(o.x, q.hkey) | sub_sat2(q.hkey, o.y)) | (sub_sat2(o.z, q.hdiag) | sub_sat2(q.hdiag, o.w))) == 0u;
}

// With the cut, the octagon that decides about a node: under the cut (e^l <= t) only
// its own two cluster triangles are tested, so theirs; a node whose children are all
// under the cut can only lead to those children's cluster tests, so the union of
// their own; else everything beneath.
__device__ __forceinline__ uint32_t oct_class(bool cut, bool kids_cut)
{
    return cut ? kOctOwn : (kids_cut ? kOctKids : kOctSub);
}
__device__ __forceinline__ uint4 load_octagon(const HierDev& H, uint32_t cls, uint32_t node)
{
    // (a 32-bit byte offset: 3 x 22.4 M nodes x 16 B at 8192^2)
    return *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(H.oct_c) + (cls * H.nodes + node) * 16u);
}

// Cluster queue entry: level (4 bits) << 24 | Morton code of the node (< 2^24).
constexpr int kCluShift = 24;

// A wavefront's node lists in LDS (see list_words): 32-bit items for the levels below
// S, 16-bit items (code in bits 0..13, the flags kAllCut and kInside in bits 14, 15)
// from S up (only with the cut).  The level is wave-uniform wherever a list is read
// or written.
template <bool CUT>
struct NodeLists {
    uint32_t* w;
    uint16_t* h;
    int S;
    __device__ NodeLists(uint32_t* lds, int L)
        : w(lds), h(reinterpret_cast<uint16_t*>(lds + (size_t)(short_list_level(L, CUT) - 1) * kListCap)),
          S(short_list_level(L, CUT))
    {
    }
    __device__ __forceinline__ uint32_t get(int lev, int i) const
    {
        if (!CUT || lev < S) return w[(lev - 1) * kListCap + i];
        const uint32_t v = h[(lev - S) * kListCap + i];
        return (v & 0x3fffu) | ((v & 0xc000u) << 16);
    }
    __device__ __forceinline__ void put(int lev, int i, uint32_t item) const
    {
        if (!CUT || lev < S)
            w[(lev - 1) * kListCap + i] = item;
        else
            h[(lev - S) * kListCap + i] = (uint16_t)((item & 0x3fffu) | ((item >> 16) & 0xc000u));
    }
};

enum { kTilesNone = 0, kTilesEmit = 1, kTilesItem = 2, kTilesSplit = 3 };

// Reserve n items of the wave's segment; the first one's place, or -1 when they do
// not all fit (what the failed reservation covers is marked unused).  Every lane
// calls it with the same n > 0.
__device__ __forceinline__ int64_t tile_reserve(const TileWork& T, int n)
{
    const uint32_t seg = blockIdx.x & (kTileSegs - 1);
    uint32_t at = 0;
    if (lane_id() == 0) at = atomicAdd(&T.ctl->seg[seg].v, (uint32_t)n);
    at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
    unsigned long long* const raw = T.raw + (size_t)seg * T.segcap;
    if (at + (uint32_t)n <= T.segcap) return (int64_t)seg * T.segcap + at;
    for (uint32_t i = at + lane_id(); i < T.segcap; i += 64) raw[i] = ~0ull;
    return -1;
}

// Does node m of level lev >= kTileLevel, whose box holds h and which is not under the
// cut, become an item?  Residuals grow with the level (a node's fit restricted to a
// child is no better than the child's own), so the largest one some levels beneath
// tells whether the descent gets that far.
template <bool CUT>
__device__ __forceinline__ bool tile_item(const HierDev& H, const TileWork& T, const QuerySetup& q, int lev, uint32_t m)
{
    if (!CUT) return lev == kTileLevel;
    const float2 e = H.tile_e[(uint32_t)(level_offset(H.logn, lev) - level_offset(H.logn, kTileLevel)) + m];
    return e.x > q.t && (lev == kTileLevel || (T.coarse && e.y <= q.t));
}

// An item's word: the query's place, the node's level less kTileLevel (bits 24..27
// of the low half: Morton codes of these levels take at most 10) and its list item.
constexpr int kItemLevelShift = 24;
__device__ __forceinline__ unsigned long long tile_word(unsigned long long place, int lev, uint32_t item)
{
    return (place << 32) | ((uint32_t)(lev - kTileLevel) << kItemLevelShift) | item;
}
__device__ __forceinline__ int tile_word_level(unsigned long long w)
{
    return kTileLevel + (int)(((uint32_t)w >> kItemLevelShift) & 0xfu);
}
// the first tile beneath an item's node
__device__ __forceinline__ uint32_t tile_word_bin(unsigned long long w)
{
    return ((uint32_t)w & 0xffffu) << (2 * (tile_word_level(w) - kTileLevel));
}

// The shared descent.  List items are nodes (Morton codes) whose box contains h,
// whose region meets the support box and which are not under the cluster cut.  A
// lane takes one item: a level-1 node tests its 2 x 2 cells from its leaf record;
// any other node loads its (up to) four overlapping children's boxes together and
// keeps those that contain h: children under the cut go to the wave's cluster
// queue if the box of their own two cluster triangles contains h, the others to
// the list of the level below.  The cluster queue is taken 64
// nodes at a time, one per lane, each testing its node's two cluster triangles, so
// the cluster tests and the descent never share a step (a step runs every branch
// any lane takes).  Roots: every lane with root_ok holds a root of level
// root_level (level 0: texel cell packed i | j << 16; else a Morton code),
// box-tested here unless roots_tested.  With SPAWN (persistent workers), while
// some worker of the plan is idle the wave gives away part of its pending work
// before each step: half of the items of its highest non-empty list (the largest
// subtrees it holds), if that level is at least split_level, become tasks of the
// global queue.  A full queue simply leaves them here.
// With TILES == kTilesEmit, children (or roots) of level kTileLevel with enough
// beneath them become items of the tile queue instead of list entries; what does not
// fit there stays here.  With TILES == kTilesItem the root is one such item, ready to expand.
template <int MODE, bool CUT, bool SPAWN, int KER, int TILES = kTilesNone>
__device__ void descend(const HierDev& H, const QuerySetup& q, uint32_t* lists, int root_level,
                        bool root_ok, uint32_t root_item, bool roots_tested, int split_level,
                        unsigned long long qidx, const TaskQueue& Q, Acc& acc, Rec& rec,
                        const TileWork& T = TileWork{}, int lane_level = 0)
{
    static_assert(!SPAWN || MODE == kModeValue, "donation is only used by value-mode workers");
    const int lane = threadIdx.x & 63;
    const NodeLists<CUT> nl(lists, H.L);
    uint32_t* hq = lists + list_words(H.L, CUT);  // hit queue
    uint32_t* cq = hq + kHitCap;            // cluster queue (CUT)
    int hn = 0;                             // queued hits (wave-uniform)
    int cn = 0;                             // queued cluster nodes (wave-uniform)
    uint32_t pend = 0, ebase = 0;           // this lane's float32 hits not yet queued
    uint32_t nonempty = 0;   // bit l: list of level l non-empty (wave-uniform)
    int cntv = 0;            // lane l holds the size of list l
    const AxisRuns rx0 = axis_runs(q.cxlo, q.cxhi, 0, H.n), ry0 = axis_runs(q.cylo, q.cyhi, 0, H.n);
    if constexpr (TILES == kTilesItem) {
        if (lane == 0) nl.put(root_level, 0, root_item);
        if (lane == root_level) cntv = 1;
        nonempty = 1u << root_level;
        wave_sync();
    } else if (root_level == 0) {
        const int i = (int)(root_item & 0xffffu), j = (int)(root_item >> 16);
        if (root_ok) {
            pend = plane_cell_mask(H, q, i, j, acc);
            ebase = kHitPlane | ((uint32_t)j << 14) | ((uint32_t)i << 1);
        }
    } else {
        bool ok = root_ok;
        const uint32_t m = root_item & kCodeMask;
        const int rl = TILES == kTilesSplit && CUT ? lane_level : root_level;
        const uint32_t idx = (uint32_t)level_offset(H.logn, rl) + m;
        bool cut = false, kids_cut = false;
        if (CUT && ok) {
            const float2 em = H.clu_em[idx];
            cut = em.x <= q.t;
            kids_cut = em.y <= q.t;
        }
        if (ok && !roots_tested) {
            acc.nodes += 1;
            ok = in_octagon(q, CUT ? load_octagon(H, oct_class(cut, kids_cut), idx) : H.oct_k[idx]);
        }
        cut = cut && ok;
        const uint32_t entry = root_item | (kids_cut ? kAllCut : 0u);
        if (TILES == kTilesEmit && root_level >= kTileLevel) {
            const uint64_t be = __ballot(ok && !cut && tile_item<CUT>(H, T, q, root_level, m));
            const int64_t out = be ? tile_reserve(T, __popcll(be)) : -1;
            if (out >= 0 && ((be >> lane) & 1ull)) {
                T.raw[out + __popcll(be & ((1ull << lane) - 1ull))] = tile_word(qidx, root_level, entry);
                ok = false;
            }
        }
        const uint64_t bl = __ballot(ok && !cut);
        if (ok && !cut) nl.put(root_level, __popcll(bl & ((1ull << lane) - 1ull)), entry);
        if (CUT) {
            const uint64_t bc = __ballot(cut);
            if (cut) cq[__popcll(bc & ((1ull << lane) - 1ull))] = ((uint32_t)rl << kCluShift) | m;
            cn = __popcll(bc);
        }
        const int tot = __popcll(bl);
        if (lane == root_level) cntv = tot;
        if (tot) nonempty |= 1u << root_level;
        wave_sync();
    }
    // SPAWN: the starving flag, loaded at the start of a step (its latency hides behind
    // the step's own loads) and acted on before the next one
    unsigned hungry = 0;
    while (true) {
        queue_hits(hq, hn, pend, ebase);
        if (hn >= 64 || (hn > 0 && !nonempty && cn == 0)) {
            // (lanes still holding hits imply a full queue, so they get here too)
            const int c = min(hn, 64);
            hn -= c;
            hit_round<MODE, KER>(H, q, hq + hn, c, acc, rec);
            continue;
        }
        if (CUT && (cn >= 64 || (cn > 0 && !nonempty))) {
            // a round of cluster nodes, one per lane (every lane's hits are queued)
            const int c = min(cn, 64);
            cn -= c;
            if (lane < c) {
                const uint32_t e = cq[cn + lane];
                const int lev = (int)(e >> kCluShift);
                const uint32_t m = e & ((1u << kCluShift) - 1u);
                pend = cluster_mask(H, q, lev, level_offset(H.logn, lev) + m, acc);
                ebase = kHitCluster | ((uint32_t)lev << 25) | (m << 1);
            }
            wave_sync();
            continue;
        }
        if (!nonempty) break;
        if (SPAWN && hungry) {
            // some workers wait for tasks: give away up to half of the highest list,
            // at most one node per waiting worker
            const int lh = 31 - __builtin_clz(nonempty);
            if (lh >= split_level) {
                const int ch = __builtin_amdgcn_readlane(cntv, lh);
                // keep at least one item: a lone top item is given only when lower lists hold work
                int d = min(ch >= 2 ? ch / 2 : ((nonempty & ~(1u << lh)) ? 1 : 0), 64);
                unsigned long long slot = 0;
                if (lane == 0 && d > 0) {
                    const long long waiting = (long long)__hip_atomic_load(&Q.ctl->head, __ATOMIC_RELAXED,
                                                                           __HIP_MEMORY_SCOPE_AGENT) -
                                              (long long)__hip_atomic_load(&Q.ctl->tail, __ATOMIC_RELAXED,
                                                                           __HIP_MEMORY_SCOPE_AGENT);
                    d = (int)min((long long)d, max(0ll, waiting));
                    if (d > 0) {
                        slot = __hip_atomic_fetch_add(&Q.ctl->tail, (unsigned long long)d, __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_AGENT);
                        // slots past the capacity are not used: those nodes stay here
                        const long long room = (long long)Q.capacity - (long long)slot;
                        const int dd = (int)max(0ll, min((long long)d, room));
                        if (dd < d) atomicAdd(&Q.ctl->refused, (unsigned long long)(d - dd));
                        d = dd;
                        if (d > 0) {
                            // counted before they become visible
                            __hip_atomic_fetch_add(&Q.ctl->outstanding, (unsigned long long)d, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT);
                            atomicAdd(&Q.ctl->spawned, (unsigned long long)d);
                        }
                    }
                    if (d == 0)
                        __hip_atomic_store(&Q.ctl->starving[blockIdx.x & (kStarveCopies - 1)].v, 0u,
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                d = __builtin_amdgcn_readfirstlane(d);
                slot = uniform_u64(slot);
                if (d > 0) {
                    if (lane < d) {
                        const uint32_t mm = nl.get(lh, ch - 1 - lane) & kCodeMask;  // the top d items
                        Q.tasks[slot + lane] = (qidx << 32) | ((unsigned long long)lh << 26) | (unsigned long long)mm;
                        // the release store orders the task word before its flag
                        __hip_atomic_store(&Q.flags[slot + lane], Q.ctl->epoch, __ATOMIC_RELEASE,
                                           __HIP_MEMORY_SCOPE_AGENT);
                    }
                    if (lane == lh) cntv = ch - d;
                    if (ch == d) nonempty &= ~(1u << lh);
                    acc.donated = true;
                    wave_sync();
                    if (!nonempty) continue;  // (cannot happen: one item is always kept)
                }
            }
        }
        int l = __builtin_ctz(nonempty);
        int cnt = __builtin_amdgcn_readlane(cntv, l);
        if (cnt < 32) {
            // the lowest list would fill less than half a wave: expand the next higher
            // level first, so the lower levels run with fuller waves (what does not fit
            // is re-queued).  Measured on powerlaw2048: thresholds 8 to 32 all take
            // 3 % less time than deferring every list shorter than a full wave.
            const uint32_t higher = nonempty & ~((2u << l) - 1u);
            if (higher) {
                l = __builtin_ctz(higher);
                cnt = __builtin_amdgcn_readlane(cntv, l);
            }
        }
        const int k = min(cnt, 64), base = cnt - k;
        unsigned hv = 0;
        if (SPAWN && lane == 0 && 31 - __builtin_clz(nonempty) >= split_level)
            hv = __hip_atomic_load(&Q.ctl->starving[blockIdx.x & (kStarveCopies - 1)].v, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        if (lane == l) cntv = base;
        if (base == 0) nonempty &= ~(1u << l);
        uint32_t chm = 0;     // children whose boxes contain h (bit c: child 4m + c)
        uint32_t cin = 0;     // children wholly inside the box (bit c)
        uint32_t m4 = 0;      // 4m: the first child's code
        uint32_t tested = 0;  // child boxes read by this lane
        uint32_t cut4 = 0;    // children under the cut (bit c)
        uint32_t all4 = 0;    // children whose own children are all under the cut (bit c)
        uint32_t entry = 0;   // the lane's list item (Morton code | kInside)
        if (lane < k) {
            entry = nl.get(l, base + lane);
            const uint32_t m = entry & kCodeMask;
            const bool inside = (entry & kInside) != 0u;
            if (l == 1) {
                pend = leaf_quad_mask(H, q, m, inside, rx0, ry0, acc);
                ebase = m << 3;
            } else {
                // the four children are one Morton segment; children outside the support
                // are masked afterwards.  Without the cut their octagons (64 B) are read
                // at once.  With it, first their residuals and their children's largest
                // (32 B, four sibling groups to a line) unless all are known to be under
                // the cut, then for each child the one octagon that decides about it: a
                // second round trip, but 96 B at most instead of the three boxes of every
                // child, and from level 3 up mostly one class for the whole group.
                const uint32_t c0 = (uint32_t)level_offset(H.logn, l - 1) + 4u * m;
                uint4 o0, o1, o2, o3;
                if (CUT) {
                    uint32_t k0 = kOctOwn, k1 = kOctOwn, k2 = kOctOwn, k3 = kOctOwn;
                    cut4 = 0xfu;
                    if (!(entry & kAllCut)) {
                        const float4* ep = reinterpret_cast<const float4*>(
                            reinterpret_cast<const char*>(H.clu_em) + c0 * 8u);
                        const float4 ea = ep[0], eb = ep[1];
                        cut4 = (uint32_t)(ea.x <= q.t) | ((uint32_t)(ea.z <= q.t) << 1) |
                               ((uint32_t)(eb.x <= q.t) << 2) | ((uint32_t)(eb.z <= q.t) << 3);
                        all4 = (uint32_t)(ea.y <= q.t) | ((uint32_t)(ea.w <= q.t) << 1) |
                               ((uint32_t)(eb.y <= q.t) << 2) | ((uint32_t)(eb.w <= q.t) << 3);
                        k0 = oct_class(ea.x <= q.t, ea.y <= q.t);
                        k1 = oct_class(ea.z <= q.t, ea.w <= q.t);
                        k2 = oct_class(eb.x <= q.t, eb.y <= q.t);
                        k3 = oct_class(eb.z <= q.t, eb.w <= q.t);
                    }
                    o0 = load_octagon(H, k0, c0);
                    o1 = load_octagon(H, k1, c0 + 1);
                    o2 = load_octagon(H, k2, c0 + 2);
                    o3 = load_octagon(H, k3, c0 + 3);
                } else {
                    const uint4* op = reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(H.oct_k) + c0 * 16u);
                    o0 = op[0]; o1 = op[1]; o2 = op[2]; o3 = op[3];
                }
                uint32_t ov = 0xfu;  // children meeting the support box
                cin = 0xfu;
                if (!inside) {
                    const int I = (int)morton_compact(m), J = (int)morton_compact(m >> 1);
                    const int mk = (H.n >> (l - 1)) - 1;
                    const AxisRuns rx = axis_runs(q.cxlo, q.cxhi, l - 1, mk + 1);
                    const AxisRuns ry = axis_runs(q.cylo, q.cyhi, l - 1, mk + 1);
                    ov = quad_bits(pair_in_run(I, rx.a, rx.n, mk), pair_in_run(J, ry.a, ry.n, mk));
                    cin = quad_bits(pair_in_run(I, rx.ai, rx.ni, mk), pair_in_run(J, ry.ai, ry.ni, mk));
                }
                tested = (uint32_t)__popc(ov);
                chm = ((uint32_t)in_octagon(q, o0) | ((uint32_t)in_octagon(q, o1) << 1) |
                       ((uint32_t)in_octagon(q, o2) << 2) | ((uint32_t)in_octagon(q, o3) << 3)) & ov;
                m4 = 4 * m;
            }
        }
        if (l >= 2) {
            // Children under the cut go to the cluster queue (which holds fewer than 64
            // entries here, so up to 64 x 4 more fit), the others are appended to the
            // level below (which holds fewer than 64 items: it is empty or the short
            // lowest list).  A parent whose list children would run past the list's end
            // goes back to its own list whole and is expanded again later.  Child
            // positions grow with the lane, so the parents that fit are a prefix and the
            // first one with children always fits.
            uint32_t chl = CUT ? chm & ~cut4 : chm;
            const uint32_t chc = CUT ? chm & cut4 : 0u;
            uint32_t che = 0;  // of the list children, those to leave as items
            if (TILES == kTilesEmit && l - 1 >= kTileLevel) {
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if ((chl & (1u << c)) && tile_item<CUT>(H, T, q, l - 1, m4 + c)) che |= 1u << c;
                chl &= ~che;
            }
            const int below = __builtin_amdgcn_readlane(cntv, l - 1);
            int total, nch = __popc(chl), pos = wave_prefix_small(nch, &total);
            bool back = nch > 0 && below + pos + nch > kListCap;
            if (TILES == kTilesEmit && l - 1 >= kTileLevel) {
                // (a parent that goes back leaves no items now: it is expanded again)
                int n;
                const int at = wave_prefix_small(back ? 0 : __popc(che), &n);
                const int64_t out = n ? tile_reserve(T, n) : -1;
                if (out >= 0) {
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        if (!back && (che & (1u << c)))
                            T.raw[out + at + __popc(che & ((1u << c) - 1u))] =
                                tile_word(qidx, l - 1, (m4 + c) | ((cin >> c) & 1u ? kInside : 0u) |
                                                           ((all4 >> c) & 1u ? kAllCut : 0u));
                } else if (n) {
                    // no room: all of them are evaluated here
                    chl |= che;
                    nch = __popc(chl);
                    pos = wave_prefix_small(nch, &total);
                    back = nch > 0 && below + pos + nch > kListCap;
                }
            }
            const uint64_t bb = __ballot(back);
            if (!back) {
                // child c goes to below + pos + (number of list children before it)
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (chl & (1u << c))
                        nl.put(l - 1, below + pos + __popc(chl & ((1u << c) - 1u)),
                               (m4 + c) | ((cin >> c) & 1u ? kInside : 0u) | ((all4 >> c) & 1u ? kAllCut : 0u));
                acc.nodes += tested;
            }
            if (CUT) {
                const uint32_t mine = back ? 0u : chc;
                int ctot;
                const int cpos = cn + wave_prefix_small(__popc(mine), &ctot);
                const uint32_t lev = (uint32_t)(l - 1) << kCluShift;
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (mine & (1u << c)) cq[cpos + __popc(mine & ((1u << c) - 1u))] = lev | (m4 + c);
                cn += ctot;
            }
            const int pushed = bb ? __builtin_amdgcn_readlane(pos, __builtin_ctzll(bb)) : total;
            if (lane == l - 1) cntv = below + pushed;
            if (pushed) nonempty |= 1u << (l - 1);
            if (bb) {
                const int nb = __popcll(bb);
                if (back) nl.put(l, base + __popcll(bb & ((1ull << lane) - 1ull)), entry);
                if (lane == l) cntv = base + nb;
                nonempty |= 1u << l;
            }
        }
        if (SPAWN) hungry = (unsigned)__builtin_amdgcn_readfirstlane((int)hv);
        wave_sync();
    }
}

// Root items of a query: the level-lr nodes overlapping the box, one per lane of an
// 8 x 8 lane grid where *ok is set; Morton codes (level >= 1) or packed texel cells
// (level 0).  At the entry level l0 (node side >= r) at most 3 nodes per axis overlap
// the box, at l0 - 1 at most 5.
__device__ __forceinline__ uint32_t root_item(const HierDev& H, const QuerySetup& q, int lr, bool* ok)
{
    const int lane = threadIdx.x & 63;
    const int M = H.n >> lr, mm = M - 1;
    const int kx0 = q.cxlo >> lr, ky0 = q.cylo >> lr;
    const int nkx = min((q.cxhi >> lr) - kx0 + 1, M), nky = min((q.cyhi >> lr) - ky0 + 1, M);
    const int ra = lane & 7, rb = lane >> 3;
    *ok = ra < nkx && rb < nky;
    const uint32_t I = (uint32_t)((kx0 + ra) & mm), J = (uint32_t)((ky0 + rb) & mm);
    if (lr == 0) return I | (J << 16);
    const int side = 1 << lr;
    const bool inside = axis_inside((int)I * side, side, q.cxlo, q.cxhi, H.logn) &&
                        axis_inside((int)J * side, side, q.cylo, q.cyhi, H.logn);
    return morton(I, J) | (inside ? kInside : 0u);
}

// The level a query's descent starts at.  Without the cut it starts below the entry
// level: the entry level's few large boxes seldom prune, and testing their children
// (at most 5 x 5), or their grandchildren when those fit the 8 x 8 lane grid, as
// roots skips steps that would run with at most 9 or 25 of 64 lanes.  (With the cut
// the entry-level nodes' own residuals decide first, so it starts there.)
template <bool CUT>
__device__ __forceinline__ int descent_start(const HierDev& H, const QuerySetup& q)
{
    if (CUT || q.l0 == 0) return q.l0;
    int lr = q.l0 - 1;
    if (lr >= 1) {
        const int l2 = lr - 1, M2 = H.n >> l2;
        if (min((q.cxhi >> l2) - (q.cxlo >> l2) + 1, M2) <= 8 && min((q.cyhi >> l2) - (q.cylo >> l2) + 1, M2) <= 8)
            lr = l2;
    }
    return lr;
}

// Limb `lane` (32 bits) of a wave-uniform sum, for lanes below 6.
__device__ __forceinline__ unsigned long long limb_of(const Fix192& d, int lane)
{
    const uint64_t w = lane < 2 ? d.w0 : (lane < 4 ? d.w1 : d.w2);
    return lane & 1 ? w >> 32 : w & 0xffffffffull;
}

template <int MODE>
__device__ __forceinline__ void finish(const EvalArgs& a, int64_t qi, const QuerySetup& q,
                                       const Acc& acc)
{
    const Fix192 d = wave_sum_fix(acc.d);
    if (MODE == kModeCount) {
        const uint32_t nodes = wave_sum_u32(acc.nodes), cells = wave_sum_u32(acc.cells);
        const uint32_t clus = wave_sum_u32(acc.clusters), hits = wave_sum_u32(acc.hits);
        if (lane_id() == 0) {
            uint32_t* c = a.counts + 4 * qi;
            c[0] = nodes; c[1] = cells; c[2] = clus; c[3] = hits;
        }
    }
    if (lane_id() == 0) a.out[qi] = fix_to_float(d, q.fexp);
}

template <int MODE>
__device__ __forceinline__ void invalid(const EvalArgs& a, int64_t qi)
{
    if (lane_id() == 0) {
        a.out[qi] = __int_as_float(0x7fc00000);
        if (MODE == kModeCount) {
            uint32_t* c = a.counts + 4 * qi;
            c[0] = c[1] = c[2] = c[3] = 0;
        }
    }
}

// ------------------------------------------------------------ brute force
template <int MODE, int KER>
__global__ __launch_bounds__(256) void k_eval_brute(HierDev H, EvalArgs a)
{
    const int64_t local = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (local >= a.slots) return;
    const int64_t qi = a.slot0 + local;
    const int lane = threadIdx.x & 63;
    const QuerySetup q = setup_wave<KER>(a.q[qi], a.s2r, 0.f, H);
    if (!q.valid) { invalid<MODE>(a, qi); return; }
    const int n = H.n, msk = n - 1;
    const int spanx = q.cxhi - q.cxlo + 1, spany = q.cyhi - q.cylo + 1;
    const int nx = spanx >= n ? n : spanx, ny = spany >= n ? n : spany;
    const int total = nx * ny;  // <= 8192^2
    Acc acc;
    Rec rec{a.ids, a.terms, MODE == kModeRecord ? a.offsets[qi] : 0,
            MODE == kModeRecord ? a.offsets[qi + 1] : 0};
    __shared__ uint32_t hq_all[4 * kHitCap];
    uint32_t* hq = hq_all + (threadIdx.x >> 6) * kHitCap;
    int hn = 0;
    uint32_t pend = 0, ebase = 0;
    int base = 0;
    while (true) {
        queue_hits(hq, hn, pend, ebase);
        if (hn >= 64 || (hn > 0 && base >= total)) {
            const int c = min(hn, 64);
            hn -= c;
            hit_round<MODE, KER>(H, q, hq + hn, c, acc, rec);
            continue;
        }
        if (base >= total) break;
        const int idx = base + lane;
        if (idx < total) {
            const int ca = idx % nx, cb = idx / nx;
            const int i = spanx >= n ? ca : ((q.cxlo + ca) & msk);
            const int j = spany >= n ? cb : ((q.cylo + cb) & msk);
            pend = plane_cell_mask(H, q, i, j, acc);
            ebase = kHitPlane | ((uint32_t)j << 14) | ((uint32_t)i << 1);
        }
        base += 64;
    }
    finish<MODE>(a, qi, q, acc);
}

// ------------------------------------------------------------ hierarchical

// The slot of block b's query.  In a batch with tiles the last slots hold the queries that run
// tiled: of the others the wide ones come first, then the narrow ones, each spread over
// the XCDs by themselves (in eighths of all slots the last XCDs had nothing to do: 2^21
// queries at 8192^2 93.1 ms, so 88.9).  False when none is left.
template <int MODE>
__device__ __forceinline__ bool whole_slot(const EvalArgs& a, int64_t b, int64_t* slot)
{
    if (MODE != kModeValue || !a.narrow) {
        *slot = a.slot0 + xcd_contiguous(b, gridDim.x);
        return *slot < a.slot0 + a.slots;
    }
    const int64_t end = a.slot0 + a.slots;
    const int64_t mid = min(max((int64_t)a.narrow[2], a.slot0), end), last = min(max((int64_t)a.narrow[0], mid), end);
    const int64_t wide = last - mid;
    if (b >= last - a.slot0) return false;
    *slot = b < wide ? mid + xcd_contiguous(b, wide) : a.slot0 + xcd_contiguous(b - wide, mid - a.slot0);
    return true;
}

// One wavefront per workgroup (a long query holds only its own LDS).  LDS: the node
// lists of levels 1..L (NodeLists), the hit queue and, with the cut, the cluster queue.
template <int MODE, bool CUT, int KER>
__global__ __launch_bounds__(64) void k_eval_plain(HierDev H, EvalArgs a)
{
    extern __shared__ uint32_t lds[];
    int64_t slot;
    if (!whole_slot<MODE>(a, blockIdx.x, &slot)) return;
    const int64_t qi = a.order ? (int64_t)a.order[slot] : slot;
    uint32_t* lists = lds;
    const QuerySetup q = setup_wave<KER>(a.q[qi], a.s2r, CUT ? a.tau : 0.f, H);
    if (!q.valid) { invalid<MODE>(a, qi); return; }
    Acc acc;
    Rec rec{a.ids, a.terms, MODE == kModeRecord ? a.offsets[qi] : 0,
            MODE == kModeRecord ? a.offsets[qi + 1] : 0};
    const int lr = descent_start<CUT>(H, q);
    bool ok;
    const uint32_t item = root_item(H, q, lr, &ok);
    TaskQueue none{};
    descend<MODE, CUT, false, KER>(H, q, lists, lr, ok, item, false, 0, 0, none, acc, rec);
    finish<MODE>(a, qi, q, acc);
}

// ------------------------------------------------------------ split
// Small batches: W wavefronts of one workgroup share a query, so that a picked pixel
// or a few hundred rays do not wait for single waves' chains of dependent steps.  The
// roots go down as far as their grid fits W lane grids (8 W' per axis, W' = sqrt(W)),
// and a wave takes every W'-th row and column of it, which spreads the hits.  A query
// of half-width kSplitAlone or less is one wave's work: the others leave at once (with
// them 2048 queries of sigma 1 to 4 took 55 us with 16 waves each, plain 11).
constexpr float kSplitAlone = 16.f;
template <int W>
constexpr int kSplitAxis = W == 16 ? 4 : 2;

// The grid of level-lr nodes over the included cells of one axis: first column
// (unrolled) and count; all of the torus from column 0.
__device__ __forceinline__ void split_axis(int clo, int chi, int lr, int M, int* k0, int* nk)
{
    *k0 = clo >> lr;
    *nk = (chi >> lr) - *k0 + 1;
    if (*nk >= M) {
        *k0 = 0;
        *nk = M;
    }
}

// Do the grid's columns have each ancestor d levels up once (and not at both ends of
// the torus)?
__device__ __forceinline__ bool split_once(int k0, int nk, int d, int M)
{
    return ((k0 + nk - 1) >> d) - (k0 >> d) + 1 <= (M >> d);
}

template <bool CUT, int KER, int W>
__global__ __launch_bounds__(64 * W) void k_eval_split(HierDev H, EvalArgs a)
{
    extern __shared__ uint32_t lds[];
    __shared__ Fix192 sums[W];
    const int64_t qi = a.slot0 + blockIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = lane_id();
    const QuerySetup u = setup_support(a.q[qi], a.s2r);
    const bool alone = !(u.valid && fmaxf(u.rx, u.ry) > kSplitAlone);
    if (alone && wave != 0) return;
    const QuerySetup q = setup_wave<KER>(a.q[qi], a.s2r, CUT ? a.tau : 0.f, H);
    if (!q.valid) {
        invalid<kModeValue>(a, qi);
        return;
    }
    constexpr int S = kSplitAxis<W>;
    int lr = descent_start<CUT>(H, q), kx, nkx, ky, nky;
    split_axis(q.cxlo, q.cxhi, lr, H.n >> lr, &kx, &nkx);
    split_axis(q.cylo, q.cyhi, lr, H.n >> lr, &ky, &nky);
    while (!alone && lr > (CUT ? 1 : 0)) {
        int x, nx, y, ny;
        const int M = H.n >> (lr - 1);
        split_axis(q.cxlo, q.cxhi, lr - 1, M, &x, &nx);
        split_axis(q.cylo, q.cyhi, lr - 1, M, &y, &ny);
        if (nx > 8 * S || ny > 8 * S) break;
        if (CUT && !(split_once(x, nx, q.l0 - lr + 1, M) && split_once(y, ny, q.l0 - lr + 1, M))) break;
        --lr;
        kx = x; nkx = nx; ky = y; nky = ny;
    }
    const int ca = (lane & 7) * (alone ? 1 : S) + wave % S, cb = (lane >> 3) * (alone ? 1 : S) + wave / S;
    bool ok = ca < nkx && cb < nky;
    const int mm = (H.n >> lr) - 1;
    const uint32_t I = (uint32_t)((kx + ca) & mm), J = (uint32_t)((ky + cb) & mm);
    uint32_t item = I | (J << 16);
    int lev = lr;
    if (lr > 0) {
        const int side = 1 << lr;
        const bool inside = axis_inside((int)I * side, side, q.cxlo, q.cxhi, H.logn) &&
                            axis_inside((int)J * side, side, q.cylo, q.cyhi, H.logn);
        const uint32_t m = morton(I, J);
        item = m | (inside ? kInside : 0u);
        if (CUT) {
            // the highest ancestor from the entry level down that is under the cut stands
            // in for its nodes, once: at the first of them that the grid has
            for (int l = lr + 1; l <= q.l0; ++l) {
                const int d = l - lr;
                if (ok && H.clu_em[(uint32_t)level_offset(H.logn, l) + (m >> (2 * d))].x <= q.t) {
                    lev = l;
                    item = m >> (2 * d);
                }
            }
            const int d = lev - lr;
            if (d > 0)
                ok = ok && kx + ca == max(kx, ((kx + ca) >> d) << d) && ky + cb == max(ky, ((ky + cb) >> d) << d);
        }
    }
    Acc acc;
    Rec rec{nullptr, nullptr, 0, 0};
    TaskQueue none{};
    descend<kModeValue, CUT, false, KER, kTilesSplit>(H, q, lds + wave * wave_lds_words(H.L, CUT), lr, ok, item, false, 0, 0,
                                                      none, acc, rec, TileWork{}, lev);
    const Fix192 d = wave_sum_fix(acc.d);
    if (lane == 0) sums[wave] = d;
    __syncthreads();
    if (threadIdx.x == 0) {
        Fix192 t = sums[0];
        for (int w = 1; w < (alone ? 1 : W); ++w) fix_add(t, sums[w]);
        a.out[qi] = fix_to_float(t, q.fexp);
    }
}

// ------------------------------------------------------------ tiles
// Both kernels below run on a fixed grid (the counts are known on the device only):
// a wave claims runs of consecutive pieces of work, from its XCD's eighth of them
// first, so that the waves of an XCD stay on neighbouring queries or on the same few
// tiles.  Claims shrink towards the end of a share.
constexpr unsigned kTileWaves = 256 * 24;  // 24 waves per compute unit are resident

// A plan's kernels read the batch from its control block.
__device__ __forceinline__ void batch_args(EvalArgs& a)
{
    if (a.batch) {
        a.q = a.batch->q;
        a.nq = a.batch->nq;
        a.out = a.batch->out;
    }
}

// A round's wide queries, [first, first + count) of them.  Their number and their items
// are known on the device only, the rounds are launched by the host: round a.slot0 of
// a.slots.  Each round's sort sets how many the next one takes: all that a round can
// hold or, if their items (at this round's number per query) would not fit, as many
// as fill three quarters of the room; no fewer than the rounds that are left need.  What
// does not fit is evaluated where it was found, each query at its own pace through the
// memory: 2^22 queries of sigma 4 to 1024 at 4096^2, tau = 1e-4, with 2^24 items for each
// 2^19 queries 6970 ms, with rounds that fit 3040 (15/16 of the room: 3380).  Many
// rounds start with a small one; a few do not, as one round more costs what it
// reads again (2^21 queries at 8192^2, tau = 1e-3, whose items fit: 92.5 and 94.7 ms).
struct TileRange {
    uint32_t first, count;
};
__device__ __forceinline__ TileRange tile_range(const EvalArgs& a)
{
    const TileCtl* c = a.tile.ctl;
    const int r = (int)a.slot0, rounds = (int)a.slots;
    const uint32_t first = c->first[r & 1];
    const int64_t left = max(a.nq - (int64_t)*a.narrow - (int64_t)first, (int64_t)0);
    const int64_t least = (left + (rounds - r) - 1) / (rounds - r);
    const uint32_t count = r > 0 ? c->count[r & 1] : (rounds > kTileFewRounds ? kTileFirst : a.tile.round);
    return TileRange{first, (uint32_t)min(min(left, (int64_t)a.tile.round), max((int64_t)count, least))};
}

struct Claim {
    uint32_t at, end;
};

// The wave's next run of [0, total), at most `most` long; at == end when none is
// left.  `x` counts the shares already exhausted.
__device__ __forceinline__ Claim claim_run(TileCtl::Count* ctr, uint32_t total, uint32_t most, int* x)
{
    const uint32_t workers = max(1u, gridDim.x / kXcd);
    for (; *x < kXcd; ++*x) {
        const int s = ((int)(blockIdx.x & (kXcd - 1)) + *x) & (kXcd - 1);
        const uint32_t lo = (uint32_t)((uint64_t)total * s / kXcd);
        const uint32_t len = (uint32_t)((uint64_t)total * (s + 1) / kXcd) - lo;
        uint32_t at = len, n = 0;
        if (lane_id() == 0) {
            const uint32_t seen = __hip_atomic_load(&ctr[s].v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (seen < len) {
                n = max(1u, min(most, (len - seen) / (2u * workers)));
                at = atomicAdd(&ctr[s].v, n);
            }
        }
        at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
        n = (uint32_t)__builtin_amdgcn_readfirstlane((int)n);
        if (at < len) return Claim{lo + at, lo + min(at + n, len)};
    }
    return Claim{0, 0};
}

// At one query a claim the counters' atomics, about 70 ns each on one address, set
// the pace (2^19 queries: 4.8 ms).
constexpr uint32_t kWideClaim = 8;

// The wide queries of a round: each leaves its tiles as items and stores its set-up
// and its sum so far (of what it evaluated above or instead of items).
// (5 waves per SIMD: 96 vector registers)
template <bool CUT, int KER>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(5, 8))) void k_tile_emit(HierDev H, EvalArgs a)
{
    extern __shared__ uint32_t lds[];
    batch_args(a);
    a.tile.coarse = a.narrow[1] != 0u;
    const TileWork& T = a.tile;
    const int lane = lane_id();
    const TileRange range = tile_range(a);
    const int64_t first = (int64_t)*a.narrow + range.first;
    if (range.count == 0) return;
    TaskQueue none{};
    Rec rec{nullptr, nullptr, 0, 0};
    int x = 0;
    while (true) {
        const Claim c = claim_run(T.ctl->qclaim, range.count, kWideClaim, &x);
        if (c.at >= c.end) break;
        for (uint32_t local = c.at; local < c.end; ++local) {
            const int64_t qi = (int64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)a.order[first + local]);
            const QuerySetup q = setup_wave<KER>(a.q[qi], a.s2r, CUT ? a.tau : 0.f, H);
            Acc acc;
            const int lr = max(descent_start<CUT>(H, q), kTileLevel);
            bool ok;
            const uint32_t item = root_item(H, q, lr, &ok);
            descend<kModeValue, CUT, false, KER, kTilesEmit>(H, q, lds, lr, ok, item, false, 0, (unsigned long long)local,
                                                             none, acc, rec, T);
            const Fix192 d = wave_sum_fix(acc.d);
            if (lane < 6) T.acc[6 * (size_t)local + lane] = limb_of(d, lane);
            if (lane == 0) T.setup[local] = q;
        }
    }
}

// The items, in tile order.  An item's sum is added limb by limb, which needs no
// carries between waves and nothing to wait for.
constexpr uint32_t kTileClaim = 8;

template <bool CUT, int KER>
__global__ __launch_bounds__(64) void k_eval_tiles(HierDev H, EvalArgs a)
{
    extern __shared__ uint32_t lds[];
    const TileWork& T = a.tile;
    const int lane = lane_id();
    const uint32_t total = T.ctl->total;
    if (total == 0) return;
    batch_args(a);
    // (shorter claims of few items, which the batch waits for at its end, and shortest where
    // queries left up to four of them, whole nodes: 131072 queries at 4096^2, tau = 1e-3, 11.2 and
    // 10.5 ms; items of one tile are too short for so many claims: 8192 queries at 2048^2
    // 1.6 and 3.3 ms)
    const uint32_t most = max(1u, min(kTileClaim, total / ((total / 4u < tile_range(a).count ? 16u : 4u) * gridDim.x)));
    TaskQueue none{};
    Rec rec{nullptr, nullptr, 0, 0};
    int x = 0;
    while (true) {
        const Claim c = claim_run(T.ctl->claim, total, most, &x);
        if (c.at >= c.end) break;
        for (uint32_t i = c.at; i < c.end; ++i) {
            const unsigned long long w = uniform_u64(T.items[i]);
            const uint32_t slot = (uint32_t)(w >> 32);
            const QuerySetup q = uniform_query(T.setup[slot]);
            Acc acc;
            descend<kModeValue, CUT, false, KER, kTilesItem>(H, q, lds, tile_word_level(w), true,
                                                             (uint32_t)w & ~(0xfu << kItemLevelShift), true, 0, 0, none,
                                                             acc, rec);
            if (__ballot((acc.d.w0 | acc.d.w1 | acc.d.w2) != 0ull)) {
                const Fix192 d = wave_sum_fix(acc.d);
                if (lane < 6) atomicAdd(&T.acc[6 * (size_t)slot + lane], limb_of(d, lane));
            }
        }
    }
}

__device__ __forceinline__ void tile_reset(TileCtl* c, int t)
{
    if (t < kTileSegs) c->seg[t].v = 0;
    if (t < kXcd) c->qclaim[t].v = c->claim[t].v = 0;
    if (t == 0) c->total = 0;
    if (t < kMaxTiles) c->hist[t] = c->cursor[t] = 0;
}

// Before a batch.
__device__ __forceinline__ void tile_start(TileCtl* c, int t)
{
    if (t == 0) c->first[0] = 0;
}

constexpr int kTileParts = 8;  // blocks per segment of the sorting passes

// Count the items of each tile (LDS first: one global atomic per tile and block).
__global__ __launch_bounds__(256) void k_tile_hist(TileWork T)
{
    __shared__ uint32_t loc[kMaxTiles];
    const uint32_t seg = blockIdx.x & (kTileSegs - 1), part = blockIdx.x / kTileSegs;
    const uint32_t cnt = min(T.ctl->seg[seg].v, T.segcap);
    if (part * 256u >= cnt) return;
    for (int b = threadIdx.x; b < T.tiles; b += 256) loc[b] = 0u;
    __syncthreads();
    const unsigned long long* raw = T.raw + (size_t)seg * T.segcap;
    for (uint32_t i = part * 256u + threadIdx.x; i < cnt; i += 256u * kTileParts) {
        const unsigned long long w = raw[i];
        if (w != ~0ull) atomicAdd(&loc[tile_word_bin(w)], 1u);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < T.tiles; b += 256)
        if (loc[b]) atomicAdd(&T.ctl->hist[b], loc[b]);
}

// Place the items by tile: each block counts its share again, reserves its range of
// every tile (the tiles' first places are a scan of the counts) and writes.
__global__ __launch_bounds__(256) void k_tile_scatter(EvalArgs a)
{
    batch_args(a);
    const TileWork& T = a.tile;
    const TileRange range = tile_range(a);
    const int next = ((int)a.slot0 + 1) & 1;
    if (range.count == 0) {
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            T.ctl->first[next] = range.first;
            T.ctl->count[next] = 0;
        }
        return;
    }
    __shared__ uint32_t loc[kMaxTiles], first[kMaxTiles], part_sum[256];
    const uint32_t seg = blockIdx.x & (kTileSegs - 1), part = blockIdx.x / kTileSegs;
    const uint32_t cnt = min(T.ctl->seg[seg].v, T.segcap);
    const bool none = part * 256u >= cnt;
    if (none && blockIdx.x != 0) return;
    const int t = threadIdx.x, per = (T.tiles + 255) / 256;
    uint32_t sum = 0;
    for (int k = 0; k < per; ++k)
        if (t * per + k < T.tiles) sum += T.ctl->hist[t * per + k];
    part_sum[t] = sum;
    __syncthreads();
    for (int o = 1; o < 256; o <<= 1) {
        const uint32_t v = t >= o ? part_sum[t - o] : 0u;
        __syncthreads();
        part_sum[t] += v;
        __syncthreads();
    }
    if (blockIdx.x == 0 && t == 255) T.ctl->total = part_sum[255];
    if (blockIdx.x == 0 && t < 64) {
        const uint32_t asked = wave_sum_u32(t < kTileSegs ? T.ctl->seg[t].v : 0u);
        const uint64_t room = (uint64_t)T.segcap * kTileSegs;
        if (t == 0) {
            T.ctl->first[next] = range.first + range.count;
            const bool fits = (uint64_t)asked * T.round <= room * range.count;
            T.ctl->count[next] = fits ? T.round : (uint32_t)((uint64_t)range.count * (room / 4 * 3) / asked);
        }
    }
    uint32_t run = part_sum[t] - sum;
    for (int k = 0; k < per; ++k)
        if (t * per + k < T.tiles) {
            first[t * per + k] = run;
            loc[t * per + k] = 0u;
            run += T.ctl->hist[t * per + k];
        }
    __syncthreads();
    if (none) return;
    const unsigned long long* raw = T.raw + (size_t)seg * T.segcap;
    for (uint32_t i = part * 256u + t; i < cnt; i += 256u * kTileParts) {
        const unsigned long long w = raw[i];
        if (w != ~0ull) atomicAdd(&loc[tile_word_bin(w)], 1u);
    }
    __syncthreads();
    for (int b = t; b < T.tiles; b += 256)
        if (loc[b]) loc[b] = first[b] + atomicAdd(&T.ctl->cursor[b], loc[b]);
    __syncthreads();
    for (uint32_t i = part * 256u + t; i < cnt; i += 256u * kTileParts) {
        const unsigned long long w = raw[i];
        if (w != ~0ull) T.items[atomicAdd(&loc[tile_word_bin(w)], 1u)] = w;
    }
}

// Results of the round's wide queries: the limbs' carries into the 192-bit sum.  The
// last thing of a round, so it clears the control block for the next one.
__global__ __launch_bounds__(256) void k_tile_finish(EvalArgs a)
{
    batch_args(a);
    const int t = blockIdx.x * 256 + threadIdx.x;
    tile_reset(a.tile.ctl, t);
    const TileRange range = tile_range(a);
    const int64_t first = (int64_t)*a.narrow + range.first;
    for (int64_t local = t; local < (int64_t)range.count; local += (int64_t)gridDim.x * 256) {
        const unsigned long long* w = a.tile.acc + 6 * local;
        uint64_t limb[6], carry = 0;
        for (int k = 0; k < 6; ++k) {
            const uint64_t lo = (w[k] & 0xffffffffull) + (carry & 0xffffffffull);
            limb[k] = lo & 0xffffffffull;
            carry = (lo >> 32) + (w[k] >> 32) + (carry >> 32);
        }
        const Fix192 d{limb[0] | (limb[1] << 32), limb[2] | (limb[3] << 32), limb[4] | (limb[5] << 32)};
        a.out[a.order[first + local]] = fix_to_float(d, a.tile.setup[local].fexp);
    }
}

// ------------------------------------------------------------ persistent
// Exact atomic accumulation of a 192-bit value: each word is added atomically and
// every carry out of a word is added to the next one, so once all atomics have
// completed the sum is exact whatever their interleaving.
__device__ __forceinline__ void acc_atomic_add(Fix192* dst, const Fix192& v)
{
    unsigned long long* w = (unsigned long long*)dst;
    unsigned long long c1 = 0, c2 = 0;
    if (v.w0) {
        const unsigned long long old = atomicAdd(&w[0], (unsigned long long)v.w0);
        c1 = (old + v.w0 < old) ? 1ull : 0ull;
    }
    if (v.w1) {
        const unsigned long long old = atomicAdd(&w[1], (unsigned long long)v.w1);
        c2 += (old + v.w1 < old) ? 1ull : 0ull;
    }
    if (c1) {
        const unsigned long long old = atomicAdd(&w[1], 1ull);
        c2 += (old + 1ull < old) ? 1ull : 0ull;
    }
    if (v.w2 + c2) atomicAdd(&w[2], (unsigned long long)(v.w2 + c2));
}

__global__ void k_persist_reset(QueueCtl* ctl, Fix192* acc, int* fexp, const pndf_query* q,
                                long long nq, float* out, unsigned epoch, uint32_t* hist, int nb, TileCtl* tiles)
{
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    for (long long i = t; i < nq; i += (long long)gridDim.x * blockDim.x) {
        acc[i].w0 = 0;
        acc[i].w1 = 0;
        acc[i].w2 = 0;
        fexp[i] = 0;
    }
    if (hist)
        for (long long i = t; i < 2 * nb; i += (long long)gridDim.x * blockDim.x) hist[i] = 0;
    if (tiles)
        for (long long i = t; i < kMaxTiles; i += (long long)gridDim.x * blockDim.x) {
            tile_reset(tiles, (int)i);
            tile_start(tiles, (int)i);
        }
    if (t == 0) {
        for (int x = 0; x < kXcds; ++x) ctl->qhead[x].v = 0;
        ctl->head = 0;
        ctl->tail = 0;
        ctl->outstanding = 0;
        for (int c = 0; c < kStarveCopies; ++c) ctl->starving[c].v = ctl->done[c].v = 0;
        ctl->spawned = ctl->refused = ctl->spins = 0;
        ctl->epoch = epoch;
        ctl->error = 0;
        ctl->q = q;
        ctl->out = out;
        ctl->nq = nq;
    }
}

// Queries taken by one worker per claim: an eighth of the share's remaining queries
// per worker of the XCD, at most kMaxChunk, down to single queries for the share's
// last part (so that no wave ends up holding several large footprints at the end).
// Every claim is an atomic on the share's counter, which all the XCD's workers
// hit: at one claim per few cheap queries its line serialised them (powerlaw2048
// took 18.2 ms with at most 4 queries per claim, 13.6 ms with up to 32; claims
// sized by the time of the previous chunk, or without reading the counter first,
// were slower on the scratched map's heavy tail).
constexpr int kMaxChunk = 32;
constexpr int kChunkDiv = 8;

__device__ __forceinline__ unsigned long long ld_relaxed(const unsigned long long* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void add_relaxed(unsigned long long* p, long long v)
{
    __hip_atomic_fetch_add(p, (unsigned long long)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ bool all_taken(QueueCtl* ctl, long long nq)
{
    for (int x = 0; x < kXcds; ++x)
        if ((long long)ld_relaxed(&ctl->qhead[x].v) < nq * (x + 1) / kXcds - nq * x / kXcds) return false;
    return true;
}

// A unit of work is over: a worker's whole query phase (counted when the worker
// starts, ended when it finds no query left), or a donated task (counted by its
// donor before it is published).  The decrement that leaves nothing outstanding
// after every query was taken ends the run: it raises the done flags the waiting
// workers poll.  (A worker that starts late counts itself before looking for
// queries and finds none, so the count cannot leave zero while work remains.)
__device__ __forceinline__ void unit_done(QueueCtl* ctl, long long nq)
{
    const unsigned long long old = __hip_atomic_fetch_add(&ctl->outstanding, (unsigned long long)-1ll,
                                                          __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (old == 1 && all_taken(ctl, nq))
        for (int c = 0; c < kStarveCopies; ++c)
            __hip_atomic_store(&ctl->done[c].v, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Worker waves of a persistent run.  A wave takes chunks of consecutive queries of
// the processing order, from its XCD's eighth of the order first (shrinking towards
// single queries as a share runs out, so the last ones spread over all workers).
// Once no query is left it takes a ticket of the task queue and waits for that
// slot's task (a subtree some busy wave gave away), polling only that slot's flag
// with a short exponential back-off and, now and then, whether the run is over
// (every query taken and nothing outstanding).
// (5 waves per SIMD fit without spilling vector registers)
template <bool CUT, int KER>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5, 8))) void k_persist(HierDev H, PersistArgs pa)
{
    extern __shared__ uint32_t lds[];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    uint32_t* lists = lds + (size_t)wave * wave_lds_words(H.L, CUT);
    QueueCtl* ctl = pa.Q.ctl;
    const long long nall = ctl->nq, nq = pa.narrow ? (long long)*pa.narrow : nall;  // (the wide ones run tiled)
    const pndf_query* qs = ctl->q;
    const unsigned epoch = ctl->epoch;
    // worker waves per XCD (block b runs on XCD b mod 8)
    const long long xworkers = max(1ll, (long long)gridDim.x * (blockDim.x >> 6) / kXcds);
    const int home = blockIdx.x & (kXcds - 1);
    Rec rec{nullptr, nullptr, 0, 0};
    // a wave that has waited pa.wait_ticks of the constant-rate clock without any
    // work arriving gives up and flags the run (a broken count would otherwise hang)
    long long idle_since = -1;
    int backoff = 1;
    unsigned long long spins = 0;
    long long qb = 0, qe = 0;  // the wave's current chunk of query slots
    long long ticket = -1;     // the wave's place in the task queue while it waits for a task
    int polls = 0;
    bool querying = true;      // in the query phase (counted as one outstanding unit)
    if (lane == 0) add_relaxed(&ctl->outstanding, 1);
    while (true) {
        long long task_slot = -1;
        if (qb >= qe) {
            long long nb = -1, ne = -1;
            if (lane == 0) {
                if (ticket < 0) {
                    // a chunk of queries: from this XCD's share of the processing order
                    // first (neighbouring queries, so the XCD's L2 holds their nodes), then
                    // from the other shares (one atomic per chunk, on the share's own line)
                    for (int k = 0; querying && nb < 0 && k < kXcds; ++k) {
                        const int x = (home + k) & (kXcds - 1);
                        const long long lo = nq * x / kXcds, len = nq * (x + 1) / kXcds - lo;
                        const long long qh = (long long)ld_relaxed(&ctl->qhead[x].v);
                        if (qh >= len) continue;
                        const long long c =
                            max(1ll, min((long long)kMaxChunk, (len - qh) / (kChunkDiv * xworkers)));
                        const long long qn = (long long)__hip_atomic_fetch_add(
                            &ctl->qhead[x].v, (unsigned long long)c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        if (qn < len) {
                            nb = lo + qn;
                            ne = lo + min(qn + c, len);
                        }
                    }
                    if (nb < 0 && querying) {
                        // every query is taken: the query phase is over
                        querying = false;
                        unit_done(ctl, nq);
                    }
                    if (nb < 0) {
                        // no query left: take a ticket (the next task slot in order) and tell
                        // the busy waves that workers are waiting
                        ticket = (long long)__hip_atomic_fetch_add(&ctl->head, 1ull, __ATOMIC_RELAXED,
                                                                   __HIP_MEMORY_SCOPE_AGENT);
                        polls = 0;
                        for (int c = 0; c < kStarveCopies; ++c)
                            __hip_atomic_store(&ctl->starving[c].v, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
                }
                // a relaxed poll (an acquire load would invalidate this CU's L1 under the
                // busy waves at every poll); the acquire fence only once the task is there
                if (nb < 0 && ticket >= 0 && ticket < (long long)pa.Q.capacity &&
                    __hip_atomic_load(&pa.Q.flags[ticket], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == epoch) {
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                    task_slot = ticket;
                    ticket = -1;
                }
            }
            task_slot = (long long)uniform_u64((unsigned long long)task_slot);
            nb = (long long)uniform_u64((unsigned long long)nb);
            ne = (long long)uniform_u64((unsigned long long)ne);
            ticket = (long long)uniform_u64((unsigned long long)ticket);
            if (task_slot < 0 && nb < 0) {
                // waiting for the ticket's task (a slot past the capacity never gets one);
                // the run is over once every query is taken and nothing is outstanding
                int done = 0;
                if (lane == 0) {
                    ++spins;
                    done = __hip_atomic_load(&ctl->done[home].v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u;
                    if (!done && (++polls & 63) == 0) {
                        // now and then the full condition too, and a reminder to the busy waves
                        done = (all_taken(ctl, nq) && ld_relaxed(&ctl->outstanding) == 0) ? 1 : 0;
                        if (!done)
                            for (int c = 0; c < kStarveCopies; ++c)
                                __hip_atomic_store(&ctl->starving[c].v, 1u, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT);
                    }
                    const long long now = wall_clock64();
                    if (idle_since < 0) idle_since = now;
                    if (!done && now - idle_since > pa.wait_ticks) {
                        atomicOr(&ctl->error, 1u);
                        done = 1;
                    }
                }
                done = __builtin_amdgcn_readfirstlane(done);
                if (done) break;
                for (int k = 0; k < backoff; ++k) __builtin_amdgcn_s_sleep(16);
                backoff = min(backoff * 2, 8);
                continue;
            }
            idle_since = -1;
            backoff = 1;
            if (nb >= 0) {
                qb = nb;
                qe = ne;
            }
        }
        // one work item: a stolen subtree, or the next query of the chunk
        long long qi;
        int lev;
        uint32_t item;
        bool root_ok, tested;
        if (task_slot >= 0) {
            // the slot is published (its flag carries this run's epoch); never use a
            // malformed task word
            unsigned long long word = 0;
            int ok = 0;
            if (lane == 0) {
                word = pa.Q.tasks[task_slot];
                const long long wq = (long long)(word >> 32);
                const int wl = (int)((word >> 26) & 0x3fu);
                const uint64_t wm = word & 0x3ffffffu;
                ok = 1;
                if (wq >= nall || wl < 1 || wl > H.L || wm >= (uint64_t)(H.n >> wl) * (uint64_t)(H.n >> wl)) {
                    atomicOr(&ctl->error, 4u);
                    ok = 0;
                }
            }
            ok = __builtin_amdgcn_readfirstlane(ok);
            word = uniform_u64(word);
            if (!ok) {
                if (lane == 0) unit_done(ctl, nq);
                continue;
            }
            qi = (long long)(word >> 32);
            lev = (int)((word >> 26) & 0x3fu);
            item = (uint32_t)(word & 0x3ffffffu);
            root_ok = lane == 0;
            tested = true;
        } else {
            qi = pa.order ? (long long)pa.order[qb] : qb;
            qi = (long long)uniform_u64((unsigned long long)qi);
            ++qb;
            lev = -1;  // set below from the query
            item = 0;
            root_ok = false;
            tested = false;
        }
        const QuerySetup q = setup_wave<KER>(qs[qi], pa.s2r, CUT ? pa.tau : 0.f, H);
        Acc acc;
        if (lev < 0) {
            lev = descent_start<CUT>(H, q);
            item = root_item(H, q, lev, &root_ok);
        }
        // a query whose levels are all below split_level never donates; a stolen
        // subtree may be split again
        if (q.valid)
            descend<kModeValue, CUT, true, KER>(H, q, lists, lev, root_ok, item, tested, pa.split_level,
                                           (unsigned long long)qi, pa.Q, acc, rec);
        const Fix192 d = wave_sum_fix(acc.d);
        if (lane == 0) {
            if (task_slot >= 0) {
                acc_atomic_add(&pa.acc[qi], d);
            } else {
                pa.fexp[qi] = q.valid ? q.fexp : 0x7fffffff;
                if (acc.donated)
                    acc_atomic_add(&pa.acc[qi], d);  // tasks of this query add theirs too
                else
                    pa.acc[qi] = d;                  // the only contribution
            }
        }
        if (task_slot >= 0) {
            // the task is finished.  No fence: the count only decides when workers stop;
            // the sums are read after the kernel ends.
            if (lane == 0) unit_done(ctl, nq);
        }
    }
    if (lane == 0 && spins) atomicAdd(&ctl->spins, spins);
}

__global__ void k_persist_finalize(const QueueCtl* ctl, const Fix192* acc, const int* fexp)
{
    const long long nq = ctl->nq;
    float* out = ctl->out;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < nq;
         i += (long long)gridDim.x * blockDim.x) {
        const int e = fexp[i];
        out[i] = e == 0x7fffffff ? __int_as_float(0x7fc00000) : fix_to_float(acc[i], e);
    }
}

template <bool CUT, int KER>
void launch_split(const HierDev& H, const EvalArgs& a, hipStream_t s)
{
    const size_t lds = sizeof(uint32_t) * wave_lds_words(H.L, CUT);
    const dim3 grid((unsigned)a.slots);
    if (a.split == 16)
        hipLaunchKernelGGL((k_eval_split<CUT, KER, 16>), grid, dim3(1024), 16 * lds, s, H, a);
    else
        hipLaunchKernelGGL((k_eval_split<CUT, KER, 4>), grid, dim3(256), 4 * lds, s, H, a);
}

// Launches cover at most launch_chunk() queries (grid dimensions stay far below
// 2^32 work-items).
template <int MODE, int KER>
hipError_t launch_mode(const HierDev& H, const EvalArgs& a0, int algo, hipStream_t s)
{
    const int64_t chunk = launch_chunk();
    for (int64_t off = 0; off < a0.nq; off += chunk) {
        EvalArgs a = a0;
        a.slot0 = off;
        a.slots = std::min<int64_t>(chunk, a0.nq - off);
        if (algo == PNDF_ALGO_BRUTE) {
            const unsigned blocks = (unsigned)((a.slots + 3) / 4);
            hipLaunchKernelGGL((k_eval_brute<MODE, KER>), dim3(blocks), dim3(256), 0, s, H, a);
        } else if (MODE == kModeValue && a.split) {
            if (a.tau > 0.f) launch_split<true, KER>(H, a, s);
            else launch_split<false, KER>(H, a, s);
        } else {
            const unsigned blocks = (unsigned)a.slots;
            const size_t lds = sizeof(uint32_t) * wave_lds_words(H.L, a.tau > 0.f);
            if (a.tau > 0.f)
                hipLaunchKernelGGL((k_eval_plain<MODE, true, KER>), dim3(blocks), dim3(64), lds, s, H, a);
            else
                hipLaunchKernelGGL((k_eval_plain<MODE, false, KER>), dim3(blocks), dim3(64), lds, s, H, a);
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int MODE>
hipError_t launch_kernel(const HierDev& H, const EvalArgs& a, int algo, hipStream_t s)
{
    if (a.kernel == PNDF_KERNEL_BOX) return launch_mode<MODE, PNDF_KERNEL_BOX>(H, a, algo, s);
    if (a.kernel == PNDF_KERNEL_DISK) return launch_mode<MODE, PNDF_KERNEL_DISK>(H, a, algo, s);
    return launch_mode<MODE, PNDF_KERNEL_GAUSSIAN>(H, a, algo, s);
}

// ------------------------------------------------------------ query order
constexpr int kOrderBits = 6;  // 64 x 64 buckets

__global__ void k_order_zero(OrderArgs o)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    for (int i = t; i < 2 * o.bins; i += gridDim.x * blockDim.x) o.hist[i] = 0;
    if (o.ctl) {
        tile_reset(o.ctl, t);
        tile_start(o.ctl, t);
    }
}

constexpr int kOrderMaxBins = (1 << (2 * kOrderBits)) + 2 * (1 << (2 * kOrderBits - kOrderWideShift));
constexpr int kOrderThreads = 1024;

__device__ __forceinline__ uint32_t order_bucket(const pndf_query& q, int n, int bshift)
{
    if (!(fabsf(q.x) <= 16777216.0f && fabsf(q.y) <= 16777216.0f)) return 0;  // (NaN too)
    const uint32_t cx = (uint32_t)((int)floorf(q.x) & (n - 1)) >> bshift;
    const uint32_t cy = (uint32_t)((int)floorf(q.y) & (n - 1)) >> bshift;
    return morton(cx, cy);
}

// Does a wide query take few nodes (see kLightNodes)?  Its descent goes to about the level
// where half of the nodes are under the cut, between the levels whose means its threshold lies
// between.
__device__ __forceinline__ bool is_light(const OrderArgs& o, const QuerySetup& u)
{
    if (!(u.t > 0.f)) return false;
    const float t = log2f(u.t);
    float below = o.level_e[1], level = 1.f;
    for (int l = 2; l <= o.logn; ++l) {
        const float e = o.level_e[l];
        if (t <= below) break;
        level = t < e ? (float)(l - 1) + (t - below) / (e - below) : (float)l;
        below = e;
    }
    const float n = (float)o.n;
    return log2f(fminf(2.f * u.rx, n) * fminf(2.f * u.ry, n)) - 2.f * level <= kLightNodes;
}

// The bucket of a query; with tiles (bins > nb) the wide ones' come last, the light ones before the others.
__device__ __forceinline__ uint32_t order_key(const pndf_query& q, const OrderArgs& o)
{
    const uint32_t k = order_bucket(q, o.n, o.bshift);
    if (o.bins > o.nb) {
        // (a query the evaluation rejects is not wide: k_eval_plain answers it)
        QuerySetup u = setup_support(q, o.s2r);
        if (u.valid && fmaxf(u.rx, u.ry) > (float)(1 << kTileLevel)) {
            u.t = o.tau > 0.f ? __fmul_rn(__fmul_rn(u.rx, u.ry), o.tau) : -1.f;
            return o.nb + (is_light(o, u) ? 0 : o.nb >> kOrderWideShift) + (k >> kOrderWideShift);
        }
    }
    return k;
}

// How the wide queries run (one thread); first holds the bins' first places.
__device__ __forceinline__ void order_narrow(const OrderArgs& o, int64_t nq, const uint32_t* first)
{
    const uint32_t narrow = first[o.nb], heavy = first[o.nb + (o.nb >> kOrderWideShift)];
    const uint32_t tiled = (uint64_t)nq - narrow > (o.logn > 11 ? 2 * kLightMin : kLightMin) ? heavy : narrow;
    o.narrow[0] = tiled;
    o.narrow[1] = ((uint64_t)nq - tiled) << (2 * (o.logn - kTileLevel)) > (tiled == narrow ? 3 * kTileFine : kTileFine);
    o.narrow[2] = narrow;
}

// The histogram and the scatter count in LDS first, so the global counters see one
// atomic per non-empty bin per workgroup instead of one per query; a workgroup takes
// a strided share of the batch (order_blocks).
__device__ __forceinline__ void order_hist(const pndf_query* __restrict__ q, int64_t nq, const OrderArgs& o)
{
    __shared__ uint32_t loc[kOrderMaxBins];
    for (int b = threadIdx.x; b < o.bins; b += blockDim.x) loc[b] = 0u;
    __syncthreads();
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nq;
         i += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t k = order_key(q[i], o);
        o.key[i] = k;
        atomicAdd(&loc[k], 1u);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < o.bins; b += blockDim.x)
        if (loc[b]) atomicAdd(&o.hist[b], loc[b]);
}

// exclusive scan of `bins` counters into LDS (in place if they are there) by a workgroup of
// 1024 threads: each thread's run of counters, the wave's threads by shuffles, the waves'
// sums from LDS
__device__ __forceinline__ void order_scan(const uint32_t* hist, int bins, uint32_t* first)
{
    constexpr int per = (kOrderMaxBins + kOrderThreads - 1) / kOrderThreads;
    __shared__ uint32_t part[kOrderThreads / 64];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    uint32_t v[per], sum = 0;
#pragma unroll
    for (int k = 0; k < per; ++k) {
        v[k] = t * per + k < bins ? hist[t * per + k] : 0u;
        sum += v[k];
    }
    uint32_t run = sum;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t u = __shfl_up(run, o);
        if (lane >= o) run += u;
    }
    if (lane == 63) part[wave] = run;
    __syncthreads();
    run -= sum;
    for (int w = 0; w < wave; ++w) run += part[w];
#pragma unroll
    for (int k = 0; k < per; ++k)
        if (t * per + k < bins) {
            first[t * per + k] = run;
            run += v[k];
        }
    __syncthreads();
}

// Each workgroup reserves, per bin, a range of the exact size of its share's count
// (one global atomic per non-empty bin), then places its queries in it.  Within a
// bucket the order is whatever the atomics give: results do not depend on it.
// first: the bins' first places (LDS).
__device__ __forceinline__ void order_scatter(const uint32_t* __restrict__ key, int64_t nq, int bins, const uint32_t* first,
                                              uint32_t* __restrict__ cursor, uint32_t* __restrict__ order)
{
    __shared__ uint32_t loc[kOrderMaxBins];
    for (int b = threadIdx.x; b < bins; b += blockDim.x) loc[b] = 0u;
    __syncthreads();
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = i0; i < nq; i += stride) atomicAdd(&loc[key[i]], 1u);
    __syncthreads();
    for (int b = threadIdx.x; b < bins; b += blockDim.x)
        if (loc[b]) loc[b] = first[b] + atomicAdd(&cursor[b], loc[b]);
    __syncthreads();
    for (int64_t i = i0; i < nq; i += stride) order[atomicAdd(&loc[key[i]], 1u)] = (uint32_t)i;
}

__global__ __launch_bounds__(kOrderThreads) void k_order_hist(OrderArgs o)
{
    order_hist(o.batch ? o.batch->q : o.q, o.batch ? o.batch->nq : o.nq, o);
}

__global__ __launch_bounds__(kOrderThreads) void k_order_scatter(OrderArgs o)
{
    __shared__ uint32_t first[kOrderMaxBins];
    order_scan(o.hist, o.bins, first);
    const int64_t nq = o.batch ? o.batch->nq : o.nq;
    if (o.narrow && blockIdx.x == 0 && threadIdx.x == 0) order_narrow(o, nq, first);
    order_scatter(o.key, nq, o.bins, first, o.hist + o.bins, o.order);
}

// The whole order of a batch of up to kOrderSmall queries by one workgroup, keys and places
// within the buckets in registers: such a batch waits for the order as long as for its
// queries (4096 narrow ones: 15 us in three launches, 8.5 in this one).
constexpr int kOrderSmallPer = 8;
constexpr int64_t kOrderSmall = (int64_t)kOrderSmallPer * kOrderThreads;
__global__ __launch_bounds__(kOrderThreads) void k_order_small(OrderArgs o)
{
    __shared__ uint32_t loc[kOrderMaxBins];
    const pndf_query* q = o.batch ? o.batch->q : o.q;
    const int nq = (int)(o.batch ? o.batch->nq : o.nq), t = threadIdx.x;
    for (int b = t; b < o.bins; b += kOrderThreads) loc[b] = 0u;
    if (o.ctl && !o.batch) {  // (a plan's reset has done it)
        tile_reset(o.ctl, t);
        tile_start(o.ctl, t);
    }
    __syncthreads();
    uint32_t key[kOrderSmallPer], at[kOrderSmallPer];
#pragma unroll
    for (int k = 0; k < kOrderSmallPer; ++k) {
        const int i = t + k * kOrderThreads;
        if (i < nq) key[k] = order_key(q[i], o);
    }
#pragma unroll
    for (int k = 0; k < kOrderSmallPer; ++k)
        if (t + k * kOrderThreads < nq) at[k] = atomicAdd(&loc[key[k]], 1u);
    __syncthreads();
    order_scan(loc, o.bins, loc);
    if (o.narrow && t == 0) order_narrow(o, nq, loc);
#pragma unroll
    for (int k = 0; k < kOrderSmallPer; ++k) {
        const int i = t + k * kOrderThreads;
        if (i < nq) o.order[loc[key[k]] + at[k]] = (uint32_t)i;
    }
}

}  // namespace

void order_shape(int logn, int* nb, int* bshift)
{
    const int bits = logn < kOrderBits ? logn : kOrderBits;
    *nb = 1 << (2 * bits);
    *bshift = logn - bits;
}

// Workgroups of the histogram and scatter passes: 4 queries a thread in small batches
// (64 x 64 buckets and one workgroup per 16384 queries took 65 us of a 16384-query
// tile's 253), at most one workgroup per compute unit.
static unsigned order_blocks(int64_t nq)
{
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>(256, (nq + 4095) / 4096));
}

// The three passes of the spatial order into buf = order[nq] | key[nq] | hist[2 bins] |
// narrow[3] (the counters are cleared by a kernel, never a memset node).
static OrderArgs order_args(const HierDev& H, int64_t nq, float s2r, float tau, TileCtl* ctl, uint32_t* buf)
{
    OrderArgs o{};
    order_shape(H.logn, &o.nb, &o.bshift);
    o.nq = nq;
    o.n = H.n;
    o.bins = order_bins(o.nb, ctl != nullptr);
    o.s2r = s2r;
    o.tau = tau;
    o.logn = H.logn;
    o.level_e = H.level_e;
    o.order = buf;
    o.key = buf + nq;
    o.hist = o.key + nq;
    o.ctl = ctl;
    o.narrow = ctl ? o.hist + 2 * o.bins : nullptr;
    return o;
}

static hipError_t order_passes(const HierDev& H, const pndf_query* q, int64_t nq, float s2r, float tau, TileCtl* ctl, uint32_t* buf,
                               const uint32_t** narrow, hipStream_t s)
{
    OrderArgs o = order_args(H, nq, s2r, tau, ctl, buf);
    o.q = q;
    if (narrow) *narrow = o.narrow;
    if (nq <= kOrderSmall) {
        hipLaunchKernelGGL(k_order_small, dim3(1), dim3(kOrderThreads), 0, s, o);
        return hipGetLastError();
    }
    const unsigned g = order_blocks(nq);
    hipLaunchKernelGGL(k_order_zero, dim3(8), dim3(kOrderThreads), 0, s, o);
    hipLaunchKernelGGL(k_order_hist, dim3(g), dim3(kOrderThreads), 0, s, o);
    hipLaunchKernelGGL(k_order_scatter, dim3(g), dim3(kOrderThreads), 0, s, o);
    return hipGetLastError();
}

hipError_t make_order(const HierDev& H, const pndf_query* q, int64_t nq, float s2r, float tau, OrderWork* w, hipStream_t s)
{
    *w = OrderWork{};
    int nb, bshift;
    order_shape(H.logn, &nb, &bshift);
    // tiles | order[nq] | key[nq] | counters
    size_t tiles = tiles_bytes(H, nq);
    auto bytes = [&] { return tiles + sizeof(uint32_t) * (2 * (size_t)nq + order_words(nb, tiles != 0)); };
    hipError_t e = stream_alloc(&w->mem, bytes(), s);
    if (e != hipSuccess && tiles) {
        (void)hipGetLastError();
        tiles = 0;
        e = stream_alloc(&w->mem, bytes(), s);
    }
    if (e != hipSuccess) {
        w->mem = nullptr;
        return e;
    }
    if (tiles) tiles_place(H, nq, w->mem, &w->tile);
    w->order = reinterpret_cast<uint32_t*>(static_cast<char*>(w->mem) + tiles);
    return order_passes(H, q, nq, s2r, tau, w->tile.ctl, w->order, &w->narrow, s);
}

// Workspace of the spatial order for callers that cannot allocate: one array per
// GPU, held until the process ends, for batches of up to kStaticOrderQueries
// queries (order, keys and the largest histogram: 32 MiB + 16 KiB).  Its device
// address is looked up once per device; host code uses that address, never the
// array's name.  Every call on a GPU shares it, so calls that overlap on one GPU
// race.
static __device__ __align__(256) uint32_t scratch[2 * kStaticOrderQueries + 2 * 4096 + 64];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
uint32_t* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t make_order_static(const HierDev& H, const pndf_query* q, int64_t nq, uint32_t** order, hipStream_t s)
{
    *order = nullptr;
    if (nq > kStaticOrderQueries) return hipErrorInvalidValue;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    uint32_t* buf = nullptr;
    {
        std::lock_guard<std::mutex> g(g_scratch_mu);
        if (!g_scratch_ptr[dev]) {
            void* p = nullptr;
            e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
            if (e != hipSuccess) return e;
            g_scratch_ptr[dev] = static_cast<uint32_t*>(p);
        }
        buf = g_scratch_ptr[dev];
    }
    int nb, bshift;
    order_shape(H.logn, &nb, &bshift);
    if (nb > 4096) return hipErrorInvalidValue;
    e = order_passes(H, q, nq, 0.f, 0.f, nullptr, buf, nullptr, s);
    if (e == hipSuccess) *order = buf;
    return e;
}

static size_t tiles_layout(const HierDev& H, int64_t nq, char* base, TileWork* w)
{
    *w = TileWork{};
    if (!has_tiles(H.logn)) return 0;
    const int64_t chunk = std::min(kTileChunk, launch_chunk()), slots = std::min(nq, chunk);
    w->round = (uint32_t)chunk;
    w->tiles = 1 << (2 * (H.logn - kTileLevel));
    // twice every tile of every query (the segments fill unevenly), up to kTileItems for
    // a whole chunk; the rest is evaluated where it was found
    const int64_t items = std::min<int64_t>(2 * slots * w->tiles, kTileItems / kTileChunk * chunk);
    w->segcap = (uint32_t)((items + kTileSegs - 1) / kTileSegs);
    Arena mem;
    mem.base = base;
    mem.place(&w->ctl, 1);
    mem.place(&w->raw, (size_t)w->segcap * kTileSegs);
    mem.place(&w->items, (size_t)w->segcap * kTileSegs);
    mem.place(&w->acc, 6 * (size_t)slots);
    mem.place(&w->setup, (size_t)slots);
    return mem.size;
}

size_t tiles_bytes(const HierDev& H, int64_t nq)
{
    TileWork w;
    return tiles_layout(H, nq, nullptr, &w);
}

void tiles_place(const HierDev& H, int64_t nq, void* base, TileWork* w) { tiles_layout(H, nq, static_cast<char*>(base), w); }

static hipError_t launch_tiles(const HierDev& H, EvalArgs a, hipStream_t s);

hipError_t launch_eval(const HierDev& H, const EvalArgs& a, int algo, hipStream_t s)
{
    if (a.nq <= 0) return hipSuccess;
    if (a.offsets) return launch_kernel<kModeRecord>(H, a, algo, s);
    if (a.counts) return launch_kernel<kModeCount>(H, a, algo, s);
    const hipError_t e = launch_kernel<kModeValue>(H, a, algo, s);
    return e == hipSuccess && a.narrow ? launch_tiles(H, a, s) : e;
}

// ---------------------------------------------------------------- persistent
// The launch sequence reset -> workers -> finalize, as a HIP graph.  Only the
// reset node's arguments (queries, count, output, epoch) change between runs; the
// workers and the finalizer read them from the control block.
static void reset_params(PersistPlan& P, const pndf_query* q, long long nq, float* out)
{
    P.rq = q;
    P.rnq = nq;
    P.rout = out;
    P.rargs[0] = &P.ctl;
    P.rargs[1] = &P.acc;
    P.rargs[2] = &P.fexp;
    P.rargs[3] = &P.rq;
    P.rargs[4] = &P.rnq;
    P.rargs[5] = &P.rout;
    P.rargs[6] = &P.epoch;
    P.rargs[7] = &P.ohist;
    P.rargs[8] = &P.order_bins;
    P.rargs[9] = &P.tile.ctl;
    P.reset.func = (void*)k_persist_reset;
    P.reset.gridDim = dim3((unsigned)std::min<long long>(1024, (P.max_nq + 255) / 256 + 1));
    P.reset.blockDim = dim3(256);
    P.reset.sharedMemBytes = 0;
    P.reset.kernelParams = P.rargs;
    P.reset.extra = nullptr;
}

// The worker kernel for a plan's cut setting and footprint kernel.
static void* persist_func(const PersistPlan& P)
{
    const bool cut = P.tau > 0.f;
    if (P.kernel == PNDF_KERNEL_BOX) return cut ? (void*)k_persist<true, PNDF_KERNEL_BOX> : (void*)k_persist<false, PNDF_KERNEL_BOX>;
    if (P.kernel == PNDF_KERNEL_DISK)
        return cut ? (void*)k_persist<true, PNDF_KERNEL_DISK> : (void*)k_persist<false, PNDF_KERNEL_DISK>;
    return cut ? (void*)k_persist<true, PNDF_KERNEL_GAUSSIAN> : (void*)k_persist<false, PNDF_KERNEL_GAUSSIAN>;
}

// Worker blocks of the plan's kernel that fit on one compute unit at once
// (registers and LDS), 0 if the runtime cannot tell.
int persist_resident_blocks(const HierDev& H, const PersistPlan& P)
{
    int nb = 0;
    const size_t lds = sizeof(uint32_t) * 4 * wave_lds_words(H.L, P.tau > 0.f);
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, persist_func(P), 256, lds) != hipSuccess) return 0;
    return nb;
}

// The tile kernels for a plan's or call's cut setting and footprint kernel.
struct TileFuncs {
    void *emit, *tiles;
};
static TileFuncs tile_funcs(bool cut, int kernel)
{
    if (kernel == PNDF_KERNEL_BOX)
        return cut ? TileFuncs{(void*)k_tile_emit<true, PNDF_KERNEL_BOX>, (void*)k_eval_tiles<true, PNDF_KERNEL_BOX>}
                   : TileFuncs{(void*)k_tile_emit<false, PNDF_KERNEL_BOX>, (void*)k_eval_tiles<false, PNDF_KERNEL_BOX>};
    if (kernel == PNDF_KERNEL_DISK)
        return cut ? TileFuncs{(void*)k_tile_emit<true, PNDF_KERNEL_DISK>, (void*)k_eval_tiles<true, PNDF_KERNEL_DISK>}
                   : TileFuncs{(void*)k_tile_emit<false, PNDF_KERNEL_DISK>, (void*)k_eval_tiles<false, PNDF_KERNEL_DISK>};
    return cut ? TileFuncs{(void*)k_tile_emit<true, PNDF_KERNEL_GAUSSIAN>, (void*)k_eval_tiles<true, PNDF_KERNEL_GAUSSIAN>}
               : TileFuncs{(void*)k_tile_emit<false, PNDF_KERNEL_GAUSSIAN>, (void*)k_eval_tiles<false, PNDF_KERNEL_GAUSSIAN>};
}

// The five launches of one round of wide queries (arguments a, kernels f); `add`
// launches a kernel or appends it to a graph: add(function, grid, block, LDS bytes,
// arguments).
template <typename Add>
static hipError_t tile_round(const HierDev& H, EvalArgs& a, const TileFuncs& f, Add add)
{
    const size_t lds = sizeof(uint32_t) * wave_lds_words(H.L, a.tau > 0.f);
    const int64_t left = std::min<int64_t>(a.nq, a.tile.round);
    void* both[] = {(void*)&H, (void*)&a};
    void* tile[] = {(void*)&a.tile};
    void* all[] = {(void*)&a};
    const dim3 sort(kTileSegs * kTileParts), b64(64), b256(256);
    const unsigned fin = (unsigned)std::max<int64_t>(kMaxTiles / 256, std::min<int64_t>(1024, (left + 255) / 256));
    hipError_t e = add(f.emit, dim3((unsigned)std::min<int64_t>(kTileWaves, left)), b64, lds, both);
    if (e == hipSuccess) e = add((void*)k_tile_hist, sort, b256, 0, tile);
    if (e == hipSuccess) e = add((void*)k_tile_scatter, sort, b256, 0, all);
    if (e == hipSuccess) e = add(f.tiles, dim3(kTileWaves), b64, lds, both);
    if (e == hipSuccess) e = add((void*)k_tile_finish, dim3(fin), b256, 0, all);
    return e;
}

// Rounds of a batch's wide queries (their number is known on the device only: a round
// without any costs its five launches, 13 us).  As many as hold all queries; in large
// batches twice that, so that rounds may be smaller where queries leave many items.
static int64_t tile_rounds(int64_t nq, int64_t round)
{
    const int64_t n = (nq + round - 1) / round, half = std::max<int64_t>(1, round / 2);
    return n <= kTileFewRounds ? n : (nq + half - 1) / half;
}

static hipError_t launch_tiles(const HierDev& H, EvalArgs a, hipStream_t s)
{
    const TileFuncs f = tile_funcs(a.tau > 0.f, a.kernel);
    a.slots = tile_rounds(a.nq, a.tile.round);
    for (a.slot0 = 0; a.slot0 < a.slots; ++a.slot0) {
        const hipError_t e = tile_round(H, a, f, [&](void* fn, dim3 g, dim3 b, size_t lds, void** args) {
            return hipLaunchKernel(fn, g, b, args, lds, s);
        });
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

void persist_prepare(const HierDev& H, PersistPlan& P)
{
    P.H = H;
    P.pa.Q.ctl = P.ctl;
    P.pa.Q.tasks = P.tasks;
    P.pa.Q.flags = P.flags;
    P.pa.Q.capacity = P.capacity;
    P.pa.order = P.order;
    P.pa.acc = P.acc;
    P.pa.fexp = P.fexp;
    P.pa.tau = P.tau;
    P.pa.s2r = P.s2r;
    P.pa.kernel = P.kernel;
    P.pa.split_level = P.split_level;
    P.pa.wait_ticks = P.wait_ticks;
    P.ohist = nullptr;
    P.pa.narrow = nullptr;
    P.targs.clear();
    if (!P.order) return;
    P.oargs = order_args(H, P.max_nq, P.s2r, P.tau, P.tile.ctl, P.order);
    P.oargs.batch = P.ctl;
    P.ohist = P.oargs.hist;
    P.order_bins = P.oargs.bins;
    P.pa.narrow = P.oargs.narrow;
    if (!P.tile.ctl) return;
    const int64_t rounds = tile_rounds(P.max_nq, P.tile.round);
    for (int64_t r = 0; r < rounds; ++r) {
        EvalArgs a{nullptr, P.order, P.max_nq, r,       rounds, nullptr,  nullptr,     nullptr,
                   nullptr, nullptr, P.tau,    P.s2r, P.kernel, P.pa.narrow, P.tile};
        a.batch = P.ctl;
        P.targs.push_back(a);
    }
}

hipError_t persist_graph_build(const HierDev& H, PersistPlan& P)
{
    persist_prepare(H, P);
    reset_params(P, nullptr, 0, nullptr);
    P.wargs[0] = &P.H;
    P.wargs[1] = &P.pa;
    hipKernelNodeParams work{};
    work.func = persist_func(P);
    work.gridDim = dim3((unsigned)P.blocks);
    work.blockDim = dim3(256);
    work.sharedMemBytes = (unsigned)(sizeof(uint32_t) * 4 * wave_lds_words(H.L, P.tau > 0.f));
    work.kernelParams = P.wargs;
    work.extra = nullptr;
    P.fargs[0] = &P.ctl;
    P.fargs[1] = &P.acc;
    P.fargs[2] = &P.fexp;
    hipKernelNodeParams fin{};
    fin.func = (void*)k_persist_finalize;
    fin.gridDim = dim3((unsigned)std::min<long long>(1024, (P.max_nq + 255) / 256 + 1));
    fin.blockDim = dim3(256);
    fin.sharedMemBytes = 0;
    fin.kernelParams = P.fargs;
    fin.extra = nullptr;
    hipError_t e = hipGraphCreate(&P.graph, 0);
    if (e == hipSuccess) e = hipGraphAddKernelNode(&P.reset_node, P.graph, nullptr, 0, &P.reset);
    hipGraphNode_t last = P.reset_node;
    auto chain = [&](const hipKernelNodeParams& p) {
        hipGraphNode_t node = nullptr;
        const hipError_t r = hipGraphAddKernelNode(&node, P.graph, &last, 1, &p);
        last = node;
        return r;
    };
    auto add = [&](void* fn, dim3 g, dim3 b, size_t lds, void** args) {
        hipKernelNodeParams p{};
        p.func = fn;
        p.gridDim = g;
        p.blockDim = b;
        p.sharedMemBytes = (unsigned)lds;
        p.kernelParams = args;
        return chain(p);
    };
    P.hargs[0] = &P.oargs;
    if (P.order) {
        const dim3 g(order_blocks(P.max_nq)), b(kOrderThreads);
        if (P.max_nq <= kOrderSmall) {
            if (e == hipSuccess) e = add((void*)k_order_small, dim3(1), b, 0, P.hargs);
        } else {
            if (e == hipSuccess) e = add((void*)k_order_hist, g, b, 0, P.hargs);
            if (e == hipSuccess) e = add((void*)k_order_scatter, g, b, 0, P.hargs);
        }
    }
    if (e == hipSuccess) e = chain(work);
    if (e == hipSuccess) e = chain(fin);  // (writes zeros for the wide queries, which the tiles then overwrite)
    const TileFuncs f = tile_funcs(P.tau > 0.f, P.kernel);
    for (size_t r = 0; r < P.targs.size() && e == hipSuccess; ++r) e = tile_round(P.H, P.targs[r], f, add);
    if (e == hipSuccess) e = hipGraphInstantiate(&P.exec, P.graph, nullptr, nullptr, 0);
    return e;
}

hipError_t persist_run(PersistPlan& P, const pndf_query* q, long long nq, float* out, bool use_graph,
                       hipStream_t s)
{
    ++P.epoch;
    reset_params(P, q, nq, out);
    if (use_graph) {
        hipError_t e = hipGraphExecKernelNodeSetParams(P.exec, P.reset_node, &P.reset);
        if (e == hipSuccess) e = hipGraphLaunch(P.exec, s);
        return e;
    }
    hipLaunchKernelGGL(k_persist_reset, P.reset.gridDim, P.reset.blockDim, 0, s, P.ctl, P.acc, P.fexp,
                       q, nq, out, P.epoch, P.ohist, P.order_bins, P.tile.ctl);
    if (P.order && P.max_nq <= kOrderSmall) {
        hipLaunchKernelGGL(k_order_small, dim3(1), dim3(kOrderThreads), 0, s, P.oargs);
    } else if (P.order) {
        hipLaunchKernelGGL(k_order_hist, dim3(order_blocks(P.max_nq)), dim3(kOrderThreads), 0, s, P.oargs);
        hipLaunchKernelGGL(k_order_scatter, dim3(order_blocks(P.max_nq)), dim3(kOrderThreads), 0, s, P.oargs);
    }
    const size_t lds = sizeof(uint32_t) * 4 * wave_lds_words(P.H.L, P.tau > 0.f);
    void* args[] = {&P.H, &P.pa};
    hipError_t e = hipLaunchKernel(persist_func(P), dim3((unsigned)P.blocks), dim3(256), args, lds, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_persist_finalize, P.reset.gridDim, dim3(256), 0, s, P.ctl, P.acc, P.fexp);
    e = hipGetLastError();
    const TileFuncs f = tile_funcs(P.tau > 0.f, P.kernel);
    for (size_t r = 0; r < P.targs.size() && e == hipSuccess; ++r)
        e = tile_round(P.H, P.targs[r], f, [&](void* fn, dim3 g, dim3 b, size_t l, void** x) {
            return hipLaunchKernel(fn, g, b, x, l, s);
        });
    return e;
}

}  // namespace pndf
