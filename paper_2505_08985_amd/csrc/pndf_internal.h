// Internal definitions of the gfx950 P-NDF library: handle layouts, the device
// view passed to kernels, and the device helpers shared by the evaluation
// kernels (query setup, periodic-image arithmetic, triangle tests, hit terms).
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>

#include <atomic>
#include <cstdint>
#include <string>
#include <vector>

#include "../../include/pndf.h"

namespace pndf {

constexpr int kMaxLevels = 13;   // N <= 8192
constexpr int kWave = 64;
#ifndef PNDF_LIST_CAP
#define PNDF_LIST_CAP 128
#endif
// Per-level traversal list entries.  A wave expands up to 64 parents at a time;
// parents whose children do not fit wait in their own list.  The roots of a query
// fill up to an 8 x 8 lane grid (64 entries of one list), and children are appended
// to a list that is empty or holds fewer than 32 entries (the short lowest list,
// expanded after the level above it), so with at least 64 entries the first
// parent's four children always fit and the descent progresses.  (Fewer entries
// would mean more waves per CU, but roots would overflow.)
constexpr int kListCap = PNDF_LIST_CAP;
static_assert(kListCap >= 64, "a list holds up to 64 roots; a short list (< 32) plus four children must fit");

// Kernel launches cover at most this many queries (one workgroup or one wavefront
// each), so grids stay far below 2^32 work-items.  PNDF_LAUNCH_CHUNK in the
// environment lowers it (any positive value; used by the tests to force several
// launches per call, which must give the same bits).
constexpr int64_t kLaunchChunk = (int64_t)1 << 24;
int64_t launch_chunk();

// Hit queue of a wavefront: float32 hits wait here for the FP64 stage, which takes
// them 64 at a time (fewer than 64 wait between steps; one step adds at most 64 x 8).
constexpr int kHitCap = 128;

// Cluster queue of a wavefront (with the cluster cut): nodes under the cut wait here
// to be tested 64 at a time; it holds fewer than 64 before a descent step, which adds
// at most 64 x 4.
constexpr int kCluCap = 64 + 4 * 64;

// With the cluster cut, list items of the levels from short_list_level(L, true) up
// take 16 bits: a level-l Morton code is below 4^(L - l), so from l = L - 7 it fits
// 14 bits beside the two flag bits.  Fewer LDS bytes per wavefront let more
// wavefronts reside, which pays where LDS limits them (the cut kernel: powerlaw8192
// 1169 -> 1015 ms); without the cut the kernel is not LDS-limited and the extra
// registers of the 16-bit path cost a wavefront per SIMD, so all its lists stay
// 32-bit (short level L + 1).
__host__ __device__ inline int short_list_level(int L, bool cut)
{
    return !cut ? L + 1 : (L - 7 > 1 ? L - 7 : 1);
}

// 32-bit LDS words of a wavefront's node lists: 32-bit lists of levels 1..S-1, then
// 16-bit lists of levels S..L.
__host__ __device__ inline size_t list_words(int L, bool cut)
{
    const int S = short_list_level(L, cut);
    return (size_t)(S - 1) * kListCap + (size_t)(L - S + 1) * (kListCap / 2);
}
static_assert(kListCap % 2 == 0, "16-bit lists fill whole words");

// 32-bit LDS words per wavefront of the descent: the node lists of levels 1..L, the
// hit queue, and with the cut the cluster queue.
__host__ __device__ inline size_t wave_lds_words(int L, bool cut)
{
    return list_words(L, cut) + kHitCap + (cut ? kCluCap : 0);
}

// Level-1 leaf record: the 3 x 3 texel normals of a 2 x 2 cell block (row-major,
// texel (2I + x, 2J + y) at t[3 y + x], periodic) and the clamp bits of its four
// cells (cell (di, dj) at deg[2 dj + di]), 80 bytes = five 16-byte loads.
struct QuadRec {
    float2 t[9];
    uint8_t deg[4];
    uint32_t pad;
};
static_assert(sizeof(QuadRec) == 80, "QuadRec is five 16-byte words");

// Device-side view of a mesh + hierarchy, passed to kernels by value.  Every
// per-node array is stored per level in Morton (Z) order: node (I, J) of level l at
// level_offset(logn, l) + morton(I, J), so the four children of node m are 4m .. 4m + 3.
struct HierDev {
    const float2* nrm;      // (n+1) x (n+1) padded texel normals (last row/column wrap)
    const uint8_t* deg;     // n x n clamp bits (bit0 lower, bit1 upper)
    const float2* det;      // n x n Jacobians (lower, upper), eps when clamped (projected area)
    const QuadRec* quad;    // level-1 leaf records (Morton order)
    // the cluster test record, 2 float4 per node: (N0.x, N0.y, N1.x, N1.y), (N2.x,
    // N2.y, N3.x, N3.y), except that a clamped triangle's free vertex (N0 of the
    // lower, N3 of the upper: its replacement is built from the shared edge N1 N2
    // alone) holds NaN, so the record carries the clamp bits (clamp_bits)
    const float4* clu_t;
    const float* clu_e;     // e^l per node
    int n, L, logn;
    float eps;
    float rho;              // circumradius of the clamp replacement triangle (area eps / 2)
    uint32_t nodes;         // nodes of all levels
    // octagons of the traversal (see kOctSub): oct_k the map triangles beneath the node
    // (tau = 0); with clusters oct_c holds three arrays of `nodes` octagons, indexed
    // cls * nodes + node: kOctSub the map and cluster triangles beneath the node,
    // kOctOwn its own two cluster triangles, kOctKids (from level 2) the union of its
    // four children's kOctOwn
    const uint4* oct_k;
    const uint4* oct_c;
    const float2* clu_em;   // per node e^l and the largest e^l of its four children (+inf at level 1)
    const float2* tile_e;   // maps with tiles: per node of level kTileLevel and above (packed like the others, from
                            // level kTileLevel on) the largest e^l kTileDepth and kTileSpan levels beneath
    const float* level_e;   // with tiles, per level from 1: logarithm (base 2) of a middle residual
};

// Clamp bits of a cluster test record (a, b) = clu_t[2 idx], clu_t[2 idx + 1]: bit 0
// the lower triangle (N0 stored as NaN), bit 1 the upper (N3 stored as NaN).  (The
// build keeps IEEE semantics, so x != x is the NaN test.)
__device__ __forceinline__ uint32_t clamp_bits(float4 a, float4 b)
{
    return (a.x != a.x ? 1u : 0u) | (b.z != b.z ? 2u : 0u);
}

// Order key of a half-precision value (IEEE binary16 bits): unsigned keys compare
// like the values (negative values mirrored below 0x8000, zero signs aside), so
// bounds are tested two at a time with packed 16-bit integer operations.  Octagon
// bounds are normalised so that the two zeros never exclude: a minimum of +0 is
// stored as -0 (key 0x7fff) and a maximum of -0 as +0 (key 0x8000).
__host__ __device__ __forceinline__ uint32_t half_key(uint32_t bits)
{
    return (bits & 0x8000u) ? (~bits & 0xffffu) : (bits | 0x8000u);
}

// Octagon of a set of normals (16 B): the bounds of x, y, u = x + y and v = x - y,
// each rounded outward to half precision and stored as order keys,
//   .x = min x | min y << 16, .y = max x | max y << 16, .z = min u | min v << 16,
//   .w = max u | max v << 16.
// The two diagonal slabs cut the corners that an axis-aligned box leaves empty: on
// the power-law maps a descent expands 26 % fewer nodes than with boxes, on the
// scratched maps, whose grooves put a node's normals along a slanted line, 28 to
// 36 % fewer and tests 45 % fewer clusters and leaf records (counted on the CPU,
// 2048^2 maps).  2^20 queries of sigma 1 to 64 on the 2048^2 power-law map, tau = 0:
// 8.93 -> 7.67 ms; 2^21 of sigma 1 to 8192 at 8192^2, tau = 1e-3: 108 -> 97 ms (both
// with the hit stage's Jacobians formed instead of read).  Rounding is monotone: u and v are rounded to FP64 both here and for
// the query's normal, so an octagon never excludes a normal of its set.
enum { kOctSub = 0, kOctOwn = 1, kOctKids = 2 };

// First node of level l (1 <= l <= logn + 1) in the packed per-level arrays: the
// levels below hold sum_{k=1}^{l-1} (n / 2^k)^2 = (n^2 - (n / 2^(l-1))^2) / 3 nodes.
__host__ __device__ __forceinline__ int64_t level_offset(int logn, int l)
{
    // 32-bit arithmetic suffices (n <= 8192: 4^13 = 2^26 nodes at most)
    return (int64_t)(((1u << (2 * logn)) - (1u << (2 * (logn - l + 1)))) / 3u);
}

// ---- exact accumulation: unsigned 192-bit fixed point w0 + 2^64 w1 + 2^128 w2, in
// units of 2^fexp.  Adding the float32 terms of a query in any order gives the same
// integer, so every evaluation algorithm (brute force, descent, split across waves)
// returns the same D.
struct Fix192 {
    uint64_t w0, w1, w2;
};

// Global task queue of the persistent traversal, a ticket queue: a worker with no
// query left takes a ticket (fetch-add on `head`) and waits for that slot only; a
// busy wave that sees workers waiting (head > tail) reserves slots with a fetch-add
// on `tail`, writes the tasks and publishes each by storing the launch's epoch into
// its flag.  No CAS retry loop, so thousands of waiting workers do not serialise on
// one word.  `outstanding` counts query chunks and tasks taken or published but not
// finished; a worker exits once every query is taken and nothing is outstanding.
// Every word of the control block that many waves touch sits on its own 128-byte
// line, so the pollers of one do not queue behind the users of another.
constexpr int kStarveCopies = 8;  // replicas of the starving flag (by block index)
constexpr int kXcds = 8;          // workgroups are dispatched to the 8 XCDs round-robin
struct QueueCtl {
    struct alignas(128) Head {
        unsigned long long v;
    } qhead[kXcds];                               // next query slot of each XCD's share of the order
    alignas(128) unsigned long long head;         // tickets handed out (task slots waited for)
    alignas(128) unsigned long long tail;         // task slots reserved by donors
    alignas(128) unsigned long long outstanding;  // query chunks and tasks taken or published, not finished
    struct alignas(128) Flag {
        unsigned int v;
    } starving[kStarveCopies];                    // set by idle workers, cleared by a donation
    Flag done[kStarveCopies];                     // set once every query is taken and nothing is outstanding
    alignas(128) unsigned long long spawned, refused, spins;  // statistics
    unsigned int epoch, error;      // error bit0: idle wait gave up, bit1: slot wait gave up, bit2: bad task
    const pndf_query* q;
    float* out;
    long long nq;
};

struct TaskQueue {
    QueueCtl* ctl;
    unsigned long long* tasks;  // (query << 32) | (level << 26) | Morton code of the node
    unsigned int* flags;        // epoch of the launch that published the slot
    unsigned long long capacity;
};

struct QuerySetup;

// Tiled evaluation of wide footprints.  The nodes of level kTileLevel (256 x 256
// texels) are tiles: everything the descent reads beneath one is about 3.7 MB, the
// size of an XCD's L2.  The spatial order puts the queries that enter above that
// level last; k_tile_emit descends them to it and leaves their surviving tiles as
// items, the items are sorted by tile, and the waves of an XCD work through
// neighbouring items, so that a tile's nodes come from memory about once per launch
// instead of once per query.  An item holds the place of its query and the list item
// (Morton code and flags) of its node, with the node's level.
//
// Under the cut the descent ends higher up and a tile may hold a few nodes only,
// while an item costs about 700 vector instructions before its first useful one.  So
// a node above the tile level becomes an item as a whole when all nodes kTileSpan
// levels beneath it are under the cut (its part of the hierarchy is then as large as
// a tile's at most), and a node all of whose descendants kTileDepth levels down are
// under it is evaluated on the spot.  Measured (spans 7, 8, 9, 11; one item a tile of
// level 8 otherwise): 2^21 queries at 8192^2, tau = 1e-3: 130, 98, 94, 106 ms (97
// untiled); 60001 queries of sigma 4 to 1024 on the 4096^2 scratched map, tau = 1e-4:
// 158 -> 47 ms at any span, L2 misses 7.7e9 -> 4e7, the vector ALU then always busy.
//
// A batch of few wide queries has every item one tile: a whole node's item is one wave's work
// and decides when the batch ends.  Wide queries x tiles up to 3 kTileFine (tau = 1e-3, sigma 90
// to an eighth of the map, with items of whole nodes and with tiles alone): 8192 queries at
// 2048^2 2276 and 1533 us; 128 at 8192^2 1714 and 456 us, 8192 3.7 and 4.0 ms, 16384 5.5 and
// 7.1; 10000 at 4096^2 (sigma 90 to 1000) 5.1 and 3.7 ms, 16384 of sigma 90 to 4000 5.0 and 6.1.
// Without the light queries (see OrderArgs), which are most of those that whole nodes make
// long, up to kTileFine: 15000 others at 4096^2 9.6 and 12.5 ms.
constexpr int kTileLevel = 8;
constexpr int kTileDepth = 3, kTileSpan = 9;
constexpr uint64_t kTileFine = (uint64_t)1 << 20;
constexpr int kTileSegs = 64;                        // item segments, each with a counter of its own
constexpr int kMaxTiles = 1 << (2 * (13 - kTileLevel));
constexpr int64_t kTileChunk = (int64_t)1 << 19;     // most wide queries per round
constexpr int kTileFewRounds = 4;
constexpr uint32_t kTileFirst = 1u << 17;            // the first of more rounds, before their items are known
constexpr int64_t kTileItems = (int64_t)1 << 24;     // items per round
// Maps with tiles: below 1024^2 there are fewer than 16 and the caches hold the map.
__host__ __device__ inline bool has_tiles(int logn) { return logn >= kTileLevel + 2; }
struct TileCtl {
    struct alignas(128) Count {
        uint32_t v;
    } seg[kTileSegs], qclaim[8], claim[8];           // items written per segment; queries, items claimed per XCD's share
    alignas(128) uint32_t total;                     // items after sorting
    uint32_t first[2], count[2];                     // wide queries of the even and the odd rounds (see tile_range)
    alignas(128) uint32_t hist[kMaxTiles], cursor[kMaxTiles];
};
struct TileWork {
    TileCtl* ctl;                   // nullptr: evaluate every query as a whole
    unsigned long long* raw;        // kTileSegs segments of segcap items
    unsigned long long* items;      // sorted by tile
    unsigned long long* acc;        // per wide query: six 32-bit limbs of its exact sum, each in a 64-bit word
    QuerySetup* setup;              // per wide query
    uint32_t segcap, round;         // room of a segment; most wide queries per round
    int tiles;                      // tiles of the map
    bool coarse;                    // nodes above the tile level become items (set by k_tile_emit)
};

struct EvalArgs {
    const pndf_query* q;
    const uint32_t* order;     // optional processing order (query index per slot)
    int64_t nq;
    int64_t slot0, slots;      // the launch covers processing slots [slot0, slot0 + slots)
    float* out;
    uint32_t* counts;          // nullptr unless counting
    const uint64_t* offsets;   // hit-record pass only
    uint64_t* ids;
    float* terms;
    float tau;
    float s2r;
    int kernel;                // PNDF_KERNEL_*
    const uint32_t* narrow;    // with tiles: slots from *narrow on hold the queries that run tiled (see OrderArgs)
    TileWork tile;
    int split = 0;                    // wavefronts per query of a small batch (4 or 16; 0: one)
    const QueueCtl* batch = nullptr;  // a plan's tile kernels: the batch (q, nq, out) is read from here
};
struct PersistArgs {
    TaskQueue Q;
    const uint32_t* order;  // processing order of the queries (nullptr: input order)
    const uint32_t* narrow; // with tiles: slots from *narrow on hold the wide queries (nullptr: none)
    Fix192* acc;     // per-query exact sums
    int* fexp;       // per-query binary point (written by the query's root task)
    float tau, s2r;
    int kernel;           // PNDF_KERNEL_*
    int split_level;      // smallest level whose nodes may be donated (>= 1)
    long long wait_ticks; // give-up bound of a worker's waits, in wall_clock64 ticks
};

// Arguments of the spatial order's passes.  With tiles, the buckets from nb on hold the
// wide queries, 8 x 8 coarser than the others' (k_tile_emit reads the upper levels only,
// and its items are sorted by tile).  As many as the others have made the passes
// longer (a 16384-query tile 188 us and 180) and
// gained nothing (60001 wide queries 46.8 and 46.9 ms).
//
// Wide queries that the cut leaves few nodes lose by tiles, whose items cost more than such
// a query's cache misses.  The nodes that a query visits (counted on power-law and scratched
// maps of 1024^2 to 8192^2, tau 1e-4 to 1e-2) are 0.8 to 1.6 times the area of its
// support in nodes of the level at which half of the nodes are under the cut (2 to 3 times on
// the scratched ones); up to 2^kLightNodes of them a wide query is light.  In batches of more
// than kLightMin wide queries (twice that above 2048^2) the light ones are evaluated whole;
// fewer leave the GPU idle that way.  tau = 1e-3, power law, sigma 1 to the map's side, with
// all of the wide ones tiled, with this rule, and before there were tiles: 131072 queries at
// 2048^2 9.4, 5.7 and 7.9 ms, at 1024^2 5.7, 3.1 and 4.9; 2^21 at 8192^2 88.9, 78.0 and
// 107.5.  A limit of 2^14.6 takes 12 % longer at 2048^2, one of 2^15.4 15 % at 8192^2.
constexpr int kOrderWideShift = 6;
constexpr float kLightNodes = 15.f;
constexpr uint64_t kLightMin = 8192;
struct OrderArgs {
    const pndf_query* q;
    int64_t nq;
    const QueueCtl* batch;     // a plan's passes: q and nq are read from here
    int n, bshift, nb, bins;   // bins = order_bins()
    float s2r, tau;
    int logn;
    const float* level_e;
    uint32_t* key;
    uint32_t* hist;            // bins counters, then bins cursors
    uint32_t* order;
    uint32_t* narrow;          // with tiles: the first slot that runs tiled, whether items may be whole nodes, narrow queries
    TileCtl* ctl;
};
// 32-bit words of the order's counters (the passes' histogram, cursors and narrow).
inline int order_bins(int nb, bool tiles) { return tiles ? nb + 2 * (nb >> kOrderWideShift) : nb; }
inline size_t order_words(int nb, bool tiles) { return 2 * (size_t)order_bins(nb, tiles) + 3; }

// Device resources and the instantiated launch graph of a persistent plan.
struct PersistPlan {
    QueueCtl* ctl = nullptr;
    Fix192* acc = nullptr;
    int* fexp = nullptr;
    unsigned long long* tasks = nullptr;
    unsigned int* flags = nullptr;
    unsigned long long capacity = 0;
    uint32_t* order = nullptr;  // order[max_nq] | key[max_nq] | order_words(...) counters (nullptr: input order)
    int order_bins = 0;
    void* tile_mem = nullptr;
    TileWork tile{};            // wide queries run tiled on maps with tiles (ctl nullptr: none)
    std::vector<EvalArgs> targs;  // per round: arguments of its tile kernels
    long long max_nq = 0;
    int blocks = 0, split_level = 1;
    long long wait_ticks = 0;
    float tau = 0.f, s2r = 3.f;
    int kernel = 0;
    unsigned epoch = 0;
    HierDev H{};
    PersistArgs pa{};
    // graph and the argument storage its kernel nodes point to
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    hipGraphNode_t reset_node = nullptr;
    hipKernelNodeParams reset{};
    const pndf_query* rq = nullptr;
    long long rnq = 0;
    float* rout = nullptr;
    uint32_t* ohist = nullptr;  // view into `order`
    void* rargs[10];
    void* wargs[2];
    void* fargs[3];
    OrderArgs oargs{};  // order passes: histogram, scatter
    void* hargs[1];
};

// Fill the device arguments of a plan whose buffers are allocated.
void persist_prepare(const HierDev& H, PersistPlan& P);
// Worker blocks of the plan's kernel (cut setting and footprint kernel) resident per
// compute unit at once; 0 if unknown.
int persist_resident_blocks(const HierDev& H, const PersistPlan& P);
// persist_prepare, then build and instantiate the launch graph.
hipError_t persist_graph_build(const HierDev& H, PersistPlan& P);
hipError_t persist_run(PersistPlan& P, const pndf_query* q, long long nq, float* out, bool use_graph,
                       hipStream_t s);

}  // namespace pndf

struct pndf_mesh {
    std::atomic<int> refs{1};
    int device = 0;
    int n = 0, L = 0;
    float eps = 0.f;
    float2* nrm = nullptr;
    uint8_t* deg = nullptr;
    float2* det = nullptr;
    int64_t bytes = 0;
    void* mem = nullptr;   // the one allocation behind the arrays
};

struct pndf_hier {
    pndf_mesh* mesh = nullptr;
    int cluster = 0;
    int L = 0;
    int64_t nodes = 0;
    float4* bbox = nullptr;
    float4* bbox_all = nullptr;
    uint4* oct_k = nullptr;
    uint4* oct_c = nullptr;       // 3 x nodes (kOctSub, kOctOwn, kOctKids)
    float2* clu_em = nullptr;
    float2* tile_e = nullptr;
    float* level_e = nullptr;
    float4* bbox_clu = nullptr;   // box of the node's own cluster triangles (float32)
    float4* clu_n = nullptr;      // the fitted normals as float32 (exported; the kernels read clu_t)
    float4* clu_t = nullptr;
    float* clu_e = nullptr;
    float2* clu_det = nullptr;
    pndf::QuadRec* quad = nullptr;
    int64_t bytes = 0;
    void* mem = nullptr;          // the one allocation behind the arrays
    pndf::HierDev dev;
};

namespace pndf {

// ---------------------------------------------------------------- host side
// Device memory of the handles and of the hierarchy build.  A hipMalloc and a hipFree
// cost about 0.3 ms together whatever their size, and memory that goes back to the
// driver is cleared before it is handed out again (about 29 GB/s: 14 ms for a 2048^2
// map's 0.4 GB when maps are loaded one after the other; 1.6 ms from kept blocks).
// Released blocks are therefore kept for later handles: at most 1 / kBlockKeepShare of
// the device's memory, none for longer than kBlockKeepSeconds (a thread of the library
// frees them, which exists while there are any; a hipFree that waits for the device
// does not hold up other threads), and all of them go back when an allocation of the library
// fails.  A block is kept only once the device is idle (as hipFree itself waits), so any stream
// may have it next.  Safe from several threads.  block_alloc uses the current device.
constexpr size_t kBlockKeepShare = 128;   // 1 / 128
#ifndef PNDF_BLOCK_KEEP_SECONDS
#define PNDF_BLOCK_KEEP_SECONDS 10.0
#endif
constexpr double kBlockKeepSeconds = PNDF_BLOCK_KEEP_SECONDS;
hipError_t block_alloc(size_t bytes, void** p);
void block_free(void* p);
// hipMalloc, tried once more without what the library keeps on the device.
hipError_t device_alloc(void** p, size_t bytes);

// Workspace of one call, in stream order: the call's stream may write it at once, and
// stream_free gives it back behind what that stream has by then.  The driver's
// stream-ordered allocation costs a call more than its launches: a hipFreeAsync takes 15
// to 20 us of the caller's time, and with calls on four streams a 16 MB allocation 150 to
// 300 us, from the default pool or from one of our own with any of its reuse attributes.
// So the library keeps the spaces that calls have used, each with an event behind its last
// call (a record takes 1 us), and a later call has one on the same stream or once that
// call is over; streams never wait for each other.  Batches of 4608 narrow queries at
// 2048^2 on four streams: 26 us each, 71 with two allocations from a pool of our own, 36
// with one from the default pool; 16 served tiles of them: 0.60, 1.65 and 0.75 ms.  At
// most kStreamKeep bytes per device are kept (the largest workspace, of a round of 2^19
// wide queries in a batch of 2^24, is 0.5 GB), until the last handle on the device is
// released or an allocation of the library fails.  Safe from several threads.  Under capture, and on a
// stream of another device than the current one, the driver's calls serve (under capture
// they become nodes of the graph).
constexpr uint64_t kStreamKeep = (uint64_t)512 << 20;
hipError_t stream_alloc(void** p, size_t bytes, hipStream_t s);
void stream_free(void* p, hipStream_t s);
// Lays arrays out in one allocation (256 B aligned): sizes first, then pointers.
struct Arena {
    char* base = nullptr;
    size_t size = 0;
    template <typename T>
    void place(T** p, size_t count)
    {
        if (base) *p = reinterpret_cast<T*>(base + size);
        size += (sizeof(T) * count + 255) & ~(size_t)255;
    }
};
void set_error(const std::string& msg);
pndf_status hip_fail(hipError_t e, const char* what);

// launchers implemented in the .hip files
hipError_t launch_build_mesh(const float* in, int n, float eps, float2* nrm, uint8_t* deg,
                             float2* det, unsigned* d_flag, hipStream_t s);
hipError_t build_hierarchy_levels(pndf_hier* h, hipStream_t s);
// Row-major copies of Morton-ordered per-node arrays (of `words` 32-bit words per node).
constexpr int kExports = 6;
struct ExportArgs {
    int count = 0;
    const uint32_t* src[kExports];
    uint32_t* dst[kExports];
    int words[kExports];
};
hipError_t export_rowmajor(const ExportArgs& x, int m, hipStream_t s);

hipError_t launch_eval(const HierDev& H, const EvalArgs& a, int algo, hipStream_t s);

// One sample of the P-NDF per query (sample.hip).
struct SampleArgs {
    const pndf_query* q;
    const double* xi;          // attempts x nq pairs of uniforms, attempt-major
    int64_t nq;
    int64_t first, end;        // the launch covers queries [first, end)
    int attempts;
    float tau;
    float s2r;
    int kernel;                // PNDF_KERNEL_*
    float2* m;                 // sampled normal per query
    uint64_t* tri;             // optional: triangle id
    double2* u;                // optional: unrolled texture coordinates
};
hipError_t launch_sample(const HierDev& H, const SampleArgs& a, hipStream_t s);

// Projected area P(w) per query (projarea.hip).
struct ProjArgs {
    const pndf_query* q;       // x, y, sx, sy, and w_x, w_y in place of the query normal
    int64_t nq;
    float s2r;
    int kernel;                // PNDF_KERNEL_*
    float* P;
    float* lambda;             // optional: P / w_z - 1
    const uint32_t* order;     // processing order within the launch (heaviest first), or nullptr
};
hipError_t launch_projected_area(const HierDev& H, const ProjArgs& a, hipStream_t s);

// Spatial processing order of a batch: queries bucketed by the Morton code of their
// centre cell (64 x 64 buckets over the torus), stream-ordered workspace.
// With tiles the wide queries come last and *narrow counts the others (device memory),
// else narrow is nullptr.  The order and the tiles' workspace are one allocation, which
// the caller returns (stream_free(w->mem)); without memory for the tiles w->tile.ctl is nullptr.
struct OrderWork {
    void* mem = nullptr;
    uint32_t* order = nullptr;
    const uint32_t* narrow = nullptr;
    TileWork tile{};
};
hipError_t make_order(const HierDev& H, const pndf_query* q, int64_t nq, float s2r, float tau, OrderWork* w, hipStream_t s);
// The same in the library's static per-GPU workspace (no allocation), for batches of
// at most kStaticOrderQueries queries; the order must not be freed.
constexpr int64_t kStaticOrderQueries = (int64_t)1 << 22;
hipError_t make_order_static(const HierDev& H, const pndf_query* q, int64_t nq, uint32_t** order, hipStream_t s);
// Bucket count and coordinate shift of the spatial order for a map of side 2^logn.
void order_shape(int logn, int* nb, int* bshift);
// Size of the tiled evaluation's workspace for batches of nq queries (0: no tiles), and
// its layout at `base`.
size_t tiles_bytes(const HierDev& H, int64_t nq);
void tiles_place(const HierDev& H, int64_t nq, void* base, TileWork* w);

// ---------------------------------------------------------------- device side
#if defined(__HIPCC__)

__device__ __forceinline__ float cross2(float ax, float ay, float bx, float by)
{
    return fmaf(ax, by, -(ay * bx));
}

__device__ __forceinline__ int floor_div_pow2(int a, int logn) { return a >> logn; }
__device__ __forceinline__ int ceil_div_pow2(int a, int logn) { return -((-a) >> logn); }

// Per-query constants, identical for every lane of the wave that owns the query.
struct QuerySetup {
    int kernel;                  // PNDF_KERNEL_*
    float rx, ry;                // support half-widths (disk / box radii)
    float x, y, hx, hy;
    int cxlo, cxhi, cylo, cyhi;  // included unrolled cell range per axis
    int l0;                      // entry level
    float t;                     // cut threshold fl(fl(rx ry) tau)
    uint32_t hkey, hdiag;        // order keys (half_key) of h rounded to halves: x | y << 16, x + y | x - y << 16
    double kx, ky;               // Gaussian: log2(e) / (2 sigma^2)
    double norm;                 // the kernel's peak: 1 / (2 pi sx sy), 1 / (pi rx ry) or 1 / (4 rx ry)
    int fexp;                    // binary point of the exact accumulator (units of 2^fexp)
    bool valid;
};

// Validity and support half-widths of one query (the other fields are not set).
__device__ __forceinline__ QuerySetup setup_support(const pndf_query& qr, float s2r)
{
    QuerySetup q;
    const float lim = 16777216.0f;
    bool ok = isfinite(qr.x) && isfinite(qr.y) && isfinite(qr.sx) && isfinite(qr.sy) &&
              isfinite(qr.hx) && isfinite(qr.hy) && qr.sx > 0.f && qr.sy > 0.f;
    q.rx = __fmul_rn(s2r, qr.sx);
    q.ry = __fmul_rn(s2r, qr.sy);
    q.valid = ok && fabsf(qr.x) <= lim && fabsf(qr.y) <= lim && q.rx <= lim && q.ry <= lim;
    return q;
}

__device__ __forceinline__ double readlane_f64(double v, int lane)
{
    const long long b = __double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, lane);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), lane);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Support box, entry level and kernel constants of one query (see pndf.h).
// WAVE: the query is the same in all 64 lanes, which are active; three of them take one
// of the three divisions each.
template <bool WAVE>
__device__ __forceinline__ QuerySetup setup_as(const pndf_query& qr, float s2r, float tau, int L, float eps, int kernel)
{
    QuerySetup q = setup_support(qr, s2r);
    const bool ok = q.valid;
    const float rx = q.rx, ry = q.ry;
    q.kernel = kernel;
    q.x = qr.x; q.y = qr.y; q.hx = qr.hx; q.hy = qr.hy;
    q.hkey = half_key(__half_as_ushort(__float2half_rn(qr.hx))) |
             (half_key(__half_as_ushort(__float2half_rn(qr.hy))) << 16);
    const double hu = (double)qr.hx + (double)qr.hy, hv = (double)qr.hx - (double)qr.hy;
    q.hdiag = half_key(__half_as_ushort(__float2half_rn((float)hu))) |
              (half_key(__half_as_ushort(__float2half_rn((float)hv))) << 16);
    if (!ok) {
        q.cxlo = q.cylo = 0; q.cxhi = q.cyhi = -1; q.l0 = 0; q.t = -1.f;
        q.kx = q.ky = q.norm = 0.0;
        q.fexp = 0;
        return q;
    }
    float lox = __fsub_rn(qr.x, rx), hix = __fadd_rn(qr.x, rx);
    float loy = __fsub_rn(qr.y, ry), hiy = __fadd_rn(qr.y, ry);
    q.cxlo = (int)ceilf(lox) - 1; q.cxhi = (int)floorf(hix);
    q.cylo = (int)ceilf(loy) - 1; q.cyhi = (int)floorf(hiy);
    float rmax = fmaxf(rx, ry);
    // the smallest l0 with 2^l0 >= rmax
    const int up = (int)((__float_as_uint(rmax) + 0x7fffffu) >> 23) - 127;
    q.l0 = min(max(up, 0), L);
    q.t = tau > 0.f ? __fmul_rn(__fmul_rn(rx, ry), tau) : -1.f;
    const double log2e = 1.4426950408889634074;
    const double pi = 3.14159265358979323846;
    const double peak = kernel == PNDF_KERNEL_BOX ? 4.0 : (kernel == PNDF_KERNEL_DISK ? pi : 2.0 * pi);
    const float ex = kernel == PNDF_KERNEL_GAUSSIAN ? qr.sx : rx, ey = kernel == PNDF_KERNEL_GAUSSIAN ? qr.sy : ry;
    if constexpr (WAVE) {
        const int lane = (int)(threadIdx.x & 63);
        const double f = lane == 2 ? peak : 2.0, num = lane == 2 ? 1.0 : log2e;
        const float u = lane == 2 ? ex : (lane == 1 ? qr.sy : qr.sx), v = lane == 2 ? ey : (lane == 1 ? qr.sy : qr.sx);
        const double d = num / (f * (double)u * (double)v);
        q.kx = readlane_f64(d, 0);
        q.ky = readlane_f64(d, 1);
        q.norm = readlane_f64(d, 2);
    } else {
        q.kx = log2e / (2.0 * (double)qr.sx * (double)qr.sx);
        q.ky = log2e / (2.0 * (double)qr.sy * (double)qr.sy);
        q.norm = 1.0 / (peak * (double)ex * (double)ey);
    }
    // Every term is at most norm / eps per included cell image and triangle (node
    // images of a cluster reach at most one cell beyond the box per side), so
    // D < bound = 2 (nx + 2) (ny + 2) norm / eps.  The exact accumulator counts in
    // units of 2^fexp with bound < 2^(fexp + 190): 192 bits hold any D, and every
    // float32 term down to bound 2^-190 is represented exactly.
    const double bound = 2.0 * ((double)(q.cxhi - q.cxlo) + 3.0) * ((double)(q.cyhi - q.cylo) + 3.0) *
                         q.norm / (double)eps;
    int e2;
    frexp(bound, &e2);
    q.fexp = e2 + 1 - 190;
    return q;
}
__device__ inline QuerySetup setup_query(const pndf_query& qr, float s2r, float tau, int L, float eps, int kernel)
{
    return setup_as<false>(qr, s2r, tau, L, eps, kernel);
}

// The setup of a query owned by a whole wave is the same in every lane: keep it in
// scalar registers (frees vector registers for the traversal).
__device__ __forceinline__ float uniform_f32(float v)
{
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}
__device__ __forceinline__ double uniform_f64(double v)
{
    const long long b = __double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)b);
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(b >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ unsigned long long uniform_u64(unsigned long long v)
{
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)v);
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(v >> 32));
    return ((unsigned long long)hi << 32) | lo;
}
__device__ __forceinline__ QuerySetup uniform_query(const QuerySetup& q)
{
    QuerySetup u;
    u.kernel = __builtin_amdgcn_readfirstlane(q.kernel);
    u.rx = uniform_f32(q.rx); u.ry = uniform_f32(q.ry);
    u.x = uniform_f32(q.x); u.y = uniform_f32(q.y); u.hx = uniform_f32(q.hx); u.hy = uniform_f32(q.hy);
    u.cxlo = __builtin_amdgcn_readfirstlane(q.cxlo); u.cxhi = __builtin_amdgcn_readfirstlane(q.cxhi);
    u.cylo = __builtin_amdgcn_readfirstlane(q.cylo); u.cyhi = __builtin_amdgcn_readfirstlane(q.cyhi);
    u.l0 = __builtin_amdgcn_readfirstlane(q.l0);
    u.t = uniform_f32(q.t);
    u.hkey = (uint32_t)__builtin_amdgcn_readfirstlane((int)q.hkey);
    u.hdiag = (uint32_t)__builtin_amdgcn_readfirstlane((int)q.hdiag);
    u.kx = uniform_f64(q.kx); u.ky = uniform_f64(q.ky); u.norm = uniform_f64(q.norm);
    u.fexp = __builtin_amdgcn_readfirstlane(q.fexp);
    u.valid = __builtin_amdgcn_readfirstlane((int)q.valid) != 0;
    return u;
}
// The setup of the query of a whole wave.
template <int KER>
__device__ __forceinline__ QuerySetup setup_wave(const pndf_query& qr, float s2r, float tau, const HierDev& H)
{
    return uniform_query(setup_as<true>(qr, s2r, tau, H.L, H.eps, KER));
}

// Bits [64 w, 64 w + 64) of m 2^sh for s = sh - 64 w (m < 2^53): m << s for
// 0 <= s < 64, m >> -s for -64 < s < 0, else 0 (the hardware takes shift counts
// mod 64, hence the selects).
__device__ __forceinline__ uint64_t fix_word(uint64_t m, int s)
{
    const uint64_t up = m << (s & 63), dn = m >> ((-s) & 63);
    return s >= 0 ? (s < 64 ? up : 0ull) : (s > -64 ? dn : 0ull);
}

// FP64 term t >= 0 added exactly down to 2^fexp: t = m 2^(ex - 1075) = (m 2^sh) 2^fexp,
// sh <= 136 since t < 2^(fexp + 189).  Branch-free: the lanes of a wave hold terms of
// different magnitudes, and a branch per word range would run every range.
__device__ __forceinline__ void fix_add_term(Fix192& a, double t, int fexp)
{
    const uint64_t b = (uint64_t)__double_as_longlong(t);
    int ex = (int)((b >> 52) & 0x7ffu);
    uint64_t m = b & 0xfffffffffffffull;
    if (ex) m |= 0x10000000000000ull; else ex = 1;
    const int sh = ex - 1075 - fexp;
    const uint64_t v0 = fix_word(m, sh), v1 = fix_word(m, sh - 64), v2 = fix_word(m, sh - 128);
    const uint64_t r0 = a.w0 + v0;
    const uint64_t c0 = r0 < v0 ? 1u : 0u;
    const uint64_t t1 = a.w1 + v1;
    const uint64_t c1 = t1 < v1 ? 1u : 0u;
    const uint64_t r1 = t1 + c0;
    const uint64_t c1b = r1 < c0 ? 1u : 0u;
    a.w0 = r0;
    a.w1 = r1;
    a.w2 += v2 + c1 + c1b;
}

__device__ __forceinline__ void fix_add(Fix192& a, const Fix192& b)
{
    const uint64_t r0 = a.w0 + b.w0;
    const uint64_t c0 = r0 < b.w0 ? 1u : 0u;
    const uint64_t t1 = a.w1 + b.w1;
    const uint64_t c1 = t1 < b.w1 ? 1u : 0u;
    const uint64_t r1 = t1 + c0;
    const uint64_t c1b = r1 < c0 ? 1u : 0u;
    a.w0 = r0;
    a.w1 = r1;
    a.w2 += b.w2 + c1 + c1b;
}

__device__ __forceinline__ float fix_to_float(const Fix192& a, int fexp)
{
    const double d = ((double)a.w2 * 18446744073709551616.0 + (double)a.w1) * 18446744073709551616.0 +
                     (double)a.w0;
    return (float)ldexp(d, fexp);
}

// Does a node of side `side` starting at torus cell `start` have a periodic image
// [start + pN, start + side - 1 + pN] wholly inside the unrolled cell range
// [clo, chi]?  Yes iff the first image starting at or after clo ends by chi.
__device__ __forceinline__ bool axis_inside(int start, int side, int clo, int chi, int logn)
{
    return start + (ceil_div_pow2(clo - start, logn) << logn) + side - 1 <= chi;
}

// Sum over the included periodic images of one axis of exp(-d^2 / (2 sigma^2)),
// d = start + p N + uoff - x; node of side `side` (1 for a texel cell).  The
// exponent a = d^2 log2(e) / (2 sigma^2) is split into floor(a) (an exact power of
// two, ldexp) and a fraction (float32 exp2), so nothing underflows before the
// FP64 product.
__device__ __forceinline__ double exp2_neg_split(double a)
{
    const double ai = floor(a);
    return ldexp((double)exp2f(-(float)(a - ai)), -(int)fmin(ai, 2000.0));
}

__device__ inline double gauss_axis(float x, double k, int start, int side, double uoff, int clo,
                                    int chi, int logn)
{
    int p0 = ceil_div_pow2(clo - start - side + 1, logn);
    int p1 = floor_div_pow2(chi - start, logn);
    double g = 0.0;
    double base = (double)start + uoff - (double)x;
    for (int p = p0; p <= p1; ++p) {
        const double d = base + (double)p * (double)(1 << logn);
        g += exp2_neg_split(d * d * k);
    }
    return g;
}

// Both axes of the Gaussian footprint.  When each axis has a single included image
// (every footprint narrower than the map, away from none of its wraps) the product
// of the two factors is one exponential of the summed exponents.
__device__ inline double gauss_2d(const QuerySetup& q, int sx, int sy, int side, double ux, double uy, int logn)
{
    const int px = ceil_div_pow2(q.cxlo - sx - side + 1, logn), py = ceil_div_pow2(q.cylo - sy - side + 1, logn);
    if (px == floor_div_pow2(q.cxhi - sx, logn) && py == floor_div_pow2(q.cyhi - sy, logn)) {
        const double period = (double)(1 << logn);
        const double dx = (double)sx + ux - (double)q.x + (double)px * period;
        const double dy = (double)sy + uy - (double)q.y + (double)py * period;
        return exp2_neg_split(dx * dx * q.kx + dy * dy * q.ky);
    }
    return gauss_axis(q.x, q.kx, sx, side, ux, q.cxlo, q.cxhi, logn) *
           gauss_axis(q.y, q.ky, sy, side, uy, q.cylo, q.cyhi, logn);
}

// Replacement-triangle vertices (circumradius rho around c, at 90/210/330 degrees).
__device__ __forceinline__ void eqtri_f32(float cx, float cy, float rho, float v[6])
{
    const float c30 = 0.86602540378443864676f;
    v[0] = cx;                     v[1] = cy + rho;
    v[2] = cx - rho * c30;         v[3] = cy - 0.5f * rho;
    v[4] = cx + rho * c30;         v[5] = cy - 0.5f * rho;
}

__device__ __forceinline__ void eqtri_f64(double cx, double cy, double rho, double v[6])
{
    const double c30 = 0.86602540378443864676;
    v[0] = cx;                     v[1] = cy + rho;
    v[2] = cx - rho * c30;         v[3] = cy - 0.5 * rho;
    v[4] = cx + rho * c30;         v[5] = cy - 0.5 * rho;
}

// Inclusive point-in-triangle test in float32 with the cyclic edge functions of the
// vertex offsets q_k = v_k - h: lambda_0 ~ q_b x q_c, lambda_1 ~ q_c x q_a,
// lambda_2 ~ q_a x q_b (all of one sign inside, whatever the orientation).
__device__ __forceinline__ bool tri_hit_f32(const float v[6], float hx, float hy)
{
    float ax = v[0] - hx, ay = v[1] - hy, bx = v[2] - hx, by = v[3] - hy;
    float cx = v[4] - hx, cy = v[5] - hy;
    float e0 = cross2(bx, by, cx, cy), e1 = cross2(cx, cy, ax, ay), e2 = cross2(ax, ay, bx, by);
    return (e0 >= 0.f && e1 >= 0.f && e2 >= 0.f) || (e0 <= 0.f && e1 <= 0.f && e2 <= 0.f);
}

// Contribution of a hit: the triangle's uv vertices are (a, b, c) =
// lower: (U0, U0 + s e_x, U0 + s e_y), upper: (U3, U3 - s e_x, U3 - s e_y) of the node
// (I, J) of side s = 2^lev (lev = 0: texel cell), so u* = corner +- s (l1, l2).
// Box footprint along one axis: the number of included periodic images of the
// point start + uoff within r of x.
__device__ inline double box_axis(float x, float r, int start, int side, double uoff, int clo, int chi, int logn)
{
    const int p0 = ceil_div_pow2(clo - start - side + 1, logn);
    const int p1 = floor_div_pow2(chi - start, logn);
    const double base = (double)start + uoff - (double)x;
    double c = 0.0;
    for (int p = p0; p <= p1; ++p) c += fabs(base + (double)p * (double)(1 << logn)) <= (double)r ? 1.0 : 0.0;
    return c;
}

// Disk footprint: the number of included periodic images of the point inside the
// ellipse of half-axes (rx, ry) around x.
__device__ inline double disk_images(const QuerySetup& q, int sx0, int sy0, int side, double ux, double uy, int logn)
{
    const int p0 = ceil_div_pow2(q.cxlo - sx0 - side + 1, logn), p1 = floor_div_pow2(q.cxhi - sx0, logn);
    const int r0 = ceil_div_pow2(q.cylo - sy0 - side + 1, logn), r1 = floor_div_pow2(q.cyhi - sy0, logn);
    const double bx = (double)sx0 + ux - (double)q.x, by = (double)sy0 + uy - (double)q.y;
    const double period = (double)(1 << logn);
    double c = 0.0;
    for (int p = p0; p <= p1; ++p) {
        const double dx = (bx + (double)p * period) / (double)q.rx;
        for (int r = r0; r <= r1; ++r) {
            const double dy = (by + (double)r * period) / (double)q.ry;
            c += dx * dx + dy * dy <= 1.0 ? 1.0 : 0.0;
        }
    }
    return c;
}

// (the footprint kernel KER is a template parameter: each kernel's evaluation code
// is compiled separately, so the Gaussian path carries none of the others' registers)
// The footprint weight of a hit, norm k(u*), without the division by the Jacobian.
template <int KER>
__device__ inline double hit_weight(const QuerySetup& q, int I, int J, int lev, int half, double l1,
                                    double l2, int logn)
{
    const int s = 1 << lev;
    double ux = half ? (double)s * (1.0 - l1) : (double)s * l1;
    double uy = half ? (double)s * (1.0 - l2) : (double)s * l2;
    double w;
    if constexpr (KER == PNDF_KERNEL_BOX) {
        w = box_axis(q.x, q.rx, I * s, s, ux, q.cxlo, q.cxhi, logn) *
            box_axis(q.y, q.ry, J * s, s, uy, q.cylo, q.cyhi, logn);
    } else if constexpr (KER == PNDF_KERNEL_DISK) {
        w = disk_images(q, I * s, J * s, s, ux, uy, logn);
    } else {
        w = gauss_2d(q, I * s, J * s, s, ux, uy, logn);
    }
    return q.norm * w;
}

template <int KER>
__device__ inline double hit_term(const QuerySetup& q, int I, int J, int lev, int half, double l1,
                                  double l2, float det_used, int logn)
{
    return hit_weight<KER>(q, I, J, lev, half, l1, l2, logn) / (double)det_used;
}

__device__ __forceinline__ uint64_t tri_id(int lev, int I, int J, int half)
{
    return ((uint64_t)lev << 58) | ((uint64_t)J << 29) | ((uint64_t)I << 1) | (uint64_t)half;
}

__host__ __device__ __forceinline__ uint32_t morton_spread(uint32_t v)
{
    v &= 0xffffu;
    v = (v | (v << 8)) & 0x00ff00ffu;
    v = (v | (v << 4)) & 0x0f0f0f0fu;
    v = (v | (v << 2)) & 0x33333333u;
    v = (v | (v << 1)) & 0x55555555u;
    return v;
}

__host__ __device__ __forceinline__ uint32_t morton_compact(uint32_t v)
{
    v &= 0x55555555u;
    v = (v | (v >> 1)) & 0x33333333u;
    v = (v | (v >> 2)) & 0x0f0f0f0fu;
    v = (v | (v >> 4)) & 0x00ff00ffu;
    v = (v | (v >> 8)) & 0x0000ffffu;
    return v;
}

__host__ __device__ __forceinline__ uint32_t morton(uint32_t i, uint32_t j)
{
    return morton_spread(i) | (morton_spread(j) << 1);
}

// Block index -> logical index so that each XCD (workgroups are dispatched to the
// kXcd dies round-robin) walks a contiguous range of the processing order.
constexpr int kXcd = 8;
__device__ __forceinline__ int64_t xcd_contiguous(int64_t b, int64_t nblocks)
{
    const int64_t x = b % kXcd, k = b / kXcd;
    const int64_t per = (nblocks + kXcd - 1) / kXcd, r = nblocks % kXcd;
    if (r == 0) return x * per + k;
    return (x < r ? x * per : r * per + (x - r) * (per - 1)) + k;
}

// Wave-level helpers (wave64).
__device__ __forceinline__ int lane_id() { return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0)); }

__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Exclusive prefix over the wave of a per-lane count in [0, 7], and the total.
__device__ __forceinline__ int wave_prefix_small(int c, int* total)
{
    uint64_t b0 = __ballot(c & 1), b1 = __ballot(c & 2), b2 = __ballot(c & 4);
    uint64_t lt = (1ull << lane_id()) - 1ull;
    *total = __popcll(b0) + 2 * __popcll(b1) + 4 * __popcll(b2);
    return __popcll(b0 & lt) + 2 * __popcll(b1 & lt) + 4 * __popcll(b2 & lt);
}

__device__ __forceinline__ double wave_sum_f64(double v)
{
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Wave sum of a 32-bit value, in lane 63: row shifts 1, 2, 4, 8 (lane 15 of each row
// of 16 then holds its sum), then lane 15 to the next row's and lane 31 to the upper half.
__device__ __forceinline__ uint32_t dpp_sum_u32(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);
    return v;
}

__device__ __forceinline__ uint64_t readlane_u64(uint64_t v, int lane)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane);
    return ((uint64_t)hi << 32) | lo;
}

// Exact sum over the wave (every lane must be active), modulo 2^192.  In eight limbs of
// 26 bits, as 64 of them sum within 32: one instruction per limb and step and no carries
// until the sums are in scalar registers (about 90 vector instructions; as three
// 64-bit words with carries 176).
__device__ __forceinline__ Fix192 wave_sum_fix(const Fix192& v)
{
    const uint32_t d[6] = {(uint32_t)v.w0, (uint32_t)(v.w0 >> 32), (uint32_t)v.w1, (uint32_t)(v.w1 >> 32),
                           (uint32_t)v.w2, (uint32_t)(v.w2 >> 32)};
    uint64_t sum[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int at = 26 * k, i = at >> 5, sh = at & 31;
        const uint32_t t = sh == 0 ? d[i] : (i == 5 ? d[5] >> sh : __builtin_amdgcn_alignbit(d[i + 1], d[i], sh));
        sum[k] = (uint32_t)__builtin_amdgcn_readlane((int)dpp_sum_u32(t & 0x3ffffffu), 63);
    }
    const uint64_t a0 = sum[0] + (sum[1] << 26), a1 = sum[2] + (sum[3] << 26);  // at bits 0, 52, 104, 156
    const uint64_t a2 = sum[4] + (sum[5] << 26), a3 = sum[6] + (sum[7] << 26);
    Fix192 s;
    s.w0 = a0 + (a1 << 52);
    const uint64_t c0 = s.w0 < a0 ? 1ull : 0ull, m = (a1 >> 12) + c0;  // < 2^48
    s.w1 = m + (a2 << 40);
    const uint64_t c1 = s.w1 < m ? 1ull : 0ull;
    s.w2 = (a2 >> 24) + (a3 << 28) + c1;
    return s;
}

__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v)
{
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

#endif  // __HIPCC__

}  // namespace pndf
