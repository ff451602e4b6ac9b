// Internal declarations of the gx engine (host + device).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <mutex>
#include <cstdint>
#include <cstring>
#include <string>
#include <vector>

#include "gx.h"

namespace gx {

constexpr uint32_t INF = 0xFFFFFFFFu;
constexpr size_t ALIGN = 256;

// ---------------------------------------------------------------- errors
void set_error(const char *fmt, ...);
void clear_error();

#define GX_CHECK_HIP(expr, handle)                                                       \
    do {                                                                                 \
        hipError_t _e = (expr);                                                          \
        if (_e != hipSuccess) {                                                          \
            ::gx::set_error("%s failed: %s (%s:%d)", #expr, hipGetErrorString(_e),        \
                            __FILE__, __LINE__);                                         \
            if (handle) (handle)->dev_error = true;                                      \
            return GX_EDEVICE;                                                           \
        }                                                                                \
    } while (0)

#define GX_REQUIRE(cond, code, ...)        \
    do {                                   \
        if (!(cond)) {                     \
            ::gx::set_error(__VA_ARGS__);  \
            return (code);                 \
        }                                  \
    } while (0)

inline size_t align_up(size_t x, size_t a = ALIGN) { return (x + a - 1) / a * a; }

// Bump allocator over a caller-owned device arena.
struct Carver {
    char *base;
    size_t cap, used = 0;
    bool measure_only;
    Carver(void *b, size_t c) : base(static_cast<char *>(b)), cap(c), measure_only(b == nullptr) {}
    template <class T>
    T *take(size_t count) {
        size_t off = used;
        used = align_up(used + count * sizeof(T) + (count == 0 ? 1 : 0));
        return measure_only ? nullptr : reinterpret_cast<T *>(base + off);
    }
    bool fits() const { return used <= cap; }
};

// ---------------------------------------------------------------- graph
// Edge tile of the PageRank pull (in-edges per workgroup tile): PR_BLOCK
// threads times 1, 2, 4 or 8 edges, chosen per graph at load.
constexpr int PR_BLOCK = 256;
// What is gathered per in-edge from its source (contributions, SSSP values)
// lives in slots: the HOT_SLOTS vertices with the most out-edges
// first, 2 MiB of 4-byte values that an L2 keeps while the in-edges stream
// past (on R-MAT graphs they are the sources of 70 to 93% of the in-edges).
constexpr int64_t HOT_SLOTS = int64_t(1) << 19;
constexpr int PR_TILE_MAX = PR_BLOCK * 8;
// The PageRank pull of a graph with at least PR_LDS_EDGES edges may keep the
// contributions of the first slots in LDS (120 KiB, one workgroup per CU).
// 20 supersteps without and with: R-MAT scale 16 (1 M edges) 312 and 363 us,
// 17 (2 M) 375 and 373, 18 (4 M) 566 and 506, 20 1.74 and 1.29 ms, 22 7.70 and
// 5.63 ms; uniform, 4 M edges: 2^15 vertices 550 and 423 us, 2^17 644 and 586.
// Those slots must also be the sources of 1 in PR_LDS_PART in-edges: where they
// are of few, one workgroup per CU is only fewer waves.  10 supersteps without
// and with, uniform graphs of 8 M edges: 125 000 vertices 544 and 476 us, 500 000
// (11 % of the edges) 586 and 566, 1 M (6 %) 681 and 676, 2 M (4 %) 1036 and 1077;
// of 4.3 M edges and 2 M vertices 666 and 787; of 5 M and 8 M 1.52 and 1.65 ms;
// R-MAT, whose slots hold hubs: scale 22 with 1 edge per vertex 563 and 556 us,
// with 2 806 and 706.
constexpr int32_t PR_LDS_SLOTS = 30720;
constexpr int64_t PR_LDS_EDGES = int64_t(1) << 22;
constexpr int64_t PR_LDS_PART = 16;
// Row pull of SSSP / CC: rows of at most PULL_SMALL entries are taken in
// blocks, longer ones in segments of at most PULL_SEG entries from a table
// built at load.  The rows (and the segments) are dealt to PULL_SLICES slices
// in runs of blocks; a launch's workgroups take the slice of the XCD they run
// on.
constexpr int PULL_SLICES = 8;
constexpr int PULL_SMALL = 32;
constexpr int PULL_SEG = 256;
constexpr int PULL_PACK = 32;  // batched pull: a pack of short rows ends when it has this many entries
constexpr int PULL_BLOCK = 256;     // rows a workgroup takes at a time (one per thread)
constexpr int PULL_SEG_BLOCK = 64;  // segments (16 per wave)
constexpr int PULL_RUN_LOG = 2;     // blocks per run (1 below PULL_RUN_FROM blocks, to reach every XCD)
constexpr int PULL_RUN_FROM = 2048;
// SSSP: slots whose frontier bits a pulling workgroup keeps in LDS (16 KiB;
// on R-MAT scale 22 the sources of 75% of the in-edges).
constexpr int PULL_BITS = 1 << 17;
constexpr int PULL_BIT_WORDS = PULL_BITS / 32;

// The other pull of SSSP / CC, a sweep over every in-edge (CC: neighbour) as a
// record {destination, source and weight}: destinations are dealt to bins of
// at most SWEEP_BIN_BYTES of values, each bin to one of PULL_SLICES slices; a
// bin's records are grouped by source band (source >> SWEEP_BAND_BITS), groups
// are padded to whole SWEEP_VT records with sentinels and cut into units of at
// most SWEEP_UNIT records.  It costs the same whatever the values are, and its
// random reads stay in LDS and one L2.  The row pull reads a value per entry
// from anywhere, so it needs its rows to stop early and most of its sources to
// be among a few; sweep_rule says which graphs sweep.
constexpr int SWEEP_SLICE_SHIFT = 6;  // destinations are dealt in blocks of 64
constexpr int64_t SWEEP_BIN_BYTES = int64_t(2) << 20;
constexpr int SWEEP_BAND_BITS = 13;  // 8192 sources: 32 KiB of values in LDS
constexpr int SWEEP_BAND = 1 << SWEEP_BAND_BITS;
constexpr int SWEEP_VT = 8;
constexpr int SWEEP_UNIT = 8192;
constexpr uint32_t SWEEP_SENTINEL = 0xFFFFFFFFu;  // destination of a padding record
constexpr int64_t SWEEP_V_MIN = int64_t(1) << 19, SWEEP_V_MAX = int64_t(1) << 28;
struct Sweep {
    const uint2 *rec = nullptr;    // {destination, (source mod SWEEP_BAND) << 8 | weight}; NULL: the row pull is used
    const uint4 *units = nullptr;  // {first record, records, first source of the band, 0}
    int64_t uoff[PULL_SLICES + 1] = {};  // slice x owns units uoff[x] .. uoff[x + 1] - 1
};
inline int64_t sweep_bins(int64_t V) {
    return PULL_SLICES *
           std::max<int64_t>(1, (V * 4 + PULL_SLICES * SWEEP_BIN_BYTES - 1) / (PULL_SLICES * SWEEP_BIN_BYTES));
}
inline int64_t sweep_groups(int64_t V) { return sweep_bins(V) * ((V >> SWEEP_BAND_BITS) + 1); }
// Capacities of the records and units of E entries (known before the layout is).
inline int64_t sweep_rec_cap(int64_t V, int64_t E) { return E + (SWEEP_VT - 1) * sweep_groups(V) + SWEEP_VT; }
inline int64_t sweep_unit_cap(int64_t V, int64_t E) { return sweep_rec_cap(V, E) / SWEEP_UNIT + sweep_groups(V) + 1; }
// Capacity of the segment table of E entries (known before the rows are: a
// row in it has more than PULL_SMALL entries).
inline int64_t pull_seg_cap(int64_t E) { return E / PULL_SMALL + 1; }
inline int64_t pull_pack_cap(int64_t V, int64_t E) { return std::min(E, E / PULL_PACK + (V + 63) / 64) + 1; }

// Row ends of the in-CSR (PageRank, batched PPR): rows without in-edges are
// left out, a bit per in-edge marks the last one of its row.  The in-edges are cut into
// tiles, rows that cross tiles are listed.
// (A row of at least ROWS_LONG partials is summed by a wave, batched by a
// workgroup, a piece per wave of it: with 32 every case takes the same; with 256
// batched PPR of 5 lanes on R-MAT scale 17 takes 890 us for 20 supersteps, 790 so;
// with no row cut, a star of 2 M vertices takes 1357 us for 20 PageRank supersteps,
// 832 so, and one of 200 000 3.76 ms for 20 of batched PPR, 64 lanes, 1.30 so.)
constexpr int ROWS_PIECES = 16;     // a sum of at least ROWS_LONG partials is cut into this many pieces
constexpr int ROWS_LONG = 64;
constexpr int ROWS_MID = 4;         // (a single step of loads covers fewer)
struct RowTiles {
    int64_t T = 0, n = 0;              // in-edges per tile, tiles
    const int32_t *tile_nz = nullptr;  // per tile: position in nz of the row its first edge belongs to
    const int4 *cross = nullptr;       // rows crossing tiles: {row, out-degree, first tile, last tile},
    int32_t n_cross = 0;               // those with at least ROWS_LONG further tiles first, then those
    int32_t n_long = 0, n_mid = 0;     // with at least ROWS_MID
};
// Batched PPR, a lane group's tile: a graph of few edges has too few longer
// ones to occupy the chip, a large one saves partials, the more the wider the
// batch.  20 supersteps with 64 and 256 in-edges: R-MAT scale 16 (1 M edges), 5
// lanes 690 and 1455 us, 64 lanes 1.02 and 1.24 ms; scale 18 (4 M, the last below
// the line) 5 lanes 1.20 and 1.73, 64 2.92 and 2.68, 128 4.68 and 4.60; scale 19,
// 5 lanes 1.87 and 2.11, 64 6.24 and 5.25, 128 10.1 and 9.6; scale 20, 5 lanes 3.0 and
// 3.74, 64 13.1 and 11.4; uniform, 6 M edges, 64 lanes 6.24 and 5.30.  (Up to 16 lanes
// the shorter tile would be the better one above the line too.)
inline int64_t bp_rows_tile(int64_t E) { return E >= (int64_t(1) << 22) ? 256 : 64; }
constexpr int ROWS_DANGLING = 512;  // tiles of dangling vertices at most

// Label propagation: vertices are grouped by the number of distinct
// neighbours d.  Classes 0..4 take d <= 4, 8, 16, 32, 64 and run as lane
// groups of that width; class 5 (d <= LP_MID_MAX) runs one wave or workgroup
// per vertex with a hash table of labels in LDS; class 6 (hubs) counts in hash
// tables in device memory, cut into chunks of LP_HUB_CHUNK neighbours.
constexpr int LP_CLASSES = 7;
constexpr int LP_MID_MAX = 2048;
constexpr int LP_MID_SLOTS = 4096;   // LDS table of the mid class (load at most 1/2)
constexpr int LP_HUB_CHUNK = 8192;
constexpr uint32_t LP_NONE = 0xFFFFFFFFu;

struct DevGraph {
    int64_t V = 0, E = 0, E_sym = 0;
    int32_t W = 0;                 // bitmap words: ceil(V / 32)
    // out-CSR (SSSP push): row_ptr + interleaved (dst, weight)
    const int32_t *out_rp = nullptr;
    const uint2 *out_adj = nullptr;
    // in-CSR and out-degree; its row ends and tiles (PageRank, batched PPR)
    const int32_t *in_rp = nullptr;
    const int32_t *outdeg = nullptr;
    // slot[v]: where vertex v's gathered values live, the HOT_SLOTS vertices
    // with the most out-edges first (by out-degree, then id), every other
    // vertex after them in id order; pr_src = the slot of each in-edge's source
    const int32_t *pr_src = nullptr;
    const int32_t *slot = nullptr;
    const int2 *nz = nullptr;          // {row, out-degree} of the rows with in-edges, ascending
    const int32_t *nz_slot = nullptr;  // their slots
    int64_t n_nz = 0;
    const int2 *ez = nullptr;          // {row, out-degree} of the other rows
    int64_t n_ez = 0;
    const uint64_t *row_last = nullptr;  // bit e: in-edge e is its row's last
    RowTiles pr_rows, bp_rows;         // of PageRank's tiles and of the batched PPR's
    const int32_t *dang = nullptr;     // slots of the vertices with in-edges and without out-edges
    int64_t n_dang = 0;
    int32_t pr_tile = PR_TILE_MAX;  // in-edges per PageRank workgroup tile (PR_BLOCK / 64 wave tiles)
    bool pr_hot = false;            // the PageRank pull keeps the first PR_LDS_SLOTS contributions in LDS
    // in-edges of the SSSP pull, {source slot, (destination mod 64) << 8 | weight}:
    // the entries of the rows of at most PULL_SMALL, in row order (block b of
    // 64 rows owns in_blk[b] .. in_blk[b + 1]), then the longer rows, each by
    // ascending weight; null when a weight exceeds 255 (the engine then only
    // pushes).  pull_segs: {row, first entry, end entry, first weight, bit 8:
    // the row's only one} of the long rows.
    const uint2 *in_adj = nullptr;
    const int32_t *in_blk = nullptr;
    const uint4 *pull_segs = nullptr;
    int64_t pull_nsegs = 0;
    // batched pull: runs of whole short rows of one block of 64, {first entry,
    // end entry, first row of the block, 0}
    const uint4 *packs = nullptr;
    int64_t n_packs = 0;
    // symmetric adjacency (CC push and pull, label propagation) and the
    // segments of its long rows
    const int32_t *sym_rp = nullptr;
    const int32_t *sym_col = nullptr;
    bool sym_ascending = true;  // every row's neighbours ascend (rows of the host CSR that do not are merged as they are)
    const uint4 *sym_segs = nullptr;
    int64_t sym_nsegs = 0;
    // records of the sweep, on graphs where it is the faster pull
    Sweep sweep_in, sweep_sym;
    bool sssp_pushes = false;  // SSSP pushes unless the caller names a pull fraction
    // partition metadata
    const int32_t *l2g = nullptr;          // nullptr = identity
    const uint32_t *remote_out = nullptr;  // bitmaps of W words (nullptr = none remote)
    const int32_t *part_list = nullptr;  // replicas with in-edges whose master is elsewhere (PageRank over parts)
    int64_t n_part = 0;
    const uint32_t *remote_any = nullptr;
    const uint32_t *master = nullptr;      // this part holds the master copy
    const uint32_t *master_rep = nullptr;  // ... of a vertex another part holds a replica of
    // PageRank exchanged between the parts: out-degrees in the whole graph
    const int32_t *outdeg_g = nullptr;
    int64_t V_global = 0;
};

// Label propagation's class sizes (off[c]: first list slot of class c), hubs
// and their chunks.
struct LpPlan {
    bool made = false;
    int64_t off[LP_CLASSES + 1] = {};
    int64_t nwave = 0, tab_slots = 0;
    int64_t slot_bound = 0;       // upper bound of the hub table slots
    std::vector<uint32_t> hubs;   // vertices, ascending
    std::vector<uint4> chunks;    // {hub, first entry, end entry, 0}
    std::vector<uint2> hub;       // per hub {first table slot, slots}
};

}  // namespace gx

struct gx_graph {
    gx::DevGraph d;
    uint32_t needs = 0;
    void *arena = nullptr;
    size_t arena_bytes = 0;
    int device = 0;
    int num_cus = 0;
    bool dev_error = false;
    std::vector<int32_t> host_outdeg;  // out-degree (host copy, for sources and stats)
    std::mutex lp_mu;
    gx::LpPlan lp;
    std::vector<uint32_t> sweep_in_recs, sweep_sym_recs;  // records of each of the sweep's units (size its fix-up regions)
    std::vector<int32_t> host_symdeg;  // distinct neighbours (with GX_NEED_SYM; label propagation classes)
    // supersteps of the last converged SSSP / CC run on this graph: the size
    // of the next run's first speculative group (solves on one graph tend to
    // need similar superstep counts)
    std::atomic<uint32_t> last_supersteps[2] = {0u, 0u};
    // PageRank runs replayed as HIP graphs: n supersteps from ring slot `slot`
    // (which also fixes the buffer parity) of a state laid out in `mem` with
    // damping `damping`; a state re-created in the same memory finds its graph
    // again.  Captured on `cap_stream`; the oldest entry goes past PR_GRAPHS.
    struct PrGraph {
        const void *mem;
        double damping;
        int64_t slot;
        uint32_t n;
        hipGraphExec_t exec;
    };
    static constexpr size_t PR_GRAPHS = 8;
    std::mutex pr_mu;
    std::vector<PrGraph> pr_graphs;
    hipStream_t cap_stream = nullptr;
    ~gx_graph() {
        for (auto &e : pr_graphs) (void)hipGraphExecDestroy(e.exec);
        if (cap_stream) (void)hipStreamDestroy(cap_stream);
    }
};

namespace gx {

// Host-side build + upload of the device images (gx_graph.hip).
gx_status graph_layout(const gx_graph_desc *desc, Carver &c, DevGraph *d);

// Per-superstep statistics slot kept in device memory.
// The compaction's workgroups each add to `list` and to `frontier`; adds to
// one address serialise, so the two counters live on different 128-byte
// lines and do not queue behind each other.
struct DevStep {
    unsigned long long list;      // (entries << 32) | edges, via one 64-bit add per workgroup
    unsigned long long changed;   // PageRank changed values
    unsigned long long pad;       // 1 when the superstep pulled
    unsigned long long rot_mixed; // pull: 1 when its workgroups saw different XCD rotations
    unsigned long long spare0[12];
    unsigned long long frontier;  // |F_k|
    uint32_t inv_min;             // ~(smallest active value), so that a cleared slot says "none"
    uint32_t pad1;
    unsigned long long spare1[14];
};
static_assert(sizeof(DevStep) == 256, "DevStep spans two 128-byte lines");
constexpr int STEP_RING = 4096;

// Tiles of the push relaxation (active out-edges per workgroup tile).
constexpr int PUSH_BLOCK = 256;
constexpr int PUSH_VT = 8;
constexpr int PUSH_TILE = PUSH_BLOCK * PUSH_VT;

int device_cus(int device);

// Workgroups per CU the occupancy query reports for (kernel, block size) on
// the current device; cached, because the query is slow.
int occupancy_per_cu(const void *kernel, int block);

}  // namespace gx

// Engine state of one algorithm run on a graph (gx_plain.hip, gx_lp.hip).
struct gx_state {
    gx_graph *g = nullptr;
    gx_params p{};
    int64_t k = 0;
    bool dev_error = false;
    int relax_grid = 0;   // persistent grid of the relaxation kernel
    uint32_t xcd_shift = 0;  // added to the XCD a workgroup is expected on (non-zero only to exercise the check)
    uint32_t *rot = nullptr;      // XCD rotation each workgroup of the last pull saw
    // SSSP / CC
    uint32_t *val = nullptr;
    uint8_t *front8[2] = {nullptr, nullptr};  // frontier byte maps: A_k lives in front8[k & 1]
    uint8_t *dirty8 = nullptr;                // changed since the last sync (byte per vertex)
    uint4 *list = nullptr;
    uint32_t *tile_start = nullptr;
    uint32_t *snap = nullptr;      // start-of-superstep values of every vertex (pull; SSSP's row pull: by slot)
    uint32_t *hot[2] = {nullptr, nullptr};  // SSSP: at least A_k's bits of the first PULL_BITS slots, hot[k & 1]
    uint32_t pull_edges = 0xFFFFFFFFu;
    uint2 *fix = nullptr;          // sweep: fix-up regions, fix_cap entries per relaxation workgroup
    uint32_t *fixn = nullptr;      // and the entries recorded in each
    uint32_t fix_cap = 0;
    const gx::Sweep *sweep = nullptr;  // the pull sweeps these (NULL: the row pull); snapshots are then by vertex
    bool merged = false;           // other parts' values were merged (gx_apply_delta)
    // PageRank
    float *x[2] = {nullptr, nullptr};
    float *contrib[2] = {nullptr, nullptr};
    uint32_t *synced = nullptr;
    double *head = nullptr, *tailp = nullptr;
    double *dpart = nullptr;
    uint32_t *cpart = nullptr;   // per-wave changed counts (PageRank)
    double *Dval = nullptr;
    int pr_grid = 1;                  // workgroups of k_pr_pull
    int pr_parts = 1;                 // its waves (entries of dpart and cpart)
    int pr_fix_grid = 1;              // workgroups of k_pr_fix
    int pr_fix_block = 256;           // and their threads
    double *fix_d = nullptr;          // their dangling-mass partials
    unsigned long long *fix_c = nullptr;  // and changed counts
    uint32_t *fix_done = nullptr;     // workgroups finished (the last resets it)
    void *mem = nullptr;              // the caller's state buffer (keys the graph's replay cache)
    // label propagation: lab[k & 1] holds the labels at the start of superstep k
    uint32_t *lab[2] = {nullptr, nullptr};
    uint32_t *lp_list = nullptr;              // vertices with neighbours, grouped by degree class
    int64_t lp_off[gx::LP_CLASSES + 1] = {};  // class c owns lp_list[lp_off[c] .. lp_off[c + 1])
    uint4 *lp_chunks = nullptr;               // hub edge chunks {hub index, first entry, end entry, 0}
    int64_t lp_nchunks = 0;
    uint2 *lp_hub = nullptr;                  // per hub {first table slot, slots (a power of two)}
    uint2 *lp_tab = nullptr;                  // hub tables {label, count}; label LP_NONE = free
    int64_t lp_tab_slots = 0;
    int64_t lp_nwave = 0;                     // vertices of class 5 that take one wave (listed first)
    unsigned long long *lp_best = nullptr;    // per hub: largest (count, ~label) so far (0 between supersteps)
    uint32_t *lp_log = nullptr;               // hub table slots taken in a superstep ([0]: how many)
    uint32_t *lp_cursor = nullptr;            // next slot of every list while they are filled
    uint8_t *lp_touch = nullptr;              // a neighbour's label changed: recompute
    uint2 *lp_changed = nullptr;              // the vertices the last superstep changed {vertex, neighbour chunk}
    // separate template calls (gx_params.phases): merged messages per vertex,
    // the index of the pending map in front8, and what is waiting
    uint32_t *acc = nullptr;         // SSSP / CC: min of the merged messages (INF = none)
    double *acc_d = nullptr;         // PageRank: sum of the merged messages
    uint8_t *junk8 = nullptr;        // marks the relaxation makes against the accumulator (never read)
    double *Dscratch = nullptr;      // dangling-mass slot the merge's fix-up writes (never read)
    gx::DevStep *ph_steps = nullptr; // counter slots the merge's fix-up writes (never read)
    int ph_p = 0;                    // front8[ph_p] collects the vertices the next MSGGen sends from
    bool ph_msgs = false, ph_merged = false;
    // shared
    gx::DevStep *steps = nullptr;
    uint32_t *blk_cnt = nullptr;
    int delta_blocks = 0, delta_words = 0;
    // edge-kernel timing
    std::vector<hipEvent_t> ev_pool;
    struct Pending {
        int64_t k;
        hipEvent_t a, b;
    };
    std::vector<Pending> ev_pending;
    double kernel_ms = 0;
    int64_t kernel_launches = 0;
    gx::DevStep *host_steps = nullptr;  // pinned, HOST_STEPS entries (from a process-wide pool)
    ~gx_state();
};

namespace gx {
// Label propagation (gx_lp.hip): state layout (also sizes the arena with a
// measuring Carver), initialisation, one superstep.
const LpPlan &lp_plan(gx_graph *g);
size_t lp_layout(gx_graph *g, Carver &c, gx_state *s);
gx_status lp_init(gx_state *s, hipStream_t hs);
void lp_enqueue(gx_state *s, hipStream_t hs, DevStep *step, DevStep *next);
int64_t lp_active(const gx_state *s);
}  // namespace gx
