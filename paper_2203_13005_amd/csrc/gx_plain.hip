// One worker's superstep engine: PageRank (pull), Bellman-Ford SSSP and
// min-label CC (frontier push), the lazy-upload sync set, and iteration
// control.
//
// A superstep is the algorithm template MSGGen -> MSGMerge -> MSGApply of
// Section "Algorithm Template", in BSP order.  Messages of one superstep
// are generated from the state at its start (no dependency between the
// edge triplets of one iteration, Section "Pipeline Shuffling"), so the
// frontier compaction stores a snapshot of every active vertex's value.
//
// SSSP / CC superstep k (A_k = vertices active in superstep k), one
// launch of k_relax that runs one of two forms:
//   push      : every workgroup tile relaxes exactly PUSH_TILE active
//               out-edges: Gen = snapshot (+ weight), Merge + Apply =
//               integer atomicMin on the destination, filtered by a plain
//               read; a candidate that passes marks the destination in the
//               next frontier (a plain, idempotent byte store; the next
//               compaction carries the marks into the dirty map).
//   pull      : for large frontiers instead: every row of in-edges (CC:
//               neighbours) takes the minimum over its entries itself, in an
//               order that lets it stop early, and is its value's only
//               writer.  On large graphs without hubs the pull sweeps over
//               every in-edge instead, destination slice by source band
//               (k_relax_sweep, and k_fixup after it).  The device picks push
//               or pull from the frontier's out-edge count; no host round trip.
//   k_compact : frontier byte map A_{k+1} -> active list of (edge offset,
//               CSR base, snapshot) for active vertices with out-edges; one
//               64-bit atomic per workgroup reserves list slots and edge
//               offsets; every PUSH_TILE-edge tile records the entry where it
//               starts; |A_{k+1}| is the count of vertices superstep k changed.
//               It runs after the relaxation, so the next superstep's form
//               is known on the device when its launch starts.
//               The frontier stands in for the paper's synchronisation
//               skipping (Section "Synchronization Skipping") and the equal
//               edge tiles for its fixed-size edge blocks (Section "Data Flows
//               & Management") under the balanced objective of Section
//               "Workload Balancing".
// PageRank superstep:
//   k_pr_pull : a wave per tile of consecutive in-edges; the contributions
//               are gathered and summed per destination row in a fixed order;
//               rows that cross a tile boundary leave fixed partials.
//   k_pr_fix  : completes the crossing rows (a thread each, in tile order;
//               a wave for those of many tiles) and reduces the dangling mass
//               for the next superstep: per-workgroup partials, then the last
//               workgroup to finish sums them in workgroup order.  No
//               floating-point atomics: results are bitwise reproducible.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdlib>
#include <mutex>

#include "gx_device.h"
#include "gx_internal.h"

using namespace gx;


static void pool_return(hipEvent_t e);
static void host_steps_return(gx::DevStep *p);

gx_state::~gx_state() {
    for (auto e : ev_pool) pool_return(e);
    for (auto &pr : ev_pending) {
        pool_return(pr.a);
        pool_return(pr.b);
    }
    if (host_steps) host_steps_return(host_steps);
}

namespace {

// ------------------------------------------------------------ SSSP / CC

__global__ __launch_bounds__(256) void k_min_init(uint32_t *val, uint32_t *snap, uint8_t *f0, uint8_t *f1,
                                                  uint8_t *dirty, const int32_t *l2g, const int32_t *rp, int64_t V, int32_t algo,
                                                  int32_t source, DevStep *step0, uint32_t *hot0, uint32_t *hot1) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) *step0 = DevStep{};
    if (i < PULL_BIT_WORDS && hot0) hot0[i] = hot1[i] = 0u;
    if (i < V) {
        uint32_t x;
        uint8_t f;
        if (algo == GX_CC) {
            x = l2g ? (uint32_t)l2g[i] : (uint32_t)i;
            f = rp[i + 1] > rp[i];
        } else {
            x = (i == source) ? 0u : INF;
            f = i == source;
        }
        val[i] = x;
        snap[i] = algo == GX_CC ? x : INF;  // (by slot for SSSP: the source's is written when it is compacted)
        f0[i] = f;
        f1[i] = 0;
        dirty[i] = 0;
    }
}

// Frontier byte map -> active list.  Each thread takes CVT consecutive
// vertices: one load of their frontier bytes (and one store clearing the
// byte map the next relaxation fills, which held A_{k-1}); a thread with an
// active vertex loads its CVT+1 row pointers, CVT values and slots as whole
// vectors, so no load waits on another.  A workgroup covers
// CBLOCK*CVT vertices and issues two counter atomics (list, |A|).  Active
// vertices with out-edges get a list entry (edge offset, CSR base,
// snapshot, vertex) and the tiles that start inside an entry's edges record
// it.  When the next superstep may pull (snap_all), threads with an active
// vertex also store their vertices' values as snapshots, and the smallest
// active value is left in the step: a value changes only when its vertex is
// active next, so after every compaction `snap` holds the value of every
// vertex at the start of the superstep (k_min_init wrote the first ones).
// |A_{k+1}| is the number of vertices superstep k changed.
// CVT is COMPACT_WIDE from COMPACT_WIDE_FROM vertices on and 4 below: a small
// graph then still has several workgroups, and a thread with hubs writes few
// list entries one after another (scale-15 solve: 155 us against 212 us with
// 16, together with idle pull workgroups leaving before they stage the
// frontier bits; R-MAT scale 20: 436 us with 8, 515 with 16; scale 22: 1055 and
// 1069, scale 23 of degree 8 1.58 and 1.60 ms; 16 leaves no registers for the slots).
// Without slots it is COMPACT_WIDEST where half as many reservations count
// more: from COMPACT_WIDEST_FROM vertices on, half of that on graphs of fewer
// than COMPACT_SPARSE edges per vertex, whose many supersteps have active
// vertices everywhere (SSSP with 8 and 16: 2^22 vertices of degree 1 1.61 and
// 1.50 ms, 2 1.64 and 1.55, 3 1.86 and 1.81; 2^23 of degree 2 2.56 and 2.42, 4 4.32 and
// 4.20; CC, R-MAT scale 23 of degree 8 755 and 742 us).
constexpr int COMPACT_WIDE = 8, COMPACT_WIDEST = 16;
constexpr int64_t COMPACT_WIDE_FROM = int64_t(1) << 20, COMPACT_WIDEST_FROM = int64_t(1) << 23;
constexpr int64_t COMPACT_SPARSE = 4;
// Threads per compaction workgroup: each workgroup makes one list
// reservation (an add with return on a single counter, which serialises
// across workgroups), so fewer, larger workgroups shorten that chain.
constexpr int CBLOCK = 1024;

// Flags the superstep if the workgroups of its pull saw different XCD
// rotations (one workgroup of the launch that follows the pull calls this).
__device__ __forceinline__ void check_rotations(DevStep *step, const uint32_t *__restrict__ rot, int n) {
    if (step->pad == 0) return;  // it pushed
    const uint32_t r0 = rot[0];
    bool mixed = false;
    for (int i = threadIdx.x; i < n; i += blockDim.x) mixed |= rot[i] != r0;
    if (mixed) step->rot_mixed = 1ull;
}

template <int CVT>
__global__ __launch_bounds__(CBLOCK) void k_compact(const uint8_t *__restrict__ front, uint8_t *__restrict__ front_clear,
                                                 const int32_t *__restrict__ rp, const uint32_t *__restrict__ val,
                                                 uint32_t *__restrict__ snap, int64_t V,
                                                 uint4 *__restrict__ list, uint32_t *__restrict__ tile_start,
                                                 DevStep *__restrict__ step, DevStep *__restrict__ next_step,
                                                 int snap_all, DevStep *__restrict__ prev,
                                                 uint8_t *__restrict__ dirty, uint32_t pull_edges,
                                                 const uint32_t *__restrict__ rot, int nrot,
                                                 const int32_t *__restrict__ slot, uint32_t *__restrict__ hot,
                                                 uint32_t *__restrict__ hot_clear) {
    __shared__ unsigned long long s_scan[CBLOCK / 64];
    __shared__ unsigned long long s_base;
    __shared__ int s_nf[CBLOCK / 64];
    __shared__ uint32_t s_min[CBLOCK / 64];
    const int tid = threadIdx.x;
    // The last workgroup has no vertices: its chain of reads runs beside the
    // others', which on a small graph are no longer (scale-12 solve: 228 us
    // with both in the first workgroup and the frontier read after the
    // counter, 218 us so).
    if (blockIdx.x == gridDim.x - 1) {
        if (tid == 0) *next_step = DevStep{};
        if (prev != nullptr) check_rotations(prev, rot, nrot);
        return;
    }
    // The previous superstep had no active vertex: nothing was relaxed, the
    // map read here is still the cleared one and the map cleared here is
    // empty, so A_{k+1} is empty without a sweep (its counters stay zero).
    // (A small graph's map is read as fast as the counter.)
    if (CVT >= COMPACT_WIDE && prev != nullptr && prev->frontier == 0) return;
    if (slot != nullptr)  // the bits of the superstep after the one compacted here
        for (int64_t i = (int64_t)blockIdx.x * CBLOCK + tid; i < PULL_BIT_WORDS; i += (int64_t)(gridDim.x - 1) * CBLOCK)
            hot_clear[i] = 0u;
    const int64_t u0 = ((int64_t)blockIdx.x * CBLOCK + tid) * CVT;
    uint32_t actmask = 0;
    if (u0 < V) {  // byte maps are padded to whole 32-vertex words: the CVT bytes at u0 exist
        constexpr int NW = CVT / 4;
        uint32_t fw[NW], any = 0;
#pragma unroll
        for (int q = 0; q < NW; q++) {
            fw[q] = reinterpret_cast<const uint32_t *>(front + u0)[q];
            any |= fw[q];
        }
#pragma unroll
        for (int q = 0; q < NW; q++) reinterpret_cast<uint32_t *>(front_clear + u0)[q] = 0u;
        if (dirty != nullptr && any) {  // changed vertices become dirty here
            uint32_t *d4 = reinterpret_cast<uint32_t *>(dirty + u0);
#pragma unroll
            for (int q = 0; q < NW; q++) d4[q] |= fw[q];
        }
#pragma unroll
        for (int q = 0; q < NW; q++)
#pragma unroll
            for (int b = 0; b < 4; b++)
                if ((fw[q] >> (8 * b)) & 0xFFu) actmask |= 1u << (4 * q + b);
        if (V - u0 < CVT) actmask &= (1u << (V - u0)) - 1u;  // padding bytes are no vertices
    }
    if (!__syncthreads_or(actmask != 0)) return;
    int32_t r[CVT + 1];
    uint32_t x[CVT];
    int32_t sl[CVT];
    const bool by_slot = CVT <= COMPACT_WIDE && snap_all && slot != nullptr;
#pragma unroll
    for (int i = 0; i < CVT; i++) {
        r[i] = 0;
        x[i] = 0;
        sl[i] = 0;
    }
    r[CVT] = 0;
    if (actmask) {
        if (u0 + CVT <= V) {  // rows u0 .. u0+CVT of the V+1 row pointers
            const int4 *r4 = reinterpret_cast<const int4 *>(rp + u0);
            const uint4 *x4 = reinterpret_cast<const uint4 *>(val + u0);
#pragma unroll
            for (int q = 0; q < CVT / 4; q++) {
                const int4 a = r4[q];
                const uint4 b = x4[q];
                r[4 * q] = a.x, r[4 * q + 1] = a.y, r[4 * q + 2] = a.z, r[4 * q + 3] = a.w;
                x[4 * q] = b.x, x[4 * q + 1] = b.y, x[4 * q + 2] = b.z, x[4 * q + 3] = b.w;
            }
            r[CVT] = rp[u0 + CVT];
            if (by_slot)
#pragma unroll
                for (int q = 0; q < CVT / 4; q++) {
                    const int4 a = reinterpret_cast<const int4 *>(slot + u0)[q];
                    sl[4 * q] = a.x, sl[4 * q + 1] = a.y, sl[4 * q + 2] = a.z, sl[4 * q + 3] = a.w;
                }
        } else {
#pragma unroll
            for (int i = 0; i < CVT; i++) {
                if (u0 + i < V) x[i] = val[u0 + i];
                if (by_slot && u0 + i < V) sl[i] = slot[u0 + i];
                if (u0 + i <= V) r[i] = rp[u0 + i];
            }
        }
    }
    uint32_t cnt = 0, edges = 0, low = INF;
#pragma unroll
    for (int i = 0; i < CVT; i++) {
        const int32_t dg = r[i + 1] - r[i];
        if (((actmask >> i) & 1u) && dg > 0) {
            cnt++;
            edges += (uint32_t)dg;
            low = min(low, x[i]);
        }
    }
    unsigned long long mine = ((unsigned long long)cnt << 32) | edges, total;
    unsigned long long pre = block_excl_scan_u64(mine, &total, s_scan);
    int nf = __popc(actmask);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        nf += __shfl_down(nf, o, 64);
        low = min(low, (uint32_t)__shfl_down(low, o, 64));
    }
    if ((tid & 63) == 0) {
        s_nf[tid >> 6] = nf;
        s_min[tid >> 6] = low;
    }
    if (tid == 0) s_base = total ? atomicAdd(&step->list, total) : 0ull;
    // Snapshots for the pull.  SSSP: the active vertices' values go to their
    // slots, and their bits with them (a bit too many only costs a read).
    // CC: a thread with an active vertex stores the values of all its CVT
    // vertices (whole vectors; an inactive vertex's value is the one its
    // snapshot holds already).
    if (by_slot) {
#pragma unroll
        for (int i = 0; i < CVT; i++) {
            if (!((actmask >> i) & 1u)) continue;
            snap[sl[i]] = x[i];
            if (sl[i] < PULL_BITS) atomicOr(&hot[sl[i] >> 5], 1u << (sl[i] & 31));
        }
    } else if (snap_all && actmask) {
        if (u0 + CVT <= V) {
            uint4 *s4 = reinterpret_cast<uint4 *>(snap + u0);
#pragma unroll
            for (int q = 0; q < CVT / 4; q++) s4[q] = make_uint4(x[4 * q], x[4 * q + 1], x[4 * q + 2], x[4 * q + 3]);
        } else {
#pragma unroll
            for (int i = 0; i < CVT; i++)
                if (u0 + i < V) snap[u0 + i] = x[i];
        }
    }
    __syncthreads();
    if (tid == 0) {
        int nfb = 0;
#pragma unroll
        for (int w = 0; w < CBLOCK / 64; w++) {
            nfb += s_nf[w];
            low = min(low, s_min[w]);
        }
        atomicAdd(&step->frontier, (unsigned long long)nfb);
        if (snap_all && low != INF) atomicMax(&step->inv_min, ~low);
    }
    // The out-edges counted up to this workgroup are a lower bound of the
    // frontier's: once it reaches pull_edges the next superstep pulls and
    // never reads the list, so the rest of the workgroups skip writing it.
    if ((uint32_t)(s_base + total) >= pull_edges) return;
    unsigned long long pos = s_base + pre;
#pragma unroll
    for (int i = 0; i < CVT; i++) {
        const int32_t dg = r[i + 1] - r[i];
        if (!((actmask >> i) & 1u) || dg <= 0) continue;
        const int64_t u = u0 + i;
        const uint32_t idx = (uint32_t)(pos >> 32), off = (uint32_t)pos;
        list[idx] = make_uint4(off, (uint32_t)(r[i] - (int32_t)off), x[i], (uint32_t)u);
        const uint32_t t0 = (off + PUSH_TILE - 1) / PUSH_TILE, t1 = (off + (uint32_t)dg - 1) / PUSH_TILE;
        for (uint32_t t = t0; t <= t1; t++) tile_start[t] = idx;
        pos += (1ull << 32) + (uint32_t)dg;
    }
}

// Relaxes the active out-edges, PUSH_TILE per workgroup tile (persistent
// grid; the tile count comes from the compaction's counter).
struct PushLds {
    uint32_t base[PUSH_TILE + 1];
    uint32_t snap[PUSH_TILE + 1];
    int32_t own[PUSH_TILE];
    int32_t red[4];
};

template <bool WEIGHTED>
__device__ __forceinline__ void push_body(const uint4 *__restrict__ list, const uint32_t *__restrict__ tile_start,
                                          const void *__restrict__ adj, uint32_t *__restrict__ val,
                                          uint8_t *__restrict__ front_next, unsigned long long le, PushLds &lds) {
    uint32_t *s_base = lds.base;
    uint32_t *s_snap = lds.snap;
    int32_t *s_own = lds.own;
    int32_t *s_red = lds.red;
    const int tid = threadIdx.x;
    const uint32_t L = (uint32_t)(le >> 32), EF = (uint32_t)le;
    const uint32_t ntiles = (EF + PUSH_TILE - 1) / PUSH_TILE;
    for (uint32_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const uint32_t e0 = t * PUSH_TILE;
        const int n = (int)min((uint32_t)PUSH_TILE, EF - e0);
        const uint32_t s0 = tile_start[t];
        const uint32_t s1 = (t + 1 < ntiles) ? tile_start[t + 1] : L - 1;
        const int m = (int)(s1 - s0) + 1;
        for (int p = tid; p < n; p += PUSH_BLOCK) s_own[p] = 0;
        __syncthreads();
        for (int i = tid; i < m; i += PUSH_BLOCK) {
            uint4 en = list[s0 + i];
            s_base[i] = en.y + e0;  // CSR index of the tile's edge p is s_base[j] + p
            s_snap[i] = en.z;
            uint32_t rel = en.x - e0;
            if (i > 0 && rel < (uint32_t)n) s_own[rel] = i;
        }
        __syncthreads();
        block_max_scan<PUSH_VT>(s_own, n, s_red);
        // Batched memory access: every load is unconditional (slots past the
        // tile's end repeat its last edge and are dropped at the end), so the
        // thread issues all its edge loads, then all destination reads, with
        // one wait each and no load behind another edge's atomic.
        uint32_t idx[PUSH_VT], sv[PUSH_VT];
#pragma unroll
        for (int i = 0; i < PUSH_VT; i++) {
            const int p = min(tid + i * PUSH_BLOCK, n - 1);
            const int j = s_own[p];
            idx[i] = s_base[j] + (uint32_t)p;
            sv[i] = s_snap[j];
        }
        uint32_t dst[PUSH_VT], cand[PUSH_VT], cur[PUSH_VT];
#pragma unroll
        for (int i = 0; i < PUSH_VT; i++) {
            if (WEIGHTED) {
                const uint2 a = static_cast<const uint2 *>(adj)[idx[i]];
                dst[i] = a.x;
                cand[i] = a.y;
            } else {
                dst[i] = (uint32_t) static_cast<const int32_t *>(adj)[idx[i]];
            }
        }
#pragma unroll
        for (int i = 0; i < PUSH_VT; i++) cur[i] = val[dst[i]];
#pragma unroll
        for (int i = 0; i < PUSH_VT; i++) {
            cand[i] = WEIGHTED ? sat_add(sv[i], cand[i]) : sv[i];
            if (tid + i * PUSH_BLOCK >= n) cand[i] = INF;
        }
        // A candidate below a value read during this superstep is below the
        // destination's start-of-superstep value (values only fall), so the
        // destination changes in this superstep whichever atomic lands last:
        // mark it with an idempotent plain store and let the atomic go
        // without waiting for its result.  (Destinations here are written
        // from every XCD, so the merge stays an atomic minimum.)
#pragma unroll
        for (int i = 0; i < PUSH_VT; i++) {
            if (cand[i] < cur[i]) {
                atomicMin(&val[dst[i]], cand[i]);
                front_next[dst[i]] = 1;
            }
        }
        __syncthreads();
    }
}

// Pull form of the same superstep, for large frontiers: every row takes the
// minimum over its in-edges (CC: its neighbours) of the values at the
// superstep's start.  What an inactive source sends was merged into the row
// when that source last changed, so no frontier test is needed per entry,
// and a row needs only those of its entries that could still lower it: no
// message is below `low`, the smallest active value, plus the entry's
// weight.  A row is its value's only writer and stores plainly; the segments
// of a long row, and a merge into an accumulator, use an atomic minimum.
//
// Long rows (segments), and every row of CC: one per thread is tested, the
// survivors are queued in LDS and scanned by groups of G lanes, 2 G
// consecutive entries at a time.  The entries of SSSP's long rows ascend by
// weight, so a row ends at the first entry whose bound is not below the best
// value found so far; a CC row ends as soon as it holds the smallest active
// label (hubs reach it first and, in graphs whose ids go by degree, come
// first in a row).
// SSSP's short rows: a wave streams the entries of 64 rows, whatever rows
// they belong to (an entry names its row within the 64), and takes the
// minimum per row in LDS, so no load waits for another row's.
// An entry whose source is not active (a bit in LDS for the sources with the
// most out-edges) or whose bound is too large reads no value.
//
// Bound by the latency of dependent reads (entries, then values) and, in the
// first pull of a solve, by the rate of random 4-byte reads.  R-MAT scale 22
// (65 M in-edges), the four pulls of the benchmarked solve: 241, 132, 85 and
// 75 us; the sweep takes 250-280 us for each there.  Short rows of at most 16, 32,
// 64, 128 entries: 861, 847, 1060, 1104 us for six pulls of another solve, before
// the frontier bits were kept in LDS.
struct RowItems {
    uint32_t row[64], beg[64], end[64], best[64];
};

struct PullArgs {
    const int32_t *rp;      // CC: rows; SSSP: first entry of every block of 64 short rows
    const void *adj;        // uint2 {source slot, (row mod 64) << 8 | weight} (SSSP) or int32 neighbour (CC)
    const uint4 *segs;
    int64_t nsegs;
    int first_only;         // CC before anything changed: labels ascend with the neighbours, so the first decides
    int atomic_rows;        // rows merge into an accumulator
    const uint32_t *bound;  // values that messages must be below (the vertex values)
    const uint32_t *hot;    // SSSP: frontier bits of the first slots
};

struct PullLds {
    RowItems items[4];
    uint32_t bits[PULL_BIT_WORDS];
};

// Whether slot `u` may be active (slots past the bits always may).
__device__ __forceinline__ bool may_be_active(const uint32_t *bits, uint32_t u) {
    return u >= (uint32_t)PULL_BITS || ((bits[u >> 5] >> (u & 31)) & 1u);
}

template <bool WEIGHTED, int G, int UN>
__device__ __forceinline__ void scan_items(const RowItems &it, const uint32_t *bits, int n, const PullArgs &pa, uint32_t low,
                                           const uint32_t *__restrict__ snap, uint32_t *tgt,
                                           uint8_t *__restrict__ front_next, bool atomic) {
    const int lane = threadIdx.x & 63, g = lane / G, gl = lane % G;
    for (int i0 = 0; i0 < n; i0 += 64 / G) {
        const int i = min(i0 + g, n - 1);
        bool live = i0 + g < n;
        const uint32_t row = it.row[i], end = it.end[i], start = it.best[i];
        uint32_t p = it.beg[i] + (uint32_t)gl, best = start;
        while (__any(live)) {
            // (every load is unconditional, so the chunk's loads overlap)
            uint32_t u[UN], w[UN], s[UN], bnd = INF, cand = INF;
            bool take[UN];
#pragma unroll
            for (int j = 0; j < UN; j++) {
                const uint32_t q = min(p + (uint32_t)(j * G), end - 1);
                if (WEIGHTED) {
                    const uint2 a = static_cast<const uint2 *>(pa.adj)[q];
                    u[j] = a.x, w[j] = a.y & 0xFFu;
                } else {
                    u[j] = (uint32_t) static_cast<const int32_t *>(pa.adj)[q], w[j] = 0;
                }
            }
#pragma unroll
            for (int j = 0; j < UN; j++) {
                bnd = live && p + (uint32_t)(j * G) < end ? sat_add(low, w[j]) : INF;
                take[j] = bnd < best && (!WEIGHTED || may_be_active(bits, u[j]));
                s[j] = snap[take[j] ? u[j] : row];
            }
#pragma unroll
            for (int j = 0; j < UN; j++) cand = min(cand, take[j] ? sat_add(s[j], w[j]) : INF);
#pragma unroll
            for (int o = G / 2; o > 0; o >>= 1) cand = min(cand, (uint32_t)__shfl_xor(cand, o, 64));
            best = min(best, cand);
            // the chunk's last entry has its largest bound (INF past the row's end)
            live = live && (uint32_t)__shfl(bnd, lane | (G - 1), 64) < best;
            p += UN * G;
        }
        if (gl == 0 && i0 + g < n && best < start) {
            if (atomic) atomicMin(&tgt[row], best);
            else tgt[row] = best;
            front_next[row] = 1;
        }
    }
}

// Queues the threads' rows (or segments) that pass the filter, a wave's in
// its own LDS list; returns their number.
__device__ __forceinline__ int queue_items(RowItems &it, bool take, uint32_t row, uint32_t beg, uint32_t end,
                                           uint32_t best) {
    const unsigned long long m = __ballot(take);
    if (take) {
        const int pos = __popcll(m & ((1ull << (threadIdx.x & 63)) - 1ull));
        it.row[pos] = row;
        it.beg[pos] = beg;
        it.end[pos] = end;
        it.best[pos] = best;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    return __popcll(m);
}

// The 64 rows of one wave, all short (SSSP): best[i] is row v0 + i's minimum.
__device__ __forceinline__ void stream_rows(uint32_t *best, const uint32_t *bits, int64_t v, uint32_t cur, int32_t rp0,
                                            int32_t rp1, const PullArgs &pa, uint32_t low,
                                            const uint32_t *__restrict__ snap, uint32_t *tgt,
                                            uint8_t *__restrict__ front_next) {
    constexpr int UN = 4;
    const int lane = threadIdx.x & 63;
    const uint32_t beg = (uint32_t)rp0, end = (uint32_t)rp1;
    if (!__any(low < cur) || beg == end) return;
    const uint2 *adj = static_cast<const uint2 *>(pa.adj);
    best[lane] = cur;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    for (uint32_t p0 = beg; p0 < end; p0 += 64 * UN) {
        uint2 q[UN];
        uint32_t s[UN];
        bool take[UN];
#pragma unroll
        for (int j = 0; j < UN; j++) q[j] = adj[min(p0 + 64u * j + (uint32_t)lane, end - 1)];
#pragma unroll
        for (int j = 0; j < UN; j++) {  // (an entry past the end repeats the last one: harmless)
            take[j] = sat_add(low, q[j].y & 0xFFu) < best[q[j].y >> 8] && may_be_active(bits, q[j].x);
            s[j] = snap[take[j] ? q[j].x : (uint32_t)(v - lane)];
        }
#pragma unroll
        for (int j = 0; j < UN; j++) {
            const uint32_t c = sat_add(s[j], q[j].y & 0xFFu);
            if (take[j] && c < best[q[j].y >> 8]) atomicMin(&best[q[j].y >> 8], c);
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const uint32_t b = best[lane];
    if (b < cur) {
        if (pa.atomic_rows) atomicMin(&tgt[v], b);
        else tgt[v] = b;
        front_next[v] = 1;
    }
}

// Row v takes the label of its first neighbour, the smallest.
__device__ __forceinline__ void first_neighbour(const PullArgs &pa, int64_t v, uint32_t beg, uint32_t end, uint32_t low,
                                                uint32_t cur, const uint32_t *__restrict__ snap, uint32_t *tgt,
                                                uint8_t *__restrict__ front_next) {
    if (beg >= end || low >= cur) return;
    const uint32_t c = snap[(uint32_t) static_cast<const int32_t *>(pa.adj)[beg]];
    if (c >= cur) return;
    if (pa.atomic_rows) atomicMin(&tgt[v], c);
    else tgt[v] = c;
    front_next[v] = 1;
}

// The slice of a pulling workgroup: the XCD it runs on.  The hardware deals a
// launch's workgroups to the XCDs in turn, from XCD r for workgroup 0 (r has
// been seen to differ between launches), so workgroup b runs on XCD
// (b + r) mod 8 and is the (b / 8)-th of its XCD (the grid is a multiple of
// 8).  If the workgroups of one launch saw different r, some work would be
// taken twice and some never: each leaves the r it saw, and the launch that
// follows flags the superstep if they differ.  (xcd_shift, zero outside tests,
// offsets the odd workgroups' XCD to exercise that check.)
__device__ __forceinline__ uint32_t pull_slice(DevStep *__restrict__ step, uint32_t xcd_shift,
                                               uint32_t *__restrict__ rot) {
    const uint32_t x = (xcc_id() + ((blockIdx.x & 1u) ? xcd_shift : 0u)) % PULL_SLICES;
    if (threadIdx.x == 0) rot[blockIdx.x] = (x + PULL_SLICES - blockIdx.x % PULL_SLICES) % PULL_SLICES;
    if (blockIdx.x == 0 && threadIdx.x == 0) step->pad = 1;
    return x;
}

template <bool WEIGHTED>
__device__ __forceinline__ void pull_body(const PullArgs &pa, int64_t V, const uint32_t *__restrict__ snap,
                                          uint32_t *tgt, uint8_t *__restrict__ front_next,
                                          DevStep *__restrict__ step, PullLds &lds, uint32_t xcd_shift,
                                          uint32_t *__restrict__ rot) {
    const int tid = threadIdx.x;
    RowItems &it = lds.items[tid >> 6];
    const uint32_t low = ~step->inv_min;
    // Of every 8 runs of consecutive blocks a slice takes one run (neighbouring
    // rows, whose sources often neighbour each other too, share an L2), another
    // one in each group of 8: where rows get shorter with every bit set in their
    // id, as on R-MAT, a fixed one would give one XCD many times the others'
    // entries (scale 22, first pull of a solve, in an earlier form: 380 us, with the
    // turn 335 us).
    const uint32_t x = pull_slice(step, xcd_shift, rot);
    const int64_t nper = gridDim.x / PULL_SLICES;
    const int64_t nseg = pa.first_only ? 0 : (pa.nsegs + PULL_SEG_BLOCK - 1) / PULL_SEG_BLOCK;
    const int64_t nblk = nseg + (V + PULL_BLOCK - 1) / PULL_BLOCK;
    const int lg = nblk >= PULL_RUN_FROM ? PULL_RUN_LOG : 0;
    if ((((int64_t)(blockIdx.x / PULL_SLICES) >> lg) * PULL_SLICES << lg) >= nblk) return;  // no block for it
    if (WEIGHTED) {
        const uint4 *h4 = reinterpret_cast<const uint4 *>(pa.hot);
        const int n4 = (int)min((V + 127) / 128, (int64_t)(PULL_BIT_WORDS / 4));
        for (int q = tid; q < n4; q += 256) reinterpret_cast<uint4 *>(lds.bits)[q] = h4[q];
        __syncthreads();
    }
    for (int64_t j = blockIdx.x / PULL_SLICES;; j += nper) {
        const uint32_t grp = (uint32_t)(j >> lg);
        if ((int64_t)grp * PULL_SLICES << lg >= nblk) break;
        const uint32_t turn = (x + (grp * 0x9E3779B1u >> 29)) % PULL_SLICES;
        const int64_t blk = (((int64_t)grp * PULL_SLICES + turn) << lg) + (j & ((1 << lg) - 1));
        if (blk >= nblk) continue;
        __builtin_amdgcn_wave_barrier();
        if (blk < nseg) {  // segments of long rows first: they are the longest work
            // (a wave takes few segments, so that a superstep that has to
            // read them all finds every wave at work)
            const int64_t q = blk * PULL_SEG_BLOCK + (tid >> 6) * (PULL_SEG_BLOCK / 4) + (tid & 63);
            uint4 sg = make_uint4(0u, 0u, 0u, 0u);
            uint32_t cur = 0;
            if ((tid & 63) < PULL_SEG_BLOCK / 4 && q < pa.nsegs) {
                sg = pa.segs[q];
                cur = pa.bound[sg.x];
            }
            const int n = queue_items(it, sat_add(low, sg.w & 0xFFu) < cur, sg.x, sg.y, sg.z, cur);
            scan_items<WEIGHTED, 16, 4>(it, lds.bits, n, pa, low, snap, tgt, front_next, true);
            continue;
        }
        const int64_t v = (blk - nseg) * PULL_BLOCK + tid;
        const uint32_t cur = v < V ? pa.bound[v] : 0u;
        if (WEIGHTED) {
            const int64_t b = min(v, V - 1) >> 6;
            stream_rows(it.best, lds.bits, v, cur, pa.rp[b], pa.rp[b + 1], pa, low, snap, tgt, front_next);
            continue;
        }
        uint32_t beg = 0, end = 0;
        if (v < V) {
            beg = (uint32_t)pa.rp[v];
            end = (uint32_t)pa.rp[v + 1];
        }
        if (pa.first_only) {
            first_neighbour(pa, v, beg, end, low, cur, snap, tgt, front_next);
            continue;
        }
        const int n = queue_items(it, beg < end && end - beg <= PULL_SMALL && low < cur, (uint32_t)v, beg, end, cur);
        scan_items<WEIGHTED, 4, 2>(it, lds.bits, n, pa, low, snap, tgt, front_next, pa.atomic_rows != 0);
    }
}

// CC's first superstep where the sweep is the pull: one neighbour per row.
__device__ __forceinline__ void first_body(const PullArgs &pa, int64_t V, const uint32_t *__restrict__ snap,
                                           uint32_t *tgt, uint8_t *__restrict__ front_next,
                                           DevStep *__restrict__ step, uint32_t *__restrict__ rot) {
    if (threadIdx.x == 0) rot[blockIdx.x] = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) step->pad = 1;
    for (int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x; v < V; v += (int64_t)gridDim.x * 256)
        first_neighbour(pa, v, (uint32_t)pa.rp[v], (uint32_t)pa.rp[v + 1], ~step->inv_min, pa.bound[v], snap, tgt,
                        front_next);
}

// Pull form on graphs without hubs (see Sweep): every record once.  A
// workgroup takes units of its slice, so each XCD's L2 holds one bin's
// destinations; a unit's band of source values is staged in LDS, INF where the
// frontier map says the source is inactive, so a record's gather is an LDS
// read.  The 64 lanes of a wave take 64 consecutive records (destinations
// ascending), so lanes whose destinations share a cache line make one request
// between them: those reads, one per record, bound it.  A record without a
// candidate reads nothing (its offset lies past the buffer).
//
// A candidate below a value read during the superstep is below the
// destination's start value (values only fall), so the destination changes
// whatever else lands: it is marked, its value is set with a plain store, and
// the pair goes to the workgroup's fix-up region.  Racing stores may leave a
// larger candidate; k_fixup, a later launch, re-applies every recorded one that
// is still below.  Every writer of a destination runs on the XCD of its slice,
// so one L2 sees all of its stores, and a region holds every record its
// workgroup can meet, so no candidate goes another way.  (With an atomic
// minimum instead, 2^22 vertices, 67 M uniform edges, the first pull of a solve
// takes 820 us, 590 so.)
struct FixRegion {
    uint2 *ent;       // this workgroup's region
    uint32_t *count;  // LDS: candidates so far
};

template <bool WEIGHTED>
__device__ __forceinline__ void sweep_body(const Sweep &sw, int64_t V, const uint32_t *__restrict__ snap,
                                           const uint8_t *__restrict__ front_cur, uint32_t *tgt,
                                           uint8_t *__restrict__ front_next, DevStep *__restrict__ step,
                                           uint32_t *s_val, const FixRegion &fr, uint32_t xcd_shift,
                                           uint32_t *__restrict__ rot) {
    const int tid = threadIdx.x, lane = tid & 63;
    const uint32_t x = pull_slice(step, xcd_shift, rot);
    const __amdgpu_buffer_rsrc_t trs =
        __builtin_amdgcn_make_buffer_rsrc(tgt, (short)0, (int)(uint32_t)(V * 4), 0x00020000);
    const int64_t nper = gridDim.x / PULL_SLICES;
    for (int64_t ui = sw.uoff[x] + blockIdx.x / PULL_SLICES; ui < sw.uoff[x + 1]; ui += nper) {
        const uint4 un = sw.units[ui];
        const uint32_t start = un.x, end = un.x + un.y, bb = un.z;
        __syncthreads();  // the previous unit's gathers are done
        if ((int64_t)bb + SWEEP_BAND <= V) {
            const uint4 *s4 = reinterpret_cast<const uint4 *>(snap + bb);
            const uint32_t *f4 = reinterpret_cast<const uint32_t *>(front_cur + bb);
            constexpr int N = SWEEP_BAND / 4 / 256;
            uint4 sv[N];
            uint32_t fv[N];
#pragma unroll
            for (int q = 0; q < N; q++) {
                sv[q] = s4[q * 256 + tid];
                fv[q] = f4[q * 256 + tid];
            }
#pragma unroll
            for (int q = 0; q < N; q++)
                reinterpret_cast<uint4 *>(s_val)[q * 256 + tid] =
                    make_uint4(fv[q] & 0xFFu ? sv[q].x : INF, fv[q] & 0xFF00u ? sv[q].y : INF,
                               fv[q] & 0xFF0000u ? sv[q].z : INF, fv[q] & 0xFF000000u ? sv[q].w : INF);
        } else {  // the last band ends at V
            for (int i = tid; i < SWEEP_BAND; i += 256) s_val[i] = bb + i < V && front_cur[bb + i] ? snap[bb + i] : INF;
        }
        __syncthreads();
        for (uint32_t c0 = start; c0 < end; c0 += 256 * SWEEP_VT) {
            uint32_t dst[SWEEP_VT], m[SWEEP_VT], cur[SWEEP_VT];
            uint2 q[SWEEP_VT];
#pragma unroll
            for (int i = 0; i < SWEEP_VT; i++) q[i] = sw.rec[min(c0 + (uint32_t)i * 256 + (uint32_t)tid, end - 1)];
#pragma unroll
            for (int i = 0; i < SWEEP_VT; i++) {  // (past the unit's end: no candidate, so a region holds them all)
                dst[i] = c0 + (uint32_t)i * 256 + (uint32_t)tid < end ? q[i].x : SWEEP_SENTINEL;
                const uint32_t sv = s_val[q[i].y >> 8];
                m[i] = dst[i] == SWEEP_SENTINEL ? INF : WEIGHTED ? sat_add(sv, q[i].y & 0xFFu) : sv;
                cur[i] = __builtin_amdgcn_raw_buffer_load_b32(trs, m[i] != INF ? dst[i] * 4u : 0x80000000u, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);  // every read above is issued before the first compare
            uint32_t cnt = 0;
#pragma unroll
            for (int i = 0; i < SWEEP_VT; i++) cnt += m[i] < cur[i];
            // one reservation per wave, entries in lane order
            uint32_t incl = cnt;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t y = __shfl_up(incl, o, 64);
                if (lane >= o) incl += y;
            }
            uint32_t pos = 0;
            if (lane == 63 && incl) pos = atomicAdd(fr.count, incl);
            pos = __shfl(pos, 63, 64) + incl - cnt;
#pragma unroll
            for (int i = 0; i < SWEEP_VT; i++)
                if (m[i] < cur[i]) {
                    fr.ent[pos++] = make_uint2(dst[i], m[i]);
                    tgt[dst[i]] = m[i];
                    front_next[dst[i]] = 1;
                }
        }
    }
}

// One launch per superstep: the frontier's edge count, known on the device
// after the compaction, picks the form (a second, idle launch would cost a
// dispatch and a sweep of exiting workgroups every superstep).
union RelaxLds {
    PushLds push;
    PullLds pull;
};
union SweepLds {
    PushLds push;
    uint32_t val[SWEEP_BAND];
};

// (CC's first superstep reads one neighbour per row in either pull.)
template <bool WEIGHTED>
__global__ __launch_bounds__(256) void k_relax_sweep(
    const uint4 *__restrict__ list, const uint32_t *__restrict__ tile_start, const void *__restrict__ adj, PullArgs pa,
    Sweep sw, const uint8_t *__restrict__ front_cur, int64_t V, const uint32_t *__restrict__ snap, uint32_t *val,
    uint8_t *__restrict__ front_next, DevStep *__restrict__ step, uint32_t pull_edges, uint2 *__restrict__ fix,
    uint32_t *__restrict__ fixn, uint32_t fix_cap, uint32_t *__restrict__ rot, uint32_t xcd_shift) {
    __shared__ SweepLds lds;
    __shared__ uint32_t s_fixn;
    if (threadIdx.x == 0) s_fixn = 0;
    __syncthreads();
    const unsigned long long le = step->list;
    if ((uint32_t)le < pull_edges)
        push_body<WEIGHTED>(list, tile_start, adj, val, front_next, le, lds.push);
    else if (!WEIGHTED && pa.first_only)
        first_body(pa, V, snap, val, front_next, step, rot);
    else
        sweep_body<WEIGHTED>(sw, V, snap, front_cur, val, front_next, step, lds.val,
                             FixRegion{fix + (size_t)blockIdx.x * fix_cap, &s_fixn}, xcd_shift, rot);
    __syncthreads();
    if (threadIdx.x == 0) fixn[blockIdx.x] = s_fixn;
}

// Workgroup b re-applies the candidates that relaxation workgroup b recorded
// and that are still below the stored value (after a push there are none).
__global__ __launch_bounds__(256) void k_fixup(const uint2 *__restrict__ fix, const uint32_t *__restrict__ fixn,
                                               uint32_t fix_cap, uint32_t *__restrict__ val) {
    const uint32_t n = fixn[blockIdx.x];
    const uint2 *e = fix + (size_t)blockIdx.x * fix_cap;
    for (uint32_t i = threadIdx.x; i < n; i += 256) {
        const uint2 q = e[i];
        if (q.y < val[q.x]) atomicMin(&val[q.x], q.y);
    }
}

template <bool WEIGHTED>
__global__ __launch_bounds__(256) void k_relax(const uint4 *__restrict__ list, const uint32_t *__restrict__ tile_start,
                                               const void *__restrict__ adj, PullArgs pa, int64_t V,
                                               const uint32_t *__restrict__ snap, uint32_t *val,
                                               uint8_t *__restrict__ front_next, DevStep *__restrict__ step,
                                               uint32_t pull_edges, uint32_t *__restrict__ rot, uint32_t xcd_shift) {
    __shared__ RelaxLds lds;
    const unsigned long long le = step->list;
    if ((uint32_t)le >= pull_edges)
        pull_body<WEIGHTED>(pa, V, snap, val, front_next, step, lds.pull, xcd_shift, rot);
    else
        push_body<WEIGHTED>(list, tile_start, adj, val, front_next, le, lds.push);
}

// ------------------------------------------------------------ PageRank

__global__ __launch_bounds__(256) void k_pr_init(float *x, float *contrib, uint32_t *synced,
                                                 const int32_t *__restrict__ outdeg, const int32_t *__restrict__ slot,
                                                 int64_t V, float x0, double *dpart, DevStep *step0) {
    __shared__ double s_d[4];
    int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v == 0) *step0 = DevStep{};
    double dl = 0.0;
    if (v < V) {
        int od = outdeg[v];
        x[v] = x0;
        synced[v] = __float_as_uint(x0);
        contrib[slot[v]] = od > 0 ? x0 / (float)od : 0.0f;
        if (od == 0) dl = (double)x0;
    }
    double t = block_sum<double>(dl, s_d);
    if (threadIdx.x == 0) dpart[blockIdx.x] = t;
}

// Single workgroup: D = sum of n partials in a fixed order.
__global__ __launch_bounds__(1024) void k_reduce_D(const double *__restrict__ part, int n, double *D) {
    __shared__ double s_d[16];
    double a = 0.0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) a += part[i];
    double t = block_sum<double>(a, s_d);
    if (threadIdx.x == 0) *D = t;
}

struct PrApply {
    double base, d, dD;  // x' = base + d * acc + dD, with dD = d * D / V
    const float *x_in;
    float *x_out, *c_out;
    static constexpr bool kRows = true;  // reads out-degree, slot and old rank
    __device__ __forceinline__ void row(int32_t r, double acc, int32_t od, int32_t sl, float xi, double &dsum,
                                        int &chg) const {
        float xn = (float)(base + d * acc + dD);
        x_out[r] = xn;
        if (od > 0) c_out[sl] = xn / (float)od;  // (a slot without out-edges is not gathered)
        else dsum += (double)xn;
        chg += __float_as_uint(xn) != __float_as_uint(xi);
    }
};

// The merge alone (separate template calls): the combined messages of a row
// are stored; what is applied happens later.
struct PrStore {
    double d, dD;  // (unused)
    double *acc;
    static constexpr bool kRows = false;
    static constexpr const float *x_in = nullptr;
    __device__ __forceinline__ void row(int32_t r, double total, int32_t, int32_t, float, double &, int &) const {
        acc[r] = total;
    }
};

struct PrArgs {
    const int32_t *src;        // slot of every in-edge's source
    const uint8_t *row_last;   // a bit per in-edge: the last of its row
    const int32_t *tile_nz;
    const int2 *nz, *ez;
    const int32_t *nz_slot, *slot;
    const int4 *cross;
    int32_t n_cross, n_cross_long, n_cross_mid;
    int64_t V, E, n_nz, n_ez;
    int32_t ntiles;
    const float *c_in;
    double *Dp;
    double inv_V;
    double *head, *tailp, *dpart;
    uint32_t *cpart;
    int nparts;
};

// A wave takes tiles of 64 * VT consecutive in-edges, lane l the VT edges from
// l * VT on: it loads their source slots and row-end bits, gathers all their
// contributions, and a segmented scan over the lanes gives each the sum that
// the lanes before it leave open for its first row.  The sums of the rows that
// end in the tile go through LDS, so that the rows' slots, old ranks and new
// values are read and written by consecutive lanes.  A row that began in an
// earlier tile leaves its sum in head, one that goes on in tailp.  Rows
// without in-edges come last, four per lane.
//
// HOT: the contributions of the first slots (the sources of the most edges)
// are staged in LDS, and only the other gathers go to memory: the staged
// slots' offsets lie past the buffer, which fetches nothing.
//
// Bound by the gathers that reach an L2, about one per in-edge without the LDS
// table; with it, 0.48 of the edges of R-MAT scale 22 (65 M in-edges).  There
// the pull takes 262 us: 115 without any gather, 210 if all of them hit an L2,
// 235 without the sums; the gathers' requests run at about 150 G/s whatever
// the lanes' order.  A workgroup per tile, with every value staged in LDS and
// a search for the row of each edge, took 483 us.
// Inclusive sums over the lanes: within 16, within a half, over the wave.  Of
// the lanes before this one, the nearest `from` belong to its segment.
__device__ __forceinline__ double dpp_scan(double x, int from, int lane) {
    const int at = lane & 15;
#define GX_SCAN_STEP(CTRL, ROWS, TAKE)                                                                        \
    {                                                                                                         \
        const long long b = __double_as_longlong(x);                                                          \
        const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, ROWS, 0xf, false);                        \
        const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROWS, 0xf, false);                \
        const bool take = TAKE;                                                                               \
        x += __longlong_as_double(((long long)(take ? hi : 0) << 32) | (uint32_t)(take ? lo : 0));            \
    }
    GX_SCAN_STEP(0x111, 0xf, from >= 1)  // row_shr
    GX_SCAN_STEP(0x112, 0xf, from >= 2)
    GX_SCAN_STEP(0x114, 0xf, from >= 4)
    GX_SCAN_STEP(0x118, 0xf, from >= 8)
    GX_SCAN_STEP(0x142, 0xa, from > at)         // lane 15 of the row before (row_bcast:15)
    GX_SCAN_STEP(0x143, 0xc, from > lane - 32)  // lane 31 (row_bcast:31)
#undef GX_SCAN_STEP
    return x;
}
__device__ __forceinline__ int dpp_scan(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);
    return x;
}

template <int VT, bool HOT, class AP>
__global__ __launch_bounds__(HOT ? 1024 : PR_BLOCK) void k_pr_pull(PrArgs a, AP ap) {
    constexpr int NW = (HOT ? 1024 : PR_BLOCK) / 64, T = 64 * VT, SUMS = T < 256 ? T : 256;
    constexpr int NEAR = HOT ? PR_LDS_SLOTS : 0;
    __shared__ double s_sum[NW][SUMS];
    __shared__ float s_hot[NEAR + 4];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    // from slot NEAR on; the staged slots' offsets wrap round and lie past the buffer, as does the padding's
    const __amdgpu_buffer_rsrc_t crs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(a.c_in) + NEAR, (short)0, (int)(uint32_t)((a.V - NEAR) * 4), 0x00020000);
    if (HOT) {
        for (int i = threadIdx.x; i < NEAR / 4; i += 1024)
            reinterpret_cast<float4 *>(s_hot)[i] = reinterpret_cast<const float4 *>(a.c_in)[i];
        if (threadIdx.x == 0) s_hot[NEAR] = 0.f;
        __syncthreads();
    }
    ap.dD = ap.d * (*a.Dp) * a.inv_V;
    double *sums = s_sum[wv];
    double dsum = 0.0;
    int chg = 0;
    const int gw = (int)blockIdx.x * NW + wv, nw = (int)gridDim.x * NW;
    // Three tiles are in the works: the sources, row ends and rows of the one
    // after next are loaded, the contributions and old ranks of the next one
    // gathered, and this one is summed.
    struct Rows {
        uint32_t bits = 0;
        int2 r = {0, 0};
        int32_t ord = 0, sl = 0;
        bool head = false;
    };
    const auto load = [&](int64_t t, int32_t(&u)[VT], Rows &q) {
        const int64_t e0 = t * T, e1 = e0 + lane * VT;
        // (the in-edges stream by once: kept out of the caches' way)
        constexpr int LW = VT < 4 ? VT : 4;
        typedef int32_t Wide __attribute__((ext_vector_type(LW)));
#pragma unroll
        for (int j = 0; j < VT; j += LW) {
            const Wide x = __builtin_nontemporal_load(reinterpret_cast<const Wide *>(&a.src[e1 + j]));
#pragma unroll
            for (int i = 0; i < LW; i++) u[j + i] = x[i];
        }
        q.bits = (a.row_last[e1 >> 3] >> (e1 & 7)) & ((1u << VT) - 1u);
        q.head = e0 > 0 && !((a.row_last[(e0 - 1) >> 3] >> 7) & 1u);
        q.ord = a.tile_nz[t];
        const int32_t i = min(q.ord + lane, (int32_t)a.n_nz - 1);
        q.r = a.nz[i];
        q.sl = AP::kRows ? a.nz_slot[i] : 0;
    };
    const auto gather = [&](const int32_t(&u)[VT], const Rows &q, float(&cv)[VT], float &xi) {
        xi = AP::kRows ? ap.x_in[q.r.x] : 0.f;
#pragma unroll
        for (int j = 0; j < VT; j++)
            cv[j] = HOT ? __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(crs, ((uint32_t)u[j] - NEAR) * 4u, 0, 0))
                        : a.c_in[u[j]];
    };
    int32_t u[VT], un[VT];
    float cv[VT], xi = 0.f;
    Rows q, qn;
    if (gw < a.ntiles) {
        load(gw, u, q);
        if (gw + nw < a.ntiles) load(gw + nw, un, qn);
        gather(u, q, cv, xi);
    }
    for (int64_t t = gw; t < a.ntiles; t += nw) {
        int32_t us[VT];
        float cn[VT], xn = 0.f;
        Rows qs;
        if (t + 2 * nw < a.ntiles) load(t + 2 * nw, us, qs);
        if (t + nw < a.ntiles) gather(un, qn, cn, xn);
        if (HOT)
#pragma unroll
            for (int j = 0; j < VT; j++) cv[j] += s_hot[min((uint32_t)u[j], (uint32_t)NEAR)];  // (one of them is 0)
        else if ((t + 1) * T > a.E)
#pragma unroll
            for (int j = 0; j < VT; j++) cv[j] = t * T + lane * VT + j < a.E ? cv[j] : 0.f;
        const int n = __popc(q.bits);
        const int upto = dpp_scan(n), ends = __builtin_amdgcn_readlane(upto, 63);
        const unsigned long long has = __ballot(n > 0) & (~0ull >> (63 - lane));
        // what each lane leaves open, and what the lanes before it carry into its first row
        double open = 0.0;
#pragma unroll
        for (int j = 0; j < VT; j++) open += (double)(q.bits < (1u << j) ? cv[j] : 0.f);
        open = dpp_scan(open, has ? lane - 63 + __clzll(has) : lane, lane);
        const long long ob = __double_as_longlong(open);
        const int clo = __builtin_amdgcn_update_dpp(0, (int)ob, 0x138, 0xf, 0xf, false);  // wave_shr:1
        const int chi = __builtin_amdgcn_update_dpp(0, (int)(ob >> 32), 0x138, 0xf, 0xf, false);
        const double carry = __longlong_as_double(((long long)chi << 32) | (uint32_t)clo);
        if (lane == 63) {  // what is open at the end of the tile
            if (ends > 0 || !q.head) a.tailp[t] = open;
            else a.head[t] = open;
        }
        for (int base = 0; base < ends; base += SUMS) {
            __builtin_amdgcn_wave_barrier();
            double sum = carry;
            int p = upto - n - base;
#pragma unroll
            for (int j = 0; j < VT; j++) {
                sum += (double)cv[j];
                if ((q.bits >> j) & 1u) {
                    if (T == SUMS || (uint32_t)p < (uint32_t)SUMS) sums[p] = sum;
                    p++;
                    sum = 0.0;
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (base == 0) {
                if (q.head && lane == 0) a.head[t] = sums[0];
                if (lane >= (q.head ? 1 : 0) && lane < ends) ap.row(q.r.x, sums[lane], q.r.y, q.sl, xi, dsum, chg);
            }
            for (int i = base + lane + (base ? 0 : 64); i < min(ends, base + SUMS); i += 64) {
                const int2 r = a.nz[q.ord + i];
                ap.row(r.x, sums[i - base], r.y, AP::kRows ? a.nz_slot[q.ord + i] : 0, AP::kRows ? ap.x_in[r.x] : 0.f,
                       dsum, chg);
            }
        }
#pragma unroll
        for (int j = 0; j < VT; j++) {
            u[j] = un[j];
            un[j] = us[j];
            cv[j] = cn[j];
        }
        xi = xn;
        q = qn;
        qn = qs;
    }
    // rows without in-edges
    for (int64_t i0 = (int64_t)gw * 256; i0 < a.n_ez; i0 += (int64_t)nw * 256) {
        int2 r[4];
        int32_t sl[4];
        float xi[4];
#pragma unroll
        for (int j = 0; j < 4; j++) r[j] = a.ez[min(i0 + 64 * j + lane, a.n_ez - 1)];
#pragma unroll
        for (int j = 0; j < 4; j++) {
            sl[j] = AP::kRows && r[j].y > 0 ? a.slot[r[j].x] : 0;
            xi[j] = AP::kRows ? ap.x_in[r[j].x] : 0.f;
        }
#pragma unroll
        for (int j = 0; j < 4; j++)
            if (i0 + 64 * j + lane < a.n_ez) ap.row(r[j].x, 0.0, r[j].y, sl[j], xi[j], dsum, chg);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        dsum += __shfl_down(dsum, o, 64);
        chg += __shfl_down(chg, o, 64);
    }
    if (lane == 0) {  // per-wave partials, summed by k_pr_fix (no atomics on one shared counter)
        a.dpart[gw] = dsum;
        a.cpart[gw] = (uint32_t)chg;
    }
}

// Completes the rows that cross tile boundaries and reduces the dangling mass
// of the new ranks for the next superstep: every workgroup leaves its partial
// sums, and the last one to finish adds them up in workgroup order, so the
// result does not depend on timing (a single workgroup is done with its own).
// A chain of dependent accesses bounds it, so each wave has one kind of work:
// R-MAT scale 22 43 us with a thread or sixteen lanes per row one after the
// other in 1024 workgroups of 256, whose returning atomics on one counter
// queue, 21 us in workgroups of 1024; 20 supersteps of scale 14 take 329 us with
// the kinds one after the other, 278 us so (tiles of 1024).  The kernel boundary makes every pull
// wave's partials visible here; *Dp (the old mass) is read by every workgroup
// before the last one overwrites it.
constexpr int PR_FIX_BLOCK = 1024;  // (at most)
constexpr int PR_FIX_MAX_GRID = 512;

// The work of a k_pr_fix wave, in this order; each bound is the first unit of
// the next kind.
struct PrFixUnits {
    int wave, mid, few, all;
    __host__ __device__ PrFixUnits(int n_cross, int n_long, int n_mid, int nparts)
        : wave(n_long), mid(wave + (n_mid + 3) / 4), few(mid + (n_cross - n_long - n_mid + 63) / 64),
          all(few + (nparts + 255) / 256) {}
};

template <class AP>
__global__ __launch_bounds__(PR_FIX_BLOCK) void k_pr_fix(PrArgs a, AP ap, DevStep *__restrict__ step,
                                                         DevStep *__restrict__ next_step, double *fix_d,
                                                         unsigned long long *fix_c, uint32_t *fix_done) {
    __shared__ double s_d[PR_FIX_BLOCK / 64];
    __shared__ unsigned long long s_c[PR_FIX_BLOCK / 64];
    __shared__ int s_last;
    ap.dD = ap.d * (*a.Dp) * a.inv_V;
    double dsum = 0.0;
    int chg = 0;
    unsigned long long csum = 0;
    const int lane = threadIdx.x & 63, sub = lane & 15, waves = (int)(gridDim.x * blockDim.x) / 64;
    const PrFixUnits n(a.n_cross, a.n_cross_long, a.n_cross_mid, a.nparts);
    for (int w = (int)(blockIdx.x * blockDim.x + threadIdx.x) / 64; w < n.all; w += waves) {
        if (w >= n.few) {  // the pull's partials, four per lane
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const int i = (w - n.few) * 256 + 64 * k + lane;
                if (i < a.nparts) {
                    dsum += a.dpart[i];
                    csum += a.cpart[i];
                }
            }
            continue;
        }
        // a row of many tiles takes the wave (a contiguous piece of them per
        // lane, then a fixed tree), one of some tiles sixteen lanes, one of
        // few a thread
        const int width = w < n.wave ? 64 : w < n.mid ? 16 : 1;
        const int j = w < n.wave ? w : w < n.mid ? a.n_cross_long + (w - n.wave) * 4 + lane / 16
                                                 : a.n_cross_long + a.n_cross_mid + (w - n.mid) * 64 + lane;
        const bool on = j < (w < n.mid ? a.n_cross_long + a.n_cross_mid : a.n_cross);
        if (width > 1) {
            const int4 q = on ? a.cross[j] : make_int4(0, 0, 0, -1);
            const int32_t sl = AP::kRows ? a.slot[q.x] : 0;
            const float xi = AP::kRows ? ap.x_in[q.x] : 0.f;
            const int at = width == 64 ? lane : sub;
            double s = on && at == 0 ? a.tailp[q.z] : 0.0;
            const int64_t m = q.w - q.z;
            for (int64_t i = m * at / width; i < m * (at + 1) / width; i++) s += a.head[q.z + 1 + i];
            if (width == 64) {
                s += __shfl_down(s, 32, 64);
                s += __shfl_down(s, 16, 64);
            }
#pragma unroll
            for (int o = 8; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
            if (on && at == 0) ap.row(q.x, s, q.y, sl, xi, dsum, chg);
        } else if (on) {
            const int4 q = a.cross[j];
            const int32_t sl = AP::kRows ? a.slot[q.x] : 0;
            const float xi = AP::kRows ? ap.x_in[q.x] : 0.f;
            double s = a.tailp[q.z];
            for (int32_t t = q.z + 1; t <= q.w; t++) s += a.head[t];
            ap.row(q.x, s, q.y, sl, xi, dsum, chg);
        }
    }
    const double td = block_sum<double>(dsum, s_d);
    const unsigned long long tc = block_sum<unsigned long long>(csum + (unsigned long long)chg, s_c);
    if (gridDim.x > 1 && threadIdx.x == 0) {
        fix_d[blockIdx.x] = td;
        fix_c[blockIdx.x] = tc;
        // release this workgroup's partials; acquire the others' if last
        const uint32_t before = __hip_atomic_fetch_add(fix_done, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
        s_last = before == gridDim.x - 1;
    }
    double D = td;
    unsigned long long C = tc;
    if (gridDim.x > 1) {
        __syncthreads();
        if (!s_last) return;
        __threadfence();
        double d = 0.0;
        unsigned long long c = 0;
        for (uint32_t b = threadIdx.x; b < gridDim.x; b += blockDim.x) {
            d += fix_d[b];
            c += fix_c[b];
        }
        D = block_sum<double>(d, s_d);
        C = block_sum<unsigned long long>(c, s_c);
    }
    if (threadIdx.x == 0) {
        *a.Dp = D;  // dangling mass of x_{t+1}
        step->changed = C;
        step->frontier = 0;
        *next_step = DevStep{};
        *fix_done = 0;  // for the next superstep (after this kernel ends)
    }
}

// ------------------------------------------------------------ PageRank across the parts of a vertex-cut

__device__ __forceinline__ bool bit_of(const uint32_t *bm, int64_t v) { return (bm[v >> 5] >> (v & 31)) & 1u; }

// The replicas whose merged sums another part's master needs are known with
// the graph (ascending local, hence global ids): (gid, sum) of each.  Counting
// and selecting them from the bit maps on every call, 32 vertices per thread,
// took 29 us for a part of R-MAT scale 18 (one of four), this 3 us.
__global__ __launch_bounds__(256) void k_part_emit(const int32_t *__restrict__ part_list, uint32_t n,
                                                   const int32_t *__restrict__ l2g, const double *__restrict__ acc,
                                                   int32_t *__restrict__ gid_out, double *__restrict__ val_out) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t v = part_list[i];
    gid_out[i] = l2g ? l2g[v] : v;
    val_out[i] = acc[v];
}

// Local id of a global one (-1: not held; no map: the same id): a search over 256 samples of the
// ascending map in LDS, then over one 256th of the map.  The chain of
// dependent reads bounds it: the whole search in global memory took 7.2 us
// for a part of R-MAT scale 18 (one of four; a launch alone about 3), 6.4 us so.
constexpr int MAP_SAMPLES = 256;
__device__ __forceinline__ void sample_map(const int32_t *__restrict__ l2g, int64_t V, int32_t *s_top) {
    if (!l2g) return;
    const int64_t end = (threadIdx.x + 1) * V / MAP_SAMPLES;  // (256 threads)
    s_top[threadIdx.x] = end > 0 ? l2g[end - 1] : -1;
    __syncthreads();
}
__device__ __forceinline__ int64_t local_of(const int32_t *__restrict__ l2g, int64_t V, const int32_t *s_top, int32_t g) {
    if (!l2g) return g >= 0 && g < V ? g : -1;
    int p = 0;
#pragma unroll
    for (int step = MAP_SAMPLES / 2; step > 0; step /= 2)
        if (s_top[p + step - 1] < g) p += step;
    if (s_top[p] < g) return -1;  // beyond the last
    int64_t lo = p * V / MAP_SAMPLES, hi = (p + 1) * V / MAP_SAMPLES;
    while (lo < hi) {
        const int64_t mid = (lo + hi) / 2;
        if (l2g[mid] < g) lo = mid + 1;
        else hi = mid;
    }
    return l2g[lo] == g ? lo : -1;
}

// A master adds another part's merged sum for it (one pair per vertex per
// call; the caller orders the calls, so the sum's order is fixed).
__global__ __launch_bounds__(256) void k_part_add(const int32_t *__restrict__ gid, const double *__restrict__ vals,
                                                  uint32_t n, const int32_t *__restrict__ l2g, int64_t V,
                                                  const uint32_t *__restrict__ master, double *__restrict__ acc) {
    __shared__ int32_t s_top[MAP_SAMPLES];
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    const int32_t g = i < n ? gid[i] : -1;
    sample_map(l2g, V, s_top);
    if (i >= n) return;
    const int64_t x = local_of(l2g, V, s_top, g);
    if (x >= 0 && bit_of(master, x)) acc[x] += vals[i];
}

// A replica takes its master's new rank.
__global__ __launch_bounds__(256) void k_replica_set(const int32_t *__restrict__ gid, const uint32_t *__restrict__ vals,
                                                     uint32_t n, const int32_t *__restrict__ l2g, int64_t V,
                                                     const uint32_t *__restrict__ master, uint32_t *__restrict__ x) {
    __shared__ int32_t s_top[MAP_SAMPLES];
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    const int32_t g = i < n ? gid[i] : -1;
    sample_map(l2g, V, s_top);
    if (i >= n) return;
    const int64_t v = local_of(l2g, V, s_top, g);
    if (v >= 0 && !bit_of(master, v)) x[v] = vals[i];
}

// ------------------------------------------------------------ sync set

// The vertices of a block's `words` words (32 each) that another part needs
// and whose value changed, as bits in s_word.  With a dirty map a thread reads
// the 32 bytes of a word; values are compared with the synced copy by
// consecutive lanes.
constexpr int DELTA_WORDS = 256;  // words of a block at most

__device__ __forceinline__ void delta_words(int words, int32_t W, int64_t V, const uint32_t *__restrict__ remote, bool all,
                                            const uint8_t *__restrict__ dirty, const uint32_t *__restrict__ vals,
                                            const uint32_t *__restrict__ synced, uint32_t *s_word) {
    const int32_t w0 = blockIdx.x * words;
    if (dirty) {
        const int32_t w = w0 + (int32_t)threadIdx.x;
        if ((int)threadIdx.x < words) {
            uint32_t bits = 0;
            uint32_t mask = w >= W ? 0u : all ? 0xFFFFFFFFu : remote ? remote[w] : 0u;
            if (w == W - 1 && (V & 31)) mask &= (1u << (V & 31)) - 1u;
            if (mask) {
                const uint4 *d16 = reinterpret_cast<const uint4 *>(dirty + (int64_t)w * 32);
                const uint4 a = d16[0], b = d16[1];
                const uint32_t d4[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
                for (int q = 0; q < 8; q++) {
                    const uint32_t x = d4[q];
                    bits |= (uint32_t)((x & 0xFFu) != 0) << (4 * q) | (uint32_t)((x & 0xFF00u) != 0) << (4 * q + 1) |
                            (uint32_t)((x & 0xFF0000u) != 0) << (4 * q + 2) |
                            (uint32_t)((x & 0xFF000000u) != 0) << (4 * q + 3);
                }
            }
            s_word[threadIdx.x] = bits & mask;
        }
    } else {
        for (int k = 0; k < words / 8; k++) {
            const int i = k * 256 + (int)threadIdx.x;
            const int64_t v = (int64_t)w0 * 32 + i, u = min(v, V - 1);
            const uint32_t mask = all ? 0xFFFFFFFFu : remote ? remote[u >> 5] : 0u;
            const bool pick = v < V && ((mask >> (v & 31)) & 1u) && vals[u] != synced[u];
            const unsigned long long m = __ballot(pick);
            if ((threadIdx.x & 31) == 0) s_word[i >> 5] = (uint32_t)(m >> (threadIdx.x & 32));
        }
    }
    __syncthreads();
}

__global__ __launch_bounds__(256) void k_delta_count(int words, int32_t W, int64_t V, const uint32_t *remote, int all,
                                                     const uint8_t *dirty, const uint32_t *vals,
                                                     const uint32_t *synced, uint32_t *blk_cnt) {
    __shared__ uint32_t s_word[DELTA_WORDS];
    __shared__ unsigned long long s[4];
    delta_words(words, W, V, remote, all, dirty, vals, synced, s_word);
    const unsigned long long t =
        block_sum<unsigned long long>((int)threadIdx.x < words ? __popc(s_word[threadIdx.x]) : 0, s);
    if (threadIdx.x == 0) blk_cnt[blockIdx.x] = (uint32_t)t;
}

// Pairs in ascending vertex order: a block starts at the sum of the counts
// below its own, its vertices are written by consecutive lanes.  (One thread
// per word that wrote its 32 vertices one after the other used a lane per
// cache line: for the labels of one of eight parts of R-MAT scale 24 241 us, now
// 35.)
__global__ __launch_bounds__(256) void k_delta_emit(int words, int32_t W, int64_t V, const uint32_t *remote, int all,
                                                    uint8_t *dirty, const uint32_t *__restrict__ vals,
                                                    uint32_t *synced, const int32_t *__restrict__ l2g,
                                                    const uint32_t *__restrict__ blk_cnt, int nblk, uint32_t cap,
                                                    int32_t *__restrict__ gid_out, uint32_t *__restrict__ val_out,
                                                    uint32_t *total_out) {
    __shared__ uint32_t s_word[DELTA_WORDS], s_pos[DELTA_WORDS];
    __shared__ unsigned long long s_scan[4];
    __shared__ unsigned long long s_pre[4], s_all[4];
    const int tid = threadIdx.x;
    unsigned long long pre = 0, all_ = 0;
    for (int b = tid; b < nblk; b += blockDim.x) {
        unsigned long long c = blk_cnt[b];
        all_ += c;
        if (b < (int)blockIdx.x) pre += c;
    }
    // block sums of pre / all (same tree for every block: identical totals)
    {
        const int lane = tid & 63, wid = tid >> 6;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            pre += __shfl_down(pre, o, 64);
            all_ += __shfl_down(all_, o, 64);
        }
        if (lane == 0) {
            s_pre[wid] = pre;
            s_all[wid] = all_;
        }
        __syncthreads();
        pre = s_pre[0] + s_pre[1] + s_pre[2] + s_pre[3];
        all_ = s_all[0] + s_all[1] + s_all[2] + s_all[3];
    }
    if (blockIdx.x == 0 && tid == 0) *total_out = (uint32_t)all_;
    const bool commit = all_ <= cap;
    delta_words(words, W, V, remote, all, dirty, vals, synced, s_word);
    unsigned long long tot;
    const unsigned long long at = pre + block_excl_scan_u64(tid < words ? __popc(s_word[tid]) : 0, &tot, s_scan);
    if (tid < words) s_pos[tid] = (uint32_t)at;
    __syncthreads();
    const int32_t w0 = blockIdx.x * words;
    if (tot > 0)
        for (int i = tid; i < words * 32; i += 256) {
            const uint32_t bits = s_word[i >> 5], below = (1u << (i & 31)) - 1u;
            if (!((bits >> (i & 31)) & 1u)) continue;
            const int64_t v = (int64_t)w0 * 32 + i;
            const uint32_t pos = s_pos[i >> 5] + __popc(bits & below), x = vals[v];
            if (pos < cap) {
                gid_out[pos] = l2g ? l2g[v] : (int32_t)v;
                val_out[pos] = x;
            }
            if (commit && synced) synced[v] = x;
        }
    if (commit && dirty && tid < words && w0 + tid < W) {  // the dirty bytes of this word's vertices are cleared
        uint4 *d16 = reinterpret_cast<uint4 *>(dirty + (int64_t)(w0 + tid) * 32);
        d16[0] = make_uint4(0, 0, 0, 0);
        d16[1] = make_uint4(0, 0, 0, 0);
    }
}

// Receiving side of the sync set: values other parts emitted for vertices
// this part holds (global id -> local id by binary search in the ascending
// l2g map; ids it does not hold are ignored) are merged by integer min; a
// replica whose value falls becomes active in the next superstep.
__global__ __launch_bounds__(256) void k_apply_delta(const int32_t *__restrict__ gid,
                                                     const uint32_t *__restrict__ vals, uint32_t n,
                                                     const int32_t *__restrict__ l2g, int64_t V,
                                                     uint32_t *__restrict__ val, uint8_t *__restrict__ front_next) {
    __shared__ int32_t s_top[MAP_SAMPLES];
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    const int32_t g = i < n ? gid[i] : -1;
    sample_map(l2g, V, s_top);
    if (i >= n) return;
    const int64_t x = local_of(l2g, V, s_top, g);
    if (x < 0) return;
    const uint32_t v = vals[i];
    if (v < val[x]) {  // below the value before the merge: the replica changes
        atomicMin(&val[x], v);
        front_next[x] = 1;
    }
}

__global__ void k_zero_step(DevStep *step) { *step = DevStep{}; }
__global__ void k_set_f64(double *p, double v) { *p = v; }
__global__ void k_get_f64(const double *p, double *to) { *to = *p; }
__global__ void k_set_u32(uint32_t *p, uint32_t v) { *p = v; }

// ------------------------------------------------------------ separate template calls

__global__ __launch_bounds__(256) void k_fill_u32(uint32_t *p, int64_t n, uint32_t v) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = v;
}

// MSGApply of SSSP / CC: a vertex whose merged message is below its value
// takes it, and is marked for the next MSGGen and for the sync set; the
// accumulator is reset for the next merge.
__global__ __launch_bounds__(256) void k_ph_apply(uint32_t *__restrict__ acc, uint32_t *__restrict__ val,
                                                  uint8_t *__restrict__ pend, uint8_t *__restrict__ dirty, int64_t V,
                                                  DevStep *step, const uint32_t *__restrict__ rot, int nrot) {
    __shared__ unsigned long long s_c[4];
    if (blockIdx.x == 0) check_rotations(step, rot, nrot);
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    unsigned c = 0;
    if (v < V) {
        const uint32_t a = acc[v];
        if (a != INF) {
            acc[v] = INF;
            if (a < val[v]) {
                val[v] = a;
                pend[v] = 1;
                dirty[v] = 1;
                c = 1;
            }
        }
    }
    const unsigned long long t = block_sum<unsigned long long>((unsigned long long)c, s_c);
    if (threadIdx.x == 0 && t) atomicAdd(&step->changed, t);
}

// MSGGen of PageRank: every vertex's message x[u]/outdeg(u) and the
// dangling mass (per-workgroup partials, summed in order by k_reduce_D).
// (master != NULL: a part of a vertex-cut; only its masters' dangling mass
// counts, every other part counts its own masters)
__global__ __launch_bounds__(256) void k_ph_pr_gen(const float *__restrict__ x, const int32_t *__restrict__ outdeg,
                                                   const int32_t *__restrict__ slot, float *__restrict__ contrib,
                                                   int64_t V, double *dpart, const uint32_t *__restrict__ master) {
    __shared__ double s_d[4];
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    double dl = 0.0;
    if (v < V) {
        const float xv = x[v];
        const int od = outdeg[v];
        contrib[slot[v]] = od > 0 ? xv / (float)od : 0.0f;
        if (od == 0 && (!master || bit_of(master, v))) dl = (double)xv;
    }
    const double t = block_sum<double>(dl, s_d);
    if (threadIdx.x == 0) dpart[blockIdx.x] = t;
}

// MSGApply of PageRank: x' = (1-d)/V + d * (merged + D/V), in place.  Few,
// large workgroups: each adds its count to one counter (a part of
// R-MAT scale 18, one of four: 9.2 us in workgroups of 256, whose atomics queue,
// 5.8 us so).
constexpr int PH_APPLY = 4096;  // vertices of a workgroup
__global__ __launch_bounds__(1024) void k_ph_pr_apply(const double *__restrict__ acc, float *__restrict__ x, int64_t V,
                                                      double base, double d, const double *__restrict__ Dp,
                                                      double inv_V, DevStep *step, DevStep *next,
                                                      const uint32_t *__restrict__ master) {
    __shared__ unsigned long long s_c[16];
    const double dD = d * (*Dp) * inv_V;
    unsigned c = 0;
#pragma unroll
    for (int j = 0; j < PH_APPLY / 1024; j++) {
        const int64_t v = (int64_t)blockIdx.x * PH_APPLY + j * 1024 + threadIdx.x;
        if (v < V && (!master || bit_of(master, v))) {  // a part of a vertex-cut applies at its masters
            const float xn = (float)(base + d * acc[v] + dD);
            c += __float_as_uint(xn) != __float_as_uint(x[v]);
            x[v] = xn;
        }
    }
    const unsigned long long t = block_sum<unsigned long long>((unsigned long long)c, s_c);
    if (threadIdx.x == 0) {
        if (t) atomicAdd(&step->changed, t);
        if (blockIdx.x == 0) *next = DevStep{};
    }
}

template <class T>
inline unsigned grid_for(T n, unsigned block) {
    return (unsigned)std::max<T>(1, (n + block - 1) / block);
}

}  // namespace

// ------------------------------------------------------------------ host

template <class K>
static int persistent_grid(gx_graph *g, K kernel, int block) {
    return g->num_cus * occupancy_per_cu(reinterpret_cast<const void *>(kernel), block);
}

// Persistent grid of the relaxation: whole multiples of the slice count (a
// pulling XCD's workgroups share its slice's units evenly).
static int relax_grid_for(gx_graph *g, const gx_params *p, bool sweep) {
    const int pg = sweep ? (p->algo == GX_CC ? persistent_grid(g, k_relax_sweep<false>, 256)
                                             : persistent_grid(g, k_relax_sweep<true>, 256))
                         : (p->algo == GX_CC ? persistent_grid(g, k_relax<false>, 256)
                                             : persistent_grid(g, k_relax<true>, 256));
    return std::max(PULL_SLICES, pg / PULL_SLICES * PULL_SLICES);
}

// Fix-up entries per workgroup of a sweep: the records of the units one takes
// (the j-th workgroup on the XCD of slice x takes units j, j + nper, ... of
// slice x), maximised over x and j, so a region never overflows.
static uint32_t fix_cap_for(const Sweep &sw, const std::vector<uint32_t> &recs, int grid) {
    const int64_t nper = grid / PULL_SLICES;
    int64_t most = 0;
    for (int x = 0; x < PULL_SLICES; x++)
        for (int64_t j = 0; j < nper; j++) {
            int64_t sum = 0;
            for (int64_t u = sw.uoff[x] + j; u < sw.uoff[x + 1]; u += nper) sum += recs[(size_t)u];
            most = std::max(most, sum);
        }
    return (uint32_t)most;
}

// What the pull of `s` reads; `bound`: the vertex values.  CC labels ascend
// with the neighbour ids until the first superstep ran or another part's
// labels were merged, so that superstep reads one neighbour per vertex (if
// the neighbours of every row ascend).
static PullArgs pull_args(const gx_state *s) {
    const DevGraph &d = s->g->d;
    if (s->p.algo == GX_CC)
        return {d.sym_rp, d.sym_col, d.sym_segs, d.sym_nsegs, s->k == 0 && !s->merged && d.sym_ascending,
                s->acc != nullptr, s->val, nullptr};
    return {d.in_blk, d.in_adj, d.pull_segs, d.pull_nsegs, 0, s->acc != nullptr, s->val, s->hot[s->k & 1]};
}

// The relaxation of the active list and the frontier map `front` it was built
// from, against `tgt` (the values, or an accumulator).
static void launch_relax(gx_state *s, hipStream_t hs, const uint8_t *front, uint32_t *tgt, uint8_t *front_next,
                         DevStep *step) {
    const DevGraph &d = s->g->d;
    const bool cc = s->p.algo == GX_CC;
    const void *adj = cc ? (const void *)d.sym_col : (const void *)d.out_adj;
    const PullArgs pa = pull_args(s);
    if (s->sweep) {
        hipLaunchKernelGGL(cc ? k_relax_sweep<false> : k_relax_sweep<true>, dim3(s->relax_grid), dim3(256), 0, hs, s->list,
                           s->tile_start, adj, pa, *s->sweep, front, d.V, s->snap, tgt, front_next, step,
                           s->pull_edges, s->fix, s->fixn, s->fix_cap, s->rot, s->xcd_shift);
        hipLaunchKernelGGL(k_fixup, dim3(s->relax_grid), dim3(256), 0, hs, s->fix, s->fixn, s->fix_cap, tgt);
    } else {
        hipLaunchKernelGGL(cc ? k_relax<false> : k_relax<true>, dim3(s->relax_grid), dim3(256), 0, hs, s->list,
                           s->tile_start, adj, pa, d.V, s->snap, tgt, front_next, step, s->pull_edges, s->rot,
                           s->xcd_shift);
    }
}

// Compacts the map `front` (A_{s->k + ahead}) into the active list, counting
// into `step`; clears `clear` and the slot after.  `prev`: the step that
// filled the map, `dirty`: where its changes are kept (both NULL where no
// superstep did).
static void launch_compact(gx_state *s, hipStream_t hs, const uint8_t *front, uint8_t *clear, int ahead, DevStep *prev,
                           uint8_t *dirty) {
    const DevGraph &d = s->g->d;
    const int64_t k = s->k + ahead;
    const bool slots = s->hot[0] && s->pull_edges != 0xFFFFFFFFu;
    const int cvt = !slots && (d.V >= COMPACT_WIDEST_FROM ||
                               (2 * d.V >= COMPACT_WIDEST_FROM && d.E < COMPACT_SPARSE * d.V))
                        ? COMPACT_WIDEST
                    : d.V >= COMPACT_WIDE_FROM ? COMPACT_WIDE : 4;
    auto kern = cvt == COMPACT_WIDEST ? k_compact<COMPACT_WIDEST>
              : cvt == COMPACT_WIDE ? k_compact<COMPACT_WIDE> : k_compact<4>;
    hipLaunchKernelGGL(kern, dim3(grid_for<int64_t>(d.V, CBLOCK * cvt) + 1), dim3(CBLOCK), 0, hs, front,
                       clear, s->p.algo == GX_CC ? d.sym_rp : d.out_rp, s->val, s->snap, d.V, s->list, s->tile_start,
                       s->steps + (k % STEP_RING), s->steps + ((k + 1) % STEP_RING),
                       (int)(s->pull_edges != 0xFFFFFFFFu), prev, dirty, s->pull_edges, s->rot, s->relax_grid,
                       slots ? d.slot : nullptr, s->hot[k & 1], s->hot[(k + 1) & 1]);
}

// The pull of this graph's tiles (and the fewest workgroups that hold every
// wave the CUs can, or every tile).
template <class AP>
static auto pr_pull_for(const DevGraph &d) {
    if (d.pr_hot)
        return d.pr_tile == 256 ? k_pr_pull<1, true, AP> : d.pr_tile == 512 ? k_pr_pull<2, true, AP>
             : d.pr_tile == 1024 ? k_pr_pull<4, true, AP> : k_pr_pull<8, true, AP>;
    return d.pr_tile == 256 ? k_pr_pull<1, false, AP> : d.pr_tile == 512 ? k_pr_pull<2, false, AP>
         : d.pr_tile == 1024 ? k_pr_pull<4, false, AP> : k_pr_pull<8, false, AP>;
}

static int pr_grid_for(gx_graph *g, const gx_params *p) {
    const DevGraph &d = g->d;
    if (d.pr_hot) return g->num_cus;
    const int64_t items = std::max(d.pr_rows.n, (d.n_ez + 255) / 256), waves = PR_BLOCK / 64;
    const int resident = p->phases ? persistent_grid(g, pr_pull_for<PrStore>(d), PR_BLOCK)
                                   : persistent_grid(g, pr_pull_for<PrApply>(d), PR_BLOCK);
    return (int)std::max<int64_t>(1, std::min<int64_t>(resident, (items + waves - 1) / waves));
}

static PrArgs pr_args(const gx_state *s, const float *c_in, double *Dp, double inv_V) {
    const DevGraph &d = s->g->d;
    PrArgs a{};
    a.src = d.pr_src;
    a.row_last = reinterpret_cast<const uint8_t *>(d.row_last);
    a.tile_nz = d.pr_rows.tile_nz;
    a.nz = d.nz;
    a.ez = d.ez;
    a.nz_slot = d.nz_slot;
    a.slot = d.slot;
    a.cross = d.pr_rows.cross;
    a.n_cross = d.pr_rows.n_cross;
    a.n_cross_long = d.pr_rows.n_long;
    a.n_cross_mid = d.pr_rows.n_mid;
    a.V = d.V;
    a.E = d.E;
    a.n_nz = d.n_nz;
    a.n_ez = d.n_ez;
    a.ntiles = (int32_t)d.pr_rows.n;
    a.c_in = c_in;
    a.Dp = Dp;
    a.inv_V = inv_V;
    a.head = s->head;
    a.tailp = s->tailp;
    a.dpart = s->dpart;
    a.cpart = s->cpart;
    a.nparts = s->pr_parts;
    return a;
}

static size_t state_layout(gx_graph *g, const gx_params *p, Carver &c, gx_state *s) {
    const DevGraph &d = g->d;
    int64_t V = d.V;
    int32_t W = d.W;
    if (p->algo == GX_LP) {
        lp_layout(g, c, s);
    } else if (p->algo == GX_PAGERANK) {
        const int64_t nt = std::max<int64_t>(1, d.pr_rows.n);
        s->x[0] = c.take<float>(V);
        s->x[1] = c.take<float>(V);
        s->contrib[0] = c.take<float>(V + 1);  // (the last tile's padding reads one past the slots)
        s->contrib[1] = c.take<float>(V + 1);
        s->synced = c.take<uint32_t>(V);
        s->head = c.take<double>(nt);
        s->tailp = c.take<double>(nt);
        s->pr_grid = pr_grid_for(g, p);
        s->pr_parts = s->pr_grid * (d.pr_hot ? 16 : PR_BLOCK / 64);
        s->dpart = c.take<double>(std::max<int64_t>(s->pr_parts, grid_for<int64_t>(V, 256)));
        s->cpart = c.take<uint32_t>(s->pr_parts);
        s->Dval = c.take<double>(1);
        const int units = PrFixUnits(d.pr_rows.n_cross, d.pr_rows.n_long, d.pr_rows.n_mid, s->pr_parts).all;
        // a single workgroup where one holds the units; many small ones until their
        // returning atomics queue (20 supersteps of R-MAT with 256 threads always, 1024
        // always and by this rule: scale 14 280, 262, 260 us, 16 320, 398, 320, 18 563, 593,
        // 564, 22 5.81, 5.65, 5.65 ms)
        s->pr_fix_block = units <= PR_FIX_BLOCK / 64 || units >= 1024 ? PR_FIX_BLOCK : 256;
        s->pr_fix_grid = std::min(PR_FIX_MAX_GRID, (units * 64 + s->pr_fix_block - 1) / s->pr_fix_block);
        s->fix_d = c.take<double>(s->pr_fix_grid);
        s->fix_c = c.take<unsigned long long>(s->pr_fix_grid);
        s->fix_done = c.take<uint32_t>(1);
    } else {
        int64_t Eimg = p->algo == GX_SSSP ? d.E : d.E_sym;
        s->val = c.take<uint32_t>(V);
        // byte maps padded to whole 32-vertex words (the sync set reads 32 at a time)
        s->front8[0] = c.take<uint8_t>((size_t)W * 32);
        s->front8[1] = c.take<uint8_t>((size_t)W * 32);
        s->dirty8 = c.take<uint8_t>((size_t)W * 32);
        s->list = c.take<uint4>(V);
        s->tile_start = c.take<uint32_t>(Eimg / PUSH_TILE + 2);
        s->snap = c.take<uint32_t>(V);
        const Sweep &sw = p->algo == GX_CC ? d.sweep_sym : d.sweep_in;
        s->sweep = sw.rec ? &sw : nullptr;
        s->relax_grid = relax_grid_for(g, p, s->sweep != nullptr);
        s->rot = c.take<uint32_t>(s->relax_grid);
        if (s->sweep) {
            s->fix_cap = fix_cap_for(sw, p->algo == GX_CC ? g->sweep_sym_recs : g->sweep_in_recs, s->relax_grid);
            s->fix = c.take<uint2>((size_t)s->relax_grid * s->fix_cap);
            s->fixn = c.take<uint32_t>(s->relax_grid);
        }
        if (p->algo == GX_SSSP && !s->sweep)
            for (uint32_t *&h : s->hot) h = c.take<uint32_t>(PULL_BIT_WORDS);
    }
    if (p->phases) {
        if (p->algo == GX_PAGERANK) {
            s->acc_d = c.take<double>(V);
            s->Dscratch = c.take<double>(1);
            s->ph_steps = c.take<DevStep>(2);
        } else {
            s->acc = c.take<uint32_t>(V);
            s->junk8 = c.take<uint8_t>((size_t)W * 32);
        }
    }
    s->steps = c.take<DevStep>(STEP_RING);
    // enough blocks for the chip, and few enough counts for each to add up
    s->delta_words = 32;
    while (s->delta_words < DELTA_WORDS && (W + s->delta_words - 1) / s->delta_words > 1024) s->delta_words *= 2;
    s->delta_blocks = (int)grid_for<int64_t>(W, s->delta_words);
    s->blk_cnt = c.take<uint32_t>(s->delta_blocks);
    return c.used;
}

static gx_status check_params(const gx_graph *g, const gx_params *p) {
    GX_REQUIRE(g, GX_EINVAL, "graph is NULL");
    GX_REQUIRE(p, GX_EINVAL, "params is NULL");
    GX_REQUIRE(!g->dev_error, GX_EDEVICE, "graph handle has a sticky device error");
    GX_REQUIRE(p->algo == GX_PAGERANK || p->algo == GX_SSSP || p->algo == GX_CC || p->algo == GX_LP, GX_EINVAL,
               "algo %d not supported by the plain engine", p->algo);
    GX_REQUIRE(p->delta_mode <= GX_DELTA_MASTERS, GX_EINVAL, "delta_mode %u invalid", p->delta_mode);
    GX_REQUIRE(p->delta_mode != GX_DELTA_MASTERS || g->d.master_rep, GX_EINVAL,
               "GX_DELTA_MASTERS needs a partitioned graph (flags)");
    GX_REQUIRE(p->phases <= GX_PHASES_MASTERS, GX_EINVAL, "phases %u invalid", p->phases);
    GX_REQUIRE(!p->phases || p->algo != GX_LP, GX_EINVAL, "the separate template calls serve PageRank, SSSP and CC");
    GX_REQUIRE(p->phases != GX_PHASES_MASTERS || (p->algo == GX_PAGERANK && g->d.outdeg_g && g->d.master), GX_EINVAL,
               "GX_PHASES_MASTERS is PageRank on a part loaded with flags, V_global and outdeg_global");
    if (p->algo == GX_PAGERANK) {
        GX_REQUIRE(g->needs & GX_NEED_IN, GX_EINVAL, "PageRank needs GX_NEED_IN");
        GX_REQUIRE(p->damping >= 0.f && p->damping < 1.f, GX_EINVAL, "damping %f out of [0,1)", p->damping);
    }
    if (p->algo == GX_SSSP) {
        GX_REQUIRE(g->needs & GX_NEED_OUT, GX_EINVAL, "SSSP needs GX_NEED_OUT");
        GX_REQUIRE(p->source >= -1 && p->source < g->d.V, GX_EINVAL, "source %d out of [-1,V)", p->source);
    }
    if (p->algo == GX_CC) GX_REQUIRE(g->needs & GX_NEED_SYM, GX_EINVAL, "CC needs GX_NEED_SYM");
    if (p->algo == GX_LP) {
        GX_REQUIRE(g->needs & GX_NEED_SYM, GX_EINVAL, "LP needs GX_NEED_SYM");
        int64_t slots = 0;
        try {
            slots = lp_plan(const_cast<gx_graph *>(g)).slot_bound;
        } catch (const std::bad_alloc &) {
            set_error("host allocation failed while laying out the label propagation lists");
            return GX_ENOMEM;
        }
        GX_REQUIRE(slots < (int64_t(1) << 32), GX_EINVAL, "LP hub tables would exceed 2^32 slots");
    }
    return GX_OK;
}

extern "C" gx_status gx_state_bytes(const gx_graph *g, const gx_params *p, size_t *bytes) {
    clear_error();
    GX_REQUIRE(bytes, GX_EINVAL, "bytes is NULL");
    gx_status st = check_params(g, p);
    if (st != GX_OK) return st;
    Carver c(nullptr, 0);
    gx_state tmp;
    *bytes = state_layout(const_cast<gx_graph *>(g), p, c, &tmp);
    return GX_OK;
}

extern "C" gx_status gx_state_init(gx_graph *g, const gx_params *p, void *dev_state, size_t bytes, void *stream,
                                   gx_state **out) {
    clear_error();
    GX_REQUIRE(out, GX_EINVAL, "out is NULL");
    *out = nullptr;
    gx_status st = check_params(g, p);
    if (st != GX_OK) return st;
    GX_REQUIRE(dev_state, GX_EINVAL, "dev_state is NULL");
    GX_REQUIRE(reinterpret_cast<uintptr_t>(dev_state) % ALIGN == 0, GX_EINVAL, "dev_state not 256-byte aligned");
    {
        Carver m(nullptr, 0);
        gx_state tmp;
        size_t need = state_layout(g, p, m, &tmp);
        GX_REQUIRE(need <= bytes, GX_ENOMEM, "state buffer too small: need %zu bytes, have %zu", need, bytes);
    }
    gx_state *s = new (std::nothrow) gx_state();
    GX_REQUIRE(s, GX_ENOMEM, "host allocation failed");
    s->g = g;
    s->p = *p;
    s->mem = dev_state;
    // GX_XCD_CHECK_SHIFT (tests only) offsets the XCD the odd pull workgroups
    // see, so that the rotation check fires without a real fault
    if (const char *e = std::getenv("GX_XCD_CHECK_SHIFT")) s->xcd_shift = (uint32_t)std::strtoul(e, nullptr, 10);
    Carver c(dev_state, bytes);
    state_layout(g, p, c, s);
    if (p->algo == GX_SSSP || p->algo == GX_CC) {
        const DevGraph &dg = g->d;
        bool can_pull = p->algo == GX_SSSP ? dg.in_adj != nullptr : dg.sym_col != nullptr;
        // The default is where the sweep meets the push (4 M vertices, 67 M uniform edges:
        // a pull at 0.33 takes 305 us, a push at 0.27 306).  The row pull gets cheaper as
        // a solve goes on and meets it lower, per superstep near 0.1 on R-MAT scales 18 to
        // 22 and 0.2 on uniform graphs, but a solve has few supersteps between; whole
        // solves at 0.1, 0.2 and 0.3 from three sources: R-MAT scale 18 374, 376, 377 us,
        // 20 509, 520, 607, 22 1230, 1251, 1341, uniform of 1 M vertices and 16 M edges 1419,
        // 1395, 1403; CC scale 22 443, 451, 458.  (A state that only pushes keeps no
        // snapshots: the default where that is faster, see sweep_rule.)
        const double usual = p->algo == GX_SSSP && dg.sssp_pushes ? 1.0 : 0.3;
        double frac = p->pull_fraction > 0.f ? (double)p->pull_fraction : usual;
        double Eimg = (double)(p->algo == GX_SSSP ? dg.E : dg.E_sym);
        s->pull_edges = (!can_pull || frac >= 1.0) ? 0xFFFFFFFFu : (uint32_t)std::max(1.0, std::ceil(frac * Eimg));
    }
    hipStream_t hs = static_cast<hipStream_t>(stream);
    const DevGraph &d = g->d;
    int64_t V = d.V;
    if (p->algo == GX_LP) {
        gx_status ls = lp_init(s, hs);
        if (ls != GX_OK) {
            delete s;
            return ls;
        }
    } else if (p->algo == GX_PAGERANK) {
        const int64_t Vn = p->phases == GX_PHASES_MASTERS ? d.V_global : V;
        float x0 = V > 0 ? (float)(1.0 / (double)Vn) : 0.f;
        unsigned nb = grid_for<int64_t>(V, 256);
        hipLaunchKernelGGL(k_pr_init, dim3(nb), dim3(256), 0, hs, s->x[0], s->contrib[0], s->synced, d.outdeg,
                           d.slot, V, x0, s->dpart, s->steps);
        hipLaunchKernelGGL(k_reduce_D, dim3(1), dim3(1024), 0, hs, s->dpart, (int)nb, s->Dval);
        (void)hipMemsetAsync(s->fix_done, 0, sizeof(uint32_t), hs);
    } else {
        const int64_t n = std::max<int64_t>(V, s->hot[0] ? PULL_BIT_WORDS : 0);
        const int32_t *rp = p->algo == GX_CC ? d.sym_rp : d.out_rp;
        // (padding bytes of the maps beyond V are cleared too)
        hipLaunchKernelGGL(k_min_init, dim3(grid_for<int64_t>(n, 256)), dim3(256), 0, hs, s->val, s->snap,
                           s->front8[0], s->front8[1], s->dirty8, d.l2g, rp, V, p->algo, p->source, s->steps,
                           s->hot[0], s->hot[1]);
        if ((int64_t)d.W * 32 > V) {
            size_t pad = (size_t)d.W * 32 - (size_t)V;
            (void)hipMemsetAsync(s->front8[0] + V, 0, pad, hs);
            (void)hipMemsetAsync(s->front8[1] + V, 0, pad, hs);
            (void)hipMemsetAsync(s->dirty8 + V, 0, pad, hs);
        }
        if (p->phases && V > 0)
            hipLaunchKernelGGL(k_fill_u32, dim3(grid_for<int64_t>(V, 256)), dim3(256), 0, hs, s->acc, V, INF);
        // compaction of superstep 0 (each superstep then relaxes and compacts the
        // next); with separate template calls the first MSGGen does it
        if (V > 0 && !p->phases)
            launch_compact(s, hs, s->front8[0], s->front8[1], 0, nullptr, nullptr);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        set_error("state init launch failed: %s", hipGetErrorString(e));
        delete s;
        return GX_EDEVICE;
    }
    *out = s;
    return GX_OK;
}

extern "C" gx_status gx_state_free(gx_state *s) {
    clear_error();
    delete s;
    return GX_OK;
}

// The current vertex values (PageRank ranks move between two buffers per
// superstep, except under separate template calls, which update in place).
static uint32_t *cur_values(const gx_state *s) {
    if (s->p.algo == GX_PAGERANK)
        return reinterpret_cast<uint32_t *>(s->x[s->p.phases ? 0 : (s->k & 1)]);
    if (s->p.algo == GX_LP) return s->lab[s->k & 1];
    return s->val;
}

extern "C" gx_status gx_state_values(gx_state *s, void **dev_values) {
    clear_error();
    GX_REQUIRE(s && dev_values, GX_EINVAL, "NULL argument");
    *dev_values = cur_values(s);
    return GX_OK;
}

extern "C" gx_status gx_state_frontier(gx_state *s, void **dev_bitmap) {
    clear_error();
    GX_REQUIRE(s && dev_bitmap, GX_EINVAL, "NULL argument");
    GX_REQUIRE(s->p.algo == GX_SSSP || s->p.algo == GX_CC, GX_EINVAL, "only SSSP and CC keep a frontier");
    // (separate template calls: the vertices the next MSGGen sends from)
    *dev_bitmap = s->front8[s->p.phases ? s->ph_p : (s->k & 1)];
    return GX_OK;
}

extern "C" gx_status gx_state_superstep(gx_state *s, int64_t *k) {
    clear_error();
    GX_REQUIRE(s && k, GX_EINVAL, "NULL argument");
    *k = s->k;
    return GX_OK;
}

// Process-wide pool of timing events (creating events per superstep costs
// more than the short supersteps themselves).  They only time kernels and are
// read after a stream synchronisation, so they skip the system-scope fence: a
// fenced record writes back and invalidates the caches between the kernels
// it separates, a gap of several microseconds per superstep.
static std::mutex g_ev_mu;
static std::vector<hipEvent_t> g_ev_free;

static hipEvent_t pool_event(gx_state *s) {
    if (!s->ev_pool.empty()) {
        hipEvent_t e = s->ev_pool.back();
        s->ev_pool.pop_back();
        return e;
    }
    {
        std::lock_guard<std::mutex> lk(g_ev_mu);
        if (!g_ev_free.empty()) {
            hipEvent_t e = g_ev_free.back();
            g_ev_free.pop_back();
            return e;
        }
    }
    hipEvent_t e = nullptr;
    if (hipEventCreateWithFlags(&e, hipEventDisableSystemFence) != hipSuccess) return nullptr;
    return e;
}

static void pool_return(hipEvent_t e) {
    std::lock_guard<std::mutex> lk(g_ev_mu);
    g_ev_free.push_back(e);
}

// Process-wide pool of pinned buffers for reading superstep counters back.
constexpr int HOST_STEPS = 256;
static std::vector<DevStep *> g_hs_free;

static DevStep *host_steps_take() {
    {
        std::lock_guard<std::mutex> lk(g_ev_mu);
        if (!g_hs_free.empty()) {
            DevStep *p = g_hs_free.back();
            g_hs_free.pop_back();
            return p;
        }
    }
    void *p = nullptr;
    if (hipHostMalloc(&p, HOST_STEPS * sizeof(DevStep), hipHostMallocDefault) != hipSuccess) return nullptr;
    return static_cast<DevStep *>(p);
}

static void host_steps_return(DevStep *p) {
    std::lock_guard<std::mutex> lk(g_ev_mu);
    g_hs_free.push_back(p);
}

extern "C" gx_status gx_release_cached(void) {
    clear_error();
    std::lock_guard<std::mutex> lk(g_ev_mu);
    hipError_t first = hipSuccess;
    for (hipEvent_t e : g_ev_free) {
        hipError_t r = hipEventDestroy(e);
        if (first == hipSuccess) first = r;
    }
    g_ev_free.clear();
    for (DevStep *p : g_hs_free) {
        hipError_t r = hipHostFree(p);
        if (first == hipSuccess) first = r;
    }
    g_hs_free.clear();
    GX_REQUIRE(first == hipSuccess, GX_EDEVICE, "releasing cached resources failed: %s", hipGetErrorString(first));
    return GX_OK;
}

// Enqueues superstep s->k on `hs` and advances s->k.
static gx_status enqueue_superstep(gx_state *s, hipStream_t hs) {
    const DevGraph &d = s->g->d;
    const gx_params &p = s->p;
    DevStep *step = s->steps + (s->k % STEP_RING);
    DevStep *next = s->steps + ((s->k + 1) % STEP_RING);
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (p.timing) {
        e0 = pool_event(s);
        e1 = pool_event(s);
    }
    if (p.algo == GX_LP) {
        if (e0) (void)hipEventRecord(e0, hs);
        lp_enqueue(s, hs, step, next);
        if (e1) (void)hipEventRecord(e1, hs);
    } else if (p.algo == GX_PAGERANK) {
        int cur = (int)(s->k & 1);
        double dd = p.damping;
        const PrApply ap{(1.0 - dd) / (double)d.V, dd, 0.0, s->x[cur], s->x[cur ^ 1], s->contrib[cur ^ 1]};
        if (d.V > 0) {
            const PrArgs a = pr_args(s, s->contrib[cur], s->Dval, 1.0 / (double)d.V);
            if (e0) (void)hipEventRecord(e0, hs);
            hipLaunchKernelGGL(pr_pull_for<PrApply>(d), dim3(s->pr_grid), dim3(d.pr_hot ? 1024 : PR_BLOCK), 0, hs, a, ap);
            if (e1) (void)hipEventRecord(e1, hs);
            hipLaunchKernelGGL(k_pr_fix<PrApply>, dim3(s->pr_fix_grid), dim3(s->pr_fix_block), 0, hs, a, ap, step, next,
                               s->fix_d, s->fix_c, s->fix_done);
        }
    } else {
        // superstep k: relax A_k (list built by the previous compaction), then
        // compact A_{k+1} for superstep k+1
        const int cur = (int)(s->k & 1);
        if (d.V > 0) {
            if (e0) (void)hipEventRecord(e0, hs);
            launch_relax(s, hs, s->front8[cur], s->val, s->front8[cur ^ 1], step);
            if (e1) (void)hipEventRecord(e1, hs);
            launch_compact(s, hs, s->front8[cur ^ 1], s->front8[cur], 1, step, s->dirty8);
        }
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        set_error("superstep launch failed: %s", hipGetErrorString(e));
        s->dev_error = true;
        return GX_EDEVICE;
    }
    if (e0 && e1) s->ev_pending.push_back({s->k, e0, e1});
    s->k++;
    return GX_OK;
}

// After a stream synchronisation: fold the pending kernel timings of
// supersteps before k_end (later ones were enqueued speculatively after
// convergence and do no work of the solve); with `per_step`, superstep k's
// time goes to per_step[k - k0] when in range.
static void collect_timings(gx_state *s, gx_step_stats *per_step = nullptr, int64_t k0 = 0, int64_t n = 0,
                            int64_t k_end = INT64_MAX) {
    for (auto &pr : s->ev_pending) {
        float ms = 0.f;
        if (pr.k < k_end && hipEventElapsedTime(&ms, pr.a, pr.b) == hipSuccess) {
            s->kernel_ms += ms;
            s->kernel_launches++;
            if (per_step && pr.k >= k0 && pr.k < k0 + n) per_step[pr.k - k0].kernel_ms = ms;
        }
        s->ev_pool.push_back(pr.a);
        s->ev_pool.push_back(pr.b);
    }
    s->ev_pending.clear();
}

// `next` is the slot of the following superstep: for SSSP/CC the number of
// vertices a superstep changed is the size of the next frontier.
static void to_stats(const gx_state *s, const DevStep &ds, const DevStep &next, gx_step_stats *o) {
    if (s->p.algo == GX_PAGERANK) {
        o->frontier = s->g->d.V;
        o->edges = s->g->d.E;
        o->pulled = 1;
        o->changed = (int64_t)ds.changed;
    } else if (s->p.algo == GX_LP) {
        o->frontier = lp_active(s);
        o->edges = s->g->d.E_sym;
        o->pulled = 1;
        o->changed = (int64_t)ds.changed;
    } else {
        o->frontier = (int64_t)ds.frontier;
        o->edges = (int64_t)(uint32_t)ds.list;
        o->pulled = ds.pad ? 1 : 0;
        o->changed = (int64_t)next.frontier;
    }
    o->kernel_ms = 0.0;
}

static gx_status read_steps(gx_state *s, int64_t kfirst, uint32_t n, hipStream_t hs, std::vector<DevStep> &out);

extern "C" gx_status gx_superstep(gx_state *s, void *stream, gx_step_stats *stats) {
    clear_error();
    GX_REQUIRE(s, GX_EINVAL, "state is NULL");
    GX_REQUIRE(!s->p.phases, GX_EINVAL, "this state is driven by gx_msg_gen / gx_msg_merge / gx_msg_apply");
    GX_REQUIRE(!s->dev_error && !s->g->dev_error, GX_EDEVICE, "sticky device error");
    hipStream_t hs = static_cast<hipStream_t>(stream);
    int64_t k = s->k;
    gx_status st = enqueue_superstep(s, hs);
    if (st != GX_OK) return st;
    if (stats) {
        std::vector<DevStep> ds;
        st = read_steps(s, k, 2, hs, ds);
        if (st != GX_OK) return st;
        to_stats(s, ds[0], ds[1], stats);
        collect_timings(s, stats, k, 1);
    }
    return GX_OK;
}

// Copies the counters of supersteps [kfirst, kfirst + n) to out[] through the
// state's pinned buffer (ring-contiguous pieces, one synchronisation).
static gx_status read_steps(gx_state *s, int64_t kfirst, uint32_t n, hipStream_t hs, std::vector<DevStep> &out) {
    out.resize(n);
    if (!s->host_steps) s->host_steps = host_steps_take();
    GX_REQUIRE(s->host_steps, GX_ENOMEM, "pinned host allocation failed");
    for (uint32_t done = 0; done < n;) {
        uint32_t chunk = std::min<uint32_t>(n - done, HOST_STEPS);
        uint32_t copied = 0;
        while (copied < chunk) {
            int64_t k = kfirst + done + copied;
            uint32_t slot = (uint32_t)(k % STEP_RING);
            uint32_t run = std::min<uint32_t>(chunk - copied, STEP_RING - slot);
            GX_CHECK_HIP(hipMemcpyAsync(s->host_steps + copied, s->steps + slot, run * sizeof(DevStep),
                                        hipMemcpyDeviceToHost, hs),
                         s);
            copied += run;
        }
        GX_CHECK_HIP(hipStreamSynchronize(hs), s);
        std::memcpy(out.data() + done, s->host_steps, chunk * sizeof(DevStep));
        done += chunk;
    }
    for (uint32_t i = 0; i < n; i++)
        if (out[i].rot_mixed) {
            s->dev_error = true;
            set_error("superstep %lld pulled with workgroups dealt to the XCDs in more than one rotation; some "
                      "work units may have run on an XCD other than the one owning their destinations, so the "
                      "values may be wrong; run with pull_fraction >= 1 (push only) on this device",
                      (long long)(kfirst + i));
            return GX_EDEVICE;
        }
    return GX_OK;
}

// PageRank supersteps k .. k+n-1 as one HIP graph launch on `hs`.  The
// kernels' arguments depend only on the state's memory, the damping and the
// ring slot of k (which also fixes the buffer parity), so the graph is
// captured once, on the graph handle's private stream, and replayed by every
// run that starts from the same slot with the same count, also by a state
// created again in the same memory (what a reset does).  A superstep
// enqueues two kernels and no memory set.  Returns false, having enqueued
// nothing, when timing events are on, for a single superstep, or when capture
// is not available; the caller then enqueues the supersteps one by one.
static bool pr_replay(gx_state *s, uint32_t n, hipStream_t hs) {
    gx_graph *g = s->g;
    if (s->p.timing || n < 2 || g->d.V == 0) return false;
    const int64_t slot = s->k % STEP_RING, k0 = s->k;
    const double damping = s->p.damping;
    std::lock_guard<std::mutex> lk(g->pr_mu);
    hipGraphExec_t exec = nullptr;
    for (auto &e : g->pr_graphs)
        if (e.mem == s->mem && e.damping == damping && e.slot == slot && e.n == n) exec = e.exec;
    if (!exec) {
        if (!g->cap_stream && hipStreamCreateWithFlags(&g->cap_stream, hipStreamNonBlocking) != hipSuccess) {
            g->cap_stream = nullptr;
            return false;
        }
        if (hipStreamBeginCapture(g->cap_stream, hipStreamCaptureModeThreadLocal) != hipSuccess) return false;
        bool ok = true;
        for (uint32_t i = 0; i < n && ok; i++) ok = enqueue_superstep(s, g->cap_stream) == GX_OK;
        hipGraph_t graph = nullptr;
        ok = hipStreamEndCapture(g->cap_stream, &graph) == hipSuccess && ok && graph;
        ok = ok && hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0) == hipSuccess;
        if (graph) (void)hipGraphDestroy(graph);
        s->k = k0;
        (void)hipGetLastError();
        if (!ok) {
            s->dev_error = false;  // a capture that failed launched nothing
            clear_error();
            return false;
        }
        if (g->pr_graphs.size() >= gx_graph::PR_GRAPHS) {
            (void)hipGraphExecDestroy(g->pr_graphs.front().exec);
            g->pr_graphs.erase(g->pr_graphs.begin());
        }
        g->pr_graphs.push_back({s->mem, damping, slot, n, exec});
    }
    if (hipGraphLaunch(exec, hs) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    s->k = k0 + n;
    return true;
}

extern "C" gx_status gx_run_until_converged(gx_state *s, uint32_t max_supersteps, void *stream, gx_run_stats *out,
                                            gx_step_stats *per_step) {
    clear_error();
    GX_REQUIRE(s, GX_EINVAL, "state is NULL");
    GX_REQUIRE(!s->p.phases, GX_EINVAL, "this state is driven by gx_msg_gen / gx_msg_merge / gx_msg_apply");
    GX_REQUIRE(!s->dev_error && !s->g->dev_error, GX_EDEVICE, "sticky device error");
    hipStream_t hs = static_cast<hipStream_t>(stream);
    auto t0 = std::chrono::steady_clock::now();
    double ms0 = s->kernel_ms;
    int64_t l0 = s->kernel_launches;
    gx_run_stats rs{};
    std::vector<DevStep> host;
    gx_status result = GX_OK;
    const int64_t k_begin = s->k;
    if (s->p.algo == GX_PAGERANK) {
        // In chunks that leave the counter ring room for the chunk's slots
        // plus the following one, so no slot is reused before it is read.
        for (uint32_t done = 0; done < max_supersteps;) {
            const uint32_t g = std::min<uint32_t>(max_supersteps - done, STEP_RING - 2);
            const int64_t kfirst = s->k;
            if (!pr_replay(s, g, hs)) {
                for (uint32_t i = 0; i < g; i++) {
                    gx_status st = enqueue_superstep(s, hs);
                    if (st != GX_OK) return st;
                }
            }
            gx_status st = read_steps(s, kfirst, g + 1, hs, host);
            if (st != GX_OK) return st;
            for (uint32_t i = 0; i < g; i++) {
                gx_step_stats o;
                to_stats(s, host[i], host[i + 1], &o);
                if (per_step) per_step[done + i] = o;
                rs.edges += o.edges;
            }
            done += g;
        }
        rs.supersteps = max_supersteps;
        rs.converged = 0;
    } else {
        // Supersteps are enqueued in speculative groups and the host
        // synchronises once per group; supersteps enqueued after convergence
        // find an empty frontier, change nothing and cost a few microseconds
        // each, less than a host round trip.  The first group covers the
        // superstep count of the last converged run on this graph (which
        // includes the superstep that changed nothing, so a repeat of that
        // run converges inside the group; at least 6, at most 16), the later
        // ones 8 at a time.
        // (label propagation keeps no history: its first group covers 16, the
        // evaluation's cap of 15 plus one)
        const int hist = s->p.algo == GX_CC ? 1 : 0;
        const bool lp = s->p.algo == GX_LP;
        const uint32_t last = lp ? 16u : s->g->last_supersteps[hist].load(std::memory_order_relaxed);
        uint32_t done = 0, spec = std::min<uint32_t>(16, std::max<uint32_t>(6, last));
        bool conv = false;
        while (done < max_supersteps && !conv) {
            uint32_t g = std::min(spec, max_supersteps - done);
            int64_t kfirst = s->k;
            for (uint32_t i = 0; i < g; i++) {
                gx_status st = enqueue_superstep(s, hs);
                if (st != GX_OK) return st;
            }
            gx_status st = read_steps(s, kfirst, g + 1, hs, host);
            if (st != GX_OK) return st;
            for (uint32_t i = 0; i < g; i++) {
                gx_step_stats o;
                to_stats(s, host[i], host[i + 1], &o);
                if (per_step) per_step[done] = o;
                rs.edges += o.edges;
                done++;
                if (o.changed == 0) {
                    conv = true;
                    s->k = kfirst + i + 1;
                    break;
                }
            }
            spec = 8;
        }
        rs.supersteps = done;
        rs.converged = conv ? 1 : 0;
        if (conv && k_begin == 0 && !lp) s->g->last_supersteps[hist].store(done, std::memory_order_relaxed);
        if (!conv) {
            set_error("not converged after %u supersteps", max_supersteps);
            result = GX_ENOTCONVERGED;
        }
    }
    collect_timings(s, per_step, k_begin, rs.supersteps, k_begin + rs.supersteps);
    rs.edge_kernel_ms = s->kernel_ms - ms0;
    rs.edge_kernel_launches = s->kernel_launches - l0;
    rs.wall_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    if (out) *out = rs;
    return result;
}

extern "C" gx_status gx_sync_delta(gx_state *s, int32_t *dev_gid, uint32_t *dev_val, uint32_t cap, uint32_t *count,
                                   int32_t *skippable, void *stream) {
    clear_error();
    GX_REQUIRE(s && count, GX_EINVAL, "NULL argument");
    GX_REQUIRE(cap == 0 || (dev_gid && dev_val), GX_EINVAL, "output buffers are NULL");
    GX_REQUIRE(!s->dev_error && !s->g->dev_error, GX_EDEVICE, "sticky device error");
    hipStream_t hs = static_cast<hipStream_t>(stream);
    const DevGraph &d = s->g->d;
    *count = 0;
    if (skippable) *skippable = 1;
    if (d.W == 0) return GX_OK;
    bool all = s->p.delta_mode == GX_DELTA_ALL;
    const uint32_t *remote = s->p.delta_mode == GX_DELTA_MASTERS              ? d.master_rep
                           : (s->p.algo == GX_CC || s->p.algo == GX_LP) ? d.remote_any
                                                                        : d.remote_out;
    // PageRank and LP compare with the synced copy (LP labels can return to an
    // earlier value); SSSP / CC values only fall, so the dirty map decides
    const bool by_copy = s->p.algo == GX_PAGERANK || s->p.algo == GX_LP;
    const uint32_t *vals = cur_values(s);
    uint8_t *dirty = by_copy ? nullptr : s->dirty8;
    uint32_t *synced = by_copy ? s->synced : nullptr;
    // the count is written to pinned memory by the kernel itself
    if (!s->host_steps) s->host_steps = host_steps_take();
    GX_REQUIRE(s->host_steps, GX_ENOMEM, "pinned host allocation failed");
    uint32_t *const total_at = reinterpret_cast<uint32_t *>(s->host_steps);
    hipLaunchKernelGGL(k_delta_count, dim3(s->delta_blocks), dim3(256), 0, hs, s->delta_words, d.W, d.V, remote, (int)all, dirty,
                       vals, synced, s->blk_cnt);
    hipLaunchKernelGGL(k_delta_emit, dim3(s->delta_blocks), dim3(256), 0, hs, s->delta_words, d.W, d.V, remote, (int)all, dirty,
                       vals, synced, d.l2g, s->blk_cnt, s->delta_blocks, cap, dev_gid, dev_val, total_at);
    GX_CHECK_HIP(hipGetLastError(), s);
    GX_CHECK_HIP(hipStreamSynchronize(hs), s);
    const uint32_t total = *total_at;
    *count = total;
    if (skippable) *skippable = total == 0;
    if (total > cap) {
        set_error("sync set has %u entries, capacity %u", total, cap);
        return GX_ENOMEM;
    }
    return GX_OK;
}

// ------------------------------------------------------------ sync set, no allocation
// The per-workgroup counts of gx_sync_delta_noalloc live in this array: one
// copy per GPU, held until the process ends, shared by every call on that
// GPU.  Host code never passes its name to a kernel (on the host it is only a
// stand-in symbol): the device address of each GPU's copy is looked up once
// with hipGetSymbolAddress, with that GPU current, and kept in g_scratch_ptr.
// Every count a launch reads is written earlier in the same call, so nothing
// in the array has to start at zero.
constexpr int NOALLOC_SCRATCH_WORDS = 65536;  // 256 KiB: sync sets of up to 2^29 vertices
static __device__ __align__(256) uint32_t scratch[NOALLOC_SCRATCH_WORDS];

constexpr int NOALLOC_MAX_DEVICES = 64;
static std::mutex g_scratch_mu;
static uint32_t *g_scratch_ptr[NOALLOC_MAX_DEVICES] = {};

static gx_status scratch_for_device(int device, uint32_t **out) {
    GX_REQUIRE(device >= 0 && device < NOALLOC_MAX_DEVICES, GX_EINVAL, "device ordinal %d out of range", device);
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        int cur = 0;
        hipError_t e = hipGetDevice(&cur);
        if (e == hipSuccess && cur != device) e = hipSetDevice(device);
        void *ptr = nullptr;
        if (e == hipSuccess) e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (cur != device) (void)hipSetDevice(cur);
        if (e != hipSuccess || !ptr) {
            set_error("hipGetSymbolAddress(scratch) on device %d failed: %s", device,
                      hipGetErrorString(e == hipSuccess ? hipErrorInvalidSymbol : e));
            return GX_EDEVICE;
        }
        g_scratch_ptr[device] = static_cast<uint32_t *>(ptr);
    }
    *out = g_scratch_ptr[device];
    return GX_OK;
}

extern "C" gx_status gx_sync_delta_noalloc(gx_state *s, int32_t *dev_gid, uint32_t *dev_val, uint32_t cap,
                                           uint32_t *dev_count, void *stream) {
    clear_error();
    GX_REQUIRE(s && dev_count, GX_EINVAL, "NULL argument");
    GX_REQUIRE(cap == 0 || (dev_gid && dev_val), GX_EINVAL, "output buffers are NULL");
    GX_REQUIRE(!s->dev_error && !s->g->dev_error, GX_EDEVICE, "sticky device error");
    GX_REQUIRE(s->delta_blocks <= NOALLOC_SCRATCH_WORDS, GX_EINVAL,
               "gx_sync_delta_noalloc handles at most %lld vertices (graph has %lld)",
               (long long)NOALLOC_SCRATCH_WORDS * DELTA_WORDS * 32, (long long)s->g->d.V);
    uint32_t *cnt = nullptr;
    gx_status st = scratch_for_device(s->g->device, &cnt);
    if (st != GX_OK) return st;
    hipStream_t hs = static_cast<hipStream_t>(stream);
    const DevGraph &d = s->g->d;
    if (d.W == 0) {  // no vertices: the count is zero (a one-thread kernel, not a memset node)
        hipLaunchKernelGGL(k_set_u32, dim3(1), dim3(1), 0, hs, dev_count, 0u);
        GX_CHECK_HIP(hipGetLastError(), s);
        return GX_OK;
    }
    bool all = s->p.delta_mode == GX_DELTA_ALL;
    const uint32_t *remote = s->p.delta_mode == GX_DELTA_MASTERS              ? d.master_rep
                           : (s->p.algo == GX_CC || s->p.algo == GX_LP) ? d.remote_any
                                                                        : d.remote_out;
    // PageRank and LP compare with the synced copy (LP labels can return to an
    // earlier value); SSSP / CC values only fall, so the dirty map decides
    const bool by_copy = s->p.algo == GX_PAGERANK || s->p.algo == GX_LP;
    const uint32_t *vals = cur_values(s);
    uint8_t *dirty = by_copy ? nullptr : s->dirty8;
    uint32_t *synced = by_copy ? s->synced : nullptr;
    hipLaunchKernelGGL(k_delta_count, dim3(s->delta_blocks), dim3(256), 0, hs, s->delta_words, d.W, d.V, remote, (int)all, dirty,
                       vals, synced, cnt);
    hipLaunchKernelGGL(k_delta_emit, dim3(s->delta_blocks), dim3(256), 0, hs, s->delta_words, d.W, d.V, remote, (int)all, dirty,
                       vals, synced, d.l2g, cnt, s->delta_blocks, cap, dev_gid, dev_val, dev_count);
    GX_CHECK_HIP(hipGetLastError(), s);
    return GX_OK;
}

extern "C" gx_status gx_apply_delta(gx_state *s, const int32_t *dev_gid, const uint32_t *dev_val, uint32_t n,
                                    int64_t *active_next, void *stream) {
    clear_error();
    GX_REQUIRE(s, GX_EINVAL, "state is NULL");
    GX_REQUIRE(n == 0 || (dev_gid && dev_val), GX_EINVAL, "input buffers are NULL");
    GX_REQUIRE(!s->dev_error && !s->g->dev_error, GX_EDEVICE, "sticky device error");
    hipStream_t hs = static_cast<hipStream_t>(stream);
    const DevGraph &d = s->g->d;
    if (s->p.phases == GX_PHASES_MASTERS) {  // PageRank replicas take their masters' new ranks
        if (n > 0 && d.V > 0)
            hipLaunchKernelGGL(k_replica_set, dim3(grid_for<uint32_t>(n, 256)), dim3(256), 0, hs, dev_gid, dev_val, n,
                               d.l2g, d.V, d.master, reinterpret_cast<uint32_t *>(s->x[0]));
        GX_CHECK_HIP(hipGetLastError(), s);
        if (active_next) *active_next = 0;
        return GX_OK;
    }
    GX_REQUIRE(s->p.algo == GX_SSSP || s->p.algo == GX_CC, GX_EINVAL,
               "gx_apply_delta merges SSSP / CC values (and PageRank ranks under GX_PHASES_MASTERS)");
    GX_REQUIRE(!s->p.phases, GX_EINVAL, "gx_apply_delta serves SSSP / CC states driven by gx_superstep");
    if (d.V > 0) {
        // A_{k+1} (the frontier of the superstep about to run) and its counter slot
        uint8_t *front = s->front8[s->k & 1];
        DevStep *slot = s->steps + (s->k % STEP_RING);
        s->merged |= n > 0;
        if (n > 0)
            hipLaunchKernelGGL(k_apply_delta, dim3(grid_for<uint32_t>(n, 256)), dim3(256), 0, hs, dev_gid, dev_val, n,
                               d.l2g, d.V, s->val, front);
        // rebuild the active list of A_{k+1} from the merged values
        hipLaunchKernelGGL(k_zero_step, dim3(1), dim3(1), 0, hs, slot);
        launch_compact(s, hs, front, s->front8[(s->k & 1) ^ 1], 0, nullptr, nullptr);
        GX_CHECK_HIP(hipGetLastError(), s);
    }
    if (active_next) {
        *active_next = 0;
        if (d.V > 0) {
            DevStep ds{};
            GX_CHECK_HIP(hipMemcpyAsync(&ds, s->steps + (s->k % STEP_RING), sizeof ds, hipMemcpyDeviceToHost, hs), s);
            GX_CHECK_HIP(hipStreamSynchronize(hs), s);
            *active_next = (int64_t)ds.frontier;
        }
    }
    return GX_OK;
}

// ------------------------------------------------------------ separate template calls

static gx_status ph_check(gx_state *s) {
    GX_REQUIRE(s, GX_EINVAL, "state is NULL");
    GX_REQUIRE(s->p.phases, GX_EINVAL, "state was not initialised with gx_params.phases");
    GX_REQUIRE(!s->dev_error && !s->g->dev_error, GX_EDEVICE, "sticky device error");
    return GX_OK;
}

extern "C" gx_status gx_msg_gen(gx_state *s, void *stream) {
    clear_error();
    gx_status st = ph_check(s);
    if (st != GX_OK) return st;
    GX_REQUIRE(!s->ph_msgs, GX_EINVAL, "MSGGen: the previous messages have not been merged");
    hipStream_t hs = static_cast<hipStream_t>(stream);
    const DevGraph &d = s->g->d;
    if (d.V > 0) {
        if (s->p.algo == GX_PAGERANK) {
            const unsigned nb = grid_for<int64_t>(d.V, 256);
            const bool parts = s->p.phases == GX_PHASES_MASTERS;
            hipLaunchKernelGGL(k_ph_pr_gen, dim3(nb), dim3(256), 0, hs, s->x[0], parts ? d.outdeg_g : d.outdeg,
                               d.slot, s->contrib[0], d.V, s->dpart, parts ? d.master : nullptr);
            hipLaunchKernelGGL(k_reduce_D, dim3(1), dim3(1024), 0, hs, s->dpart, (int)nb, s->Dval);
        } else {
            // the pending map's vertices become the active list (with the values
            // they send); the other map is cleared to collect the next changes
            launch_compact(s, hs, s->front8[s->ph_p], s->front8[s->ph_p ^ 1], 0, nullptr, nullptr);
        }
        GX_CHECK_HIP(hipGetLastError(), s);
    }
    s->ph_p ^= 1;
    s->ph_msgs = true;
    return GX_OK;
}

extern "C" gx_status gx_msg_merge(gx_state *s, void *stream) {
    clear_error();
    gx_status st = ph_check(s);
    if (st != GX_OK) return st;
    if (!s->ph_msgs) return GX_OK;  // nothing generated since the last merge
    hipStream_t hs = static_cast<hipStream_t>(stream);
    const DevGraph &d = s->g->d;
    if (d.V > 0) {
        if (s->p.algo == GX_PAGERANK) {
            const PrStore ap{(double)s->p.damping, 0.0, s->acc_d};
            const PrArgs a = pr_args(s, s->contrib[0], s->Dscratch, 1.0 / (double)d.V);
            hipLaunchKernelGGL(pr_pull_for<PrStore>(d), dim3(s->pr_grid), dim3(d.pr_hot ? 1024 : PR_BLOCK), 0, hs, a, ap);
            hipLaunchKernelGGL(k_pr_fix<PrStore>, dim3(s->pr_fix_grid), dim3(s->pr_fix_block), 0, hs, a, ap, s->ph_steps,
                               s->ph_steps + 1, s->fix_d, s->fix_c, s->fix_done);
        } else {
            // the relaxation of the fused superstep, against the accumulator:
            // it combines the messages by minimum and changes no vertex value
            // (MSGGen has turned the maps round)
            launch_relax(s, hs, s->front8[s->ph_p ^ 1], s->acc, s->junk8, s->steps + (s->k % STEP_RING));
        }
        GX_CHECK_HIP(hipGetLastError(), s);
    }
    s->ph_msgs = false;
    s->ph_merged = true;
    return GX_OK;
}

extern "C" gx_status gx_msg_apply(gx_state *s, void *stream, gx_step_stats *stats) {
    clear_error();
    gx_status st = ph_check(s);
    if (st != GX_OK) return st;
    hipStream_t hs = static_cast<hipStream_t>(stream);
    if (stats) *stats = gx_step_stats{};
    if (!s->ph_merged) return GX_OK;  // nothing merged since the last apply
    const DevGraph &d = s->g->d;
    const int64_t k = s->k;
    DevStep *step = s->steps + (k % STEP_RING), *next = s->steps + ((k + 1) % STEP_RING);
    if (d.V > 0) {
        if (s->p.algo == GX_PAGERANK) {
            const bool parts = s->p.phases == GX_PHASES_MASTERS;
            const double Vn = (double)(parts ? d.V_global : d.V);
            hipLaunchKernelGGL(k_ph_pr_apply, dim3(grid_for<int64_t>(d.V, PH_APPLY)), dim3(1024), 0, hs, s->acc_d, s->x[0],
                               d.V, (1.0 - (double)s->p.damping) / Vn, (double)s->p.damping, s->Dval, 1.0 / Vn, step,
                               next, parts ? d.master : nullptr);
        } else {
            hipLaunchKernelGGL(k_ph_apply, dim3(grid_for<int64_t>(d.V, 256)), dim3(256), 0, hs, s->acc, s->val,
                               s->front8[s->ph_p], s->dirty8, d.V, step, s->rot, s->relax_grid);
        }
        GX_CHECK_HIP(hipGetLastError(), s);
    }
    s->ph_merged = false;
    s->k++;
    if (stats && d.V > 0) {
        std::vector<DevStep> ds;
        st = read_steps(s, k, 1, hs, ds);
        if (st != GX_OK) return st;
        const bool pr = s->p.algo == GX_PAGERANK;
        stats->frontier = pr ? d.V : (int64_t)ds[0].frontier;
        stats->edges = pr ? d.E : (int64_t)(uint32_t)ds[0].list;
        stats->changed = (int64_t)ds[0].changed;
        stats->pulled = pr ? 1 : (ds[0].pad ? 1 : 0);
    }
    return GX_OK;
}

// ------------------------------------------------------------ PageRank across the parts of a vertex-cut

static gx_status parts_check(gx_state *s) {
    GX_REQUIRE(s, GX_EINVAL, "state is NULL");
    GX_REQUIRE(s->p.phases == GX_PHASES_MASTERS, GX_EINVAL, "state was not initialised with GX_PHASES_MASTERS");
    GX_REQUIRE(!s->dev_error && !s->g->dev_error, GX_EDEVICE, "sticky device error");
    return GX_OK;
}

extern "C" gx_status gx_dangling_get(gx_state *s, double *mass, void *stream) {
    clear_error();
    gx_status st = parts_check(s);
    if (st != GX_OK) return st;
    GX_REQUIRE(mass, GX_EINVAL, "mass is NULL");
    hipStream_t hs = static_cast<hipStream_t>(stream);
    // stored to pinned memory: a copy to pageable memory took 10 us more (PageRank
    // over four parts of R-MAT scale 18, 40 calls: 6.2 ms with it, 5.8 ms so)
    if (!s->host_steps) s->host_steps = host_steps_take();
    GX_REQUIRE(s->host_steps, GX_ENOMEM, "pinned host allocation failed");
    double *const at = reinterpret_cast<double *>(s->host_steps);
    hipLaunchKernelGGL(k_get_f64, dim3(1), dim3(1), 0, hs, s->Dval, at);
    GX_CHECK_HIP(hipGetLastError(), s);
    GX_CHECK_HIP(hipStreamSynchronize(hs), s);
    *mass = *at;
    return GX_OK;
}

extern "C" gx_status gx_dangling_set(gx_state *s, double mass, void *stream) {
    clear_error();
    gx_status st = parts_check(s);
    if (st != GX_OK) return st;
    hipStream_t hs = static_cast<hipStream_t>(stream);
    hipLaunchKernelGGL(k_set_f64, dim3(1), dim3(1), 0, hs, s->Dval, mass);
    GX_CHECK_HIP(hipGetLastError(), s);
    return GX_OK;
}

extern "C" gx_status gx_partial_emit(gx_state *s, int32_t *dev_gid, double *dev_val, uint32_t cap, uint32_t *count,
                                     void *stream) {
    clear_error();
    gx_status st = parts_check(s);
    if (st != GX_OK) return st;
    GX_REQUIRE(count, GX_EINVAL, "count is NULL");
    GX_REQUIRE(cap == 0 || (dev_gid && dev_val), GX_EINVAL, "output buffers are NULL");
    GX_REQUIRE(s->ph_merged, GX_EINVAL, "no merged messages to send");
    hipStream_t hs = static_cast<hipStream_t>(stream);
    const DevGraph &d = s->g->d;
    *count = 0;
    if (d.W == 0) return GX_OK;
    const uint32_t total = (uint32_t)d.n_part, n = std::min(total, cap);
    if (n > 0)
        hipLaunchKernelGGL(k_part_emit, dim3(grid_for<uint32_t>(n, 256)), dim3(256), 0, hs, d.part_list, n, d.l2g, s->acc_d,
                           dev_gid, dev_val);
    GX_CHECK_HIP(hipGetLastError(), s);
    GX_CHECK_HIP(hipStreamSynchronize(hs), s);
    *count = total;
    if (total > cap) {
        set_error("%u merged sums to send, capacity %u", total, cap);
        return GX_ENOMEM;
    }
    return GX_OK;
}

extern "C" gx_status gx_partial_add(gx_state *s, const int32_t *dev_gid, const double *dev_val, uint32_t n,
                                    void *stream) {
    clear_error();
    gx_status st = parts_check(s);
    if (st != GX_OK) return st;
    GX_REQUIRE(n == 0 || (dev_gid && dev_val), GX_EINVAL, "input buffers are NULL");
    GX_REQUIRE(s->ph_merged, GX_EINVAL, "merge this part's messages before adding other parts' sums");
    hipStream_t hs = static_cast<hipStream_t>(stream);
    const DevGraph &d = s->g->d;
    if (n > 0 && d.V > 0)
        hipLaunchKernelGGL(k_part_add, dim3(grid_for<uint32_t>(n, 256)), dim3(256), 0, hs, dev_gid, dev_val, n, d.l2g,
                           d.V, d.master, s->acc_d);
    GX_CHECK_HIP(hipGetLastError(), s);
    return GX_OK;
}
