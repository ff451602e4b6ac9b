// Label propagation (community-detection form) on the symmetric adjacency.
//
// The paper's evaluation runs "LP" capped at 15 iterations (Section "Setup",
// first footnote) through the algorithm template (Section "Algorithm
// Template"): MSGGen sends a vertex's label along each of its edges in both
// directions, MSGMerge gathers the labels bound for a vertex, MSGApply keeps
// the most frequent one (the smallest on a tie).  One superstep reads the
// labels of its start (lab[k & 1]) and writes lab[(k + 1) & 1].
//
// The merge is a mode over a multiset, so it is computed where the messages
// meet: a vertex reads its distinct neighbours' labels and counts them.
// Vertices are grouped by degree so each group's counting fits its size:
//   classes 0..4 (d <= 4 .. 64): one lane group of width G = 4 .. 64 per
//     vertex, each lane one neighbour, counts by lane shuffles (G = 64: by
//     ballots, one per distinct label) and the winner by a maximum of
//     (count, ~label);
//   class 5 (64 < d <= LP_MID_MAX): labels counted in an LDS hash table at
//     most half full, one wave per vertex up to LP_WAVE_MAX neighbours, one
//     workgroup above;
//   class 6 (hubs): neighbours cut into chunks; each chunk counts in LDS and
//     adds its (label, count) pairs to the hub's table in device memory, and
//     every sum reached there to the hub's running maximum: the largest
//     (count, ~label) over all partial sums is the largest over the final
//     ones.  The table slots taken are logged, so only they are cleared.
// Counts are exact integers and the winner is the unique maximum of
// (count, ~label), so the result does not depend on the order of the atomics.
//
// Superstep 0 needs no counting where every row's neighbours ascend: the
// labels are the (distinct) global ids, so every count is 1 and the winner is
// the first neighbour's (other rows are counted).  After that only
// the vertices with a neighbour whose label changed can change: when the
// changed vertices' edges are a small part of all (LP_DENSE), their
// neighbours are marked and only the marked are recomputed; a vertex that
// changed in the superstep before is copied, every other label is in both
// buffers already.  R-MAT scale 20, shuffled ids, 15 iterations: every
// superstep recomputing every vertex took 700 us; now the first takes 107 us,
// the two that recompute all 695 and 419 us (bound by the counting in LDS),
// and the ten from the sixth on 65 us each (their six launches).
// The class lists are built on the device; counting them on the host took 19
// of the 29.7 ms of a whole run (reset included), which now takes 2.9 ms.
#include <algorithm>
#include <vector>

#include "gx_device.h"
#include "gx_internal.h"
#include "gx_limits.h"

using namespace gx;

namespace {

constexpr int LP_BLOCK = 256;

__device__ __forceinline__ unsigned long long lp_key(uint32_t count, uint32_t label) {
    return ((unsigned long long)count << 32) | (unsigned long long)(0xFFFFFFFFu - label);
}

__device__ __forceinline__ uint32_t lp_hash(uint32_t x) { return x * 0x9E3779B1u; }

// Changed vertices' entries {vertex, chunk of LP_CHANGED_CHUNK neighbours};
// step->list counts (entries << 32) | their neighbours.
constexpr int LP_CHANGED_CHUNK = 1024;
// A superstep after changes with more than E_sym / LP_DENSE neighbours
// recomputes every vertex: marking nearly all costs more than it saves (15
// iterations with 2, 4, 8, 16: R-MAT scale 20, shuffled ids 2.75, 2.67, 2.67, 2.67 ms,
// as they are 1.52, 1.45, 1.45, 1.45; scale 16 570, 558, 550, 552 us).
constexpr int64_t LP_DENSE = 4;

struct LpStep {
    const int32_t *rp, *col;
    const uint32_t *lab;
    uint32_t *nxt;
    uint8_t *touch;
    uint2 *changed;
    DevStep *step;
    const DevStep *prev;
    int64_t E_sym;
    bool first;  // superstep 0: there is no superstep before it
    __device__ __forceinline__ bool full() const {
        return first || (int64_t)(uint32_t)prev->list * LP_DENSE > E_sym;
    }
};

// The changed vertices of a workgroup, kept in LDS so that each workgroup
// reserves its list entries once (adds with a result on one counter queue up).
struct ChangedQ {
    uint32_t v[LP_BLOCK];
    uint32_t n;
    unsigned long long scan[LP_BLOCK / 64], base;
};

__device__ __forceinline__ void changed_put(ChangedQ &q, uint32_t v) { q.v[atomicAdd(&q.n, 1u)] = v; }

// (whole workgroup; q.n <= LP_BLOCK)
__device__ __forceinline__ void changed_flush(ChangedQ &q, const LpStep &a) {
    __syncthreads();
    const uint32_t n = q.n;
    if (n == 0) return;
    uint32_t v = 0, d = 0;
    if (threadIdx.x < n) {
        v = q.v[threadIdx.x];
        d = (uint32_t)(a.rp[v + 1] - a.rp[v]);
    }
    const uint32_t ne = (d + LP_CHANGED_CHUNK - 1) / LP_CHANGED_CHUNK;
    unsigned long long total;
    const unsigned long long pre = block_excl_scan_u64((unsigned long long)ne << 32 | d, &total, q.scan);
    if (threadIdx.x == 0) {
        q.base = atomicAdd(&a.step->list, total);
        atomicAdd(&a.step->changed, (unsigned long long)n);
        q.n = 0;
    }
    __syncthreads();
    const uint32_t at = (uint32_t)((q.base + pre) >> 32);
    for (uint32_t i = 0; i < ne; i++) a.changed[at + i] = make_uint2(v, i);
    __syncthreads();
}

struct LpCursors {
    uint32_t at[7];  // first slot of every list
};

__global__ __launch_bounds__(LP_BLOCK) void k_lp_init(uint32_t *lab0, uint32_t *lab1, uint32_t *synced, uint8_t *touch,
                                                      unsigned long long *best, int64_t hubs,
                                                      const int32_t *__restrict__ l2g, int64_t V, DevStep *step0, uint32_t *cursor,
                                                      LpCursors at) {
    const int64_t v = (int64_t)blockIdx.x * LP_BLOCK + threadIdx.x;
    if (v == 0) *step0 = DevStep{};
    if (v < 7) cursor[v] = at.at[v];
    if (v < hubs) best[v] = 0ull;
    if (v >= V) return;
    touch[v] = 0;
    const uint32_t l = l2g ? (uint32_t)l2g[v] : (uint32_t)v;
    lab0[v] = l;
    lab1[v] = l;
    synced[v] = l;
}

__global__ __launch_bounds__(LP_BLOCK) void k_lp_tab_clear(uint2 *tab, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * LP_BLOCK + threadIdx.x;
    if (i < n) tab[i] = make_uint2(LP_NONE, 0u);
}

// Superstep 0: the first neighbour's label (labels ascend with the ids).
__global__ __launch_bounds__(LP_BLOCK) void k_lp_first(LpStep a, int64_t V, DevStep *next) {
    __shared__ ChangedQ s_q;
    if (threadIdx.x == 0) s_q.n = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) *next = DevStep{};
    __syncthreads();
    const int64_t v = (int64_t)blockIdx.x * LP_BLOCK + threadIdx.x;
    if (v < V) {
        const int32_t b = a.rp[v], e = a.rp[v + 1];
        if (e > b) {
            a.nxt[v] = a.lab[a.col[b]];
            changed_put(s_q, (uint32_t)v);  // (a neighbour's id is another id)
        }
    }
    changed_flush(s_q, a);
}

// The vertices changed in the superstep before: copied, and their neighbours
// marked (16 lanes an entry).
__global__ __launch_bounds__(LP_BLOCK) void k_lp_mark(LpStep a, DevStep *next, uint32_t *log_n) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *next = DevStep{};
        *log_n = 0;
    }
    if (a.full()) return;
    const unsigned long long le = a.prev->list;
    const uint32_t n = (uint32_t)(le >> 32), gl = threadIdx.x & 15;
    for (uint32_t i = (blockIdx.x * LP_BLOCK + threadIdx.x) / 16; i < n; i += gridDim.x * (LP_BLOCK / 16)) {
        const uint2 q = a.changed[i];
        const int32_t b = a.rp[q.x] + (int32_t)q.y * LP_CHANGED_CHUNK, e = chunk_end(b, a.rp[q.x + 1], LP_CHANGED_CHUNK);
        if (q.y == 0 && gl == 0) a.nxt[q.x] = a.lab[q.x];
        for (int32_t p = b + (int32_t)gl; p < e; p += 64) {
            int32_t u[4];
#pragma unroll
            for (int j = 0; j < 4; j++) u[j] = a.col[min(p + 16 * j, e - 1)];
#pragma unroll
            for (int j = 0; j < 4; j++) a.touch[u[j]] = 1;
        }
    }
}

// Whether vertex v has to be recomputed (its mark is taken back).
__device__ __forceinline__ bool lp_take(const LpStep &a, bool full, uint32_t v) {
    if (full) return true;
    if (!a.touch[v]) return false;
    a.touch[v] = 0;
    return true;
}

struct LpQueue {
    uint32_t v[64];
    int32_t a[64], d[64];
};

// Classes 0..4.  A wave takes up to 64 vertices of its class's list (8 for G
// = 64), one per lane, queues the ones to recompute and gives each a lane
// group.
template <int G>
__device__ __forceinline__ void lp_groups(const LpStep &a, bool full, const uint32_t *__restrict__ list, int64_t n,
                                          int64_t wave, LpQueue &q, ChangedQ &cq) {
    constexpr int W = G <= 8 ? 64 : 512 / G;
    const int lane = threadIdx.x & 63;
    const int64_t i = wave * W + lane;
    uint32_t v = 0;
    bool take = false;
    if (lane < W && i < n) {
        v = list[i];
        take = lp_take(a, full, v);
    }
    const unsigned long long m = __ballot(take);
    if (take) {
        const int pos = __popcll(m & ((1ull << lane) - 1ull));
        const int32_t b = a.rp[v];
        q.v[pos] = v;
        q.a[pos] = b;
        q.d[pos] = a.rp[v + 1] - b;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int cnt = __popcll(m), j = lane & (G - 1), base = lane - j;
    for (int i0 = 0; i0 < cnt; i0 += 64 / G) {
        const int s = min(i0 + lane / G, cnt - 1);
        const bool ok = i0 + lane / G < cnt;
        const uint32_t u = q.v[s];
        const int32_t d = q.d[s];
        const uint32_t L = ok && j < d ? a.lab[a.col[q.a[s] + j]] : LP_NONE;
        unsigned long long key = 0ull;
        if (G == 64) {  // one ballot per distinct label
            for (unsigned long long left = __ballot(L != LP_NONE); left;) {
                const uint32_t x = (uint32_t)__builtin_amdgcn_readlane((int)L, __ffsll((unsigned long long)left) - 1);
                const unsigned long long same = __ballot(L == x);
                const unsigned long long k2 = lp_key((uint32_t)__popcll(same), x);
                key = k2 > key ? k2 : key;
                left &= ~same;
            }
        } else {
            uint32_t c = 0;
#pragma unroll
            for (int t = 0; t < G; t++) c += (uint32_t)(__shfl(L, base + t, 64) == L);
            key = L != LP_NONE ? lp_key(c, L) : 0ull;
#pragma unroll
            for (int o = G / 2; o > 0; o >>= 1) {
                const unsigned long long k2 = __shfl_xor(key, o, 64);
                key = k2 > key ? k2 : key;
            }
        }
        if (ok && j == 0) {
            const uint32_t nl = 0xFFFFFFFFu - (uint32_t)key;
            a.nxt[u] = nl;
            if (nl != a.lab[u]) changed_put(cq, u);
        }
    }
}

struct LpRanges {
    const uint32_t *list;
    int64_t off[6];   // class c owns list[off[c] .. off[c + 1])
    uint32_t blk[6];  // workgroups of class c: blk[c] .. blk[c + 1] - 1
};

__global__ __launch_bounds__(LP_BLOCK) void k_lp_groups(LpStep a, LpRanges r) {
    __shared__ LpQueue s_q[LP_BLOCK / 64];
    __shared__ ChangedQ s_c;
    if (threadIdx.x == 0) s_c.n = 0;
    __syncthreads();
    const bool full = a.full();
    int c = 0;
    while (c < 4 && blockIdx.x >= r.blk[c + 1]) c++;
    const int64_t wave = (int64_t)(blockIdx.x - r.blk[c]) * (LP_BLOCK / 64) + (threadIdx.x >> 6);
    const uint32_t *list = r.list + r.off[c];
    const int64_t n = r.off[c + 1] - r.off[c];
    LpQueue &q = s_q[threadIdx.x >> 6];
    switch (c) {
        case 0: lp_groups<4>(a, full, list, n, wave, q, s_c); break;
        case 1: lp_groups<8>(a, full, list, n, wave, q, s_c); break;
        case 2: lp_groups<16>(a, full, list, n, wave, q, s_c); break;
        case 3: lp_groups<32>(a, full, list, n, wave, q, s_c); break;
        default: lp_groups<64>(a, full, list, n, wave, q, s_c); break;
    }
    changed_flush(s_c, a);
}

// Vertices per wave of lp_groups<G>.
constexpr int lp_wave_vertices(int c) { return c <= 1 ? 64 : 512 / (4 << c); }

// Counts one label per lane (LP_NONE: none) into an LDS table of `slots`
// (a power of two, 1 << lg, at most half full): the first two labels met are
// counted for the whole wave at once (after the first supersteps most lanes
// hold the same few), the rest lane by lane.
__device__ __forceinline__ void lp_count(uint32_t *key, uint32_t *cnt, int lg, uint32_t L) {
    const int lane = threadIdx.x & 63;
    uint32_t add = L != LP_NONE ? 1u : 0u;
#pragma unroll
    for (int t = 0; t < 2; t++) {
        const unsigned long long left = __ballot(add == 1u);
        if (!left) break;
        const int lead = __ffsll(left) - 1;
        const uint32_t x = (uint32_t)__builtin_amdgcn_readlane((int)L, lead);
        const unsigned long long same = __ballot(add == 1u && L == x);
        if (add == 1u && L == x) add = lane == lead ? 0x80000000u | (uint32_t)__popcll(same) : 0u;
    }
    add &= 0x7FFFFFFFu;
    if (add) {
        uint32_t h = lp_hash(L) >> (32 - lg);
        for (;;) {
            const uint32_t k = atomicCAS(&key[h], LP_NONE, L);
            if (k == LP_NONE || k == L) {
                atomicAdd(&cnt[h], add);
                break;
            }
            h = (h + 1) & ((1u << lg) - 1u);
        }
    }
}

// Mid class, up to LP_WAVE_MAX neighbours: one wave per vertex.
constexpr int LP_WAVE_MAX = 512;

__global__ __launch_bounds__(LP_BLOCK) void k_lp_mid_wave(LpStep a, const uint32_t *__restrict__ list, int64_t n) {
    __shared__ uint32_t s_key[LP_BLOCK / 64][2 * LP_WAVE_MAX], s_cnt[LP_BLOCK / 64][2 * LP_WAVE_MAX];
    __shared__ ChangedQ s_c;
    if (threadIdx.x == 0) s_c.n = 0;
    __syncthreads();
    const bool full = a.full();
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    uint32_t *key = s_key[wv], *cnt = s_cnt[wv];
    // (a workgroup takes at most LP_BLOCK vertices: the queue holds them all)
    const int64_t per = (n + gridDim.x - 1) / gridDim.x, lo = per * blockIdx.x, hi = min(n, lo + per);
    for (int64_t i = lo + wv; i < hi; i += LP_BLOCK / 64) {
        const uint32_t v = list[i];
        if (!full && !a.touch[v]) continue;
        if (lane == 0) a.touch[v] = 0;
        const int32_t b = a.rp[v], d = a.rp[v + 1] - b;
        int lg = 7;
        while ((1 << lg) < 2 * d) lg++;
        for (int s = lane; s < (1 << lg); s += 64) {
            key[s] = LP_NONE;
            cnt[s] = 0;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        for (int e = 0; e < d; e += 256) {
            uint32_t L[4];
            int32_t u[4];
#pragma unroll
            for (int j = 0; j < 4; j++) u[j] = a.col[b + min(e + 64 * j + lane, d - 1)];
#pragma unroll
            for (int j = 0; j < 4; j++) L[j] = a.lab[u[j]];
#pragma unroll
            for (int j = 0; j < 4; j++) lp_count(key, cnt, lg, e + 64 * j + lane < d ? L[j] : LP_NONE);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        unsigned long long best = 0;
        for (int s = lane; s < (1 << lg); s += 64) {
            const uint32_t k = key[s];
            if (k != LP_NONE) {
                const unsigned long long x = lp_key(cnt[s], k);
                best = x > best ? x : best;
            }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const unsigned long long b2 = __shfl_down(best, o, 64);
            best = b2 > best ? b2 : best;
        }
        if (lane == 0) {
            const uint32_t nl = 0xFFFFFFFFu - (uint32_t)best;
            a.nxt[v] = nl;
            if (nl != a.lab[v]) changed_put(s_c, v);
        }
        __builtin_amdgcn_wave_barrier();
    }
    changed_flush(s_c, a);
}

// Mid class above that: one workgroup per vertex; the table holds the next
// power of two at or above 2d slots.
__global__ __launch_bounds__(LP_BLOCK) void k_lp_mid(LpStep a, const uint32_t *__restrict__ list, int64_t n) {
    __shared__ uint32_t s_key[LP_MID_SLOTS];
    __shared__ uint32_t s_cnt[LP_MID_SLOTS];
    __shared__ unsigned long long s_best[LP_BLOCK / 64];
    __shared__ ChangedQ s_c;
    const int tid = threadIdx.x;
    if (tid == 0) s_c.n = 0;
    __syncthreads();
    const bool full = a.full();
    const int64_t per = (n + gridDim.x - 1) / gridDim.x, lo = per * blockIdx.x, hi = min(n, lo + per);
    for (int64_t i = lo; i < hi; i++) {
        const uint32_t v = list[i];
        const bool take = full || a.touch[v];
        __syncthreads();  // (every thread has read the mark before it is taken back)
        if (!take) continue;
        if (tid == 0) a.touch[v] = 0;
        const int32_t b = a.rp[v], d = a.rp[v + 1] - b;
        int lg = 7;
        while ((1 << lg) < 2 * d) lg++;
        const int slots = 1 << lg;
        for (int s = tid; s < slots; s += LP_BLOCK) {
            s_key[s] = LP_NONE;
            s_cnt[s] = 0;
        }
        __syncthreads();
        for (int e = 0; e < d; e += 4 * LP_BLOCK) {
            uint32_t L[4];
            int32_t u[4];
#pragma unroll
            for (int j = 0; j < 4; j++) u[j] = a.col[b + min(e + LP_BLOCK * j + tid, d - 1)];
#pragma unroll
            for (int j = 0; j < 4; j++) L[j] = a.lab[u[j]];
#pragma unroll
            for (int j = 0; j < 4; j++) lp_count(s_key, s_cnt, lg, e + LP_BLOCK * j + tid < d ? L[j] : LP_NONE);
        }
        __syncthreads();
        unsigned long long best = 0;
        for (int s = tid; s < slots; s += LP_BLOCK) {
            const uint32_t k = s_key[s];
            if (k != LP_NONE) {
                const unsigned long long key = lp_key(s_cnt[s], k);
                best = key > best ? key : best;
            }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const unsigned long long b2 = __shfl_down(best, o, 64);
            best = b2 > best ? b2 : best;
        }
        if ((tid & 63) == 0) s_best[tid >> 6] = best;
        __syncthreads();
        if (tid == 0) {
            for (int w = 1; w < LP_BLOCK / 64; w++) best = s_best[w] > best ? s_best[w] : best;
            const uint32_t nl = 0xFFFFFFFFu - (uint32_t)best;
            a.nxt[v] = nl;
            if (nl != a.lab[v]) changed_put(s_c, v);
        }
    }
    changed_flush(s_c, a);
}

// Hub chunks: each workgroup counts its chunk's labels in an LDS table
// (labels that find no free slot within a few probes go straight to the
// hub's table) and adds the chunk's (label, count) pairs to the hub's table.
constexpr int LP_CHUNK_SLOTS = 4096;
constexpr int LP_CHUNK_LG = 12;
constexpr int LP_CHUNK_PROBES = 16;

// Adds c to label L of a hub and raises the hub's maximum; returns the slot
// if it was taken by this add, else LP_NONE.
__device__ __forceinline__ uint32_t lp_tab_add(uint2 *tab, uint2 hb, unsigned long long *best, uint32_t L, uint32_t c) {
    uint32_t h = (lp_hash(L) >> 7) & (hb.y - 1);
    for (;;) {
        uint2 *t = tab + hb.x + h;
        const uint32_t k = atomicCAS(&t->x, LP_NONE, L);
        if (k == LP_NONE || k == L) {
            const unsigned long long key = lp_key(atomicAdd(&t->y, c) + c, L);
            if (key > *best) atomicMax(best, key);  // (a stale read only costs an atomic)
            return k == LP_NONE ? hb.x + h : LP_NONE;
        }
        h = (h + 1) & (hb.y - 1);
    }
}

struct LpHubs {
    const uint32_t *hubs;  // vertices
    const uint4 *chunks;   // {hub, first entry, end entry, 0}
    const uint2 *hub;      // per hub {first table slot, slots}
    uint2 *tab;
    unsigned long long *best;  // per hub, 0 between supersteps
    uint32_t *log, *log_n;     // table slots taken in this superstep
};

__global__ __launch_bounds__(LP_BLOCK) void k_lp_hub_count(LpStep a, LpHubs hu) {
    __shared__ uint32_t s_key[LP_CHUNK_SLOTS];
    __shared__ uint32_t s_cnt[LP_CHUNK_SLOTS];
    __shared__ unsigned long long s_scan[LP_BLOCK / 64];
    __shared__ uint32_t s_base;
    const int tid = threadIdx.x;
    const uint4 ch = hu.chunks[blockIdx.x];
    if (!a.full() && !a.touch[hu.hubs[ch.x]]) return;  // (k_lp_hub_pick takes the mark back)
    const uint2 hb = hu.hub[ch.x];
    for (int s = tid; s < LP_CHUNK_SLOTS; s += LP_BLOCK) {
        s_key[s] = LP_NONE;
        s_cnt[s] = 0;
    }
    __syncthreads();
    for (uint32_t e0 = ch.y; e0 < ch.z; e0 += 4 * LP_BLOCK) {
        uint32_t L[4];
        int32_t u[4];
#pragma unroll
        for (int j = 0; j < 4; j++) u[j] = a.col[min(e0 + LP_BLOCK * j + tid, ch.z - 1)];
#pragma unroll
        for (int j = 0; j < 4; j++) L[j] = a.lab[u[j]];
#pragma unroll
        for (int j = 0; j < 4; j++) {
            // one add for the lanes that hold the first lane's label
            const bool in = e0 + LP_BLOCK * j + tid < ch.z;
            const unsigned long long all = __ballot(in);
            if (!in) continue;
            const int lead = __ffsll(all) - 1;
            const uint32_t x = (uint32_t)__builtin_amdgcn_readlane((int)L[j], lead);
            const unsigned long long same = __ballot(L[j] == x);
            uint32_t add = 1;
            if (L[j] == x) {
                if ((tid & 63) != lead) continue;
                add = (uint32_t)__popcll(same);
            }
            uint32_t h = lp_hash(L[j]) >> (32 - LP_CHUNK_LG);
            bool done = false;
            for (int p = 0; p < LP_CHUNK_PROBES; p++) {
                const uint32_t k = atomicCAS(&s_key[h], LP_NONE, L[j]);
                if (k == LP_NONE || k == L[j]) {
                    atomicAdd(&s_cnt[h], add);
                    done = true;
                    break;
                }
                h = (h + 1) & (LP_CHUNK_SLOTS - 1);
            }
            if (!done) {
                const uint32_t s = lp_tab_add(hu.tab, hb, &hu.best[ch.x], L[j], add);
                if (s != LP_NONE) hu.log[atomicAdd(hu.log_n, 1u)] = s;
            }
        }
    }
    __syncthreads();
    constexpr int PT = LP_CHUNK_SLOTS / LP_BLOCK;
    uint32_t took[PT], n = 0;
#pragma unroll
    for (int i = 0; i < PT; i++) {
        const int s = tid + i * LP_BLOCK;
        took[i] = s_key[s] != LP_NONE ? lp_tab_add(hu.tab, hb, &hu.best[ch.x], s_key[s], s_cnt[s]) : LP_NONE;
        n += took[i] != LP_NONE;
    }
    unsigned long long total;
    uint32_t at = (uint32_t)block_excl_scan_u64(n, &total, s_scan);
    if (tid == 0) s_base = total ? atomicAdd(hu.log_n, (uint32_t)total) : 0u;
    __syncthreads();
    at += s_base;
#pragma unroll
    for (int i = 0; i < PT; i++)
        if (took[i] != LP_NONE) hu.log[at++] = took[i];
}

// Every recomputed hub takes its maximum; the table slots taken are freed.
__global__ __launch_bounds__(LP_BLOCK) void k_lp_hub_pick(LpStep a, LpHubs hu, int64_t n) {
    __shared__ ChangedQ s_c;
    if (threadIdx.x == 0) s_c.n = 0;
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * LP_BLOCK + threadIdx.x;
    if (i < n) {
        const unsigned long long best = hu.best[i];
        if (best) {  // (a hub has neighbours: 0 says it was not recomputed)
            const uint32_t v = hu.hubs[i], nl = 0xFFFFFFFFu - (uint32_t)best;
            hu.best[i] = 0ull;
            a.touch[v] = 0;
            a.nxt[v] = nl;
            if (nl != a.lab[v]) changed_put(s_c, v);
        }
    }
    const uint32_t m = *hu.log_n;
    for (uint32_t j = blockIdx.x * LP_BLOCK + threadIdx.x; j < m; j += gridDim.x * LP_BLOCK)
        hu.tab[hu.log[j]] = make_uint2(LP_NONE, 0u);
    changed_flush(s_c, a);
}

int lp_class_of(int32_t d) {
    if (d <= 0) return -1;
    if (d <= 4) return 0;
    if (d <= 8) return 1;
    if (d <= 16) return 2;
    if (d <= 32) return 3;
    if (d <= 64) return 4;
    if (d <= LP_MID_MAX) return 5;
    return 6;
}

uint32_t lp_hub_slots(int32_t d) {
    uint32_t s = 256;
    while (s < (uint32_t)d + (uint32_t)d / 2) s *= 2;  // load at most 2/3
    return s;
}

// Fills the class lists (all but the hubs', which the plan holds): a
// workgroup reserves room in every list for its LP_FILL vertices at once.
// List c's cursor starts at its first slot; the order of the workgroups'
// pieces does not matter.
constexpr int LP_FILL = LP_BLOCK * 8;

__device__ __forceinline__ int lp_list_of(int32_t d) {  // 0..4, 5 (one wave), 6 (one workgroup), -1: none, or a hub
    if (d <= 0 || d > LP_MID_MAX) return -1;
    if (d > LP_WAVE_MAX) return 6;
    if (d > 64) return 5;
    return d <= 4 ? 0 : 30 - __clz((unsigned)d - 1u);  // 5..8: 1, 9..16: 2, 17..32: 3, 33..64: 4
}

__global__ __launch_bounds__(LP_BLOCK) void k_lp_fill(const int32_t *__restrict__ rp, int64_t V, uint32_t *list,
                                                      uint32_t *cursor) {
    __shared__ uint32_t s_n[7], s_at[7];
    if (threadIdx.x < 7) s_n[threadIdx.x] = 0;
    __syncthreads();
    int c[LP_FILL / LP_BLOCK];
    uint32_t at[LP_FILL / LP_BLOCK];
    const int64_t v0 = (int64_t)blockIdx.x * LP_FILL + threadIdx.x;
#pragma unroll
    for (int i = 0; i < LP_FILL / LP_BLOCK; i++) {
        const int64_t v = v0 + i * LP_BLOCK;
        c[i] = v < V ? lp_list_of(rp[v + 1] - rp[v]) : -1;
        // (ascending inside a wave: the lanes of a list rank themselves, one adds)
        at[i] = 0;
#pragma unroll
        for (int q = 0; q < 7; q++) {
            const unsigned long long m = __ballot(c[i] == q);
            if (c[i] != q) continue;
            const int lead = __ffsll(m) - 1;
            uint32_t b = 0;
            if ((int)(threadIdx.x & 63) == lead) b = atomicAdd(&s_n[q], (uint32_t)__popcll(m));
            at[i] = (uint32_t)__builtin_amdgcn_readlane((int)b, lead) +
                    (uint32_t)__popcll(m & ((1ull << (threadIdx.x & 63)) - 1ull));
        }
    }
    __syncthreads();
    if (threadIdx.x < 7) s_at[threadIdx.x] = s_n[threadIdx.x] ? atomicAdd(&cursor[threadIdx.x], s_n[threadIdx.x]) : 0u;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < LP_FILL / LP_BLOCK; i++)
        if (c[i] >= 0) list[s_at[c[i]] + at[i]] = (uint32_t)(v0 + i * LP_BLOCK);
}

template <class T>
unsigned blocks_for(T n, int b) {
    return (unsigned)std::max<T>(1, (n + b - 1) / b);
}

}  // namespace

namespace gx {

// The class sizes, hubs and hub chunks of a graph, from the host copy of its
// symmetric degrees: worked out by the first state on the graph and kept
// with it.
const LpPlan &lp_plan(gx_graph *g) {
    std::lock_guard<std::mutex> lk(g->lp_mu);
    if (g->lp.made) return g->lp;
    LpPlan p;
    int64_t cnt[LP_CLASSES] = {};
    int64_t acc = 0;
    for (size_t v = 0; v < g->host_symdeg.size(); v++) {
        const int32_t d = g->host_symdeg[v];
        const int c = lp_class_of(d);
        if (c >= 0) cnt[c]++;
        p.nwave += c == 5 && d <= LP_WAVE_MAX;
        if (c == LP_CLASSES - 1) {
            const uint32_t slots = lp_hub_slots(d);
            for (int64_t e = 0; e < d; e += LP_HUB_CHUNK)
                p.chunks.push_back(make_uint4((uint32_t)p.hubs.size(), (uint32_t)(acc + e),
                                              (uint32_t)(acc + std::min<int64_t>(d, e + LP_HUB_CHUNK)), 0u));
            p.hub.push_back(make_uint2((uint32_t)p.tab_slots, slots));
            p.hubs.push_back((uint32_t)v);
            p.tab_slots += slots;
            p.slot_bound += 3 * (int64_t)d + 256;
        }
        acc += d;
    }
    for (int c = 0; c < LP_CLASSES; c++) p.off[c + 1] = p.off[c] + cnt[c];
    p.made = true;
    return g->lp = std::move(p);
}

size_t lp_layout(gx_graph *g, Carver &c, gx_state *s) {
    const int64_t V = g->d.V;
    const LpPlan &p = lp_plan(g);
    std::copy(p.off, p.off + LP_CLASSES + 1, s->lp_off);
    s->lp_nchunks = (int64_t)p.chunks.size();
    s->lp_tab_slots = p.tab_slots;
    s->lp_nwave = p.nwave;
    s->lab[0] = c.take<uint32_t>(V);
    s->lab[1] = c.take<uint32_t>(V);
    s->synced = c.take<uint32_t>(V);
    s->lp_list = c.take<uint32_t>(std::max<int64_t>(1, s->lp_off[LP_CLASSES]));
    const int64_t hubs = s->lp_off[LP_CLASSES] - s->lp_off[LP_CLASSES - 1];
    s->lp_chunks = c.take<uint4>(std::max<int64_t>(1, s->lp_nchunks));
    s->lp_hub = c.take<uint2>(std::max<int64_t>(1, hubs));
    s->lp_tab = c.take<uint2>(std::max<int64_t>(1, s->lp_tab_slots));
    s->lp_best = c.take<unsigned long long>(std::max<int64_t>(1, hubs));
    s->lp_log = c.take<uint32_t>(s->lp_tab_slots + 1);  // [0]: entries, then the slots taken
    s->lp_touch = c.take<uint8_t>(V);
    s->lp_cursor = c.take<uint32_t>(8);
    s->lp_changed = c.take<uint2>(V + g->d.E_sym / LP_CHANGED_CHUNK + 1);
    return c.used;
}

// Initialises the labels to the global ids and builds the class lists.
gx_status lp_init(gx_state *s, hipStream_t hs) {
    gx_graph *g = s->g;
    const DevGraph &d = g->d;
    const LpPlan &p = lp_plan(g);
    const int64_t V = d.V, hubs = (int64_t)p.hubs.size();
    LpCursors at;
    for (int c = 0; c < 6; c++) at.at[c] = (uint32_t)p.off[c];
    at.at[6] = (uint32_t)(p.off[5] + p.nwave);
    hipLaunchKernelGGL(k_lp_init, dim3(blocks_for<int64_t>(V, LP_BLOCK)), dim3(LP_BLOCK), 0, hs, s->lab[0], s->lab[1],
                       s->synced, s->lp_touch, s->lp_best, hubs, d.l2g, V, s->steps, s->lp_cursor, at);
    if (p.tab_slots > 0)
        hipLaunchKernelGGL(k_lp_tab_clear, dim3(blocks_for<int64_t>(p.tab_slots, LP_BLOCK)), dim3(LP_BLOCK), 0, hs,
                           s->lp_tab, p.tab_slots);
    if (V > 0)
        hipLaunchKernelGGL(k_lp_fill, dim3(blocks_for<int64_t>(V, LP_FILL)), dim3(LP_BLOCK), 0, hs, d.sym_rp, V,
                           s->lp_list, s->lp_cursor);
    if (hubs > 0) {
        GX_CHECK_HIP(hipMemcpyAsync(s->lp_list + p.off[6], p.hubs.data(), (size_t)hubs * 4, hipMemcpyHostToDevice, hs), s);
        GX_CHECK_HIP(hipMemcpyAsync(s->lp_chunks, p.chunks.data(), p.chunks.size() * sizeof(uint4),
                                    hipMemcpyHostToDevice, hs), s);
        GX_CHECK_HIP(hipMemcpyAsync(s->lp_hub, p.hub.data(), (size_t)hubs * sizeof(uint2), hipMemcpyHostToDevice, hs), s);
    }
    GX_CHECK_HIP(hipGetLastError(), s);
    return GX_OK;
}

// One superstep: labels lab[k & 1] -> lab[(k + 1) & 1]; the changed vertices
// are counted and listed in `step`, `next` is cleared for the following
// superstep.
void lp_enqueue(gx_state *s, hipStream_t hs, DevStep *step, DevStep *next) {
    const DevGraph &d = s->g->d;
    const int cur = (int)(s->k & 1);
    const int64_t *off = s->lp_off;
    const DevStep *prev = s->steps + ((s->k + STEP_RING - 1) % STEP_RING);
    const LpStep a{d.sym_rp,     d.sym_col,     s->lab[cur], s->lab[cur ^ 1], s->lp_touch,
                   s->lp_changed, step,          prev,        d.E_sym,         s->k == 0};
    if (s->k == 0 && d.sym_ascending) {
        hipLaunchKernelGGL(k_lp_first, dim3(blocks_for<int64_t>(d.V, LP_BLOCK)), dim3(LP_BLOCK), 0, hs, a, d.V, next);
        return;
    }
    const unsigned wide = (unsigned)s->g->num_cus * 8;
    hipLaunchKernelGGL(k_lp_mark, dim3(wide), dim3(LP_BLOCK), 0, hs, a, next, s->lp_log);
    LpRanges r{};
    r.list = s->lp_list;
    for (int c = 0; c < 6; c++) {
        r.off[c] = off[c];
        if (c < 5) r.blk[c + 1] = r.blk[c] + (unsigned)((off[c + 1] - off[c] + 4 * lp_wave_vertices(c) - 1) / (4 * lp_wave_vertices(c)));
    }
    if (r.blk[5] > 0) hipLaunchKernelGGL(k_lp_groups, dim3(r.blk[5]), dim3(LP_BLOCK), 0, hs, a, r);
    // (a workgroup of the mid kernels takes at most LP_BLOCK vertices)
    auto mid = [&](auto kern, const uint32_t *list, int64_t n, int per_wg) {
        if (n > 0)
            hipLaunchKernelGGL(kern, dim3((unsigned)std::max<int64_t>(std::min<int64_t>((n + per_wg - 1) / per_wg, wide),
                                                                      (n + LP_BLOCK - 1) / LP_BLOCK)),
                               dim3(LP_BLOCK), 0, hs, a, list, n);
    };
    mid(k_lp_mid_wave, s->lp_list + off[5], s->lp_nwave, LP_BLOCK / 64);
    mid(k_lp_mid, s->lp_list + off[5] + s->lp_nwave, off[6] - off[5] - s->lp_nwave, 1);
    const int64_t nhub = off[7] - off[6];
    if (nhub > 0) {
        const LpHubs hu{s->lp_list + off[6], s->lp_chunks, s->lp_hub, s->lp_tab, s->lp_best, s->lp_log + 1, s->lp_log};
        hipLaunchKernelGGL(k_lp_hub_count, dim3((unsigned)s->lp_nchunks), dim3(LP_BLOCK), 0, hs, a, hu);
        hipLaunchKernelGGL(k_lp_hub_pick, dim3(std::max(blocks_for<int64_t>(nhub, LP_BLOCK), wide / 4)), dim3(LP_BLOCK), 0,
                           hs, a, hu, nhub);
    }
}

// Vertices an LP superstep computes (those with at least one neighbour).
int64_t lp_active(const gx_state *s) { return s->lp_off[LP_CLASSES]; }

}  // namespace gx
