// Batched lanes: B independent single-source problems over one resident
// graph, carried in a [V x B] state tile (B contiguous per vertex).  The
// evaluation of the paper runs several SSSP sources simultaneously to raise
// the arithmetic intensity (Section "Setup", first footnote); here the lanes
// are independent problems, each equal to its plain solve.
//
// SSSP: per superstep three ordinary launches
//   compaction: every (vertex, 32-lane group) whose lane mask is non-zero
//     and that has out-edges becomes one active entry and its 32 distances
//     are copied to its vertex's slot of the snapshot (Jacobi semantics per
//     lane; a distance changes only when its vertex is active next, so the
//     snapshot then holds every row); one 64-bit atomic per workgroup chunk
//     reserves entries and edge offsets; tiles of equal (entry, edge) work
//     units record where they start.
//   push (small frontiers): 8 threads per work unit handle the unit's 32
//     lanes (4 each, one 16-byte load of the destination's group);
//     improvements are folded by atomicMin per lane (no result awaited: a
//     candidate below a value read during the superstep already proves the
//     lane changes), and the group's improved-lane bits by one atomicOr into
//     the next mask.
//   pull (large frontiers): a lane group takes a run of in-edges, reads each
//     source's whole row and takes the minimum, so a row is written once and
//     without atomics; see k_bs_pull.
//   The host enqueues supersteps in groups and reads the counters back once
//   per group; a superstep without active lanes changes nothing.
// PPR: per superstep three ordinary launches: a pull over equal in-edge tiles
//   (a lane group per tile, batch lanes across the group), rows crossing
//   tiles completed in tile order, and the seeds' rows, which take the
//   teleport and the dangling mass.  Every sum has a fixed order that depends
//   on the graph alone, so a lane's arithmetic is independent of the other
//   lanes and of the launch shape.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <mutex>
#include <string>
#include <tuple>

#include "gx_device.h"
#include "gx_internal.h"
#include "gx_batch.h"

namespace gx {

// ------------------------------------------------------------------ SSSP

template <int BLOCK, int VT>
struct BsShared {
    static constexpr int T = BLOCK * VT;
    static constexpr int NW = BLOCK / 64;
    int32_t own[T];
    uint32_t base[T + 1];
    uint32_t mask[T + 1];
    uint32_t g[T + 1];
    uint32_t srow[T + 1];
    int32_t red[NW];
    unsigned long long cnt[NW];
    uint32_t lane[256];
};

// Compaction of batched superstep k: active (vertex, group) pairs -> entries,
// snapshot rows, tile starts (tiles of `tile` units).  Grid-strided over the
// V*G mask words, CW per thread (1 for a small graph, which then still has a
// workgroup per CU).  Once the units counted reach pull_units
// the superstep pulls and the rest of the entries is not written.  The rows
// are copied by 8 threads each, which also take every lane's smallest active
// distance (for the pull) into the counters.
constexpr int BS_CBLOCK = 256;
constexpr int64_t BS_WIDE_FROM = int64_t(1) << 20;  // mask words

template <int CW>
__global__ __launch_bounds__(BS_CBLOCK) void k_bs_compact(BsArgs a, uint32_t k, uint32_t tile) {
    __shared__ unsigned long long s_scan[BS_CBLOCK / 64];
    __shared__ unsigned long long s_base;
    __shared__ uint32_t s_low[256];
    __shared__ uint32_t s_word[BS_CBLOCK * CW], s_vg[BS_CBLOCK * CW], s_row[BS_CBLOCK * CW];
    const int tid = threadIdx.x;
    const int64_t VG = a.V * (int64_t)a.G;
    const int slot = k & 3;
    const uint32_t *Mc = a.M[k & 1];
    uint32_t *Mn = a.M[(k + 1) & 1];
    if (blockIdx.x == 0 && tid == 0) {
        a.ctl->list[(k + 1) & 3] = 0;
        a.ctl->changed[(k + 1) & 3] = 0;
        if (k > 0 && a.ctl->changed[(k - 1) & 3] == 0 && a.ctl->steps == 0) a.ctl->steps = k;
    }
    if (blockIdx.x == 0) a.ctl->inv_low[(k + 1) & 3][tid] = 0;
    s_low[tid] = INF;
    constexpr int64_t CHUNK = BS_CBLOCK * CW;
    for (int64_t base = (int64_t)blockIdx.x * CHUNK; base < VG; base += (int64_t)gridDim.x * CHUNK) {
        uint32_t word[CW], u[CW], g[CW], row[CW], any = 0;
        int32_t r0[CW], deg[CW];
        const int64_t i0 = base + (int64_t)tid * CW;
#pragma unroll
        for (int j = 0; j < CW; j++) word[j] = 0;
#pragma unroll
        for (int j = 0; j < CW; j++)
            if (i0 + j < VG) {
                word[j] = Mc[i0 + j];
                Mn[i0 + j] = 0u;
            }
#pragma unroll
        for (int j = 0; j < CW; j++) any |= word[j];
        if (!__syncthreads_or(any != 0)) continue;
        unsigned long long mine = 0, total;
        u[0] = VG < (int64_t(1) << 32) ? (uint32_t)i0 / a.G : (uint32_t)(i0 / a.G);
        g[0] = (uint32_t)(i0 - (int64_t)u[0] * a.G);
#pragma unroll
        for (int j = 0; j < CW; j++) {
            if (j > 0) {
                const bool wrap = g[j - 1] + 1 == a.G;
                g[j] = wrap ? 0u : g[j - 1] + 1;
                u[j] = u[j - 1] + (wrap ? 1u : 0u);
            }
            r0[j] = deg[j] = 0;
            row[j] = 0;
            if (word[j]) {
                r0[j] = a.rp[u[j]];
                deg[j] = a.rp[u[j] + 1] - r0[j];
                row[j] = (uint32_t)a.slot[u[j]] * a.G + g[j];
            }
            if (deg[j] > 0) mine += (1ull << 32) | (uint32_t)deg[j];
        }
        const unsigned long long pre = block_excl_scan_u64(mine, &total, s_scan);
        if (tid == 0) s_base = total ? atomicAdd(&a.ctl->list[slot], total) : 0ull;
        uint32_t e = (uint32_t)(pre >> 32);
#pragma unroll
        for (int j = 0; j < CW; j++)
            if (deg[j] > 0) {
                s_word[e] = word[j];
                s_vg[e] = (uint32_t)(i0 + j - base);
                s_row[e++] = row[j];
            }
        __syncthreads();
        const uint32_t n = (uint32_t)(total >> 32) * 8;
        for (uint32_t i = tid; i < n; i += BS_CBLOCK) {
            const uint32_t q = i & 7, w = s_word[i / 8] >> (4 * q);
            const uint64_t vg = (uint64_t)base + s_vg[i / 8];
            const uint64_t v = VG < (int64_t(1) << 32) ? (uint64_t)((uint32_t)vg / a.G) : vg / a.G;
            const uint32_t gg = (uint32_t)(vg - v * a.G);
            const uint4 x = *reinterpret_cast<const uint4 *>(a.D + (size_t)v * a.B + a.l0 + gg * 32 + q * 4);
            a.S[(size_t)s_row[i / 8] * 8 + q] = x;
            const uint32_t xv[4] = {x.x, x.y, x.z, x.w};
            if (a.in_adj)
#pragma unroll
                for (int j = 0; j < 4; j++)
                    if (((w >> j) & 1u) && xv[j] < s_low[gg * 32 + q * 4 + j]) atomicMin(&s_low[gg * 32 + q * 4 + j], xv[j]);
        }
        unsigned long long pos = s_base + pre;
        const bool pulls = (uint32_t)(s_base + total) >= a.pull_units;
        __syncthreads();
        if (pulls) continue;
#pragma unroll
        for (int j = 0; j < CW; j++) {
            if (deg[j] <= 0) continue;
            const uint32_t idx = (uint32_t)(pos >> 32), off = (uint32_t)pos;
            a.list[idx] = make_uint4(off, (uint32_t)(r0[j] - (int32_t)off), word[j], row[j]);
            const uint32_t t0 = (off + tile - 1) / tile, t1 = (off + (uint32_t)deg[j] - 1) / tile;
            for (uint32_t t = t0; t <= t1; t++) a.tile_start[t] = idx;
            pos += (1ull << 32) | (uint32_t)deg[j];
        }
    }
    __syncthreads();
    if (s_low[tid] != INF) {
        uint32_t *p = &a.ctl->inv_low[slot][tid];
        if (~s_low[tid] > *p) atomicMax(p, ~s_low[tid]);  // (a stale read only costs an atomic)
    }
}

// Push of batched superstep k: relax the equal tiles of (entry, edge) work
// units; `it` indexes the per-lane activation counters.
template <int BLOCK, int VT>
__device__ __forceinline__ void bs_relax(const BsArgs &a, uint32_t k, uint32_t it, BsShared<BLOCK, VT> &sh) {
    constexpr int T = BLOCK * VT;
    constexpr int UNITS = BLOCK / 8;
    const int tid = threadIdx.x;
    const int slot = k & 3;
    uint32_t *Mn = a.M[(k + 1) & 1];
    const unsigned long long le = a.ctl->list[slot];
    const uint32_t L = (uint32_t)(le >> 32), EF = (uint32_t)le;
    const uint32_t ntiles = (EF + T - 1) / T;
    unsigned long long changed = 0;
    if (a.lane_cnt)
        for (int q = tid; q < 256; q += BLOCK) sh.lane[q] = 0;
    __syncthreads();
    const int sub = tid & 7;
    // a small frontier has fewer tiles than the grid has workgroups: each tile
    // is then shared by `parts` of them
    constexpr int UB = 4;
    const uint32_t parts = min((uint32_t)(T / (UNITS * UB)), max(1u, gridDim.x / max(1u, ntiles)));
    for (uint32_t tp = blockIdx.x; tp < ntiles * parts; tp += gridDim.x) {
        const uint32_t t = tp / parts, e0 = t * T;
        const int n = (int)min((uint32_t)T, EF - e0);
        const int per = (int)((T / parts + UNITS * UB - 1) / (UNITS * UB)) * (UNITS * UB);
        const int lo = (int)(tp % parts) * per, hi = min(n, lo + per);
        if (lo >= n) continue;
        const uint32_t s0 = a.tile_start[t];
        const uint32_t s1 = (t + 1 < ntiles) ? a.tile_start[t + 1] : L - 1;
        const int m = (int)(s1 - s0) + 1;
        for (int p = tid; p < n; p += BLOCK) sh.own[p] = 0;
        __syncthreads();
        for (int q = tid; q < m; q += BLOCK) {
            uint4 en = a.list[s0 + q];
            sh.base[q] = en.y + e0;
            sh.mask[q] = en.z;
            sh.srow[q] = en.w;
            sh.g[q] = en.w % a.G;
            uint32_t rel = en.x - e0;
            if (q > 0 && rel < (uint32_t)n) sh.own[rel] = q;
        }
        __syncthreads();
        block_max_scan<VT>(sh.own, n, sh.red);
        // UB work units per 8-thread group at a time: their edge loads, then
        // their snapshot and destination loads, then the relaxations, all
        // loads unconditional (units past the tile's end repeat its last
        // unit with no lanes).  The lane minima go out as atomics whose
        // results are not awaited; only the mask atomics return, once.
        for (int p0 = lo + (tid >> 3); p0 < hi; p0 += UNITS * UB) {
            uint2 ed[UB];
            uint32_t my4[UB], gq[UB], sq[UB];
#pragma unroll
            for (int q = 0; q < UB; q++) {
                const int p = min(p0 + q * UNITS, n - 1);
                const int j = sh.own[p];
                sq[q] = sh.srow[j];
                gq[q] = sh.g[j];
                my4[q] = (p0 + q * UNITS < hi) ? (sh.mask[j] >> (sub * 4)) & 15u : 0u;
                ed[q] = a.adj[sh.base[j] + (uint32_t)p];
            }
            uint4 sn[UB], cur[UB];
#pragma unroll
            for (int q = 0; q < UB; q++) {
                sn[q] = a.S[(size_t)sq[q] * 8 + sub];
                cur[q] = *reinterpret_cast<const uint4 *>(a.D + (size_t)ed[q].x * a.B + a.l0 + gq[q] * 32 + sub * 4);
            }
            uint32_t cand[UB][4], word[UB];
#pragma unroll
            for (int q = 0; q < UB; q++) {
                const uint32_t snv[4] = {sn[q].x, sn[q].y, sn[q].z, sn[q].w};
                const uint32_t cv[4] = {cur[q].x, cur[q].y, cur[q].z, cur[q].w};
                uint32_t imp = 0;
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    cand[q][r] = sat_add(snv[r], ed[q].y);
                    // below a value read this superstep: the lane changes
                    if (((my4[q] >> r) & 1u) && cand[q][r] < cv[r]) imp |= 1u << r;
                }
                uint32_t w = imp << (sub * 4);
                w |= __shfl_xor(w, 1, 8);
                w |= __shfl_xor(w, 2, 8);
                w |= __shfl_xor(w, 4, 8);
                word[q] = w;
            }
#pragma unroll
            for (int q = 0; q < UB; q++) {
                const uint32_t imp = (word[q] >> (sub * 4)) & 15u;
                uint32_t *dp = a.D + (size_t)ed[q].x * a.B + a.l0 + gq[q] * 32 + sub * 4;
#pragma unroll
                for (int r = 0; r < 4; r++)
                    if ((imp >> r) & 1u) atomicMin(dp + r, cand[q][r]);
            }
            // The group leader ORs all UB words (a zero word changes nothing)
            // under one branch, so the returns are awaited once.
            if (sub == 0 && (word[0] | word[1] | word[2] | word[3])) {
                static_assert(UB == 4, "the branch above names the UB words");
                uint32_t prev[UB];
#pragma unroll
                for (int q = 0; q < UB; q++) prev[q] = atomicOr(&Mn[(size_t)ed[q].x * a.G + gq[q]], word[q]);
#pragma unroll
                for (int q = 0; q < UB; q++) {
                    const uint32_t nb = word[q] & ~prev[q];
                    changed += __popc(nb);
                    if (a.lane_cnt)
                        for (uint32_t mm = nb; mm; mm &= mm - 1) atomicAdd(&sh.lane[gq[q] * 32 + __ffs(mm) - 1], 1u);
                }
            }
        }
        __syncthreads();
    }
    unsigned long long tot = block_sum<unsigned long long>(changed, sh.cnt);
    if (tid == 0 && tot) atomicAdd(&a.ctl->changed[slot], tot);
    if (a.lane_cnt) {
        __syncthreads();
        for (int q = tid; q < (int)(a.G * 32); q += BLOCK)
            if (sh.lane[q]) atomicAdd(&a.lane_cnt[(size_t)it * a.B + a.l0 + q], sh.lane[q]);
    }
}

template <int BLOCK, int VT>
__global__ __launch_bounds__(BLOCK) void k_bs_relax(BsArgs a, uint32_t k, uint32_t it) {
    __shared__ BsShared<BLOCK, VT> sh;
    const uint32_t units = (uint32_t)a.ctl->list[k & 3];
    if (units > 0 && units < a.pull_units) bs_relax<BLOCK, VT>(a, k, it, sh);
}

// Pull of batched superstep k.  A group of W lanes (W = 32 for one 32-lane
// group, else 64 with LPT lanes per thread) takes the in-edges of a segment
// of a long row or of a pack of short rows, 8 at a time: the rows of the 8
// sources are loaded (by slot, so the rows of the vertices with the most
// out-edges lie together), then folded in turn; an entry names its row.  A
// finished row's improved lanes are stored and their bits, a ballot, become
// its next mask; rows of several segments merge by atomics.  What an inactive
// lane of a source sends was merged before and lowers nothing.  The entries
// of a segment ascend by weight: 64 lanes of it end where none of them can
// still fall, the smallest active distance of each lane plus the weight being
// no smaller than the lane's best (a lane without active vertices needs
// nothing).
//
// Bound by the gathered rows.  R-MAT scale 20, 256 lanes: the first pull of a
// solve takes 2.33 ms (16 M rows of 1 KiB: 7 TB/s), the eight after it 1.73 to
// 0.56 ms.  The solve took 97 ms when every superstep pushed, with an atomic
// per improving lane, in one persistent launch of 8 waves per CU; 14.7 ms now.
template <int W, int LPT>
__global__ __launch_bounds__(256) void k_bs_pull(BsArgs a, uint32_t k, uint32_t it) {
    if ((uint32_t)a.ctl->list[k & 3] < a.pull_units) return;
    constexpr int NG = 64 / W, EB = LPT == 1 ? 16 : 8;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, g = lane / W;
    const uint32_t b0 = (uint32_t)(lane % W), width = a.G * 32;
    uint32_t *Mn = a.M[(k + 1) & 1];
    const uint32_t *S = reinterpret_cast<const uint32_t *>(a.S);
    uint32_t cl[LPT], cnt[LPT], low[LPT];
    bool has[LPT];
#pragma unroll
    for (int i = 0; i < LPT; i++) {
        has[i] = b0 + 64u * i < width;
        cl[i] = min(b0 + 64u * i, width - 1);
        cnt[i] = 0;
        low[i] = has[i] ? ~a.ctl->inv_low[k & 3][cl[i]] : INF;
    }
    const int64_t total = a.nsegs + a.npacks, nwaves = (int64_t)gridDim.x * 4;
    for (int64_t t0 = ((int64_t)blockIdx.x * 4 + wv) * NG; t0 < total; t0 += nwaves * NG) {
        const int64_t t = W == 64 ? (int64_t)__builtin_amdgcn_readfirstlane((int)t0) : t0 + g;
        const bool on = t < total;
        const int64_t tq = on ? t : total - 1;
        const bool seg = tq < a.nsegs;
        const uint4 un = seg ? a.segs[tq] : a.packs[tq - a.nsegs];
        const bool atomic = seg && !(un.w & 0x100u);
        uint32_t row = seg ? un.x : 0xFFFFFFFFu, p = seg ? un.y : un.x;
        const uint32_t end = seg ? un.z : un.y;
        uint32_t acc[LPT], cur[LPT];
#pragma unroll
        for (int i = 0; i < LPT; i++) {
            acc[i] = INF;
            cur[i] = seg ? a.D[(size_t)un.x * a.B + a.l0 + cl[i]] : 0u;
        }
        auto close = [&]() {  // the row's lanes below their value
#pragma unroll
            for (int i = 0; i < LPT; i++) {
                const bool imp = on && has[i] && acc[i] < cur[i];
                const unsigned long long m = __ballot(imp);
                uint32_t *dp = a.D + (size_t)row * a.B + a.l0 + cl[i];
                uint32_t *mp = Mn + (size_t)row * a.G + cl[i] / 32;
                const uint32_t word = (uint32_t)(m >> (lane & 32));
                if (imp) {
                    if (!atomic) {
                        *dp = acc[i];
                        cnt[i]++;
                    } else {
                        atomicMin(dp, acc[i]);
                    }
                }
                if (word) {
                    uint32_t before = 0;
                    if (!atomic) {
                        if ((lane & 31) == 0) *mp = word;
                    } else {
                        if ((lane & 31) == 0) before = atomicOr(mp, word);
                        before = __shfl(before, lane & 32, 64);
                        cnt[i] += ((word & ~before) >> (lane & 31)) & 1u;  // counted by the segment that set it
                    }
                }
            }
        };
        // which of the row's 64-lane slices go on (a short row's all do)
        bool sl[LPT], live = false;
        auto go_on = [&](uint32_t w) {
            live = false;
#pragma unroll
            for (int i = 0; i < LPT; i++) {
                const unsigned long long m = __ballot(min(acc[i], cur[i]) > sat_add(low[i], w));
                sl[i] = on && (W == 64 ? m != 0 : (uint32_t)(m >> (lane & 32)) != 0);
                live |= sl[i];
            }
        };
        if (seg) {
            go_on(un.w & 0xFFu);
        } else {
            live = on;
#pragma unroll
            for (int i = 0; i < LPT; i++) sl[i] = true;
        }
        uint2 q[EB];  // the next entries, loaded a round ahead
#pragma unroll
        for (int j = 0; j < EB; j++) q[j] = a.in_adj[min(p + (uint32_t)j, end - 1)];
        while (W == 64 ? live : __any(live)) {
            if (live) {
                uint32_t tw[EB], s[EB][LPT];
#pragma unroll
                for (int i = 0; i < LPT; i++)
                    if (LPT == 1 || sl[i])
#pragma unroll
                        for (int j = 0; j < EB; j++) s[j][i] = S[(size_t)q[j].x * width + cl[i]];
                p += EB;
#pragma unroll
                for (int j = 0; j < EB; j++) {
                    tw[j] = q[j].y;
                    q[j] = a.in_adj[min(p + (uint32_t)j, end - 1)];
                }
#pragma unroll
                for (int j = 0; j < EB; j++) {
                    const uint32_t r = seg ? row : un.z + (tw[j] >> 8);
                    if (r != row) {  // (an entry past the end repeats the last one: the same row, the same minimum)
                        if (row != 0xFFFFFFFFu) close();
                        row = r;
#pragma unroll
                        for (int i = 0; i < LPT; i++) {
                            acc[i] = INF;
                            cur[i] = a.D[(size_t)row * a.B + a.l0 + cl[i]];
                        }
                    }
#pragma unroll
                    for (int i = 0; i < LPT; i++)
                        if (LPT == 1 || sl[i]) acc[i] = min(acc[i], sat_add(s[j][i], tw[j] & 0xFFu));
                }
                if (p >= end) live = false;
                else if (seg) go_on(tw[EB - 1] & 0xFFu);
            }
        }
        if (row != 0xFFFFFFFFu) close();
    }
    // one add per workgroup to the shared counter; lane_cnt only has to tell
    // the lanes that changed from the others
    __shared__ uint32_t s_sum, s_lane[256];
    if (threadIdx.x == 0) s_sum = 0;
    s_lane[threadIdx.x] = 0;
    __syncthreads();
    uint32_t sum = 0;
#pragma unroll
    for (int i = 0; i < LPT; i++) {
        sum += cnt[i];
        if (has[i] && cnt[i]) s_lane[cl[i]] = 1;
    }
    if (sum) atomicAdd(&s_sum, sum);
    __syncthreads();
    if (threadIdx.x == 0 && s_sum) atomicAdd(&a.ctl->changed[k & 3], (unsigned long long)s_sum);
    if (a.lane_cnt && threadIdx.x < width && s_lane[threadIdx.x])
        a.lane_cnt[(size_t)it * a.B + a.l0 + threadIdx.x] = 1;
}

__global__ __launch_bounds__(256) void k_bs_fill(uint32_t *D, size_t n, uint32_t x) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) D[i] = x;
}

// Lane b of the pass starting at lane l0: D[src][b] = 0 and its mask bit.
__global__ __launch_bounds__(256) void k_bs_sources(uint32_t *D, uint32_t *M0, const int32_t *src, uint32_t B,
                                                    uint32_t l0, uint32_t width, uint32_t G) {
    uint32_t q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= width) return;
    int32_t s = src[l0 + q];
    if (s < 0) return;
    D[(size_t)s * B + l0 + q] = 0u;
    atomicOr(&M0[(size_t)s * G + q / 32], 1u << (q & 31));
}

// Serving: re-initialise lane b (column of D over all V, its masks) and seed it.
__global__ __launch_bounds__(256) void k_bs_lane_reset(uint32_t *D, uint32_t *S, const int32_t *slot, uint32_t *Mc,
                                                       uint32_t *Mn, int64_t V, uint32_t B, uint32_t G, uint32_t lane,
                                                       int32_t src) {
    const uint32_t bit = 1u << (lane & 31), g = lane / 32;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < V; v += (int64_t)gridDim.x * blockDim.x) {
        D[(size_t)v * B + lane] = (v == src) ? 0u : INF;
        S[(size_t)slot[v] * G * 32 + lane] = INF;  // (the source's is written when it is compacted)
        uint32_t w = Mc[(size_t)v * G + g];
        uint32_t want = (v == src) ? (w | bit) : (w & ~bit);
        if (want != w) Mc[(size_t)v * G + g] = want;
        uint32_t w2 = Mn[(size_t)v * G + g];
        if (w2 & bit) Mn[(size_t)v * G + g] = w2 & ~bit;
    }
}

// ------------------------------------------------------------------ PPR
//
// x' = d * sum of contributions, plus (1 - d) + d * D at the lane's seed, D =
// the lane's dangling mass.  Rows without in-edges keep the 0 they start with
// (a seed among them is the seed kernel's), so only rows with in-edges are
// visited.  A vertex without out-edges keeps its rank in its contribution
// slot, which no edge reads, so D is one more row whose in-edges are the
// dangling vertices.  Ranks are written only in a lane's last superstep.

// Per-lane constants of one PPR superstep: lane b is live when it is inside
// the processed width, holds a query and has not reached its end superstep (a
// finished lane is frozen).
template <int LPT>
struct PprLanes {
    uint32_t bl[LPT];  // load column (clamped into the processed width)
    bool live[LPT], last[LPT];
    int32_t seed[LPT];
    __device__ PprLanes(const BpArgs &a, uint32_t k, uint32_t b0) {
#pragma unroll
        for (int i = 0; i < LPT; i++) {
            const uint32_t b = b0 + 64u * i;
            bl[i] = min(b, a.Bw - 1);
            seed[i] = b < a.Bw ? a.seed[b] : -1;
            const uint32_t end = a.end && b < a.Bw ? (uint32_t)a.end[b] : a.last;
            live[i] = seed[i] >= 0 && (int32_t)(end - k) > 0;
            last[i] = end == k + 1;
        }
    }
};

// A finished row sum: the contribution, the rank if it is the lane's last,
// and the sum itself where the seed kernel goes on with it.
template <int LPT>
__device__ __forceinline__ void ppr_apply(const BpArgs &a, int32_t r, int32_t sl, int od, const double (&acc)[LPT],
                                          const PprLanes<LPT> &L, float *__restrict__ c_out, uint32_t b0) {
#pragma unroll
    for (int i = 0; i < LPT; i++) {
        if (!L.live[i]) continue;
        const uint32_t b = b0 + 64u * i;
        const float xn = (float)((double)a.d * acc[i]);
        c_out[(size_t)(uint32_t)sl * a.B + b] = od > 0 ? xn / (float)od : xn;
        if (L.last[i]) a.x[(size_t)r * a.B + b] = xn;
        if (L.seed[i] == r) a.seed_acc[b] = acc[i];
    }
}

// Pull of superstep k.  A group of W lanes (W = 64 for more than 32 lanes,
// with LPT lanes per thread) streams one tile of consecutive in-edges; the
// wave holds 64 / W tiles.  Edges come 16 at a time: their contribution rows
// are all loaded before any is added, whatever rows they belong to, and after
// each add one bit says whether the row ends there.  The ending rows' ids and
// out-degrees are staged in LDS, 64 edges at a time.  The first sum of a
// tile may finish a row begun in an earlier tile (head), the last may go on
// in the next one (tail).  Tiles of dangling vertices come first.
//
// Bound by the gathered contribution rows.  R-MAT scale 20, 64 lanes (16 M
// edges, 4.1 GB gathered per superstep): one wave per 256-edge tile that
// also closed every empty row, walked the 16 loaded rows once per ending row
// and wrote ranks every superstep took 2360 us (2500 us with the other three
// launches); this one takes 520 us (555 us with the other two), 7.9 TB/s of
// gathered rows.  Contributions are stored by slot: by vertex number the hubs
// of R-MAT (numbers with few bits set) lay power-of-two strides apart and the
// superstep took 680 us, and with 256 lanes 3.05 ms where it takes 2.16 now.
__device__ __forceinline__ double *bp_partial(double *p, int64_t t, uint32_t B, uint32_t b) { return p + t * B + b; }

template <int W, int LPT>
__global__ __launch_bounds__(256) void k_bp_pull(BpArgs a, uint32_t k) {
    constexpr int NG = 64 / W, EB = 16;
    __shared__ int2 s_nz[4][NG][64];
    __shared__ int32_t s_sl[4][NG][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, g = lane / W;
    const uint32_t b0 = (uint32_t)(lane % W);
    const float *__restrict__ c_in = a.c[k & 1];
    float *__restrict__ c_out = a.c[(k + 1) & 1];
    const PprLanes<LPT> L(a, k, b0);
    const int64_t total = a.ndtiles + a.ntiles;
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    for (int64_t t0 = ((int64_t)blockIdx.x * 4 + wv) * NG; t0 < total; t0 += nwaves * NG) {
        const int64_t tt = W == 64 ? (int64_t)__builtin_amdgcn_readfirstlane((int)t0) : t0 + g;
        const bool on = W == 64 || tt < total;
        const int64_t tq = on ? tt : total - 1;
        const bool dng = tq < a.ndtiles;
        const int64_t t = dng ? tq : tq - a.ndtiles;
        const int tile = dng ? a.dtile : a.tile;
        const int64_t e0 = t * tile;
        const int n = (int)min((int64_t)tile, (dng ? a.n_dang : a.E) - e0);
        const int32_t *__restrict__ ids = (dng ? a.dang : a.src) + e0;
        int32_t ord = dng ? 0 : a.tile_nz[t];
        bool head = !dng && e0 > 0 && !((a.row_last[(e0 - 1) >> 6] >> ((e0 - 1) & 63)) & 1ull);
        bool open = true;  // the sum in acc has not been written
        double acc[LPT];
#pragma unroll
        for (int i = 0; i < LPT; i++) acc[i] = 0.0;
        for (int w0 = 0; W == 64 ? w0 < n : __any(w0 < n); w0 += 64) {
            const bool in = w0 < n;
            const uint64_t m = in && !dng ? a.row_last[(e0 + w0) >> 6] : 0ull;
            const int ends = __popcll(m);
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int q = 0; q < 64; q += W)
                if (q + (int)b0 < ends) {
                    s_nz[wv][g][q + b0] = a.nz[ord + q + (int)b0];
                    s_sl[wv][g][q + b0] = a.nz_slot[ord + q + (int)b0];
                }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            int idx = 0;
#pragma unroll 1
            for (int c0 = 0; c0 < 64; c0 += EB) {
                const int p0 = w0 + c0;
                if (W == 64 ? p0 >= n : !__any(p0 < n)) break;
                const bool have = p0 < n;
                const int4 *i4 = reinterpret_cast<const int4 *>(ids + (have ? p0 : 0));
                int32_t u[EB];
#pragma unroll
                for (int q = 0; q < EB / 4; q++) {
                    const int4 v = i4[q];
                    u[4 * q] = v.x, u[4 * q + 1] = v.y, u[4 * q + 2] = v.z, u[4 * q + 3] = v.w;
                }
                float v[EB][LPT];
#pragma unroll
                for (int j = 0; j < EB; j++) {
                    const int32_t uj = p0 + j < n ? u[j] : 0;
                    const float *row = c_in + (size_t)(uint32_t)uj * a.B;
#pragma unroll
                    for (int i = 0; i < LPT; i++) v[j][i] = row[L.bl[i]];
                }
                const uint32_t mm = (uint32_t)(m >> c0) & 0xFFFFu;
#pragma unroll
                for (int j = 0; j < EB; j++) {
                    const bool add = p0 + j < n;
#pragma unroll
                    for (int i = 0; i < LPT; i++) acc[i] += add ? (double)v[j][i] : 0.0;
                    if ((mm >> j) & 1u) {  // the row ends with this edge
                        const int2 rw = s_nz[wv][g][idx];
                        const int32_t sl = s_sl[wv][g][idx++];
                        if (head) {
                            head = false;
                            if (on)
#pragma unroll
                                for (int i = 0; i < LPT; i++)
                                    if (b0 + 64u * i < a.Bw) *bp_partial(a.head, t, a.B, b0 + 64u * i) = acc[i];
                        } else if (on) {
                            ppr_apply<LPT>(a, rw.x, sl, rw.y, acc, L, c_out, b0);
                        }
#pragma unroll
                        for (int i = 0; i < LPT; i++) acc[i] = 0.0;
                    }
                }
            }
            ord += ends;
            if (in && !dng && n - w0 <= 64) open = !((m >> (n - w0 - 1)) & 1ull);
        }
        if (on && open) {
            double *p = dng ? a.dpart : head ? a.head : a.tailp;
#pragma unroll
            for (int i = 0; i < LPT; i++)
                if (b0 + 64u * i < a.Bw) *bp_partial(p, t, a.B, b0 + 64u * i) = acc[i];
        }
    }
}

// s plus p[i * stride] over i = 0 .. n-1 in index order; the loads go out AT
// at a time, the adds stay in order.
template <int AT>
__device__ __forceinline__ double ordered_sum(double s, const double *p, int64_t stride, int64_t n) {
    for (int64_t i0 = 0; i0 < n; i0 += AT) {
        double v[AT];
#pragma unroll
        for (int j = 0; j < AT; j++) v[j] = p[std::min<int64_t>(i0 + j, n - 1) * stride];
#pragma unroll
        for (int j = 0; j < AT; j++)
            if (i0 + j < n) s += v[j];
    }
    return s;
}

// The sums of p[i * stride + column] over n partials, cut into ROWS_PIECES
// contiguous pieces that are summed by one wave each and added in order; the
// 64 columns start at `col`.  Valid in the first wave.
__device__ __forceinline__ double pieces_sum(double s, const double *p, uint32_t B, uint32_t col, uint32_t Bw, int64_t n,
                                             double (*s_p)[64]) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const uint32_t b = col + (uint32_t)lane;
    const int64_t lo = n * wv / ROWS_PIECES, hi = n * (wv + 1) / ROWS_PIECES;
    __syncthreads();
    s_p[wv][lane] = b < Bw ? ordered_sum<16>(0.0, p + lo * B + b, B, hi - lo) : 0.0;
    __syncthreads();
    if (wv == 0)
        for (int i = 0; i < ROWS_PIECES; i++) s += s_p[i][lane];
    return s;
}

// Rows crossing tiles: the first tile's tail and the later tiles' heads in
// tile order.  One workgroup per long row, a lane group per other row, with
// 16 loads in flight for the rows of several tiles (the chain of loads bounds
// the kernel: 100003 vertices, 1.6 M edges, 5 lanes: 9.1 us with 4
// for all rows, 7.6 us so).
constexpr int BP_FIX_BLOCK = 64 * ROWS_PIECES;

template <int W, int LPT>
__global__ __launch_bounds__(BP_FIX_BLOCK) void k_bp_fix(BpArgs a, uint32_t k) {
    __shared__ double s_p[ROWS_PIECES][64];
    const int lane = threadIdx.x & 63;
    float *c_out = a.c[(k + 1) & 1];
    if ((int)blockIdx.x < a.n_cross_long) {
        const int4 q = a.cross[blockIdx.x];
        const int32_t sl = a.slot[q.x];
        const PprLanes<LPT> L(a, k, (uint32_t)lane);
        double acc[LPT];
#pragma unroll
        for (int i = 0; i < LPT; i++) {
            const uint32_t b = (uint32_t)lane + 64u * i;
            const double s = b < a.Bw ? a.tailp[(int64_t)q.z * a.B + b] : 0.0;
            acc[i] = pieces_sum(s, a.head + (int64_t)(q.z + 1) * a.B, a.B, 64u * i, a.Bw, q.w - q.z, s_p);
        }
        if (threadIdx.x < 64) ppr_apply<LPT>(a, q.x, sl, q.y, acc, L, c_out, (uint32_t)lane);
        return;
    }
    const uint32_t b0 = (uint32_t)(lane % W);
    const PprLanes<LPT> L(a, k, b0);
    const int groups = BP_FIX_BLOCK / W;
    for (int64_t j = a.n_cross_long + (int64_t)(blockIdx.x - a.n_cross_long) * groups + threadIdx.x / W; j < a.n_cross;
         j += (int64_t)(gridDim.x - a.n_cross_long) * groups) {
        const int4 q = a.cross[j];
        const int32_t sl = a.slot[q.x];
        double acc[LPT];
#pragma unroll
        for (int i = 0; i < LPT; i++) {
            const uint32_t b = b0 + 64u * i;
            acc[i] = 0.0;
            if (b >= a.Bw) continue;
            const double s = a.tailp[(int64_t)q.z * a.B + b];
            const double *p = a.head + (int64_t)(q.z + 1) * a.B + b;
            acc[i] = j < a.n_cross_wide ? ordered_sum<16>(s, p, a.B, q.w - q.z) : ordered_sum<ROWS_MID>(s, p, a.B, q.w - q.z);
        }
        ppr_apply<LPT>(a, q.x, sl, q.y, acc, L, c_out, b0);
    }
}

// The lanes' dangling mass and their seeds' rows (a workgroup per 64 lanes).
__global__ __launch_bounds__(BP_FIX_BLOCK) void k_bp_seed(BpArgs a, uint32_t k) {
    __shared__ double s_p[ROWS_PIECES][64];
    const uint32_t b = blockIdx.x * 64 + (threadIdx.x & 63);
    double D = pieces_sum(0.0, a.dpart, a.B, blockIdx.x * 64, a.Bw, a.ndtiles, s_p);
    if (threadIdx.x >= 64 || b >= a.Bw) return;
    const int32_t r = a.seed[b];
    const uint32_t end = a.end ? (uint32_t)a.end[b] : a.last;
    if (r < 0 || (int32_t)(end - k) <= 0) return;
    const int od = a.outdeg[r];
    const size_t at = (size_t)r * a.B + b, at_c = (size_t)(uint32_t)a.slot[r] * a.B + b;
    const bool no_in = a.in_rp[r + 1] == a.in_rp[r];
    if (od == 0 && no_in) D += (double)a.c[k & 1][at_c];  // a seed that no list of dangling vertices holds
    const double v = (double)a.d * (no_in ? 0.0 : a.seed_acc[b]) + ((1.0 - (double)a.d) + (double)a.d * D);
    const float xn = (float)v;
    a.c[(k + 1) & 1][at_c] = od > 0 ? xn / (float)od : xn;
    if (end == k + 1) a.x[at] = xn;
}

// Superstep 0: ranks e_seed (in the contributions; in x too if there are no
// supersteps), 0 in every row no superstep writes.
__global__ __launch_bounds__(256) void k_bp_init(float *x, float *c0, float *c1, const int32_t *seed,
                                                 const int32_t *in_rp, const int32_t *outdeg, const int32_t *slot,
                                                 int64_t V, uint32_t B, uint32_t iters) {
    const size_t n = (size_t)V * B;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const int64_t v = (int64_t)(i / B);
        const uint32_t b = (uint32_t)(i % B);
        const bool here = seed[b] == v;
        const int od = outdeg[v];
        const size_t at = (size_t)(uint32_t)slot[v] * B + b;
        c0[at] = !here ? 0.0f : od > 0 ? 1.0f / (float)od : 1.0f;
        if (iters == 0 || in_rp[v + 1] == in_rp[v]) {
            c1[at] = 0.0f;
            x[i] = here && iters == 0 ? 1.0f : 0.0f;
        }
    }
}

// Serving: lane b restarts from its new seed.  The other buffer and x hold
// this lane's old values: rows with in-edges are rewritten before they are
// read, so only the old seed's (perhaps without in-edges) are cleared.
__global__ __launch_bounds__(256) void k_bp_lane_reset(float *x, float *c, float *c_other, double *seed_acc,
                                                       const int32_t *outdeg, const int32_t *slot, int64_t V,
                                                       uint32_t B, uint32_t lane, int32_t seed, int32_t old) {
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < V; v += (int64_t)gridDim.x * blockDim.x) {
        const int od = outdeg[v];
        c[(size_t)(uint32_t)slot[v] * B + lane] = v != seed ? 0.0f : od > 0 ? 1.0f / (float)od : 1.0f;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        seed_acc[lane] = 0.0;
        if (old >= 0) c_other[(size_t)(uint32_t)slot[old] * B + lane] = x[(size_t)old * B + lane] = 0.0f;
    }
}

// Gathers lane b of a [V x B] tile into a contiguous vector.
__global__ __launch_bounds__(256) void k_lane_extract(const uint32_t *tile, int64_t V, uint32_t B, uint32_t lane,
                                                      uint32_t *out) {
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < V; v += (int64_t)gridDim.x * blockDim.x)
        out[v] = tile[(size_t)v * B + lane];
}

// ------------------------------------------------------------------ host

const BsVariant *bs_variants(int *n) {
    static const BsVariant v[] = {
        {256, 4, (const void *)k_bs_relax<256, 4>},  {256, 8, (const void *)k_bs_relax<256, 8>},
        {512, 4, (const void *)k_bs_relax<512, 4>},  {512, 8, (const void *)k_bs_relax<512, 8>},
        {1024, 2, (const void *)k_bs_relax<1024, 2>}, {1024, 4, (const void *)k_bs_relax<1024, 4>},
    };
    static_assert(BS_MAX_TILE >= 1024 * 4 && BS_MAX_TILE >= 512 * 8, "the largest tile above");
    *n = (int)(sizeof v / sizeof v[0]);
    return v;
}

void bs_layout(const DevGraph &d, uint32_t B, Carver &c, BsWork *w) {
    const uint32_t G = B / 32;
    const int64_t VG = d.V * (int64_t)G;
    w->M[0] = c.take<uint32_t>(VG);
    w->M[1] = c.take<uint32_t>(VG);
    w->list = c.take<uint4>(VG);
    w->S = c.take<uint4>(VG * 8);
    w->tile_start = c.take<uint32_t>((d.E * (int64_t)G) / BS_MIN_TILE + 2);
    w->ctl = c.take<BsCtl>(1);
    w->src = c.take<int32_t>(B);
}

void bp_layout(const DevGraph &d, uint32_t B, Carver &c, BpWork *w) {
    const int64_t nt = std::max<int64_t>(1, d.bp_rows.n);
    w->c[0] = c.take<float>((size_t)d.V * B);
    w->c[1] = c.take<float>((size_t)d.V * B);
    w->head = c.take<double>(nt * B);
    w->tailp = c.take<double>(nt * B);
    w->dpart = c.take<double>((size_t)ROWS_DANGLING * B);
    w->seed_acc = c.take<double>(B);
    w->seed = c.take<int32_t>(2 * (size_t)B);  // seeds, then per-lane end supersteps
    w->end = w->seed + B;
}

BpArgs bp_args_for(const DevGraph &d, const BpWork &w, float *x, uint32_t B, float damping) {
    BpArgs a{};
    a.src = d.pr_src;
    a.nz = d.nz;
    a.nz_slot = d.nz_slot;
    a.slot = d.slot;
    a.row_last = d.row_last;
    a.tile_nz = d.bp_rows.tile_nz;
    a.cross = d.bp_rows.cross;
    a.dang = d.dang;
    a.in_rp = d.in_rp;
    a.outdeg = d.outdeg;
    a.n_nz = d.n_nz;
    a.tile = (int32_t)d.bp_rows.T;
    a.ntiles = d.bp_rows.n;
    a.E = d.E;
    a.n_dang = d.n_dang;
    // (few tiles of dangling vertices: their partials are added by one workgroup)
    a.dtile = (int32_t)std::max<int64_t>(a.tile, ((d.n_dang + ROWS_DANGLING - 1) / ROWS_DANGLING + 63) / 64 * 64);
    a.ndtiles = (int32_t)((d.n_dang + a.dtile - 1) / a.dtile);
    a.n_cross = d.bp_rows.n_cross;
    a.n_cross_long = d.bp_rows.n_long;
    a.n_cross_wide = d.bp_rows.n_long + d.bp_rows.n_mid;
    a.B = B;
    a.Bw = B;
    a.d = damping;
    a.seed = w.seed;
    a.x = x;
    a.c[0] = w.c[0];
    a.c[1] = w.c[1];
    a.head = w.head;
    a.tailp = w.tailp;
    a.dpart = w.dpart;
    a.seed_acc = w.seed_acc;
    return a;
}

// A superstep pulls when its units are at least 1 / BS_PULL_PART of all
// (edge, group) pairs.  With 1/3, 1/6 and 1/12: 32 lanes, 50000 vertices 714, 720,
// 778 us; 256 lanes, R-MAT scale 20 15.4, 14.8, 15.2 ms; scale 16 2.17, 2.00, 2.01 ms;
// 64 lanes, scale 20 6.40, 6.40, 7.20 ms; uniform of 4 M edges, 256 lanes 13.8, 14.0,
// 14.5 ms, 32 lanes 3.40, 3.46, 3.54; a 300 x 300 grid 24.6, 25.1, 25.6 ms.
constexpr int64_t BS_PULL_PART = 6;

BsArgs bs_args_for(const DevGraph &d, const BsWork &w, uint32_t *D, uint32_t B, uint32_t l0, uint32_t G) {
    BsArgs a{};
    a.rp = d.out_rp;
    a.adj = d.out_adj;
    a.in_adj = d.in_adj;
    a.segs = d.pull_segs;
    a.packs = d.packs;
    a.slot = d.slot;
    a.nsegs = d.pull_nsegs;
    a.npacks = d.n_packs;
    a.pull_units = d.in_adj ? (uint32_t)std::min<int64_t>(0xFFFFFFFE, d.E * (int64_t)G / BS_PULL_PART + 1) : 0xFFFFFFFFu;
    a.V = d.V;
    a.B = B;
    a.l0 = l0;
    a.G = G;
    a.D = D;
    a.M[0] = w.M[0];
    a.M[1] = w.M[1];
    a.list = w.list;
    a.S = w.S;
    a.tile_start = w.tile_start;
    a.ctl = w.ctl;
    return a;
}

}  // namespace gx

using namespace gx;

static gx_status check_batch(const gx_graph *g, int32_t algo, uint32_t B) {
    GX_REQUIRE(g, GX_EINVAL, "graph is NULL");
    GX_REQUIRE(!g->dev_error, GX_EDEVICE, "sticky device error on the graph");
    GX_REQUIRE(algo == GX_SSSP || algo == GX_PPR, GX_EINVAL, "batched algo must be GX_SSSP or GX_PPR");
    GX_REQUIRE(B >= 1 && B <= 256, GX_EINVAL, "B=%u out of [1,256]", B);
    if (algo == GX_SSSP) {
        GX_REQUIRE(B % 32 == 0, GX_EINVAL, "SSSP lanes must be a multiple of 32 (B=%u)", B);
        GX_REQUIRE(g->needs & GX_NEED_OUT, GX_EINVAL, "batched SSSP needs GX_NEED_OUT");
    } else {
        GX_REQUIRE(g->needs & GX_NEED_IN, GX_EINVAL, "batched PPR needs GX_NEED_IN");
    }
    return GX_OK;
}

extern "C" gx_status gx_batch_bytes(const gx_graph *g, int32_t algo, uint32_t B, size_t *bytes) {
    clear_error();
    GX_REQUIRE(bytes, GX_EINVAL, "bytes is NULL");
    gx_status st = check_batch(g, algo, B);
    if (st != GX_OK) return st;
    Carver c(nullptr, 0);
    if (algo == GX_SSSP) {
        BsWork w;
        bs_layout(g->d, B, c, &w);
    } else {
        BpWork w;
        bp_layout(g->d, B, c, &w);
    }
    *bytes = c.used;
    return GX_OK;
}

namespace gx {

// Runs SSSP lanes with one tuning; returns GX_OK / error.  out: [V x B] u32.
gx_status run_bsssp(gx_graph *g, const int32_t *dev_src, uint32_t B, BsWork &w, uint32_t *D, const gx_tune &tn,
                    hipStream_t s, int64_t *supersteps) {
    const DevGraph &d = g->d;
    int nv = 0;
    const BsVariant *vars = bs_variants(&nv);
    const BsVariant *var = nullptr;
    for (int i = 0; i < nv; i++)
        if (vars[i].block == tn.block && vars[i].block * vars[i].vt == tn.tile) var = &vars[i];
    GX_REQUIRE(var, GX_EINVAL, "unsupported tuning block=%u tile=%u", tn.block, tn.tile);
    GX_REQUIRE(tn.width % 32 == 0 && tn.width >= 32 && B % tn.width == 0, GX_EINVAL, "width %u invalid for B=%u",
               tn.width, B);
    const size_t n = (size_t)d.V * B;
    hipLaunchKernelGGL(k_bs_fill, dim3(std::min<size_t>(4096, (n + 255) / 256 + 1)), dim3(256), 0, s, D, n, INF);
    int64_t steps_max = 0;
    const uint32_t width = bs_pass_width(d.E, tn.width);
    for (uint32_t l0 = 0; l0 < B; l0 += width) {
        const uint32_t G = width / 32;
        GX_CHECK_HIP(hipMemsetAsync(w.M[0], 0, (size_t)d.V * G * 4, s), g);
        GX_CHECK_HIP(hipMemsetAsync(w.M[1], 0, (size_t)d.V * G * 4, s), g);
        GX_CHECK_HIP(hipMemsetAsync(w.ctl, 0, sizeof(BsCtl), s), g);
        const size_t ns = (size_t)d.V * width;
        hipLaunchKernelGGL(k_bs_fill, dim3(std::min<size_t>(4096, (ns + 255) / 256 + 1)), dim3(256), 0, s,
                           reinterpret_cast<uint32_t *>(w.S), ns, INF);
        hipLaunchKernelGGL(k_bs_sources, dim3((width + 255) / 256), dim3(256), 0, s, D, w.M[0], dev_src, B, l0, width,
                           G);
        const BsArgs a = bs_args_for(d, w, D, B, l0, G);
        // supersteps in groups, one readback each (one past the end costs less
        // than the wait for a readback: groups of 6 and 6, 12 and 6, 20 and 12 take 535,
        // 500, 450 us for 32 lanes on R-MAT scale 12 and 4.73, 4.71, 4.60 ms for 256 on
        // scale 18)
        BsCtl ctl{};
        for (uint32_t k = 0, n = 12; ctl.steps == 0; n = 6) {
            for (const uint32_t to = k + n; k < to; k++)
                GX_CHECK_HIP(bs_launch_superstep(a, k, 0, *var, (int)tn.grid, g->num_cus, s), g);
            GX_CHECK_HIP(hipMemcpyAsync(&ctl, w.ctl, sizeof ctl, hipMemcpyDeviceToHost, s), g);
            GX_CHECK_HIP(hipStreamSynchronize(s), g);
            if (ctl.steps == 0 && ctl.changed[(k - 1) & 3] == 0) ctl.steps = k;
        }
        steps_max = std::max<int64_t>(steps_max, ctl.steps);
    }
    if (supersteps) *supersteps = steps_max;
    return GX_OK;
}

gx_status run_bppr(gx_graph *g, const int32_t *dev_seed, uint32_t B, BpWork &w, float d_, uint32_t iters,
                   float *out, hipStream_t s, int grid_want) {
    const DevGraph &d = g->d;
    if (dev_seed != w.seed)
        GX_CHECK_HIP(hipMemcpyAsync(w.seed, dev_seed, B * 4, hipMemcpyDeviceToDevice, s), g);
    const size_t n = (size_t)d.V * B;
    hipLaunchKernelGGL(k_bp_init, dim3((unsigned)std::min<size_t>(8192, (n + 255) / 256 + 1)), dim3(256), 0, s, out,
                       w.c[0], w.c[1], w.seed, d.in_rp, d.outdeg, d.slot, d.V, B, iters);
    BpArgs a = bp_args_for(d, w, out, B, d_);
    a.last = iters;
    // ordinary launches (measured faster than one persistent kernel with grid
    // barriers: each phase then runs at its own full occupancy)
    const int grid = grid_want > 0 ? grid_want : 2 * g->num_cus;
    for (uint32_t k = 0; k < iters; k++) GX_CHECK_HIP(bp_launch_superstep(a, k, grid, s), g);
    GX_CHECK_HIP(hipGetLastError(), g);
    GX_CHECK_HIP(hipStreamSynchronize(s), g);
    return GX_OK;
}

// ---- launchers of the ordinary-launch phases (serving)

template <int W, int LPT>
static void bs_launch_pull(const BsArgs &a, uint32_t k, uint32_t it, int cus, hipStream_t s) {
    const int64_t waves = (a.nsegs + a.npacks + 64 / W - 1) / (64 / W);
    const int64_t most = (int64_t)cus * occupancy_per_cu((const void *)k_bs_pull<W, LPT>, 256);
    hipLaunchKernelGGL((k_bs_pull<W, LPT>), dim3((unsigned)std::min(most, (waves + 3) / 4)), dim3(256), 0, s, a, k, it);
}

hipError_t bs_launch_superstep(const BsArgs &a, uint32_t k, uint32_t it, const BsVariant &v, int grid, int cus,
                               hipStream_t s) {
    const int64_t words = a.V * (int64_t)a.G;
    const bool wide = words >= BS_WIDE_FROM;
    const int64_t chunk = BS_CBLOCK * (wide ? 4 : 1);
    hipLaunchKernelGGL(wide ? k_bs_compact<4> : k_bs_compact<1>,
                       dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>(8 * (int64_t)cus, (words + chunk - 1) / chunk))),
                       dim3(BS_CBLOCK), 0, s, a, k, v.block * v.vt);
    const int g = grid > 0 ? grid : cus * occupancy_per_cu(v.fn, (int)v.block);
    BsArgs arg = a;
    void *params[] = {&arg, &k, &it};
    const hipError_t e = hipLaunchKernel(v.fn, dim3((unsigned)g), dim3(v.block), params, 0, s);
    if (e != hipSuccess) return e;
    if (a.in_adj && a.nsegs + a.npacks > 0) {
        if (a.G == 1) bs_launch_pull<32, 1>(a, k, it, cus, s);
        else if (a.G == 2) bs_launch_pull<64, 1>(a, k, it, cus, s);
        else if (a.G <= 4) bs_launch_pull<64, 2>(a, k, it, cus, s);
        else if (a.G <= 6) bs_launch_pull<64, 3>(a, k, it, cus, s);
        else bs_launch_pull<64, 4>(a, k, it, cus, s);
    }
    return hipGetLastError();
}

template <int W, int LPT>
static void bp_launch(const BpArgs &a, uint32_t k, int grid, int cus, hipStream_t s) {
    const int64_t waves = (a.ndtiles + a.ntiles + 64 / W - 1) / (64 / W);
    // the pull keeps its row gathers in flight from every wave the CUs hold
    const int64_t most = std::max(grid, cus * occupancy_per_cu((const void *)k_bp_pull<W, LPT>, 256));
    if (waves > 0)
        hipLaunchKernelGGL((k_bp_pull<W, LPT>), dim3((unsigned)std::min<int64_t>(most, (waves + 3) / 4)), dim3(256), 0, s,
                           a, k);
    const int64_t few = a.n_cross - a.n_cross_long, per = BP_FIX_BLOCK / W;
    const int64_t blocks = std::min<int64_t>(4 * (int64_t)grid, (few + per - 1) / per);
    if (a.n_cross > 0)
        hipLaunchKernelGGL((k_bp_fix<W, LPT>), dim3((unsigned)(a.n_cross_long + blocks)), dim3(BP_FIX_BLOCK), 0, s, a, k);
}

// Lane groups as narrow as the processed width allows: 5 lanes on a ragged
// scale-17 graph (1.5 M edges) take 33 us a superstep, 157 us when a wave took
// one tile whatever the width.
hipError_t bp_launch_superstep(const BpArgs &a, uint32_t k, int grid, hipStream_t s) {
    int dev = 0;
    (void)hipGetDevice(&dev);
    const int cus = device_cus(dev);
    if (a.Bw <= 8) bp_launch<8, 1>(a, k, grid, cus, s);
    else if (a.Bw <= 16) bp_launch<16, 1>(a, k, grid, cus, s);
    else if (a.Bw <= 32) bp_launch<32, 1>(a, k, grid, cus, s);
    else if (a.Bw <= 64) bp_launch<64, 1>(a, k, grid, cus, s);
    else if (a.Bw <= 128) bp_launch<64, 2>(a, k, grid, cus, s);
    else if (a.Bw <= 192) bp_launch<64, 3>(a, k, grid, cus, s);
    else bp_launch<64, 4>(a, k, grid, cus, s);
    hipLaunchKernelGGL(k_bp_seed, dim3((a.Bw + 63) / 64), dim3(BP_FIX_BLOCK), 0, s, a, k);
    return hipGetLastError();
}

hipError_t bs_lane_reset(const BsArgs &a, uint32_t k, uint32_t lane, int32_t src, hipStream_t s) {
    unsigned nb = (unsigned)std::min<int64_t>(2048, (a.V + 255) / 256 + 1);
    hipLaunchKernelGGL(k_bs_lane_reset, dim3(nb), dim3(256), 0, s, a.D, reinterpret_cast<uint32_t *>(a.S), a.slot,
                       a.M[k & 1], a.M[(k + 1) & 1], a.V, a.B, a.G, lane, src);
    return hipGetLastError();
}

hipError_t bp_lane_reset(const BpArgs &a, uint32_t k, int64_t V, uint32_t lane, int32_t seed, int32_t old, hipStream_t s) {
    unsigned nb = (unsigned)std::min<int64_t>(2048, (V + 255) / 256 + 1);
    hipLaunchKernelGGL(k_bp_lane_reset, dim3(nb), dim3(256), 0, s, a.x, a.c[k & 1], a.c[(k + 1) & 1], a.seed_acc, a.outdeg,
                       a.slot, V, a.B, lane, seed, old);
    return hipGetLastError();
}

hipError_t lane_extract(const uint32_t *tile, int64_t V, uint32_t B, uint32_t lane, uint32_t *out, hipStream_t s) {
    unsigned nb = (unsigned)std::min<int64_t>(2048, (V + 255) / 256 + 1);
    hipLaunchKernelGGL(k_lane_extract, dim3(nb), dim3(256), 0, s, tile, V, B, lane, out);
    return hipGetLastError();
}

gx_tune default_tune(uint32_t B) {
    gx_tune t{};
    t.block = 256;
    t.tile = 2048;
    t.width = B;
    t.grid = 0;
    return t;
}

}  // namespace gx

static gx_status batch_common(gx_graph *g, int32_t algo, const int32_t *sources, uint32_t B, void *dev_work,
                              size_t work_bytes, void *dev_out, BsWork *bsw, BpWork *bpw) {
    gx_status st = check_batch(g, algo, B);
    if (st != GX_OK) return st;
    GX_REQUIRE(sources && dev_work && dev_out, GX_EINVAL, "NULL argument");
    GX_REQUIRE(reinterpret_cast<uintptr_t>(dev_work) % ALIGN == 0, GX_EINVAL, "dev_work not 256-byte aligned");
    GX_REQUIRE(reinterpret_cast<uintptr_t>(dev_out) % 16 == 0, GX_EINVAL, "dev_out not 16-byte aligned");
    for (uint32_t b = 0; b < B; b++)
        GX_REQUIRE(sources[b] >= 0 && sources[b] < g->d.V, GX_EINVAL, "sources[%u]=%d out of [0,V)", b, sources[b]);
    Carver c(dev_work, work_bytes);
    if (algo == GX_SSSP) bs_layout(g->d, B, c, bsw);
    else bp_layout(g->d, B, c, bpw);
    GX_REQUIRE(c.fits(), GX_ENOMEM, "workspace too small: need %zu bytes, have %zu", c.used, work_bytes);
    return GX_OK;
}

extern "C" gx_status gx_batch_run(gx_graph *g, int32_t algo, const int32_t *sources, uint32_t B, float damping,
                                  uint32_t iters, void *dev_work, size_t work_bytes, void *dev_out,
                                  const gx_tune *tune, void *stream, gx_run_stats *out) {
    clear_error();
    BsWork bsw;
    BpWork bpw;
    gx_status st = batch_common(g, algo, sources, B, dev_work, work_bytes, dev_out, &bsw, &bpw);
    if (st != GX_OK) return st;
    hipStream_t s = static_cast<hipStream_t>(stream);
    auto t0 = std::chrono::steady_clock::now();
    gx_run_stats rs{};
    if (algo == GX_SSSP) {
        gx_tune tn = tune ? *tune : default_tune(B);
        if (tn.block == 0) tn.block = 256;
        if (tn.tile == 0) tn.tile = tn.block * 8;
        if (tn.width == 0) tn.width = B;
        GX_CHECK_HIP(hipMemcpyAsync(bsw.src, sources, B * 4, hipMemcpyHostToDevice, s), g);
        int64_t steps = 0;
        st = run_bsssp(g, bsw.src, B, bsw, static_cast<uint32_t *>(dev_out), tn, s, &steps);
        if (st != GX_OK) return st;
        rs.supersteps = steps;
        rs.converged = 1;
    } else {
        GX_REQUIRE(damping >= 0.f && damping < 1.f, GX_EINVAL, "damping %f out of [0,1)", damping);
        GX_CHECK_HIP(hipMemcpyAsync(bpw.seed, sources, B * 4, hipMemcpyHostToDevice, s), g);
        st = run_bppr(g, bpw.seed, B, bpw, damping, iters, static_cast<float *>(dev_out), s,
                      tune ? (int)tune->grid : 0);
        if (st != GX_OK) return st;
        rs.supersteps = iters;
        rs.edges = (int64_t)iters * g->d.E;
    }
    rs.wall_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    if (out) *out = rs;
    return GX_OK;
}

// Autotune results kept on disk when GX_TUNE_CACHE names a file: one line
// per (graph signature, algorithm, lanes, iterations) with the chosen shape
// and its time.  The signature hashes the graph's size, its out-degrees and
// the device's CU count (FNV-1a), so a cached shape is reused only for the
// same graph on the same kind of device.
namespace {
struct TuneKey {
    uint64_t sig;
    int32_t algo;
    uint32_t B, iters;
    bool operator<(const TuneKey &o) const {
        return std::tie(sig, algo, B, iters) < std::tie(o.sig, o.algo, o.B, o.iters);
    }
};
struct TuneCache {
    std::mutex mu;
    std::string path;  // the file the map was read from
    std::map<TuneKey, std::pair<gx_tune, double>> map;
};
TuneCache &tune_cache() {
    static TuneCache c;
    return c;
}

uint64_t graph_signature(const gx_graph *g) {
    uint64_t h = 1469598103934665603ull;
    auto mix = [&](uint64_t v) {
        for (int i = 0; i < 8; i++) {
            h ^= (v >> (8 * i)) & 0xFFu;
            h *= 1099511628211ull;
        }
    };
    mix((uint64_t)g->d.V);
    mix((uint64_t)g->d.E);
    mix((uint64_t)g->num_cus);
    for (int32_t d : g->host_outdeg) mix((uint64_t)(uint32_t)d);
    return h;
}

// Reads the file named by GX_TUNE_CACHE into the map (again when the name
// changes); returns false when the variable is not set.
bool tune_cache_open(TuneCache &c) {
    const char *p = std::getenv("GX_TUNE_CACHE");
    if (!p || !*p) return false;
    if (c.path == p) return true;
    c.path = p;
    c.map.clear();
    if (FILE *f = std::fopen(p, "r")) {
        unsigned long long sig;
        int algo;
        unsigned B, iters, block, tile, width, grid;
        double ms;
        while (std::fscanf(f, "%llx %d %u %u %u %u %u %u %lf", &sig, &algo, &B, &iters, &block, &tile, &width,
                           &grid, &ms) == 9)
            c.map[TuneKey{sig, algo, B, iters}] = {gx_tune{block, tile, width, grid}, ms};
        std::fclose(f);
    }
    return true;
}
}  // namespace

extern "C" gx_status gx_batch_autotune(gx_graph *g, int32_t algo, const int32_t *sources, uint32_t B, float damping,
                                       uint32_t iters, void *dev_work, size_t work_bytes, void *dev_out,
                                       void *stream, gx_tune *best, double *best_ms) {
    clear_error();
    GX_REQUIRE(best, GX_EINVAL, "best is NULL");
    BsWork bsw;
    BpWork bpw;
    gx_status st = batch_common(g, algo, sources, B, dev_work, work_bytes, dev_out, &bsw, &bpw);
    if (st != GX_OK) return st;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const TuneKey key{graph_signature(g), algo, B, algo == GX_PPR ? iters : 0u};
    {
        TuneCache &tc = tune_cache();
        std::lock_guard<std::mutex> lk(tc.mu);
        auto it = tune_cache_open(tc) ? tc.map.find(key) : tc.map.end();
        if (it != tc.map.end()) {  // a stored shape: run it once so dev_out holds its result
            *best = it->second.first;
            if (best_ms) *best_ms = it->second.second;
            if (algo == GX_SSSP) {
                GX_CHECK_HIP(hipMemcpyAsync(bsw.src, sources, B * 4, hipMemcpyHostToDevice, s), g);
                return run_bsssp(g, bsw.src, B, bsw, static_cast<uint32_t *>(dev_out), *best, s, nullptr);
            }
            GX_CHECK_HIP(hipMemcpyAsync(bpw.seed, sources, B * 4, hipMemcpyHostToDevice, s), g);
            return run_bppr(g, bpw.seed, B, bpw, damping, iters, static_cast<float *>(dev_out), s, (int)best->grid);
        }
    }
    std::vector<gx_tune> cands;
    if (algo == GX_SSSP) {
        int nv = 0;
        const BsVariant *vars = bs_variants(&nv);
        for (uint32_t width = 32; width <= B; width *= 2) {
            if (B % width) continue;
            for (int i = 0; i < nv; i++) cands.push_back(gx_tune{vars[i].block, vars[i].block * vars[i].vt, width, 0});
        }
        GX_CHECK_HIP(hipMemcpyAsync(bsw.src, sources, B * 4, hipMemcpyHostToDevice, s), g);
    } else {
        // (the grid only bounds the workgroups that complete the rows crossing tiles: the
        // pull takes every workgroup the CUs hold, the graph fixes its tiles)
        for (int frac : {1, 2, 4}) cands.push_back(gx_tune{256, BP_TILE, B, (uint32_t)(g->num_cus * frac)});
        GX_CHECK_HIP(hipMemcpyAsync(bpw.seed, sources, B * 4, hipMemcpyHostToDevice, s), g);
    }
    const size_t n = (size_t)g->d.V * B;
    std::vector<uint32_t> ref, cur;
    double bms = 1e300;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    GX_CHECK_HIP(hipEventCreate(&e0), g);
    GX_CHECK_HIP(hipEventCreate(&e1), g);
    gx_status result = GX_OK;
    for (size_t ci = 0; ci < cands.size() && result == GX_OK; ci++) {
        const gx_tune &tn = cands[ci];
        (void)hipEventRecord(e0, s);
        if (algo == GX_SSSP)
            result = run_bsssp(g, bsw.src, B, bsw, static_cast<uint32_t *>(dev_out), tn, s, nullptr);
        else
            result = run_bppr(g, bpw.seed, B, bpw, damping, iters, static_cast<float *>(dev_out), s, (int)tn.grid);
        (void)hipEventRecord(e1, s);
        if (result != GX_OK) break;
        if (hipEventSynchronize(e1) != hipSuccess) {
            result = GX_EDEVICE;
            break;
        }
        float ms = 0.f;
        (void)hipEventElapsedTime(&ms, e0, e1);
        // every candidate must reproduce the first candidate's tile exactly
        cur.resize(n);
        if (hipMemcpy(cur.data(), dev_out, n * 4, hipMemcpyDeviceToHost) != hipSuccess) {
            result = GX_EDEVICE;
            break;
        }
        if (ci == 0) ref.swap(cur);
        else if (std::memcmp(ref.data(), cur.data(), n * 4) != 0) {
            set_error("autotune candidate block=%u tile=%u width=%u grid=%u changed the result", tn.block, tn.tile,
                      tn.width, tn.grid);
            result = GX_EDEVICE;
            break;
        }
        if (ms < bms) {
            bms = ms;
            *best = tn;
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (result != GX_OK) return result;
    if (best_ms) *best_ms = bms;
    {
        TuneCache &tc = tune_cache();
        std::lock_guard<std::mutex> lk(tc.mu);
        if (tune_cache_open(tc)) {
            tc.map[key] = {*best, bms};
            if (FILE *f = std::fopen(tc.path.c_str(), "a")) {
                std::fprintf(f, "%llx %d %u %u %u %u %u %u %.6f\n", (unsigned long long)key.sig, key.algo, key.B,
                             key.iters, best->block, best->tile, best->width, best->grid, bms);
                std::fclose(f);
            }
        }
    }
    // leave the best candidate's result in dev_out
    if (algo == GX_SSSP)
        return run_bsssp(g, bsw.src, B, bsw, static_cast<uint32_t *>(dev_out), *best, s, nullptr);
    return run_bppr(g, bpw.seed, B, bpw, damping, iters, static_cast<float *>(dev_out), s, (int)best->grid);
}
