// Batched lanes: B independent single-source problems over one resident
// graph, carried in a [V x B] state tile (B contiguous per vertex) by one
// persistent cooperative kernel per pass.  The evaluation of the paper runs
// several SSSP sources simultaneously to raise the arithmetic intensity
// (Section "Setup", first footnote); here the lanes are independent
// problems, each equal to its plain solve.
//
// SSSP (k_bsssp): per superstep
//   compaction: every (vertex, 32-lane group) whose lane mask is non-zero
//     and that has out-edges becomes one active entry; its 32 start-of-
//     superstep distances are copied to a snapshot row (Jacobi semantics per
//     lane); one 64-bit atomic per workgroup chunk reserves entries and edge
//     offsets; tiles of equal (entry, edge) work units record where they
//     start.
//   relaxation: 8 threads per work unit handle the unit's 32 lanes (4 each,
//     one 16-byte load of the destination's group); improvements are
//     folded by atomicMin per lane (no result awaited: a candidate below a
//     value read during the superstep already proves the lane changes), and
//     the group's improved-lane bits by one atomicOr into the next mask.
//   A grid barrier separates the phases; the loop ends when a superstep
//   activates no (vertex, lane) pair.
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
    unsigned long long scan[NW];
    unsigned long long base64;
    int32_t red[NW];
    unsigned long long cnt[NW];
    uint32_t lane[256];
    unsigned int flag;
};

// Phase 1 of batched superstep k: active (vertex, group) pairs -> entries,
// snapshots, tile starts.  Grid-strided over the V*G mask words.
template <int BLOCK, int VT>
__device__ __forceinline__ void bs_compact(const BsArgs &a, uint32_t k, BsShared<BLOCK, VT> &sh) {
    constexpr int T = BLOCK * VT;
    const int tid = threadIdx.x;
    const int64_t VG = a.V * (int64_t)a.G;
    const int slot = k & 3;
    const uint32_t *Mc = a.M[k & 1];
    uint32_t *Mn = a.M[(k + 1) & 1];
    if (blockIdx.x == 0 && tid == 0) {
        a.ctl->list[(k + 1) & 3] = 0;
        a.ctl->changed[(k + 1) & 3] = 0;
    }
    for (int64_t base = (int64_t)blockIdx.x * BLOCK; base < VG; base += (int64_t)gridDim.x * BLOCK) {
        const int64_t i = base + tid;
        uint32_t word = 0, u = 0, g = 0;
        int32_t r0 = 0, deg = 0;
        if (i < VG) {
            word = Mc[i];
            Mn[i] = 0u;
            if (word) {
                u = (uint32_t)(i / a.G);
                g = (uint32_t)(i % a.G);
                r0 = a.rp[u];
                deg = a.rp[u + 1] - r0;
            }
        }
        const bool has = word && deg > 0;
        unsigned long long mine = has ? ((1ull << 32) | (uint32_t)deg) : 0ull, total;
        unsigned long long pre = block_excl_scan_u64(mine, &total, sh.scan);
        if (tid == 0) sh.base64 = total ? atomicAdd(&a.ctl->list[slot], total) : 0ull;
        __syncthreads();
        if (has) {
            unsigned long long pos = sh.base64 + pre;
            uint32_t idx = (uint32_t)(pos >> 32), off = (uint32_t)pos;
            a.list[idx] = make_uint4(off, (uint32_t)(r0 - (int32_t)off), word, g);
            const uint4 *src = reinterpret_cast<const uint4 *>(a.D + (size_t)u * a.B + a.l0 + g * 32);
            uint4 *dst = a.S + (size_t)idx * 8;
#pragma unroll
            for (int q = 0; q < 8; q++) dst[q] = src[q];
            uint32_t t0 = (off + T - 1) / T, t1 = (off + (uint32_t)deg - 1) / T;
            for (uint32_t t = t0; t <= t1; t++) a.tile_start[t] = idx;
        }
        __syncthreads();
    }
}

// Phase 2 of batched superstep k: relax the equal tiles of (entry, edge)
// work units; `it` indexes the per-lane activation counters.
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
    for (uint32_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const uint32_t e0 = t * T;
        const int n = (int)min((uint32_t)T, EF - e0);
        const uint32_t s0 = a.tile_start[t];
        const uint32_t s1 = (t + 1 < ntiles) ? a.tile_start[t + 1] : L - 1;
        const int m = (int)(s1 - s0) + 1;
        for (int p = tid; p < n; p += BLOCK) sh.own[p] = 0;
        __syncthreads();
        for (int q = tid; q < m; q += BLOCK) {
            uint4 en = a.list[s0 + q];
            sh.base[q] = en.y + e0;
            sh.mask[q] = en.z;
            sh.g[q] = en.w;
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
        constexpr int UB = 4;
        for (int p0 = tid >> 3; p0 < n; p0 += UNITS * UB) {
            uint2 ed[UB];
            uint32_t my4[UB], gq[UB], jq[UB];
#pragma unroll
            for (int q = 0; q < UB; q++) {
                const int p = min(p0 + q * UNITS, n - 1);
                const int j = sh.own[p];
                jq[q] = (uint32_t)j;
                gq[q] = sh.g[j];
                my4[q] = (p0 + q * UNITS < n) ? (sh.mask[j] >> (sub * 4)) & 15u : 0u;
                ed[q] = a.adj[sh.base[j] + (uint32_t)p];
            }
            uint4 sn[UB], cur[UB];
#pragma unroll
            for (int q = 0; q < UB; q++) {
                sn[q] = a.S[(size_t)(s0 + jq[q]) * 8 + sub];
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

// One persistent cooperative launch runs supersteps until one activates no
// (vertex, lane) pair or max_steps have run; grid barriers separate phases.
template <int BLOCK, int VT>
__global__ __launch_bounds__(BLOCK) void k_bsssp(BsArgs a) {
    __shared__ BsShared<BLOCK, VT> sh;
    uint32_t k = a.k0;
    for (uint32_t it = 0; it < a.max_steps; it++, k++) {
        bs_compact<BLOCK, VT>(a, k, sh);
        if (!grid_sync(&a.ctl->bar, gridDim.x, &sh.flag, a.bar_ticks)) return;
        bs_relax<BLOCK, VT>(a, k, it, sh);
        if (!grid_sync(&a.ctl->bar, gridDim.x, &sh.flag, a.bar_ticks)) return;
        const unsigned long long ch =
            __hip_atomic_load(&a.ctl->changed[k & 3], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (blockIdx.x == 0 && threadIdx.x == 0) a.ctl->steps = it + 1;
        if (ch == 0 && a.stop_when_idle) break;
    }
}

// The same phases as ordinary launches (serving: several pools overlap on
// their own streams, so no launch may rely on grid-wide co-residency).
template <int BLOCK, int VT>
__global__ __launch_bounds__(BLOCK) void k_bs_compact(BsArgs a, uint32_t k) {
    __shared__ BsShared<BLOCK, VT> sh;
    bs_compact<BLOCK, VT>(a, k, sh);
}
template <int BLOCK, int VT>
__global__ __launch_bounds__(BLOCK) void k_bs_relax(BsArgs a, uint32_t k, uint32_t it) {
    __shared__ BsShared<BLOCK, VT> sh;
    bs_relax<BLOCK, VT>(a, k, it, sh);
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
__global__ __launch_bounds__(256) void k_bs_lane_reset(uint32_t *D, uint32_t *Mc, uint32_t *Mn, int64_t V, uint32_t B,
                                                       uint32_t G, uint32_t lane, int32_t src) {
    const uint32_t bit = 1u << (lane & 31), g = lane / 32;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < V; v += (int64_t)gridDim.x * blockDim.x) {
        D[(size_t)v * B + lane] = (v == src) ? 0u : INF;
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
__device__ __forceinline__ void ppr_apply(const BpArgs &a, int32_t r, int od, const double (&acc)[LPT],
                                          const PprLanes<LPT> &L, float *__restrict__ c_out, uint32_t b0) {
#pragma unroll
    for (int i = 0; i < LPT; i++) {
        if (!L.live[i]) continue;
        const uint32_t b = b0 + 64u * i;
        const float xn = (float)((double)a.d * acc[i]);
        c_out[(size_t)r * a.B + b] = od > 0 ? xn / (float)od : xn;
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
// launches); this one takes 675 us (722 us with the other two), 6.1 TB/s of
// gathered rows.
__device__ __forceinline__ double *bp_partial(double *p, int64_t t, uint32_t B, uint32_t b) { return p + t * B + b; }

template <int W, int LPT>
__global__ __launch_bounds__(256) void k_bp_pull(BpArgs a, uint32_t k) {
    constexpr int NG = 64 / W, EB = 16;
    __shared__ int2 s_nz[4][NG][64];
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
        const int32_t *__restrict__ ids = (dng ? a.dang : a.in_col) + e0;
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
                if (q + (int)b0 < ends) s_nz[wv][g][q + b0] = a.nz[ord + q + (int)b0];
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
                        const int2 rw = s_nz[wv][g][idx++];
                        if (head) {
                            head = false;
                            if (on)
#pragma unroll
                                for (int i = 0; i < LPT; i++)
                                    if (b0 + 64u * i < a.Bw) *bp_partial(a.head, t, a.B, b0 + 64u * i) = acc[i];
                        } else if (on) {
                            ppr_apply<LPT>(a, rw.x, rw.y, acc, L, c_out, b0);
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

// s plus p[i * stride] over i = 0 .. n-1 in index order; the loads go out 16
// at a time, the adds stay in order.
__device__ __forceinline__ double ordered_sum(double s, const double *p, int64_t stride, int64_t n) {
    for (int64_t i0 = 0; i0 < n; i0 += 16) {
        double v[16];
#pragma unroll
        for (int j = 0; j < 16; j++) v[j] = p[std::min<int64_t>(i0 + j, n - 1) * stride];
#pragma unroll
        for (int j = 0; j < 16; j++)
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
    s_p[wv][lane] = b < Bw ? ordered_sum(0.0, p + lo * B + b, B, hi - lo) : 0.0;
    __syncthreads();
    if (wv == 0)
        for (int i = 0; i < ROWS_PIECES; i++) s += s_p[i][lane];
    return s;
}

// Rows crossing tiles: the first tile's tail and the later tiles' heads in
// tile order.  One workgroup per long row, a lane group per other row.
constexpr int BP_FIX_BLOCK = 64 * ROWS_PIECES;

template <int W, int LPT>
__global__ __launch_bounds__(BP_FIX_BLOCK) void k_bp_fix(BpArgs a, uint32_t k) {
    __shared__ double s_p[ROWS_PIECES][64];
    const int lane = threadIdx.x & 63;
    float *c_out = a.c[(k + 1) & 1];
    if ((int)blockIdx.x < a.n_cross_long) {
        const int4 q = a.cross[blockIdx.x];
        const PprLanes<LPT> L(a, k, (uint32_t)lane);
        double acc[LPT];
#pragma unroll
        for (int i = 0; i < LPT; i++) {
            const uint32_t b = (uint32_t)lane + 64u * i;
            const double s = b < a.Bw ? a.tailp[(int64_t)q.z * a.B + b] : 0.0;
            acc[i] = pieces_sum(s, a.head + (int64_t)(q.z + 1) * a.B, a.B, 64u * i, a.Bw, q.w - q.z, s_p);
        }
        if (threadIdx.x < 64) ppr_apply<LPT>(a, q.x, q.y, acc, L, c_out, (uint32_t)lane);
        return;
    }
    const uint32_t b0 = (uint32_t)(lane % W);
    const PprLanes<LPT> L(a, k, b0);
    const int groups = BP_FIX_BLOCK / W;
    for (int64_t j = a.n_cross_long + (int64_t)(blockIdx.x - a.n_cross_long) * groups + threadIdx.x / W; j < a.n_cross;
         j += (int64_t)(gridDim.x - a.n_cross_long) * groups) {
        const int4 q = a.cross[j];
        double acc[LPT];
#pragma unroll
        for (int i = 0; i < LPT; i++) {
            const uint32_t b = b0 + 64u * i;
            acc[i] = 0.0;
            if (b >= a.Bw) continue;
            double s = a.tailp[(int64_t)q.z * a.B + b];
            for (int32_t t = q.z + 1; t <= q.w; t += 4) {
                double v[4];
#pragma unroll
                for (int u = 0; u < 4; u++) v[u] = a.head[(int64_t)min(t + u, q.w) * a.B + b];
#pragma unroll
                for (int u = 0; u < 4; u++)
                    if (t + u <= q.w) s += v[u];
            }
            acc[i] = s;
        }
        ppr_apply<LPT>(a, q.x, q.y, acc, L, c_out, b0);
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
    const size_t at = (size_t)r * a.B + b;
    const bool no_in = a.in_rp[r + 1] == a.in_rp[r];
    if (od == 0 && no_in) D += (double)a.c[k & 1][at];  // a seed that no list of dangling vertices holds
    const double v = (double)a.d * (no_in ? 0.0 : a.seed_acc[b]) + ((1.0 - (double)a.d) + (double)a.d * D);
    const float xn = (float)v;
    a.c[(k + 1) & 1][at] = od > 0 ? xn / (float)od : xn;
    if (end == k + 1) a.x[at] = xn;
}

// Superstep 0: ranks e_seed (in the contributions; in x too if there are no
// supersteps), 0 in every row no superstep writes.
__global__ __launch_bounds__(256) void k_bp_init(float *x, float *c0, float *c1, const int32_t *seed,
                                                 const int32_t *in_rp, const int32_t *outdeg, int64_t V, uint32_t B,
                                                 uint32_t iters) {
    const size_t n = (size_t)V * B;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const int64_t v = (int64_t)(i / B);
        const uint32_t b = (uint32_t)(i % B);
        const bool here = seed[b] == v;
        const int od = outdeg[v];
        c0[i] = !here ? 0.0f : od > 0 ? 1.0f / (float)od : 1.0f;
        if (iters == 0 || in_rp[v + 1] == in_rp[v]) {
            c1[i] = 0.0f;
            x[i] = here && iters == 0 ? 1.0f : 0.0f;
        }
    }
}

// Serving: lane b restarts from its new seed.  The other buffer and x hold
// this lane's old values: rows with in-edges are rewritten before they are
// read, so only the old seed's (perhaps without in-edges) are cleared.
__global__ __launch_bounds__(256) void k_bp_lane_reset(float *x, float *c, float *c_other, double *seed_acc,
                                                       const int32_t *outdeg, int64_t V, uint32_t B, uint32_t lane,
                                                       int32_t seed, int32_t old) {
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < V; v += (int64_t)gridDim.x * blockDim.x) {
        const int od = outdeg[v];
        c[(size_t)v * B + lane] = v != seed ? 0.0f : od > 0 ? 1.0f / (float)od : 1.0f;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        seed_acc[lane] = 0.0;
        if (old >= 0) c_other[(size_t)old * B + lane] = x[(size_t)old * B + lane] = 0.0f;
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
        {256, 4, (const void *)k_bsssp<256, 4>},  {256, 8, (const void *)k_bsssp<256, 8>},
        {512, 4, (const void *)k_bsssp<512, 4>},  {512, 8, (const void *)k_bsssp<512, 8>},
        {1024, 2, (const void *)k_bsssp<1024, 2>}, {1024, 4, (const void *)k_bsssp<1024, 4>},
    };
    *n = (int)(sizeof v / sizeof v[0]);
    return v;
}


// Workgroups of a cooperative (grid-barrier) launch.  By default at most
// max_per_cu per CU and at most half of the occupancy bound; a kernel whose
// phases run for milliseconds (batched PPR) passes max_per_cu = 0 to use
// the whole bound (the cooperative launch itself refuses a grid that cannot
// be resident at once).
int coop_grid(const void *kernel, int block, int num_cus, int want, int max_per_cu) {
    const int occ = occupancy_per_cu(kernel, block);
    int per_cu = max_per_cu > 0 ? std::max(1, std::min(max_per_cu, occ / 2)) : std::max(1, occ);
    int cap = per_cu * num_cus;
    if (want > 0) return std::min(want, cap);
    return cap;
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
    const int64_t nt = std::max<int64_t>(1, rows_tiles(d.E));
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
    a.in_col = d.in_col;
    a.nz = d.nz;
    a.row_last = d.row_last;
    a.tile_nz = d.tile_nz;
    a.cross = d.cross;
    a.dang = d.dang;
    a.in_rp = d.in_rp;
    a.outdeg = d.outdeg;
    a.n_nz = d.n_nz;
    a.tile = (int32_t)rows_tile(d.E);
    a.ntiles = rows_tiles(d.E);
    a.E = d.E;
    a.n_dang = d.n_dang;
    // (few tiles of dangling vertices: their partials are added by one workgroup)
    a.dtile = (int32_t)std::max<int64_t>(a.tile, ((d.n_dang + ROWS_DANGLING - 1) / ROWS_DANGLING + 63) / 64 * 64);
    a.ndtiles = (int32_t)((d.n_dang + a.dtile - 1) / a.dtile);
    a.n_cross = d.n_cross;
    a.n_cross_long = d.n_cross_long;
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

// Wall-clock ticks a grid barrier may wait: BARRIER_LIMIT_S seconds at the
// device's constant wall-clock rate (a superstep phase of the batched
// kernel takes milliseconds; only a grid that is not co-resident waits that
// long).
unsigned long long barrier_limit_ticks(int device) {
    int khz = 0;
    if (hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, device) != hipSuccess || khz <= 0)
        khz = 100000;  // 100 MHz, the gfx9 constant clock
    return (unsigned long long)(BARRIER_LIMIT_S * 1e3 * (double)khz);
}

hipError_t launch_coop(const void *kernel, int grid, int block, void *args, hipStream_t s) {
    void *params[] = {args};
    return hipLaunchCooperativeKernel(kernel, dim3(grid), dim3(block), params, 0, s);
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
    const int grid = coop_grid(var->fn, var->block, g->num_cus, (int)tn.grid, 2);
    for (uint32_t l0 = 0; l0 < B; l0 += tn.width) {
        const uint32_t G = tn.width / 32;
        GX_CHECK_HIP(hipMemsetAsync(w.M[0], 0, (size_t)d.V * G * 4, s), g);
        GX_CHECK_HIP(hipMemsetAsync(w.M[1], 0, (size_t)d.V * G * 4, s), g);
        GX_CHECK_HIP(hipMemsetAsync(w.ctl, 0, sizeof(BsCtl), s), g);
        hipLaunchKernelGGL(k_bs_sources, dim3((tn.width + 255) / 256), dim3(256), 0, s, D, w.M[0], dev_src, B, l0,
                           tn.width, G);
        BsArgs a{};
        a.rp = d.out_rp;
        a.adj = d.out_adj;
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
        a.max_steps = (uint32_t)std::min<int64_t>(d.V + 2, 0x7FFFFFFF);
        a.k0 = 0;
        a.lane_cnt = nullptr;
        a.stop_when_idle = 1;
        a.bar_ticks = barrier_limit_ticks(g->device);
        GX_CHECK_HIP(launch_coop(var->fn, grid, var->block, &a, s), g);
        BsCtl ctl;
        GX_CHECK_HIP(hipMemcpyAsync(&ctl, w.ctl, sizeof ctl, hipMemcpyDeviceToHost, s), g);
        GX_CHECK_HIP(hipStreamSynchronize(s), g);
        if (ctl.bar.error) {
            set_error("grid barrier waited over %.0f s in batched SSSP (pass at lane %u, grid %d x %u)",
                      BARRIER_LIMIT_S, l0, grid, var->block);
            g->dev_error = true;
            return GX_EDEVICE;
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
                       w.c[0], w.c[1], w.seed, d.in_rp, d.outdeg, d.V, B, iters);
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

hipError_t bs_launch_superstep(const BsArgs &a, uint32_t k, uint32_t it, int grid, hipStream_t s) {
    hipLaunchKernelGGL((k_bs_compact<256, 8>), dim3(grid), dim3(256), 0, s, a, k);
    hipLaunchKernelGGL((k_bs_relax<256, 8>), dim3(grid), dim3(256), 0, s, a, k, it);
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

hipError_t bs_lane_reset(uint32_t *D, uint32_t *Mc, uint32_t *Mn, int64_t V, uint32_t B, uint32_t G, uint32_t lane,
                         int32_t src, hipStream_t s) {
    unsigned nb = (unsigned)std::min<int64_t>(2048, (V + 255) / 256 + 1);
    hipLaunchKernelGGL(k_bs_lane_reset, dim3(nb), dim3(256), 0, s, D, Mc, Mn, V, B, G, lane, src);
    return hipGetLastError();
}

hipError_t bp_lane_reset(const BpArgs &a, uint32_t k, int64_t V, uint32_t lane, int32_t seed, int32_t old, hipStream_t s) {
    unsigned nb = (unsigned)std::min<int64_t>(2048, (V + 255) / 256 + 1);
    hipLaunchKernelGGL(k_bp_lane_reset, dim3(nb), dim3(256), 0, s, a.x, a.c[k & 1], a.c[(k + 1) & 1], a.seed_acc, a.outdeg,
                       V, a.B, lane, seed, old);
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
