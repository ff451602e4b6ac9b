// Graph ingestion: host validation, host packaging of the device images, and
// block-streamed host-to-device transfer through three rotating pinned
// buffers (the n/c/u block rotation of Section "Pipeline Shuffling": while
// block i is in flight on the copy stream, block i+1 is packaged into the
// next buffer; pointers rotate instead of data being copied between stages).
#include <algorithm>
#include <atomic>
#include <cmath>
#include <condition_variable>
#include <cstdarg>
#include <cstdio>
#include <functional>
#include <map>
#include <mutex>
#include <queue>
#include <memory>
#include <thread>
#include <tuple>

#include "gx_internal.h"

namespace gx {

static thread_local std::string g_err;

void set_error(const char *fmt, ...) {
    char buf[1024];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
}
void clear_error() { g_err.clear(); }

int device_cus(int device) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || n <= 0) n = 256;
    return n;
}

int occupancy_per_cu(const void *kernel, int block) {
    static std::mutex mu;
    static std::map<std::tuple<int, const void *, int>, int> cache;
    int dev = 0;
    (void)hipGetDevice(&dev);
    std::lock_guard<std::mutex> lk(mu);
    auto key = std::make_tuple(dev, kernel, block);
    auto it = cache.find(key);
    if (it != cache.end()) return it->second;
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, block, 0) != hipSuccess || per_cu <= 0)
        per_cu = 1;
    cache[key] = per_cu;
    return per_cu;
}

// Host threads kept for the packaging passes (a load runs hundreds of them,
// one per 16 MiB block, and starting threads for each would cost more than
// the pass).  One pass at a time; a pass started from inside a pass, or
// while another load holds the workers, runs on the calling thread.
class HostWorkers {
  public:
    static HostWorkers &get() {
        static HostWorkers w;
        return w;
    }
    unsigned size() const { return (unsigned)workers_.size() + 1; }
    // Runs job(t) for t = 0 .. size()-1, share 0 on the calling thread; false
    // (nothing run) when the workers are busy.
    bool run(const std::function<void(unsigned)> &job) {
        std::unique_lock<std::mutex> busy(pass_, std::try_to_lock);
        if (!busy.owns_lock() || in_pass_) return false;
        {
            std::lock_guard<std::mutex> lk(mu_);
            job_ = &job;
            left_ = (unsigned)workers_.size();
            gen_++;
        }
        cv_.notify_all();
        in_pass_ = true;
        job(0);
        in_pass_ = false;
        std::unique_lock<std::mutex> lk(mu_);
        done_.wait(lk, [this] { return left_ == 0; });
        job_ = nullptr;
        return true;
    }
    ~HostWorkers() {
        {
            std::lock_guard<std::mutex> lk(mu_);
            stop_ = true;
            gen_++;
        }
        cv_.notify_all();
        for (auto &t : workers_) t.join();
    }

  private:
    HostWorkers() {
        const unsigned n = std::max(1u, std::min(16u, std::thread::hardware_concurrency()));
        for (unsigned t = 1; t < n; t++) workers_.emplace_back([this, t] { loop(t); });
    }
    void loop(unsigned t) {
        uint64_t seen = 0;
        std::unique_lock<std::mutex> lk(mu_);
        while (true) {
            cv_.wait(lk, [&] { return gen_ != seen; });
            seen = gen_;
            if (stop_) return;
            const std::function<void(unsigned)> *job = job_;
            lk.unlock();
            in_pass_ = true;
            (*job)(t);
            in_pass_ = false;
            lk.lock();
            if (--left_ == 0) done_.notify_all();
        }
    }
    std::vector<std::thread> workers_;
    std::mutex pass_, mu_;
    std::condition_variable cv_, done_;
    const std::function<void(unsigned)> *job_ = nullptr;
    unsigned left_ = 0;
    uint64_t gen_ = 0;
    bool stop_ = false;
    static thread_local bool in_pass_;
};
thread_local bool HostWorkers::in_pass_ = false;

template <class F>
static void parallel_for(int64_t n, F f, int64_t serial_below = 65536) {
    HostWorkers &w = HostWorkers::get();
    const unsigned nt = w.size();
    if (n < serial_below || nt == 1) {
        f(0, n);
        return;
    }
    const std::function<void(unsigned)> job = [&](unsigned t) { f(n * t / nt, n * (t + 1) / nt); };
    if (!w.run(job)) f(0, n);
}

// Host images built from the description before upload.
// Vectors whose elements start uninitialised (resize leaves them as they
// are): the edge-sized images are written in full by parallel passes, so a
// value fill on one thread first would only cost time.
template <class T>
struct NoInit : std::allocator<T> {
    template <class U>
    struct rebind {
        using other = NoInit<U>;
    };
    NoInit() = default;
    template <class U>
    NoInit(const NoInit<U> &) {}
    template <class U, class... A>
    void construct(U *p, A &&...a) {
        if constexpr (sizeof...(A) == 0) ::new ((void *)p) U;
        else ::new ((void *)p) U(std::forward<A>(a)...);
    }
};
template <class T>
using EdgeVec = std::vector<T, NoInit<T>>;

struct HostImages {
    std::vector<int32_t> in_rp, outdeg, slot, nz_slot;
    std::vector<int2> nz, ez;
    std::vector<uint64_t> row_last;
    std::vector<int32_t> dang;
    struct Tiles {
        std::vector<int32_t> tile_nz;
        std::vector<int4> cross;
        int32_t n_long = 0, n_mid = 0;
    } pr_rows, bp_rows;
    int64_t lds_edges = 0;  // edges whose source has one of the first PR_LDS_SLOTS slots
    EdgeVec<int32_t> in_col, pr_src;
    EdgeVec<uint32_t> in_w;
    EdgeVec<uint2> in_adj;
    std::vector<int32_t> sym_rp;
    EdgeVec<int32_t> sym_col;
    bool sym_ascending = true;
    std::vector<int32_t> in_blk;
    std::vector<uint4> pull_segs, sym_segs, packs;
    struct SweepRecs {
        EdgeVec<uint2> rec;
        std::vector<uint4> units;
        std::vector<uint32_t> recs;  // of every unit
        int64_t uoff[PULL_SLICES + 1] = {};
    } sweep_in, sweep_sym;
    std::vector<uint32_t> rem_out, rem_any, master, master_rep;
    std::vector<int32_t> part_list;
};

static gx_status validate(const gx_graph_desc *d) {
    GX_REQUIRE(d, GX_EINVAL, "desc is NULL");
    GX_REQUIRE(d->V >= 0 && d->V < (int64_t(1) << 31) - 64, GX_EINVAL, "V=%lld out of range", (long long)d->V);
    GX_REQUIRE(d->E >= 0 && d->E < (int64_t(1) << 31) - PR_TILE_MAX, GX_EINVAL, "E=%lld out of range",
               (long long)d->E);
    GX_REQUIRE(d->pr_tile_edges == 0 || d->pr_tile_edges == 256 || d->pr_tile_edges == 512 ||
                   d->pr_tile_edges == 1024 || d->pr_tile_edges == 2048,
               GX_EINVAL, "pr_tile_edges=%u not 0, 256, 512, 1024 or 2048", d->pr_tile_edges);
    GX_REQUIRE(d->needs != 0 && (d->needs & ~7u) == 0, GX_EINVAL, "needs=%u invalid", d->needs);
    // the symmetric image holds up to two entries per directed edge, indexed by int32 row pointers
    GX_REQUIRE(!(d->needs & GX_NEED_SYM) || 2 * d->E <= (int64_t)INT32_MAX - 512, GX_EINVAL,
               "E=%lld too large for the symmetric (CC) image: 2E must stay below 2^31", (long long)d->E);
    GX_REQUIRE(d->row_ptr || d->V == 0, GX_EINVAL, "row_ptr is NULL");
    GX_REQUIRE(d->col || d->E == 0, GX_EINVAL, "col is NULL");
    GX_REQUIRE(!(d->needs & GX_NEED_OUT) || d->w || d->E == 0, GX_EINVAL, "weights required for GX_NEED_OUT");
    if (d->V == 0) {
        GX_REQUIRE(d->E == 0, GX_EINVAL, "E > 0 with V == 0");
        return GX_OK;
    }
    GX_REQUIRE(d->row_ptr[0] == 0, GX_EINVAL, "row_ptr[0] != 0");
    GX_REQUIRE(d->row_ptr[d->V] == d->E, GX_EINVAL, "row_ptr[V]=%d != E=%lld", d->row_ptr[d->V], (long long)d->E);
    for (int64_t v = 0; v < d->V; v++)
        GX_REQUIRE(d->row_ptr[v + 1] >= d->row_ptr[v], GX_EINVAL, "row_ptr decreases at %lld", (long long)v);
    std::atomic<int64_t> badpos{INT64_MAX};  // the first column out of range, over the host threads
    parallel_for(d->E, [&](int64_t lo, int64_t hi) {
        for (int64_t e = lo; e < hi; e++)
            if ((uint32_t)d->col[e] >= (uint32_t)d->V) {
                int64_t cur = badpos.load();
                while (e < cur && !badpos.compare_exchange_weak(cur, e)) {
                }
                return;
            }
    });
    const int64_t bp = badpos.load();
    GX_REQUIRE(bp == INT64_MAX, GX_EINVAL, "col[%lld]=%d out of [0,V)", (long long)bp,
               bp == INT64_MAX ? 0 : d->col[bp]);
    GX_REQUIRE((d->V_global == 0) == (d->outdeg_global == nullptr), GX_EINVAL,
               "V_global and outdeg_global come together");
    if (d->outdeg_global) {
        GX_REQUIRE(d->V_global >= d->V && d->V_global < (int64_t(1) << 31), GX_EINVAL, "V_global=%lld out of range",
                   (long long)d->V_global);
        for (int64_t v = 0; v < d->V; v++)
            GX_REQUIRE(d->outdeg_global[v] >= d->row_ptr[v + 1] - d->row_ptr[v], GX_EINVAL,
                       "outdeg_global[%lld] below the local out-degree", (long long)v);
    }
    if (d->l2g) {
        GX_REQUIRE(d->l2g[0] >= 0, GX_EINVAL, "l2g[0] negative");
        for (int64_t v = 1; v < d->V; v++)
            GX_REQUIRE(d->l2g[v] > d->l2g[v - 1], GX_EINVAL, "l2g not strictly ascending at %lld", (long long)v);
    }
    return GX_OK;
}

static unsigned host_threads() { return std::max(1u, std::min(16u, std::thread::hardware_concurrency())); }

// Stable counting sort of the edges by destination: in-rows list their
// sources in ascending order, the same result as one sequential pass.  The
// destinations are cut into buckets of equal vertex ranges; the edges, in
// source order, are cut into one chunk per thread.  Each thread counts its
// chunk's edges per bucket, the counts are laid out bucket by bucket and
// chunk by chunk (so a bucket keeps the chunks' source order), each thread
// copies its chunk's edges to their buckets, and the buckets, handed out
// one at a time, are sorted by destination with a counting sort of their
// own.  Every edge is read a bounded number of times whatever the thread
// count.
static void build_in_csr(const gx_graph_desc *d, HostImages &h) {
    const int64_t V = d->V, E = d->E;
    h.in_rp.assign(V + 1, 0);
    h.in_col.resize(E);
    const bool wts = d->w && (d->needs & GX_NEED_OUT);
    if (wts) h.in_w.resize(E);
    if (E == 0) return;
    const unsigned nt = E < 4096 ? 1u : host_threads();
    const int64_t NB = std::max<int64_t>(1, std::min<int64_t>(256, V / 64));  // destination buckets
    const int64_t span = (V + NB - 1) / NB;                                    // vertices per bucket
    // source-ordered edge chunks: chunk t holds the out-rows of sources [src_cut[t], src_cut[t+1])
    std::vector<int64_t> src_cut(nt + 1, V);
    src_cut[0] = 0;
    for (unsigned t = 1; t < nt; t++)
        src_cut[t] = std::upper_bound(d->row_ptr, d->row_ptr + V, (int32_t)(E * t / nt)) - d->row_ptr - 1;
    for (unsigned t = 1; t <= nt; t++) src_cut[t] = std::max(src_cut[t], src_cut[t - 1]);
    std::vector<int64_t> cnt((size_t)nt * NB, 0);  // [chunk][bucket]
    auto run = [&](auto &&body) {
        std::vector<std::thread> th;
        for (unsigned t = 0; t < nt; t++) th.emplace_back([&, t] { body(t); });
        for (auto &x : th) x.join();
    };
    run([&](unsigned t) {
        int64_t *c = cnt.data() + (size_t)t * NB;
        for (int64_t e = d->row_ptr[src_cut[t]]; e < d->row_ptr[src_cut[t + 1]]; e++) c[d->col[e] / span]++;
    });
    // offsets: bucket-major, then chunk order inside a bucket
    std::vector<int64_t> boff(NB + 1, 0);
    std::vector<int64_t> off((size_t)nt * NB);
    int64_t acc = 0;
    for (int64_t bk = 0; bk < NB; bk++) {
        boff[bk] = acc;
        for (unsigned t = 0; t < nt; t++) {
            off[(size_t)t * NB + bk] = acc;
            acc += cnt[(size_t)t * NB + bk];
        }
    }
    boff[NB] = acc;
    // edges grouped by bucket: (destination, source[, weight])
    std::unique_ptr<int32_t[]> bdst(new int32_t[E]), bsrc(new int32_t[E]);  // (no zero fill)
    std::unique_ptr<uint32_t[]> bw(wts ? new uint32_t[E] : nullptr);
    run([&](unsigned t) {
        int64_t *o = off.data() + (size_t)t * NB;
        for (int64_t u = src_cut[t]; u < src_cut[t + 1]; u++)
            for (int32_t e = d->row_ptr[u]; e < d->row_ptr[u + 1]; e++) {
                const int32_t v = d->col[e];
                const int64_t p = o[v / span]++;
                bdst[p] = v;
                bsrc[p] = (int32_t)u;
                if (wts) bw[p] = d->w[e];
            }
    });
    // each bucket: counting sort by destination (stable), row pointers of its range
    std::atomic<int64_t> next{0};
    run([&](unsigned) {
        std::vector<int32_t> pos;
        for (int64_t bk; (bk = next.fetch_add(1)) < NB;) {
            const int64_t vlo = bk * span, vhi = std::min<int64_t>(V, vlo + span);
            if (vlo >= vhi) continue;
            const int64_t e0 = boff[bk], e1 = boff[bk + 1];
            pos.assign((size_t)(vhi - vlo) + 1, 0);
            for (int64_t i = e0; i < e1; i++) pos[bdst[i] - vlo + 1]++;
            for (int64_t j = 0; j < vhi - vlo; j++) {  // pos[j]: first slot of destination vlo + j
                pos[j + 1] += pos[j];
                h.in_rp[vlo + j + 1] = (int32_t)(e0 + pos[j + 1]);
            }
            for (int64_t i = e0; i < e1; i++) {
                const int64_t p = e0 + pos[bdst[i] - vlo]++;
                h.in_col[p] = bsrc[i];
                if (wts) h.in_w[p] = bw[i];
            }
        }
    });
}

// Slots: the HOT_SLOTS vertices with the most out-edges (ties by id) take
// slots 0.. in that order, the others follow in id order, so what is gathered
// from hubs falls on a few cache lines.
static void build_slots(const gx_graph_desc *d, HostImages &h) {
    const int64_t V = d->V;
    const int64_t K = std::min<int64_t>(V, HOT_SLOTS);
    auto deg = [d](int64_t v) { return d->row_ptr[v + 1] - d->row_ptr[v]; };
    // vertices per degree, then the first slot of every degree, largest first
    int32_t top = 0;
    for (int64_t v = 0; v < V; v++) top = std::max(top, deg(v));
    std::vector<int64_t> at((size_t)top + 2, 0);
    for (int64_t v = 0; v < V; v++) at[deg(v)]++;
    int64_t acc = 0;
    for (int32_t x = top; x >= 0; x--) {
        const int64_t n = at[x];
        at[x] = acc;
        acc += n;
    }
    h.slot.resize(V);
    int64_t next = K;
    for (int64_t v = 0; v < V; v++) {
        const int64_t s = at[deg(v)]++;
        h.slot[v] = (int32_t)(s < K ? s : next++);
        if (s < PR_LDS_SLOTS) h.lds_edges += deg(v);
    }
}

// The rows with in-edges, where they end, and the other rows.
static void build_rows(const gx_graph_desc *d, HostImages &h) {
    const int64_t V = d->V, E = d->E;
    h.row_last.assign((size_t)(E + PR_TILE_MAX) / 64 + 1, 0);
    h.nz.reserve((size_t)std::min(V, E));
    h.nz_slot.reserve((size_t)std::min(V, E));
    for (int64_t v = 0; v < V; v++) {
        const int32_t a = h.in_rp[v], b = h.in_rp[v + 1];
        const int32_t od = d->row_ptr[v + 1] - d->row_ptr[v];
        if (a == b) {
            h.ez.push_back(make_int2((int32_t)v, od));
            continue;
        }
        h.nz.push_back(make_int2((int32_t)v, od));
        h.nz_slot.push_back(h.slot[v]);
        h.row_last[(b - 1) >> 6] |= uint64_t(1) << ((b - 1) & 63);
        if (od == 0) h.dang.push_back(h.slot[v]);
    }
}

// The tiles of T in-edges, and the rows that cross them.
static void build_row_tiles(int64_t E, int64_t T, const HostImages &h, HostImages::Tiles &out) {
    const int64_t nt = (E + T - 1) / T;
    out.tile_nz.assign((size_t)nt + 1, 0);
    std::vector<int4> mid, few;
    int64_t t = 0;
    for (size_t i = 0; i < h.nz.size(); i++) {
        const int2 r = h.nz[i];
        const int32_t a = h.in_rp[r.x], b = h.in_rp[r.x + 1];
        for (; t * T < b && t < nt; t++) out.tile_nz[t] = (int32_t)i;  // tiles whose first edge is in this row
        const int32_t t0 = (int32_t)(a / T), t1 = (int32_t)((b - 1) / T);
        if (t1 - t0 >= ROWS_LONG) out.cross.push_back(make_int4(r.x, r.y, t0, t1));
        else if (t1 - t0 >= ROWS_MID) mid.push_back(make_int4(r.x, r.y, t0, t1));
        else if (t1 > t0) few.push_back(make_int4(r.x, r.y, t0, t1));
    }
    out.n_long = (int32_t)out.cross.size();
    out.n_mid = (int32_t)mid.size();
    out.cross.insert(out.cross.end(), mid.begin(), mid.end());
    out.cross.insert(out.cross.end(), few.begin(), few.end());
}

// PageRank workgroup tile: the caller's choice, else the largest.  Eight
// in-edges per lane leave the fewest rows that cross tiles and the least work
// per edge in the pull (20 supersteps of R-MAT, 2048 against 1024, 512, 256:
// scale 12 225, 241, 228, 276 us; 14 266, 278, 285, 302; 18 574, 592, 684,
// 972; 22 5.62, 5.86, 7.33, 10.96 ms).
static int32_t pr_tile_for(const gx_graph_desc *d) {
    return d->pr_tile_edges ? (int32_t)d->pr_tile_edges : PR_TILE_MAX;
}

// The segments of the rows with more than PULL_SMALL entries.
static void build_segs(const std::vector<int32_t> &rp, std::vector<uint4> &segs) {
    segs.clear();
    for (size_t v = 0; v + 1 < rp.size(); v++) {
        if (rp[v + 1] - rp[v] <= PULL_SMALL) continue;
        for (int32_t e = rp[v]; e < rp[v + 1]; e += PULL_SEG)
            segs.push_back(make_uint4((uint32_t)v, (uint32_t)e, (uint32_t)std::min(rp[v + 1], e + PULL_SEG), 0u));
    }
}

// A row of the SSSP pull by ascending weight, weights of at most 8 bits:
// counted over the 256 weights (rows here are longer than PULL_SMALL).
static void row_by_weight(const int32_t *src, const int32_t *slot, const uint32_t *w, int32_t n, uint32_t tag,
                          uint2 *out) {
    int32_t at[257] = {};
    for (int32_t i = 0; i < n; i++) at[w[i] + 1]++;
    for (int i = 0; i < 256; i++) at[i + 1] += at[i];
    for (int32_t i = 0; i < n; i++) out[at[w[i]]++] = make_uint2((uint32_t)slot[src[i]], tag | w[i]);
}

// In-edges of the SSSP pull, {source slot, (destination mod 64) << 8 | weight}:
// the entries of short rows first, in row order (blk_ptr: where every block
// of 64 rows starts), then the long rows by ascending weight, cut into
// segments.
static void build_in_adj(HostImages &h) {
    const int64_t V = (int64_t)h.in_rp.size() - 1, E = h.in_rp[V];
    const std::vector<int32_t> &rp = h.in_rp;
    h.in_adj.resize(E);
    h.in_blk.assign((size_t)(V + 63) / 64 + 1, 0);
    EdgeVec<int32_t> off(V), seg(V);  // first entry (and segment) of every row
    int32_t at = 0, from = 0;
    auto flush = [&](int64_t v) {  // the entries up to `at` end a pack of row v's block
        if (at > from) h.packs.push_back(make_uint4((uint32_t)from, (uint32_t)at, (uint32_t)(v & ~int64_t(63)), 0u));
        from = at;
    };
    for (int64_t v = 0; v < V; v++) {
        if ((v & 63) == 0) {
            if (v > 0) flush(v - 1);
            h.in_blk[v >> 6] = at;
        }
        off[v] = at;
        const int32_t n = rp[v + 1] - rp[v];
        if (n <= PULL_SMALL) at += n;
        if (at - from >= PULL_PACK) flush(v);
    }
    if (V > 0) flush(V - 1);
    h.in_blk.back() = at;
    h.pull_segs.clear();
    for (int64_t v = 0; v < V; v++) {
        const int32_t n = rp[v + 1] - rp[v];
        if (n <= PULL_SMALL) continue;
        off[v] = at;
        seg[v] = (int32_t)h.pull_segs.size();
        for (int32_t e = 0; e < n; e += PULL_SEG)
            h.pull_segs.push_back(
                make_uint4((uint32_t)v, (uint32_t)(at + e), (uint32_t)(at + std::min(n, e + PULL_SEG)), 0u));
        at += n;
    }
    std::atomic<int64_t> next{0};  // rows differ in length: blocks are handed out one at a time
    const int64_t step = E < (1 << 18) ? V : 4096;
    parallel_for((V + step - 1) / step, [&](int64_t, int64_t) {
        for (int64_t lo; (lo = next.fetch_add(step)) < V;)
            for (int64_t v = lo; v < std::min(V, lo + step); v++) {
                const int32_t e0 = rp[v], n = rp[v + 1] - e0;
                const uint32_t tag = (uint32_t)(v & 63) << 8;
                if (n > PULL_SMALL) {
                    row_by_weight(&h.in_col[e0], h.slot.data(), &h.in_w[e0], n, tag, &h.in_adj[off[v]]);
                    for (int32_t e = 0, i = seg[v]; e < n; e += PULL_SEG, i++)
                        h.pull_segs[i].w = (h.in_adj[off[v] + e].y & 0xFFu) | (n <= PULL_SEG ? 0x100u : 0u);
                    continue;
                }
                for (int32_t i = 0; i < n; i++)
                    h.in_adj[off[v] + i] = make_uint2((uint32_t)h.slot[h.in_col[e0 + i]], tag | h.in_w[e0 + i]);
            }
    }, 2);
}

static bool byte_weights(const gx_graph_desc *d) {
    std::atomic<bool> ok{true};
    parallel_for(d->E, [&](int64_t lo, int64_t hi) {
        for (int64_t e = lo; e < hi; e++)
            if (d->w[e] > 255u) {
                ok = false;
                return;
            }
    });
    return ok;
}

// Symmetric adjacency: sorted union of out- and in-neighbours, self
// excluded, duplicates removed (needs the in-CSR).
// Whether SSSP and CC sweep on this graph.  From about a million vertices on an L2
// no longer holds all values, and what counts is the share of the edges whose
// source is among the PULL_BITS vertices with the most out-edges: the row pull
// gains with it, the sweep does not, and a larger or denser graph needs more.
// The lines are fitted to whole solves on 75 graphs of 2^19 to 2^23 vertices and
// degrees 1 to 64, made as R-MAT is with a = 0.25 (uniform) to 0.57.  Row pull
// against sweep, ms:
//   SSSP, 2^22 vertices of degree 16, shares 0.05, 0.11, 0.21, 0.27: 9.7, 6.8, 4.2,
//     3.7 and 6.3, 5.2, 4.4, 3.9; 2^21 of degree 4, shares 0.13, 0.33, 0.39: 1.29,
//     1.34, 1.21 and 1.19, 1.23, 1.16; 2^23 of degree 8, shares 0.03, 0.14, 0.19:
//     10.8, 7.6, 6.1 and 7.0, 6.7, 6.3; degree 2, 2^22, share 0.09: 1.82 and 1.87;
//     2^20 of degree 4, 16, 64, share 0.2: 0.81, 1.44, 3.4 and 0.87, 1.33, 2.7; 2^19
//     of degree 32, 64, 100, share 0.3: 1.16, 1.65, 1.98 and 1.13, 1.49, 1.94, of degree
//     64, share 0.47: 1.34 and 1.33; 2^18 of degree 128: 1.06 and 1.20;
//   CC, 2^22 of degree 16, the same shares: 7.2, 4.6, 2.6, 1.9 and 4.4, 3.1, 2.2, 2.0;
//     2^22 of degree 4, share 0.07: 3.6 and 4.0; 2^20 of degree 8, 16, share 0.2:
//     0.62, 0.88 and 0.68, 0.79; about one edge per vertex, 3 M and 4.2 M vertices,
//     uniform: 2.80, 4.25 and 2.54, 3.63; 4.2 M, share 0.16: 2.33 and 2.42; 8.4 M,
//     share 0.08: 6.9 and 7.4.
//
// SSSP on graphs of fewer than 3 edges per vertex gains from neither: a solve
// takes some forty supersteps, few of them dense, and what a pull saves in those
// is spent on keeping every vertex's snapshot in the others.  Row pull (at the
// default fraction) against pushing only: 2^20 vertices of degree 2, share 0.29, 897
// and 834 us; 2^22 of degree 1 1.68 and 1.47 ms, 2, shares 0.09, 0.28, 0.76: 1.76, 1.62,
// 1.00 and 1.56, 1.43, 1.14 ms; 2^23 of degree 2, shares 0.05, 0.20, 0.67: 2.86, 3.18,
// 1.48 and 2.42, 2.46, 1.70 ms.
struct SweepRule {
    bool in = false, sym = false, push = false;
};
static SweepRule sweep_rule(const gx_graph_desc *d) {
    SweepRule r;
    const int64_t V = d->V, E = d->E;
    if (!(d->needs & (GX_NEED_OUT | GX_NEED_SYM)) || V < SWEEP_V_MIN || V > SWEEP_V_MAX || 2 * E < V ||
        sweep_groups(V) * SWEEP_VT > E)
        return r;
    // the edges of the PULL_BITS largest out-degrees (fewer than that many have FAR or more)
    constexpr int32_t FAR = 1 << 16;
    std::unique_ptr<int32_t[]> count(new (std::nothrow) int32_t[FAR]());
    if (!count) return r;
    int64_t left = PULL_BITS, edges = 0;
    for (int64_t v = 0; v < V; v++) {
        const int32_t n = d->row_ptr[v + 1] - d->row_ptr[v];
        if (n < FAR) count[n]++;
        else edges += n, left--;
    }
    for (int32_t x = FAR - 1; x > 0 && left > 0; x--) {
        const int64_t n = std::min<int64_t>(left, count[x]);
        edges += n * x;
        left -= n;
    }
    const double share = (double)edges / (double)E;
    const double mv = (double)V / (double)(1 << 20), degree = (double)E / (double)V;
    const bool large = mv >= 1.5;  // (below, the values fit or nearly)
    r.push = mv >= 1 && degree < 3 && share < 0.45;
    r.in = (d->needs & GX_NEED_OUT) && degree >= (large ? 3 : mv >= 1 ? 12 : 32) &&
           share * share * std::sqrt(degree) * mv < 0.8;
    const bool few = degree < 1.8 && large && mv < 6 && share * std::cbrt(mv) < 0.22;
    r.sym = (d->needs & GX_NEED_SYM) && (few || (mv >= 1 && degree >= (large ? 6 : 12) && share * std::cbrt(mv) < 0.38));
    return r;
}

// The sweep's records from a CSR over destinations (rows) listing sources.
// Destinations are taken in blocks of 2^SWEEP_SLICE_SHIFT and dealt to the
// bins greedily, heaviest in-edge count first, each to the lightest bin so far.
// Bin j belongs to slice j mod PULL_SLICES; an XCD sweeps its bins one after
// another.  Weighted records are {dst, (src mod SWEEP_BAND) << 8 | w} (the unit
// names the band); with `w` null they are {dst, src mod SWEEP_BAND}, alike.
static void build_sweep(const std::vector<int32_t> &rp, const int32_t *src, const uint32_t *w,
                        HostImages::SweepRecs &out) {
    const int64_t V = (int64_t)rp.size() - 1;
    const int64_t nb = (V >> SWEEP_BAND_BITS) + 1;
    const int64_t nbin = sweep_bins(V), S = nbin / PULL_SLICES;
    const int64_t nblk = (V + (1 << SWEEP_SLICE_SHIFT) - 1) >> SWEEP_SLICE_SHIFT;
    std::vector<int64_t> bcnt((size_t)nblk, 0);
    for (int64_t b = 0; b < nblk; b++)
        bcnt[b] = rp[std::min(V, (b + 1) << SWEEP_SLICE_SHIFT)] - rp[b << SWEEP_SLICE_SHIFT];
    std::vector<int64_t> order((size_t)nblk);
    for (int64_t i = 0; i < nblk; i++) order[i] = i;
    std::stable_sort(order.begin(), order.end(), [&](int64_t a, int64_t b) { return bcnt[a] > bcnt[b]; });
    // group index of block b's bin: slices are contiguous, their bins in order
    std::vector<int32_t> group((size_t)nblk, 0);
    std::vector<std::vector<int32_t>> blocks((size_t)PULL_SLICES);  // each slice's blocks, ascending
    using Bin = std::pair<int64_t, int64_t>;  // in-edges so far, bin
    std::priority_queue<Bin, std::vector<Bin>, std::greater<Bin>> lightest;
    for (int64_t j = 0; j < nbin; j++) lightest.push({0, j});
    for (int64_t b : order) {
        const auto [n, j] = lightest.top();
        lightest.pop();
        lightest.push({n + bcnt[b], j});
        group[b] = (int32_t)((j % PULL_SLICES) * S + j / PULL_SLICES);
    }
    for (int64_t b = 0; b < nblk; b++) blocks[group[b] / S].push_back((int32_t)b);
    const int64_t ng = nbin * nb;
    std::vector<int64_t> cnt((size_t)ng, 0);
    // one thread per slice: it owns the groups of its bins, so the counts and
    // the fill below need no shared counters
    auto per_slice = [&](auto &&body) {
        parallel_for(PULL_SLICES, [&](int64_t lo, int64_t hi) {
            for (int64_t x = lo; x < hi; x++)
                for (const int32_t b : blocks[x]) {
                    const int64_t v1 = std::min(V, (int64_t)(b + 1) << SWEEP_SLICE_SHIFT);
                    for (int64_t v = (int64_t)b << SWEEP_SLICE_SHIFT; v < v1; v++) body(v, group[b] * nb);
                }
        }, 1);
    };
    per_slice([&](int64_t v, int64_t g0) {
        for (int32_t e = rp[v]; e < rp[v + 1]; e++) cnt[g0 + (src[e] >> SWEEP_BAND_BITS)]++;
    });
    std::vector<int64_t> pos((size_t)ng + 1, 0);
    for (int64_t g = 0; g < ng; g++) pos[g + 1] = pos[g] + (cnt[g] + SWEEP_VT - 1) / SWEEP_VT * SWEEP_VT;
    out.rec.resize((size_t)pos[ng]);  // every slot is written below: a record or a sentinel
    for (int64_t g = 0; g < ng; g++)
        for (int64_t i = pos[g] + cnt[g]; i < pos[g + 1]; i++) out.rec[i] = make_uint2(SWEEP_SENTINEL, 0u);
    std::vector<int64_t> fill(pos.begin(), pos.end() - 1);
    per_slice([&](int64_t v, int64_t g0) {
        for (int32_t e = rp[v]; e < rp[v + 1]; e++) {
            const uint32_t u = (uint32_t)src[e];
            out.rec[fill[g0 + (u >> SWEEP_BAND_BITS)]++] =
                make_uint2((uint32_t)v, (u & (SWEEP_BAND - 1)) << 8 | (w ? w[e] : 0u));
        }
    });
    out.units.clear();
    for (int x = 0; x < PULL_SLICES; x++) {
        out.uoff[x] = (int64_t)out.units.size();
        for (int64_t g = x * S * nb; g < (x + 1) * S * nb; g++)
            for (int64_t s0 = pos[g]; s0 < pos[g + 1]; s0 += SWEEP_UNIT)
                out.units.push_back(make_uint4((uint32_t)s0, (uint32_t)std::min<int64_t>(SWEEP_UNIT, pos[g + 1] - s0),
                                               (uint32_t)((g % nb) << SWEEP_BAND_BITS), 0u));
    }
    out.uoff[PULL_SLICES] = (int64_t)out.units.size();
    out.recs.reserve(out.units.size());
    for (const uint4 &u : out.units) out.recs.push_back(u.y);
}

static void build_sym(const gx_graph_desc *d, HostImages &h) {
    int64_t V = d->V;
    const int32_t *orp = d->row_ptr, *oc = d->col;
    const int32_t *irp = h.in_rp.data(), *ic = h.in_col.data();
    auto merge_row = [&](int64_t u, int32_t *out, bool &up) -> int32_t {
        int32_t a = orp[u], ae = orp[u + 1], b = irp[u], be = irp[u + 1], n = 0, last = -1;
        while (a < ae || b < be) {
            int32_t x;
            if (b >= be || (a < ae && oc[a] <= ic[b])) x = oc[a++];
            else x = ic[b++];
            if (x == (int32_t)u || x == last) continue;
            if (out) out[n] = x;
            n++;
            up &= x > last;
            last = x;
        }
        return n;
    };
    // Out-rows that the caller did not sort leave rows that do not ascend and
    // may hold a neighbour twice: no one neighbour then stands for a row.
    std::atomic<bool> ascending{true};
    h.sym_rp.assign(V + 1, 0);
    parallel_for(V, [&](int64_t lo, int64_t hi) {
        bool up = true;
        for (int64_t u = lo; u < hi; u++) h.sym_rp[u + 1] = merge_row(u, nullptr, up);
        if (!up) ascending = false;
    });
    h.sym_ascending = ascending;
    for (int64_t v = 0; v < V; v++) h.sym_rp[v + 1] += h.sym_rp[v];
    h.sym_col.resize(h.sym_rp[V]);
    parallel_for(V, [&](int64_t lo, int64_t hi) {
        bool up = true;
        for (int64_t u = lo; u < hi; u++) merge_row(u, h.sym_col.data() + h.sym_rp[u], up);
    });
}

static void build_flags(const gx_graph_desc *d, int32_t W, HostImages &h) {
    h.rem_out.assign(W, 0);
    h.rem_any.assign(W, 0);
    h.master.assign(W, 0);
    h.master_rep.assign(W, 0);
    if (!d->flags) return;
    for (int64_t v = 0; v < d->V; v++) {
        uint32_t bit = 1u << (v & 31);
        const uint8_t f = d->flags[v];
        if (f & GX_FLAG_REMOTE_OUT) h.rem_out[v >> 5] |= bit;
        if (f & GX_FLAG_REMOTE_ANY) h.rem_any[v >> 5] |= bit;
        if (f & GX_FLAG_MASTER) h.master[v >> 5] |= bit;
        if ((f & GX_FLAG_MASTER) && (f & GX_FLAG_REMOTE_ANY)) h.master_rep[v >> 5] |= bit;
        if (d->outdeg_global && !(f & GX_FLAG_MASTER) && (f & GX_FLAG_REMOTE_ANY) && h.in_rp[v + 1] > h.in_rp[v])
            h.part_list.push_back((int32_t)v);
    }
}

// Device layout; with a measuring Carver it only sizes the arena.  E_sym
// must be known for the symmetric image (computed by the caller).
static void take_sweep(int64_t V, int64_t E, Carver &c, Sweep *s) {
    s->rec = c.take<uint2>(sweep_rec_cap(V, E));
    s->units = c.take<uint4>(sweep_unit_cap(V, E));
}

static void layout(const gx_graph_desc *desc, int64_t E_sym, const SweepRule &sweep, Carver &c, DevGraph *d) {
    int64_t V = desc->V, E = desc->E;
    d->V = V;
    d->E = E;
    d->E_sym = E_sym;
    d->W = (int32_t)((V + 31) / 32);
    if (desc->needs & GX_NEED_OUT) {
        d->out_rp = c.take<int32_t>(V + 1);
        d->out_adj = c.take<uint2>(E);
    }
    if (desc->needs & (GX_NEED_IN | GX_NEED_OUT)) {
        d->in_rp = c.take<int32_t>(V + 1);
        d->pr_tile = pr_tile_for(desc);
    }
    if (desc->needs & GX_NEED_IN) {
        d->nz = c.take<int2>(std::min(V, E));
        d->row_last = c.take<uint64_t>((E + PR_TILE_MAX) / 64 + 1);  // (whole tiles)
        // (byte offsets of the other slots are 32 bits)
        d->pr_hot = E >= PR_LDS_EDGES && V >= PR_LDS_SLOTS && V < (int64_t(1) << 29);
        d->pr_rows.T = d->pr_tile / (PR_BLOCK / 64);
        d->bp_rows.T = bp_rows_tile(E);
        for (RowTiles *r : {&d->pr_rows, &d->bp_rows}) {
            r->n = (E + r->T - 1) / r->T;
            r->tile_nz = c.take<int32_t>(r->n + 1);
            r->cross = c.take<int4>(r->n);
        }
        d->nz_slot = c.take<int32_t>(std::min(V, E));
        d->ez = c.take<int2>(V);
        d->dang = c.take<int32_t>(std::min(V, E) + 64);
        d->outdeg = c.take<int32_t>(V);
        d->pr_src = c.take<int32_t>(E + PR_TILE_MAX);  // (read in whole tiles)
    }
    if (desc->needs & (GX_NEED_IN | GX_NEED_OUT)) d->slot = c.take<int32_t>(V);
    if ((desc->needs & GX_NEED_OUT) && (desc->E == 0 || byte_weights(desc))) {
        d->in_adj = c.take<uint2>(E);
        d->in_blk = c.take<int32_t>((V + 63) / 64 + 1);
        d->pull_segs = c.take<uint4>(pull_seg_cap(E));
        d->packs = c.take<uint4>(pull_pack_cap(V, E));
        if (sweep.in) take_sweep(V, E, c, &d->sweep_in);
    }
    if (desc->needs & GX_NEED_SYM) {
        d->sym_rp = c.take<int32_t>(V + 1);
        d->sym_col = c.take<int32_t>(E_sym);
        d->sym_segs = c.take<uint4>(pull_seg_cap(E_sym));
        if (sweep.sym) take_sweep(V, E_sym, c, &d->sweep_sym);
    }
    if (desc->l2g) d->l2g = c.take<int32_t>(V);
    if (desc->outdeg_global) {
        d->outdeg_g = c.take<int32_t>(V);
        d->V_global = desc->V_global;
        if (desc->flags) d->part_list = c.take<int32_t>(V);
    }
    if (desc->flags) {
        d->remote_out = c.take<uint32_t>(d->W);
        d->remote_any = c.take<uint32_t>(d->W);
        d->master = c.take<uint32_t>(d->W);
        d->master_rep = c.take<uint32_t>(d->W);
    }
}

// Upper bound of the symmetric image without building it: every directed
// edge contributes at most two neighbour entries.
static int64_t sym_bound(const gx_graph_desc *d) { return 2 * d->E; }

// Streams byte ranges produced by `fill` to device memory in fixed blocks
// through three rotating pinned buffers on a dedicated copy stream.
struct Uploader {
    static constexpr size_t BLOCK = size_t(16) << 20;
    size_t block = BLOCK;  // bytes of a buffer (less for a small graph: pinning memory costs)
    size_t used = 0;       // bytes of the current buffer taken: small arrays share one
    hipStream_t copy = nullptr;
    void *buf[3] = {nullptr, nullptr, nullptr};
    hipEvent_t ev[3] = {nullptr, nullptr, nullptr};
    uint64_t idx = 0;
    hipError_t err = hipSuccess;

    hipError_t open(size_t total) {
        block = std::min(BLOCK, align_up(std::max<size_t>(total, 1), size_t(64) << 10));
        if ((err = hipStreamCreateWithFlags(&copy, hipStreamNonBlocking)) != hipSuccess) return err;
        for (int i = 0; i < 3; i++) {
            if ((err = hipHostMalloc(&buf[i], block, hipHostMallocDefault)) != hipSuccess) return err;
            if ((err = hipEventCreateWithFlags(&ev[i], hipEventDisableTiming)) != hipSuccess) return err;
        }
        return hipSuccess;
    }
    // The current buffer is full: the next one, once its last copies are done.
    void turn() {
        err = hipEventRecord(ev[idx % 3], copy);
        idx++;
        used = 0;
        if (err == hipSuccess) err = hipEventSynchronize(ev[idx % 3]);
    }
    hipError_t put(void *dev, size_t bytes, const std::function<void(char *, size_t, size_t)> &fill) {
        for (size_t off = 0, n; off < bytes && err == hipSuccess; off += n) {
            n = std::min(block, bytes - off);
            if (used + n > block) turn();
            if (err != hipSuccess) break;
            char *at = static_cast<char *>(buf[idx % 3]) + used;
            fill(at, off, n);  // package block (host)
            err = hipMemcpyAsync(static_cast<char *>(dev) + off, at, n, hipMemcpyHostToDevice, copy);
            used = std::min(block, align_up(used + n));
        }
        return err;
    }
    hipError_t put_array(void *dev, const void *host, size_t bytes) {
        return put(dev, bytes, [host](char *dst, size_t off, size_t n) {  // copied in 1 MiB pieces on the host threads
            const int64_t pieces = (int64_t)((n + (size_t(1) << 20) - 1) >> 20);
            parallel_for(
                pieces,
                [&](int64_t lo, int64_t hi) {
                    for (int64_t i = lo; i < hi; i++) {
                        const size_t a = (size_t)i << 20, len = std::min(n - a, size_t(1) << 20);
                        std::memcpy(dst + a, static_cast<const char *>(host) + off + a, len);
                    }
                },
                2);
        });
    }
    hipError_t finish(hipStream_t user) {
        hipEvent_t done = nullptr;
        if (err == hipSuccess) err = hipEventCreateWithFlags(&done, hipEventDisableTiming);
        if (err == hipSuccess) err = hipEventRecord(done, copy);
        if (err == hipSuccess) err = hipStreamWaitEvent(user, done, 0);
        if (err == hipSuccess) err = hipStreamSynchronize(copy);
        if (done) (void)hipEventDestroy(done);
        return err;
    }
    ~Uploader() {
        if (copy) (void)hipStreamSynchronize(copy);
        for (int i = 0; i < 3; i++) {
            if (ev[i]) (void)hipEventDestroy(ev[i]);
            if (buf[i]) (void)hipHostFree(buf[i]);
        }
        if (copy) (void)hipStreamDestroy(copy);
    }
};

}  // namespace gx

using namespace gx;

extern "C" const char *gx_last_error(void) { return g_err.c_str(); }
extern "C" const char *gx_version(void) { return "gx 0.1 (gfx950)"; }

extern "C" gx_status gx_graph_bytes(const gx_graph_desc *desc, size_t *arena_bytes) {
    clear_error();
    GX_REQUIRE(arena_bytes, GX_EINVAL, "arena_bytes is NULL");
    gx_status st = validate(desc);
    if (st != GX_OK) return st;
    Carver c(nullptr, 0);
    DevGraph d;
    layout(desc, sym_bound(desc), sweep_rule(desc), c, &d);
    *arena_bytes = c.used;
    return GX_OK;
}

extern "C" gx_status gx_graph_load(const gx_graph_desc *desc, void *dev_arena, size_t arena_bytes, void *stream,
                                   gx_graph **out) {
    clear_error();
    GX_REQUIRE(out, GX_EINVAL, "out is NULL");
    *out = nullptr;
    gx_status st = validate(desc);
    if (st != GX_OK) return st;
    GX_REQUIRE(dev_arena || arena_bytes == 0, GX_EINVAL, "dev_arena is NULL");
    GX_REQUIRE(reinterpret_cast<uintptr_t>(dev_arena) % ALIGN == 0, GX_EINVAL, "dev_arena not 256-byte aligned");
    const SweepRule sweep = sweep_rule(desc);
    {
        Carver m(nullptr, 0);
        DevGraph tmp;
        layout(desc, sym_bound(desc), sweep, m, &tmp);
        GX_REQUIRE(m.used <= arena_bytes, GX_ENOMEM, "arena too small: need %zu bytes, have %zu", m.used, arena_bytes);
    }

    HostImages h;
    int32_t W = (int32_t)((desc->V + 31) / 32);
    try {
        build_in_csr(desc, h);
        if (desc->needs & (GX_NEED_IN | GX_NEED_OUT)) build_slots(desc, h);
        if (desc->needs & GX_NEED_IN) {
            build_rows(desc, h);
            const int64_t T = pr_tile_for(desc) / (PR_BLOCK / 64);
            build_row_tiles(desc->E, T, h, h.pr_rows);
            build_row_tiles(desc->E, bp_rows_tile(desc->E), h, h.bp_rows);
            h.pr_src.resize((desc->E + T - 1) / T * T);
            parallel_for(desc->E, [&](int64_t lo, int64_t hi) {
                for (int64_t e = lo; e < hi; e++) h.pr_src[e] = h.slot[h.in_col[e]];
            });
            std::fill(h.pr_src.begin() + desc->E, h.pr_src.end(), (int32_t)desc->V);  // (no slot)
        }
        if ((desc->needs & GX_NEED_OUT) && desc->E > 0 && byte_weights(desc)) {
            build_in_adj(h);
            if (sweep.in) build_sweep(h.in_rp, h.in_col.data(), h.in_w.data(), h.sweep_in);
        }
        if (desc->needs & GX_NEED_SYM) {
            build_sym(desc, h);
            build_segs(h.sym_rp, h.sym_segs);
            if (sweep.sym) build_sweep(h.sym_rp, h.sym_col.data(), nullptr, h.sweep_sym);
        }
        build_flags(desc, W, h);
    } catch (const std::bad_alloc &) {
        set_error("host allocation failed while packaging the graph");
        return GX_ENOMEM;
    } catch (const std::exception &ex) {
        set_error("graph packaging failed: %s", ex.what());
        return GX_EINVAL;
    }

    gx_graph *g = new (std::nothrow) gx_graph();
    GX_REQUIRE(g, GX_ENOMEM, "host allocation failed");
    Carver c(dev_arena, arena_bytes);
    layout(desc, (int64_t)h.sym_col.size(), sweep, c, &g->d);
    g->d.pr_hot = g->d.pr_hot && h.lds_edges * PR_LDS_PART >= desc->E;
    g->d.pull_nsegs = (int64_t)h.pull_segs.size();
    g->d.n_nz = (int64_t)h.nz.size();
    g->d.n_ez = (int64_t)h.ez.size();
    g->d.n_part = (int64_t)h.part_list.size();
    for (auto [r, t] : {std::pair(&g->d.pr_rows, &h.pr_rows), std::pair(&g->d.bp_rows, &h.bp_rows)}) {
        r->n_cross = (int32_t)t->cross.size();
        r->n_long = t->n_long;
        r->n_mid = t->n_mid;
    }
    g->d.n_dang = (int64_t)h.dang.size();
    g->d.n_packs = (int64_t)h.packs.size();
    g->d.sym_nsegs = (int64_t)h.sym_segs.size();
    g->d.sym_ascending = h.sym_ascending;
    g->d.sssp_pushes = sweep.push;
    g->sweep_in_recs = std::move(h.sweep_in.recs);
    g->sweep_sym_recs = std::move(h.sweep_sym.recs);
    std::copy(h.sweep_in.uoff, h.sweep_in.uoff + PULL_SLICES + 1, g->d.sweep_in.uoff);
    std::copy(h.sweep_sym.uoff, h.sweep_sym.uoff + PULL_SLICES + 1, g->d.sweep_sym.uoff);
    g->needs = desc->needs;
    g->arena = dev_arena;
    g->arena_bytes = arena_bytes;
    if (hipGetDevice(&g->device) != hipSuccess) g->device = 0;
    g->num_cus = device_cus(g->device);
    g->host_outdeg.resize(desc->V);
    for (int64_t v = 0; v < desc->V; v++) g->host_outdeg[v] = desc->row_ptr[v + 1] - desc->row_ptr[v];
    if (!h.sym_rp.empty()) {
        g->host_symdeg.resize(desc->V);
        for (int64_t v = 0; v < desc->V; v++) g->host_symdeg[v] = h.sym_rp[v + 1] - h.sym_rp[v];
    }

    hipStream_t s = static_cast<hipStream_t>(stream);
    Uploader up;
    hipError_t e = up.open(c.used);
    const DevGraph &d = g->d;
    int64_t V = desc->V, E = desc->E;
    if (e == hipSuccess && d.out_rp) e = up.put_array((void *)d.out_rp, desc->row_ptr, (V + 1) * 4);
    if (e == hipSuccess && d.out_adj) {
        const int32_t *col = desc->col;
        const uint32_t *w = desc->w;
        // Package (destination, weight) pairs block by block.
        e = up.put((void *)d.out_adj, E * sizeof(uint2), [col, w](char *dst, size_t off, size_t n) {
            uint2 *o = reinterpret_cast<uint2 *>(dst);
            const size_t e0 = off / sizeof(uint2), cnt = n / sizeof(uint2);
            parallel_for((int64_t)cnt, [&](int64_t lo, int64_t hi) {
                for (int64_t i = lo; i < hi; i++) o[i] = make_uint2((uint32_t)col[e0 + i], w[e0 + i]);
            });
        });
    }
    if (e == hipSuccess && d.in_rp) {
        e = up.put_array((void *)d.in_rp, h.in_rp.data(), (V + 1) * 4);
    }
    if (e == hipSuccess && d.pr_src) {
        e = up.put_array((void *)d.outdeg, g->host_outdeg.data(), V * 4);
        if (e == hipSuccess) e = up.put_array((void *)d.nz, h.nz.data(), h.nz.size() * sizeof(int2));
        if (e == hipSuccess) e = up.put_array((void *)d.nz_slot, h.nz_slot.data(), h.nz_slot.size() * 4);
        if (e == hipSuccess) e = up.put_array((void *)d.ez, h.ez.data(), h.ez.size() * sizeof(int2));
        if (e == hipSuccess) e = up.put_array((void *)d.row_last, h.row_last.data(), h.row_last.size() * 8);
        for (auto [r, t] : {std::pair(&d.pr_rows, &h.pr_rows), std::pair(&d.bp_rows, &h.bp_rows)}) {
            if (e == hipSuccess) e = up.put_array((void *)r->tile_nz, t->tile_nz.data(), t->tile_nz.size() * 4);
            if (e == hipSuccess) e = up.put_array((void *)r->cross, t->cross.data(), t->cross.size() * sizeof(int4));
        }
        if (e == hipSuccess) e = up.put_array((void *)d.dang, h.dang.data(), h.dang.size() * 4);
        if (e == hipSuccess) e = up.put_array((void *)d.pr_src, h.pr_src.data(), h.pr_src.size() * 4);
    }
    if (e == hipSuccess && d.slot) e = up.put_array((void *)d.slot, h.slot.data(), V * 4);
    if (e == hipSuccess && d.in_adj && !h.in_adj.empty()) {
        e = up.put_array((void *)d.in_blk, h.in_blk.data(), h.in_blk.size() * 4);
        if (e == hipSuccess) e = up.put_array((void *)d.in_adj, h.in_adj.data(), h.in_adj.size() * sizeof(uint2));
        if (e == hipSuccess)
            e = up.put_array((void *)d.pull_segs, h.pull_segs.data(), h.pull_segs.size() * sizeof(uint4));
        if (e == hipSuccess) e = up.put_array((void *)d.packs, h.packs.data(), h.packs.size() * sizeof(uint4));
    }
    for (auto [r, t] : {std::pair(&d.sweep_in, &h.sweep_in), std::pair(&d.sweep_sym, &h.sweep_sym)}) {
        if (e == hipSuccess && r->rec) e = up.put_array((void *)r->rec, t->rec.data(), t->rec.size() * sizeof(uint2));
        if (e == hipSuccess && r->rec) e = up.put_array((void *)r->units, t->units.data(), t->units.size() * sizeof(uint4));
    }
    if (e == hipSuccess && d.sym_rp) {
        e = up.put_array((void *)d.sym_rp, h.sym_rp.data(), (V + 1) * 4);
        if (e == hipSuccess) e = up.put_array((void *)d.sym_col, h.sym_col.data(), h.sym_col.size() * 4);
        if (e == hipSuccess)
            e = up.put_array((void *)d.sym_segs, h.sym_segs.data(), h.sym_segs.size() * sizeof(uint4));
    }
    if (e == hipSuccess && d.l2g) e = up.put_array((void *)d.l2g, desc->l2g, V * 4);
    if (e == hipSuccess && d.outdeg_g) e = up.put_array((void *)d.outdeg_g, desc->outdeg_global, V * 4);
    if (e == hipSuccess && d.remote_out) {
        e = up.put_array((void *)d.remote_out, h.rem_out.data(), (size_t)W * 4);
        if (e == hipSuccess) e = up.put_array((void *)d.remote_any, h.rem_any.data(), (size_t)W * 4);
        if (e == hipSuccess) e = up.put_array((void *)d.master, h.master.data(), (size_t)W * 4);
        if (e == hipSuccess && d.part_list) e = up.put_array((void *)d.part_list, h.part_list.data(), h.part_list.size() * 4);
        if (e == hipSuccess) e = up.put_array((void *)d.master_rep, h.master_rep.data(), (size_t)W * 4);
    }
    if (e == hipSuccess) e = up.finish(s);
    if (e != hipSuccess) {
        set_error("graph upload failed: %s", hipGetErrorString(e));
        delete g;
        return GX_EDEVICE;
    }
    *out = g;
    return GX_OK;
}

extern "C" gx_status gx_graph_free(gx_graph *g) {
    clear_error();
    delete g;
    return GX_OK;
}

extern "C" gx_status gx_graph_info(const gx_graph *g, int64_t *V, int64_t *E, uint32_t *needs) {
    clear_error();
    GX_REQUIRE(g, GX_EINVAL, "graph is NULL");
    if (V) *V = g->d.V;
    if (E) *E = g->d.E;
    if (needs) *needs = g->needs;
    return GX_OK;
}
