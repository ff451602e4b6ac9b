"""The work the engine's speed is measured on: one pass of each path a program
drives through the public entry points, over the sizes those programs have.

Graphs are seeded R-MAT edge lists (a, b, c, d = 0.57, 0.19, 0.19, 0.05) with
self-loops and duplicates removed and weights in [1, 255] unless a case says
otherwise, made on the GPU and handed over as the host CSR that a program
loads.  ``V`` below 2^scale drops the vertices past it (ragged sizes), and
``shuffled`` relabels the vertices at random, as the ids of a crawled graph
are (R-MAT alone puts its hubs at the lowest ids).
"""
import math

import numpy as np
import torch

import paper_2203_13005_amd as gx

DEV = "cuda:0"
DAMPING = 0.85
CHUNK = 1 << 26  # raw edges drawn at a time


# ------------------------------------------------------------------ cases

def listed():
    return [
        # PageRank at the smallest size the benchmark runs: the graph fits in cache, latency counts
        dict(name="pagerank_rmat14", path="pagerank", scale=14, V=1 << 14, ef=16, steps=20, shuffled=False),
        # PageRank on a graph that fills the card's caches many times over
        dict(name="pagerank_rmat22", path="pagerank", scale=22, V=1 << 22, ef=16, steps=20, shuffled=False),
        # single-source distances on a small graph: a solve of a dozen short supersteps
        dict(name="sssp_rmat12", path="sssp", scale=12, V=1 << 12, ef=16, wmax=255, shuffled=False),
        # the benchmark's headline solve
        dict(name="sssp_rmat22", path="sssp", scale=22, V=1 << 22, ef=16, wmax=255, shuffled=False),
        # one worker's part (1 of 8) of a vertex-cut: components to convergence and the sync set it sends
        dict(name="cc_part_rmat24", path="cc_part", scale=24, V=1 << 24, ef=16, nparts=8, shuffled=False),
        # label propagation with the evaluation's cap of 15 iterations, arbitrary vertex ids
        dict(name="lp_rmat20_shuffled", path="lp", scale=20, V=1 << 20, ef=16, steps=15, shuffled=True),
        # 32 sources at once on a ragged mid-size graph (the narrowest batch)
        dict(name="batch_sssp_32_v50000", path="batch_sssp", scale=16, V=50_000, ef=12, lanes=32, shuffled=False),
        # the benchmark's batch: 256 sources
        dict(name="batch_sssp_256_rmat20", path="batch_sssp", scale=20, V=1 << 20, ef=16, lanes=256, shuffled=False),
        # a handful of personalised PageRank seeds on a ragged graph with arbitrary ids
        dict(name="batch_ppr_5_v100003", path="batch_ppr", scale=17, V=100_003, ef=16, lanes=5, steps=50,
             shuffled=True),
        # the benchmark's personalised PageRank batch: one pool's width
        dict(name="batch_ppr_64_rmat20", path="batch_ppr", scale=20, V=1 << 20, ef=16, lanes=64, steps=50,
             shuffled=False),
        # PageRank across the parts of a vertex-cut: the template's separate calls and the exchange
        dict(name="exchange_pagerank_rmat18", path="exchange", scale=18, V=1 << 18, ef=16, nparts=4, steps=10,
             shuffled=False),
        # a burst of mixed queries on a server that keeps two graphs resident
        dict(name="serve_48_rmat16", path="serve", scale=16, V=1 << 16, ef=16, queries=48, shuffled=False),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _sized(rng, lo, hi):
    """A vertex count spread over its logarithm, most of them no power of two."""
    V = _log(rng, lo, hi)
    scale = max(1, (V - 1).bit_length())
    if rng.random() < 0.25:
        V = 1 << scale
        if V > hi:
            V, scale = V // 2, scale - 1
    return dict(scale=scale, V=V, ef=rng.choice([8, 12, 16]), shuffled=rng.random() < 0.5)


def draw(rng):
    path = rng.choice(["pagerank", "pagerank", "sssp", "sssp", "cc_part", "lp", "batch_sssp", "batch_ppr",
                       "exchange", "serve"])
    c = dict(path=path)
    if path == "pagerank":
        c.update(_sized(rng, 1 << 11, 1 << 22), steps=rng.choice([10, 15, 20]))
    elif path == "sssp":
        c.update(_sized(rng, 1 << 11, 1 << 22), wmax=rng.choice([1, 15, 255, 255, 65535]))
    elif path == "cc_part":
        c.update(_sized(rng, 1 << 14, 1 << 24), nparts=rng.choice([2, 4, 8]))
        if c["nparts"] < 8:
            c["V"] = min(c["V"], 1 << 22)
            c["scale"] = max(1, (c["V"] - 1).bit_length())
    elif path == "lp":
        c.update(_sized(rng, 1 << 11, 1 << 20), steps=15)
    elif path == "batch_sssp":
        c.update(_sized(rng, 1 << 12, 1 << 19), lanes=rng.choice([32, 64, 96, 128, 256]))
    elif path == "batch_ppr":
        c.update(_sized(rng, 1 << 12, 1 << 19), lanes=rng.randrange(1, 129), steps=rng.choice([20, 30, 50]))
    elif path == "exchange":
        c.update(_sized(rng, 1 << 13, 1 << 18), nparts=rng.choice([2, 3, 4]), steps=10)
    else:
        c.update(_sized(rng, 1 << 13, 1 << 16), queries=rng.randrange(8, 49))
    return c


# ------------------------------------------------------------------ inputs

class _Csr:
    """The host arrays of one loaded graph (out-CSR, rows sorted by destination)."""

    def __init__(self, V, u, v, w, l2g=None, flags=None):
        rp = torch.zeros(V + 1, dtype=torch.int64, device=DEV)
        if u.numel():
            rp[1:] = torch.cumsum(torch.bincount(u, minlength=V), 0)
        self.V, self.E = int(V), int(u.numel())
        self.row_ptr = rp.to(torch.int32).cpu().numpy()
        self.col = v.to(torch.int32).cpu().numpy()
        self.w = w.to(torch.int32).cpu().numpy().view(np.uint32)
        self.l2g = None if l2g is None else l2g.to(torch.int32).cpu().numpy()
        self.flags = None if flags is None else flags.cpu().numpy()


def _keys(case, gen, keep=None, seen=None):
    """Sorted distinct edge keys u * V + v; ``keep`` filters a chunk's edges
    (after ``seen`` looked at all of them)."""
    V, scale = case["V"], case["scale"]
    E = case["ef"] * V
    perm = torch.randperm(V, generator=gen, device=DEV) if case["shuffled"] else None
    out = []
    for lo in range(0, E, CHUNK):
        n = min(CHUNK, E - lo)
        u = torch.zeros(n, dtype=torch.int64, device=DEV)
        v = torch.zeros(n, dtype=torch.int64, device=DEV)
        for _ in range(scale):
            r = torch.rand(n, generator=gen, device=DEV)
            u.mul_(2).add_(r >= 0.76)
            v.mul_(2).add_((r >= 0.95) | ((r >= 0.57) & (r < 0.76)))
        ok = (u != v) & (u < V) & (v < V)
        u, v = u[ok], v[ok]
        if perm is not None:
            u, v = perm[u], perm[v]
        if seen is not None:
            seen(u, v)
        if keep is not None:
            m = keep(u, v)
            u, v = u[m], v[m]
        out.append(torch.unique(u * V + v))
    return torch.unique(torch.cat(out)) if len(out) > 1 else out[0]


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 7919 + 17)


def _weights(n, case, gen):
    return torch.randint(1, case.get("wmax", 255) + 1, (n,), generator=gen, device=DEV)


def _edges(case, seed):
    gen = _gen(seed)
    k = _keys(case, gen)
    V = case["V"]
    return k // V, k % V, _weights(k.numel(), case, gen), gen


def _part_of(u, v, nparts):
    """The part an edge belongs to (a hash of both ends)."""
    h = (u * 0x2545F491 + v * 0x9E3779B1) & 0x7FFFFFFF
    return ((h ^ (h >> 15)) * 0x2C1B3C6D >> 12) % nparts


def _flags(l2g, out_all, any_all, part):
    """GX_FLAG_* bits from per-vertex part bit masks over the whole graph."""
    other = ~(1 << part)
    a = any_all[l2g]
    low = a & -a  # the lowest part that holds the vertex has the master copy
    f = (low == (1 << part)).to(torch.uint8)
    f |= (((out_all[l2g] & other) != 0).to(torch.uint8) << 1)
    f |= (((a & other) != 0).to(torch.uint8) << 2)
    return f


def _one_part(case, seed):
    """Part 0 of the vertex-cut, without the other parts' edges in memory."""
    V, P = case["V"], case["nparts"]
    out_all = torch.zeros(V, dtype=torch.int32, device=DEV)
    any_all = torch.zeros(V, dtype=torch.int32, device=DEV)

    def seen(u, v):
        p = _part_of(u, v, P)
        for q in range(P):
            m = p == q
            hit = torch.zeros(V, dtype=torch.bool, device=DEV)
            hit[u[m]] = True
            out_all.bitwise_or_(hit.to(torch.int32) << q)
            hit[v[m]] = True
            any_all.bitwise_or_(hit.to(torch.int32) << q)

    gen = _gen(seed)
    k = _keys(case, gen, keep=lambda u, v: _part_of(u, v, P) == 0, seen=seen)
    u, v = k // V, k % V
    held = (any_all & 1) != 0
    l2g = torch.nonzero(held).flatten()
    loc = torch.cumsum(held, 0) - 1
    fl = _flags(l2g, out_all, any_all, 0)
    return _Csr(l2g.numel(), loc[u], loc[v], _weights(k.numel(), case, gen), l2g, fl)


def _all_parts(case, seed):
    """Every part of the vertex-cut; vertices without an edge are part 0's."""
    V, P = case["V"], case["nparts"]
    u, v, w, _ = _edges(case, seed)
    p = _part_of(u, v, P)
    out_all = torch.zeros(V, dtype=torch.int32, device=DEV)
    any_all = torch.zeros(V, dtype=torch.int32, device=DEV)
    for q in range(P):
        hit = torch.zeros(V, dtype=torch.bool, device=DEV)
        hit[u[p == q]] = True
        out_all |= hit.to(torch.int32) << q
        hit[v[p == q]] = True
        any_all |= hit.to(torch.int32) << q
    any_all[any_all == 0] = 1
    parts = []
    for q in range(P):
        held = (any_all >> q) & 1 != 0
        l2g = torch.nonzero(held).flatten()
        loc = torch.cumsum(held, 0) - 1
        m = p == q
        parts.append(_Csr(l2g.numel(), loc[u[m]], loc[v[m]], w[m], l2g,
                          _flags(l2g, out_all, any_all, q)))
    return parts, torch.bincount(u, minlength=V).to(torch.int32).cpu().numpy()


def _pick(u, V, n, gen):
    """n distinct vertices with an out-edge (repeated where there are fewer)."""
    cand = torch.nonzero(torch.bincount(u, minlength=V)).flatten()
    i = torch.randperm(cand.numel(), generator=gen, device=DEV)
    i = i.repeat(-(-n // max(1, i.numel())))[:n]
    return cand[i].to(torch.int32).cpu().numpy()


def _sources(case, u, gen):
    n = case.get("lanes", case.get("queries", 1))
    return _pick(u, case["V"], n, gen)


def prepare(case, seed):
    path = case["path"]
    if path == "cc_part":
        dg = gx.DeviceGraph(_one_part(case, seed), gx.GX_NEED_SYM)
        # the caller's buffers, large enough for any part: labels, and the sync set's ids and values
        labels, gid, val = (torch.zeros(case["V"], dtype=torch.int32, device=DEV) for _ in range(3))
        return dict(path=path, st=gx.State(dg, gx.GX_CC), labels=labels, buf=(gid, val))
    if path == "exchange":
        parts, deg = _all_parts(case, seed)
        sts = [gx.State(gx.DeviceGraph(p, gx.GX_NEED_IN, V_global=case["V"], outdeg_global=deg[p.l2g]),
                        gx.GX_PAGERANK, damping=DAMPING, phases=gx.GX_PHASES_MASTERS,
                        delta_mode=gx.GX_DELTA_MASTERS) for p in parts]
        ranks = torch.zeros((len(sts), case["V"]), dtype=torch.float32, device=DEV)  # a row for each part
        return dict(path=path, sts=sts, steps=case["steps"], ranks=ranks)
    u, v, w, gen = _edges(case, seed)
    host = _Csr(case["V"], u, v, w)
    if path == "pagerank":
        dg = gx.DeviceGraph(host, gx.GX_NEED_IN)
        return dict(path=path, st=gx.State(dg, gx.GX_PAGERANK, damping=DAMPING), steps=case["steps"])
    if path == "sssp":
        dg = gx.DeviceGraph(host, gx.GX_NEED_OUT)
        return dict(path=path, st=gx.State(dg, gx.GX_SSSP, source=int(_sources(case, u, gen)[0])))
    if path == "lp":
        return dict(path=path, st=gx.State(gx.DeviceGraph(host, gx.GX_NEED_SYM), gx.GX_LP), steps=case["steps"])
    src = _sources(case, u, gen)
    if path == "serve":
        dg = gx.DeviceGraph(host, gx.GX_NEED_OUT | gx.GX_NEED_IN)
        u2, v2, w2, gen2 = _edges(case, seed + 1_000_003)
        dg2 = gx.DeviceGraph(_Csr(case["V"], u2, v2, w2), gx.GX_NEED_OUT | gx.GX_NEED_IN)
        src2 = _sources(case, u2, gen2)
        srv = gx.Server(2 << 30)
        ids = [srv.add_graph(dg), srv.add_graph(dg2)]
        qs = [(ids[i % 2], gx.GX_SSSP if i % 4 < 2 else gx.GX_PPR, int((src, src2)[i % 2][i]))
              for i in range(case["queries"])]
        return dict(path=path, srv=srv, queries=qs)
    dg = gx.DeviceGraph(host, gx.GX_NEED_OUT if path == "batch_sssp" else gx.GX_NEED_IN)
    out = torch.empty((case["V"], case["lanes"]), dtype=torch.int32 if path == "batch_sssp" else torch.float32,
                      device=DEV)
    return dict(path=path, dg=dg, src=src, out=out, steps=case.get("steps", 0))


# ------------------------------------------------------------------ one pass

def _exchange(sts, steps, ranks):
    for st in sts:
        st.reset()
    for _ in range(steps):
        for st in sts:
            st.msg_gen()
            st.msg_merge()
        D = 0.0
        for st in sts:
            D += st.dangling_get()
        for st in sts:
            st.dangling_set(D)
        sent = [st.partial_emit() for st in sts]
        for q, st in enumerate(sts):
            for p in range(len(sts)):
                if p != q and sent[p][0].numel():
                    st.partial_add(*sent[p])
        for st in sts:
            st.msg_apply(stats=False)
        bc = [st.sync_delta(on_device=True) for st in sts]
        for q, st in enumerate(sts):
            others = [b for p, b in enumerate(bc) if p != q and b[0].numel()]
            if others:
                st.apply_delta(torch.cat([o[0] for o in others]), torch.cat([o[1] for o in others]))
    for row, st in zip(ranks, sts):
        row[:st.graph.V].copy_(st.values())
    return ranks


def run(state):
    path = state["path"]
    if path == "exchange":
        return _exchange(state["sts"], state["steps"], state["ranks"])
    if path == "serve":
        srv = state["srv"]
        order = [srv.submit(*q) for q in state["queries"]]
        done = {}
        while len(done) < len(order):
            for c in srv.poll(wait_ms=100):
                if c.status != gx.GX_OK:
                    raise RuntimeError(f"query {c.id} ended with status {c.status}")
                done[c.id] = c.result
        return [done[i] for i in order]
    if path in ("batch_sssp", "batch_ppr"):
        algo = gx.GX_SSSP if path == "batch_sssp" else gx.GX_PPR
        return gx.batch_run(state["dg"], algo, state["src"], damping=DAMPING, iters=state["steps"],
                            out=state["out"])[0]
    st = state["st"]
    st.reset()
    if path == "pagerank":
        st.run(state["steps"])
        return st.values()
    if path == "lp":
        rs, _ = st.run(state["steps"], allow_cap=True)
        return st.values(), int(rs.supersteps)
    rs, _ = st.run(1 << 20)
    if path == "sssp":
        return st.values(), int(rs.supersteps), int(rs.edges)
    gid, val, _ = st.sync_delta(on_device=True, out=state["buf"])
    state["labels"][:st.graph.V].copy_(st.values())
    return state["labels"], *state["buf"], int(gid.numel()), int(rs.supersteps)


def work(case):
    """Each edge and vertex value a pass cannot do without, once per superstep
    that has to see all of them (PageRank, PPR) and once per pass otherwise."""
    V, E = case["V"], case["ef"] * case["V"]
    path = case["path"]
    if path == "pagerank":
        return dict(bytes=case["steps"] * (4 * E + 8 * V), flops=case["steps"] * 2 * E)
    if path == "sssp":
        return dict(bytes=8 * E + 8 * V, flops=2 * E)
    if path == "cc_part":
        Ep = E // case["nparts"]
        Vp = min(V, Ep)
        return dict(bytes=8 * Ep + 16 * Vp, flops=2 * Ep)
    if path == "lp":
        return dict(bytes=8 * E + 8 * V, flops=2 * E)
    if path == "batch_sssp":
        return dict(bytes=8 * E + 4 * V * case["lanes"], flops=2 * E * case["lanes"])
    if path == "batch_ppr":
        return dict(bytes=case["steps"] * (4 * E + 8 * V * case["lanes"]), flops=case["steps"] * 2 * E * case["lanes"])
    if path == "exchange":
        return dict(bytes=case["steps"] * (4 * E + 8 * V), flops=case["steps"] * 2 * E)
    n = case["queries"]
    return dict(bytes=2 * (12 * E + 8 * V) + 50 * 8 * V * n // 2 + 4 * V * n // 2, flops=(50 + 1) * 2 * E * n // 2)


# ------------------------------------------------------------------ 64-bit values

def _ranks64(V, u, v, steps, seeds=None):
    """PageRank (seeds None) or one personalised PageRank per seed, by sparse
    products in 64 bits."""
    d = float(np.float32(DAMPING))
    deg = torch.bincount(u, minlength=V).to(torch.float64)
    order = torch.argsort(v, stable=True)
    crow = torch.zeros(V + 1, dtype=torch.int32, device=DEV)
    crow[1:] = torch.cumsum(torch.bincount(v, minlength=V), 0).to(torch.int32)
    cols = u[order].to(torch.int32)
    inv = torch.where(deg > 0, 1.0 / deg.clamp(min=1), torch.zeros_like(deg))
    A = torch.sparse_csr_tensor(crow, cols, inv[cols.long()], size=(V, V))
    sink = (deg == 0).to(torch.float64)
    if seeds is None:
        x = torch.full((V, 1), 1.0 / V, dtype=torch.float64, device=DEV)
        for _ in range(steps):
            x = (1.0 - d) / V + d * (A @ x + (sink[:, None] * x).sum(0, keepdim=True) / V)
        return x[:, 0]
    s = torch.as_tensor(np.asarray(seeds), device=DEV).long()
    lane = torch.arange(len(s), device=DEV)
    x = torch.zeros((V, len(s)), dtype=torch.float64, device=DEV)
    x[s, lane] = 1.0
    for _ in range(steps):
        back = (1.0 - d) + d * (sink[:, None] * x).sum(0)
        x = d * (A @ x)
        x[s, lane] += back
    return x


def exact(case, seed):
    path = case["path"]
    if path in ("sssp", "cc_part", "lp", "batch_sssp"):
        return None  # whole numbers
    V = case["V"]
    u, v, w, gen = _edges(case, seed)
    if path == "pagerank":
        return _ranks64(V, u, v, case["steps"])
    if path == "batch_ppr":
        return _ranks64(V, u, v, case["steps"], _sources(case, u, gen))
    if path == "exchange":
        x = _ranks64(V, u, v, case["steps"])
        p = _part_of(u, v, case["nparts"])
        held = torch.zeros((case["nparts"], V), dtype=torch.bool, device=DEV)
        held[p, u] = True
        held[p, v] = True
        held[0] |= ~held.any(0)
        ranks = torch.zeros(held.shape, dtype=torch.float64, device=DEV)
        for row, h in zip(ranks, held):
            row[:int(h.sum())] = x[h]
        return ranks
    u2, v2, w2, gen2 = _edges(case, seed + 1_000_003)
    n = case["queries"]
    out = [None] * n
    for side, (a, b, g) in enumerate(((u, v, gen), (u2, v2, gen2))):
        src = _sources(case, a, g)
        at = [i for i in range(n) if i % 2 == side and i % 4 >= 2]
        if at:
            x = _ranks64(V, a, b, 50, [src[i] for i in at])
            for j, i in enumerate(at):
                out[i] = x[:, j].contiguous()
    return out
