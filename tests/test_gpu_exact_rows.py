"""Rows of exactly the lengths where the pulls change their split, each checked
on the graph as built: PageRank tiles that are full, all but full or hold one
edge, rows that cross few, some and many tiles, both sides of the edge and
vertex counts and of the share of edges from which contributions are kept in
LDS (every tile size, fused and separate calls); batched SSSP rows around the short-row and segment limits;
personalised ranks of both tile sizes.

Ranks are compared with the float64 oracle at the engine's own damping (0.85
rounded to 32 bits) by relative error.  Every rank is a sum of positive terms
in 64 bits, and each superstep rounds a rank and its contribution once to 32
bits (half an ulp each, 2^-24), the start rounds once more: after k supersteps
no rank is further off than (2 k + 1) 2^-24, and a rank is zero only where the
oracle's is."""
import numpy as np
import pytest

import gen
import oracle

from test_gpu_ppr_rows import rows_graph as ppr_rows_graph

pytestmark = pytest.mark.gpu

D = float(np.float32(0.85))


@pytest.fixture(scope="module")
def gx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2203_13005_amd as m
    return m


def near(x, ref, steps):
    x = x.astype(np.float64)
    assert np.array_equal(x == 0, ref == 0)
    m = ref != 0
    assert np.max(np.abs(x[m] - ref[m]) / ref[m], initial=0.0) <= (2 * steps + 1) * 2.0 ** -24


def row_sources(V, M, lengths, seed):
    """(sources, destinations): lengths[i] distinct sources below M, none i itself, for vertex i."""
    rng = np.random.default_rng(seed)
    lengths = np.asarray(lengths, np.int64)
    assert lengths.max() < M <= V and len(lengths) <= V
    stride = next(p for p in (7919, 7907, 7901) if (M - 1) % p)  # a prime that does not divide M - 1
    dst = np.repeat(np.arange(len(lengths)), lengths)
    nth = np.arange(len(dst)) - np.repeat(np.cumsum(lengths) - lengths, lengths)
    src = (rng.integers(0, M - 1, len(lengths))[dst] + nth * stride) % (M - 1)
    return src + (src >= dst), dst


def rows_graph(V, lengths, seed):
    """Exactly lengths[i] in-edges for vertex i; the last tenth of the vertices only receive."""
    g = gen.from_edges(V, *row_sources(V, V * 9 // 10, lengths, seed))
    assert np.array_equal(np.bincount(g.col, minlength=V)[:len(lengths)], lengths) and g.E == np.sum(lengths)
    return g


def tiles_crossed(lengths, T):
    end = np.cumsum(lengths)
    return ((end - 1) // T - (end - lengths) // T)[np.asarray(lengths) > 0]


def check_pagerank(gx, g, tile, steps, separate=False):
    ref = oracle.pagerank(g, steps, D)
    dg = gx.DeviceGraph(g, gx.GX_NEED_IN, pr_tile_edges=tile)
    st = gx.State(dg, gx.GX_PAGERANK, damping=0.85)
    st.run(steps, allow_cap=True)
    x = st.values_numpy().copy()
    near(x, ref, steps)
    if separate:
        st = gx.State(dg, gx.GX_PAGERANK, damping=0.85, phases=gx.GX_PHASES_LOCAL)
        for _ in range(steps):
            st.msg_gen()
            st.msg_merge()
            st.msg_apply(stats=False)
        near(st.values_numpy(), ref, steps)


@pytest.mark.parametrize("tile", [0, 256, 512, 1024, 2048])
@pytest.mark.parametrize("tail", [-1, 0, 1])
def test_pagerank_row_and_tile_ends(gx, tile, tail):
    T = (tile or 2048) // 4
    lengths = [1, 7, 8, 9, 63, 64, 65, 0, T - 1, T, T + 1, 0, 2 * T, 4 * T + 1, 5 * T, 17 * T + 3, 63 * T + 9, 66 * T + 5]
    lengths += [1] * (2 * T + 3)  # tiles of nothing but one-edge rows
    lengths += [T - sum(lengths) % T + T + tail]
    g = rows_graph(40_000, lengths, 3)
    assert g.E % T == tail % T
    crossed = tiles_crossed(lengths, T)
    assert crossed.max() >= 64 and {0, 1} <= set(crossed) and ((crossed >= 4) & (crossed < 64)).any()
    check_pagerank(gx, g, tile, 6, separate=True)


@pytest.mark.parametrize("E", [1, 63, 64, 511, 512, 513, 1024])
def test_pagerank_few_edges(gx, E):
    for lengths in ([0, E], [1] * E):
        g = rows_graph(1200, lengths, E)
        assert g.E == E
        check_pagerank(gx, g, 0, 6)


HOT_E, HOT_V = 1 << 22, 30720  # from here on contributions are kept in LDS


@pytest.mark.parametrize("V,E,tile", [(HOT_V - 1, HOT_E, 0), (HOT_V, HOT_E, 0), (HOT_V + 1, HOT_E - 1, 0),
                                      (HOT_V + 1, HOT_E, 256), (40_000, HOT_E + 513, 256), (40_000, HOT_E + 513, 512),
                                      (40_000, HOT_E + 513, 1024), (40_000, HOT_E + 513, 2048), (300_000, HOT_E + 1, 0)])
def test_pagerank_contributions_in_lds(gx, V, E, tile):
    rng = np.random.default_rng(V + tile)
    n = V * 3 // 4
    lengths = np.bincount((rng.random(E - 20_000) ** 1.5 * n).astype(np.int64), minlength=n)
    lengths[11] += 20_000 - 3
    lengths[-1] += 3
    g = rows_graph(V, lengths, 5)
    assert g.E == E  # (on its side of HOT_E)
    check_pagerank(gx, g, tile, 4, separate=True)


@pytest.mark.parametrize("hub_edges", [0, 200_000])
def test_pagerank_first_slots_of_few_edges(gx, hub_edges):
    """2^22 edges over two million vertices: the first 30720 slots are the sources
    of fewer than one edge in 16 (none kept in LDS), or of more, with hubs."""
    V, E = 2_000_000, HOT_E + 77
    rng = np.random.default_rng(hub_edges)
    src, dst = rng.integers(0, V, E), rng.integers(0, V, E)
    src[:hub_edges] %= 40
    g = gen.from_edges(V, src, dst)
    dst = (np.arange(V) + 1) % V  # made up to E with edges that are not there yet
    more = np.setdiff1d(np.arange(V, dtype=np.int64) * V + dst, g.src.astype(np.int64) * V + g.col)[:E - g.E]
    g = gen.from_edges(V, np.r_[g.src, more // V], np.r_[g.col, more % V])
    first = np.sort(g.outdeg())[::-1][:HOT_V].sum()
    assert g.E == E and (first * 16 >= E) == (hub_edges > 0)
    check_pagerank(gx, g, 0, 3, separate=True)


LENGTHS = [1, 31, 32, 33, 64, 65, 255, 256, 257, 512, 513, 1025]


@pytest.mark.parametrize("B,V,wmax", [(32, 1200, 255), (64, 1300, 1), (96, 4097, 15), (256, 1500, 255)])
def test_batched_rows_of_exact_lengths(gx, B, V, wmax):
    rng = np.random.default_rng(V)
    n = len(LENGTHS)
    s, d = row_sources(V, V, LENGTHS, V)
    s = np.r_[s, rng.integers(0, V, 12 * V)]
    d = np.r_[d, rng.integers(n, V, 12 * V)]
    g = gen.from_edges(V, s, d, rng.integers(1, wmax + 1, len(s)))
    assert np.bincount(g.col, minlength=V)[:n].tolist() == LENGTHS
    src = gen.pick_sources(g, B, 4)
    # most (edge, lane) pairs are active at once in some superstep, so that it pulls
    fronts = [oracle.sssp_frontiers(g, int(x))[1] for x in src[:32]]
    deg = g.outdeg()
    most = max(sum((deg * f[k]).sum() for f in fronts if k < len(f)) for k in range(12))
    assert most > 32 * g.E / 2
    out, rs = gx.batch_run(gx.DeviceGraph(g, gx.GX_NEED_OUT), gx.GX_SSSP, src)
    X = out.cpu().numpy().view(np.uint32)
    ref, K = oracle.sssp_many(g, src)
    assert np.array_equal(X, ref.T) and rs.supersteps == K.max()


@pytest.mark.parametrize("hub,dangling", [(200, 3), (4095, 700), (4097, 1), (9000, 40_000)])
@pytest.mark.parametrize("iters", [1, 2, 15])
def test_ppr_relative(gx, hub, dangling, iters):
    g, kinds = ppr_rows_graph(hub, dangling, hub)
    out, _ = gx.batch_run(gx.DeviceGraph(g, gx.GX_NEED_IN), gx.GX_PPR, kinds, iters=iters)
    X = out.cpu().numpy()
    for b, s in enumerate(kinds):
        near(X[:, b], oracle.ppr(g, int(s), iters, D), iters)


@pytest.mark.parametrize("E", [(1 << 22) - 1, 1 << 22, 4_600_001])
def test_ppr_tile_sizes_relative(gx, E):
    # both sides of the larger tile (256 in-edges from 2^22 on, 64 below)
    V = 300_000
    rng = np.random.default_rng(E)
    lengths = np.bincount(rng.integers(0, V, E - 200_256 - 9), minlength=V)
    lengths[:8] += [100, 150, 6, 50_000, 70_000, 80_000, 9, 0]
    g = rows_graph(V, lengths, 8)
    assert g.E == E and tiles_crossed(lengths, 256).max() >= 64
    src = gen.pick_sources(g, 9, seed=2)
    out, _ = gx.batch_run(gx.DeviceGraph(g, gx.GX_NEED_IN), gx.GX_PPR, src, iters=6)
    X = out.cpu().numpy()
    for b in (0, 8):
        near(X[:, b], oracle.ppr(g, int(src[b]), 6, D), 6)


def test_server_ppr_relative(gx):
    g, kinds = ppr_rows_graph(200, 50, 5)
    srv = gx.Server(256 << 20, lanes_per_pool=32, max_pools=1, epoch_supersteps=3, ppr_iters=7)
    gid = srv.add_graph(gx.DeviceGraph(g, gx.GX_NEED_OUT | gx.GX_NEED_IN))
    seeds = [int(kinds[i % len(kinds)]) if i % 2 else (37 * i) % g.V for i in range(100)]
    ids = [srv.submit(gid, gx.GX_PPR, s) for s in seeds]
    done = {}
    while len(done) < len(ids):
        for c in srv.poll(wait_ms=50):
            assert c.status == 0
            done[c.id] = c.result
    srv.close()
    for q, s in zip(ids, seeds):
        near(done[q], oracle.ppr(g, s, 7, D), 7)
