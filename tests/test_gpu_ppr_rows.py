"""Batched PPR at the sizes where its split changes: lane-group widths, rows
that end with a tile, cross one or several tiles or enough of them to be
added in pieces, many dangling vertices, and seeds of every kind (without
in-edges, without out-edges, isolated, a hub).  Within 1e-6 of the float64
oracle, and every width bit for bit the widest batch."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2203_13005_amd as m
    return m


def rows_graph(hub, dangling, seed):
    """Rows of 1, 63, 64, 65, 127, 128, 129 and `hub` in-edges, `dangling`
    vertices that only receive, 40 that only send and 10 without an edge."""
    rng = np.random.default_rng(seed)
    core = max(300, hub + 1)
    V = core + dangling + 50
    src, dst = [], []
    for i, n in enumerate([1, 63, 64, 65, 127, 128, 129, hub]):
        s = rng.choice(core - 1, n, replace=False)
        src.append(s + (s >= i))
        dst.append(np.full(n, i))
    d = core + np.arange(dangling)
    src.append(rng.integers(0, core, 2 * dangling))
    dst.append(np.r_[d, d])
    o = core + dangling + np.arange(40)
    src.append(np.repeat(o, 3))
    dst.append(rng.integers(8, core, 120))
    src.append(np.arange(8, core))
    dst.append(8 + rng.integers(0, core - 8, core - 8))
    g = gen.from_edges(V, np.concatenate(src), np.concatenate(dst))
    kinds = [0, 6, 7, 20, core, core + dangling - 1, core + dangling, V - 1]  # rows, dangling, no in-edge, isolated
    return g, np.array(kinds, np.int32)


@pytest.mark.parametrize("hub,dangling", [(200, 3), (4095, 700), (4097, 1), (9000, 40_000)])
@pytest.mark.parametrize("iters", [0, 1, 2, 15])
def test_ppr_rows_and_seeds(gx, hub, dangling, iters):
    g, kinds = rows_graph(hub, dangling, hub)
    dg = gx.DeviceGraph(g, gx.GX_NEED_IN)
    rng = np.random.default_rng(3)
    src = np.r_[kinds, rng.integers(0, g.V, 256 - len(kinds))].astype(np.int32)
    wide, _ = gx.batch_run(dg, gx.GX_PPR, src, iters=iters)
    X = wide.cpu().numpy()
    if iters:
        for b in list(range(len(kinds))) + [200]:
            assert np.max(np.abs(X[:, b].astype(np.float64) - oracle.ppr(g, int(src[b]), iters))) <= 1e-6, b
    else:
        assert np.array_equal(X, (np.arange(g.V)[:, None] == src[None, :]).astype(np.float32))
    for B in (1, 8, 9, 16, 17, 32, 33, 64, 65, 128, 129, 192, 193):
        out, _ = gx.batch_run(dg, gx.GX_PPR, src[:B], iters=iters)
        assert np.array_equal(out.cpu().numpy().view(np.uint32), X[:, :B].view(np.uint32)), B


def test_ppr_wide_tiles(gx):
    # 4.3 M in-edges: the larger tile; lanes of a batch equal the lanes alone
    rng = np.random.default_rng(8)
    V, E = 300_000, 4_600_000
    dst = rng.integers(0, V, E)
    dst[:600_000] //= 1000  # rows of thousands of in-edges
    g = gen.from_edges(V, rng.integers(0, V, E), dst)
    assert g.E >= 1 << 22
    src = gen.pick_sources(g, 9, seed=2)
    dg = gx.DeviceGraph(g, gx.GX_NEED_IN)
    out, _ = gx.batch_run(dg, gx.GX_PPR, src, iters=6)
    X = out.cpu().numpy()
    for b in (0, 8):
        assert np.max(np.abs(X[:, b].astype(np.float64) - oracle.ppr(g, int(src[b]), 6))) <= 1e-6
        alone, _ = gx.batch_run(dg, gx.GX_PPR, src[b:b + 1], iters=6)
        assert np.array_equal(alone.cpu().numpy()[:, 0].view(np.uint32), X[:, b].view(np.uint32))


def test_server_reuses_lanes_after_other_seeds(gx):
    """More queries than lanes on one graph, seeds without in-edges among them:
    a lane's earlier seed leaves nothing behind."""
    g, kinds = rows_graph(200, 50, 5)
    dg = gx.DeviceGraph(g, gx.GX_NEED_OUT | gx.GX_NEED_IN)
    srv = gx.Server(256 << 20, lanes_per_pool=32, max_pools=1, epoch_supersteps=3, ppr_iters=7)
    gid = srv.add_graph(dg)
    rng = np.random.default_rng(6)
    seeds = [int(kinds[i % len(kinds)]) if i % 2 else int(rng.integers(0, g.V)) for i in range(100)]
    ids = [srv.submit(gid, gx.GX_PPR, s) for s in seeds]
    done = {}
    while len(done) < len(ids):
        for c in srv.poll(wait_ms=50):
            assert c.status == 0
            done[c.id] = c.result
    srv.close()
    for q, s in zip(ids, seeds):
        assert np.max(np.abs(done[q].astype(np.float64) - oracle.ppr(g, s, 7))) <= 1e-6, s
