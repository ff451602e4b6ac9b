"""The batched SSSP pull at the sizes where its split changes: every lane
width, rows one short of, at and past the longest short row and whole
segments (one segment stores, several merge), packs of short rows that end
with a block, lanes that reach almost nothing, and graphs whose weights leave
only the push.  Every lane and the superstep count against the oracle."""
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


def dense_graph(V, wmax, seed):
    """Rows of 1 to 1025 in-edges, a well connected core (so that most of the
    graph is active at once), and a chain that only its own end reaches."""
    rng = np.random.default_rng(seed)
    src, dst = [], []
    for i, n in enumerate([1, 31, 32, 33, 64, 65, 255, 256, 257, 512, 513, 1025]):
        n = min(n, V - 1)
        s = rng.choice(V - 1, n, replace=False)
        src.append(s + (s >= i))
        dst.append(np.full(n, i))
    src.append(rng.integers(0, V, 12 * V))
    dst.append(rng.integers(0, V - 20, 12 * V))
    t = np.arange(V - 20, V - 1)
    src.append(t)
    dst.append(t + 1)
    s, d = np.concatenate(src), np.concatenate(dst)
    keep = ~((s >= V - 20) & (d < V - 20))  # the chain leads nowhere else
    s, d = s[keep], d[keep]
    return gen.from_edges(V, s, d, rng.integers(1, wmax + 1, len(s)))


def check(gx, g, B, seed, **kw):
    rng = np.random.default_rng(seed)
    src = rng.integers(0, g.V, B).astype(np.int32)
    src[:3] = [g.V - 5, g.V - 1, 0]  # a lane that reaches four vertices, one that reaches none
    out, rs = gx.batch_run(gx.DeviceGraph(g, gx.GX_NEED_OUT), gx.GX_SSSP, src, **kw)
    D = out.cpu().numpy().view(np.uint32)
    K = 0
    for b, s in enumerate(src):
        ref = oracle.sssp(g, int(s))
        assert np.array_equal(D[:, b], ref.state), (b, s)
        K = max(K, ref.K)
    assert rs.supersteps == K


@pytest.mark.parametrize("B", [32, 64, 96, 128, 160, 224, 256])
def test_batch_pull_widths(gx, B):
    check(gx, dense_graph(1500, 255, 1), B, B)


@pytest.mark.parametrize("V,wmax", [(1100, 255), (1152, 1), (4097, 15), (1500, 100_000)])
def test_batch_pull_rows(gx, V, wmax):
    check(gx, dense_graph(V, wmax, V), 64, V)


def test_batch_pull_in_passes(gx):
    g = dense_graph(1300, 255, 9)
    check(gx, g, 128, 4, tune=gx.Tune(512, 2048, 32, 0))


def test_batch_wide_compaction(gx):
    # more than 2^20 mask words (V * 8 groups)
    g = gen.rmat(18, edge_factor=6, seed=31)
    src = gen.pick_sources(g, 256, seed=3)
    ref, K = oracle.sssp_many(g, src)
    out, rs = gx.batch_run(gx.DeviceGraph(g, gx.GX_NEED_OUT), gx.GX_SSSP, src)
    D = out.cpu().numpy().view(np.uint32)
    for b in range(256):
        assert np.array_equal(D[:, b], ref[b]), b
    assert rs.supersteps == K.max()


def test_server_sssp_reuses_lanes(gx):
    """More queries than lanes on a dense graph: a lane's earlier source leaves
    nothing behind in the snapshot the pull reads."""
    g = dense_graph(1400, 255, 12)
    srv = gx.Server(256 << 20, lanes_per_pool=32, max_pools=1, sssp_epoch_supersteps=3)
    gid = srv.add_graph(gx.DeviceGraph(g, gx.GX_NEED_OUT | gx.GX_NEED_IN))
    rng = np.random.default_rng(2)
    srcs = [int(x) for x in rng.integers(0, g.V, 120)]
    ids = [srv.submit(gid, gx.GX_SSSP, s) for s in srcs]
    done = {}
    while len(done) < len(ids):
        for c in srv.poll(wait_ms=50):
            assert c.status == 0
            done[c.id] = c
    srv.close()
    for q, s in zip(ids, srcs):
        ref = oracle.sssp(g, s)
        assert np.array_equal(done[q].result, ref.state), s
        assert done[q].supersteps == ref.K, s
