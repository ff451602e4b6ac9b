"""Label propagation's class lists and its recomputation of changed
neighbourhoods, bit for bit against the oracle: vertices whose degree is one
short of, at and past every class limit and chunk, graphs that leave most
labels alone after a few iterations, and a run continued past its end."""
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


DEGREES = [1, 4, 5, 8, 9, 16, 17, 32, 33, 64, 65, 511, 512, 513, 1023, 1024, 1025, 2047, 2048, 2049, 4096, 4097, 8192,
           8193]


def limits_graph(leaves, seed):
    """One centre per degree joined to that many of `leaves` shared vertices,
    and pairs hanging off some of them whose labels keep swapping."""
    rng = np.random.default_rng(seed)
    n = len(DEGREES)
    src, dst = [], []
    for i, d in enumerate(DEGREES):
        src.append(np.full(min(d, leaves), i))
        dst.append(n + rng.choice(leaves, min(d, leaves), replace=False))
    V = n + leaves + 400
    p = n + leaves + np.arange(0, 400, 2)
    src.append(p)
    dst.append(p + 1)  # isolated pairs swap their labels for ever
    s, d = np.concatenate(src), np.concatenate(dst)
    return gen.from_edges(V, s, d, np.ones(len(s), np.int64))


@pytest.mark.parametrize("leaves,seed", [(9000, 1), (30000, 2)])
def test_lp_degree_limits(gx, leaves, seed):
    g = limits_graph(leaves, seed)
    assert set(DEGREES) <= set(np.bincount(np.r_[g.src, g.col], minlength=g.V)[:len(DEGREES)].tolist())
    adj = oracle.SymAdjacency(g)
    st = gx.State(gx.DeviceGraph(g, gx.GX_NEED_SYM), gx.GX_LP)
    prev = np.arange(g.V, dtype=np.uint32)
    for k in range(12):
        want = adj.lp_step(prev)
        _, _, changed = st.superstep()
        assert np.array_equal(st.values_numpy(), want), k
        assert changed == np.count_nonzero(want != prev), k
        prev = want


def test_lp_run_continued_and_reset(gx):
    g = gen.rmat(13, seed=5)
    dg = gx.DeviceGraph(g, gx.GX_NEED_SYM)
    ref = oracle.lp_steps(g, 24)
    for _ in range(2):
        st = gx.State(dg, gx.GX_LP)
        done = 0
        for n in (1, 2, 5, 16):
            rs, _ = st.run(n, allow_cap=True)
            done += rs.supersteps
            assert np.array_equal(st.values_numpy(), ref[min(done, len(ref) - 1)]), done
        st.reset()
        assert np.array_equal(st.values_numpy(), ref[0])
        st.run(3, allow_cap=True)
        assert np.array_equal(st.values_numpy(), ref[min(3, len(ref) - 1)])
        st.close()
