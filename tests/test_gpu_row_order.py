"""CC and label propagation on a host CSR whose rows are in no order: the same
labels and counts, superstep by superstep, as with sorted rows.  All edges go
up, or all go down, in id, so a neighbour is named once however the rows are
ordered (down: the smaller labels are the ones out of order); rows of every
label propagation class are among them."""
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


def graph(V, degrees, seed, down):
    """Vertex i (down: V - 1 - i) is joined to degrees[i] of the others; a random
    layer over the rest."""
    rng = np.random.default_rng(seed)
    n = len(degrees)
    src = [np.full(d, i) for i, d in enumerate(degrees)] + [rng.integers(n, V, 2 * V)]
    dst = [n + rng.choice(V - n, d, replace=False) for d in degrees] + [rng.integers(n, V, 2 * V)]
    s, d = np.concatenate(src), np.concatenate(dst)
    s, d = np.minimum(s, d), np.maximum(s, d)
    return gen.from_edges(V, V - 1 - s, V - 1 - d) if down else gen.from_edges(V, s, d)


class Shuffled:
    """The graph with every out-row in reverse or random order."""

    def __init__(self, g, how):
        rng = np.random.default_rng(1)
        key = -np.arange(g.E) if how == "reversed" else rng.permutation(g.E)
        order = np.lexsort((key, g.src))
        self.V, self.E, self.row_ptr, self.col, self.w = g.V, g.E, g.row_ptr, g.col[order], g.w[order]
        self.l2g = self.flags = None


@pytest.mark.parametrize("how", ["reversed", "random"])
@pytest.mark.parametrize("down", [False, True])
@pytest.mark.parametrize("V,degrees", [(40, [3]), (3000, [5, 9, 33, 65, 600]), (9000, [4, 64, 512, 2048, 2049, 5000])])
def test_rows_in_no_order(gx, V, degrees, down, how):
    g = graph(V, degrees, V, down)
    h = Shuffled(g, how)
    assert not np.array_equal(h.col, g.col) and np.array_equal(np.sort(h.col), np.sort(g.col))
    dg = gx.DeviceGraph(h, gx.GX_NEED_SYM)
    for frac in (1e-9, 1.0):  # every superstep pulls, every superstep pushes
        cc = gx.State(dg, gx.GX_CC, pull_fraction=frac)
        lab, front = np.arange(V, dtype=np.uint32), np.zeros(V, bool)
        front[np.unique(np.r_[g.src, g.col])] = True
        while front.any():
            lab, front = oracle.min_superstep(g, lab, front, weighted=False, both_dirs=True)
            _, _, changed = cc.superstep()
            assert changed == front.sum()
            assert np.array_equal(cc.values_numpy(), lab)
    adj = oracle.SymAdjacency(g)
    lp = gx.State(dg, gx.GX_LP)
    for _ in range(2):
        prev = np.arange(V, dtype=np.uint32)
        for k in range(10):
            want = adj.lp_step(prev)
            _, _, changed = lp.superstep()
            assert np.array_equal(lp.values_numpy(), want), k
            assert changed == np.count_nonzero(want != prev), k
            prev = want
        lp.reset()


def test_rows_in_no_order_separate_calls(gx):
    g = graph(3000, [5, 9, 33, 65, 600], 7, True)
    st = gx.State(gx.DeviceGraph(Shuffled(g, "random"), gx.GX_NEED_SYM), gx.GX_CC, pull_fraction=1e-9,
                  phases=gx.GX_PHASES_LOCAL)
    lab, front = np.arange(g.V, dtype=np.uint32), np.zeros(g.V, bool)
    front[np.unique(np.r_[g.src, g.col])] = True
    while front.any():
        lab, front = oracle.min_superstep(g, lab, front, weighted=False, both_dirs=True)
        st.msg_gen()
        st.msg_merge()
        st.msg_apply()
        assert np.array_equal(st.values_numpy(), lab)
