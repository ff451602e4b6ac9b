"""The row pull of SSSP and CC at the sizes where its split changes: rows one
short of, at and past the longest short row, whole segments and their
remainders, vertex counts around the 64 rows of a wave, the 256 of a
workgroup and the sizes where blocks are dealt in runs and sources pass the
frontier bits kept on chip; weights 0, all equal and mixed.  Every superstep
against the oracle, bit for bit."""
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


def rows_graph(V, lengths, weights, seed):
    """Vertex i of the first ones receives lengths[i] edges from distinct
    random sources; a chain and a random layer spread the distances."""
    rng = np.random.default_rng(seed)
    src, dst = [np.arange(min(V - 1, 40))], [np.arange(1, min(V, 41))]
    for i, n in enumerate(lengths):
        n = min(n, V - 1)
        s = rng.choice(V - 1, n, replace=False)
        src.append(s + (s >= i))  # every vertex but i
        dst.append(np.full(n, i))
    m = 3 * V
    src.append(rng.integers(0, V, m))
    dst.append(rng.integers(len(lengths), V, m))
    s, d = np.concatenate(src), np.concatenate(dst)
    w = {"mixed": rng.integers(0, 256, len(s)), "zero": np.zeros(len(s), int), "equal": np.full(len(s), 255)}[weights]
    return gen.from_edges(V, s, d, w)


LENGTHS = [1, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513, 1025]


@pytest.mark.parametrize("weights", ["mixed", "zero", "equal"])
@pytest.mark.parametrize("V", [63, 64, 65, 257, 1500, 140_000, 530_000])
def test_pull_row_lengths(gx, V, weights):
    g = rows_graph(V, LENGTHS[:max(1, min(len(LENGTHS), V // 4))], weights, V)
    dg = gx.DeviceGraph(g, gx.GX_NEED_OUT | gx.GX_NEED_SYM)
    dists, fronts = oracle.sssp_frontiers(g, 0)
    st = gx.State(dg, gx.GX_SSSP, source=0, pull_fraction=1e-9)
    for k in range(1, len(dists)):
        _, _, changed = st.superstep()
        assert changed == fronts[k].sum(), k
        assert np.array_equal(st.values_numpy(), dists[k]), k
    cc = gx.State(dg, gx.GX_CC, pull_fraction=1e-9)
    lab, front = np.arange(V, dtype=np.uint32), np.zeros(V, bool)
    front[np.unique(np.r_[g.src, g.col])] = True
    for k in range(200):
        lab, front = oracle.min_superstep(g, lab, front, weighted=False, both_dirs=True)
        _, _, changed = cc.superstep()
        assert changed == front.sum(), k
        assert np.array_equal(cc.values_numpy(), lab), k
        if not front.any():
            break


def test_cc_pull_after_merged_labels(gx):
    """Labels merged from another part before the first superstep: they no
    longer ascend with the ids, so the first superstep reads whole rows."""
    import torch
    p = gen.rmat_part(12, seed=3, part=1)
    rng = np.random.default_rng(4)
    pick = rng.choice(p.V, p.V // 3, replace=False)
    low = rng.integers(0, p.l2g[pick] + 1).astype(np.uint32)
    st = gx.State(gx.DeviceGraph(p, gx.GX_NEED_SYM), gx.GX_CC, pull_fraction=1e-9)
    st.apply_delta(torch.tensor(p.l2g[pick].astype(np.int32), device="cuda:0"),
                   torch.tensor(low.view(np.int32), device="cuda:0"))
    lab = p.l2g.astype(np.uint32).copy()
    lab[pick] = np.minimum(lab[pick], low)
    front = np.zeros(p.V, bool)
    front[np.unique(np.r_[p.src, p.col])] = True
    for k in range(200):
        lab, front = oracle.min_superstep(p, lab, front, weighted=False, both_dirs=True)
        st.superstep()
        assert np.array_equal(st.values_numpy(), lab), k
        if not front.any():
            break
