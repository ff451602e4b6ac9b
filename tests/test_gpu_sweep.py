"""The pull of SSSP and CC on graphs without hubs, a sweep over every in-edge:
every superstep against the oracle, bit for bit, at vertex counts around whole
bands of sources (8192) and blocks of destinations (64), weights 0, all equal,
mixed and too wide for its records, on its own and with pushes between, through
the separate calls, and after values of another part came in.  (Which graphs
sweep is tested by the arena they ask for, without a GPU.)"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

V0 = 1 << 20  # smallest vertex count that sweeps (with 12 edges per vertex)
V1 = 3 << 19  # from here on with 3, SSSP


class Csr:
    def __init__(self, V, src, dst, w=None):
        k = np.unique(src.astype(np.int64) * V + dst)
        k = k[k // V != k % V]
        self.V, self.E = V, len(k)
        self.row_ptr = np.concatenate([[0], np.cumsum(np.bincount(k // V, minlength=V))]).astype(np.int32)
        self.col = (k % V).astype(np.int32)
        self.w = np.ones(self.E, np.uint32) if w is None else w[:self.E]
        self.l2g = self.flags = None


def uniform(V, E, weights, seed):
    rng = np.random.default_rng(seed)
    w = {"mixed": lambda: rng.integers(0, 256, E), "zero": lambda: np.zeros(E), "equal": lambda: np.full(E, 255),
         "wide": lambda: rng.integers(0, 300, E)}[weights]().astype(np.uint32)
    return Csr(V, rng.integers(0, V, E), rng.integers(0, V, E), w)


@pytest.fixture(scope="module")
def gx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2203_13005_amd as m
    return m


def follow(g, step, values, state, front, weighted, both_dirs, cap=80):
    for k in range(cap):
        state, front = oracle.min_superstep(g, state, front, weighted=weighted, both_dirs=both_dirs)
        changed = step()
        assert changed == front.sum(), k
        assert np.array_equal(values(), state), k
        if not front.any():
            return
    raise AssertionError("did not settle")


def separate(st):
    def step():
        st.msg_gen()
        st.msg_merge()
        return st.msg_apply()[2]
    return step


def start(g, source):
    d = np.full(g.V, 0xFFFFFFFF, np.uint32)
    d[source] = 0
    return d, np.arange(g.V) == source


@pytest.mark.parametrize("V,E,weights", [(V1, 5_000_000, "mixed"), (V1 + 1, 5_000_000, "zero"), (V1 + 8191, 5_000_000, "equal"),
                                         (V1 + 8192, 6_000_000, "mixed"), (V0 + 63, 13_000_000, "mixed"),
                                         (V0 // 2 + 1, 17_000_000, "mixed"),
                                         (V1 + 63, 5_000_000, "wide")])
def test_sssp_sweep(gx, V, E, weights):
    g = uniform(V, E, weights, V)
    assert g.E >= (3 if V >= V1 else 12 if V >= V0 else 32) * V
    source = int(np.argmax(np.diff(g.row_ptr)))
    dg = gx.DeviceGraph(g, gx.GX_NEED_OUT)
    cap = 400
    for frac in (1e-9, 0.0):
        st = gx.State(dg, gx.GX_SSSP, source=source, pull_fraction=frac)
        follow(g, lambda: st.superstep()[2], st.values_numpy, *start(g, source), True, False, cap)
        st.close()
        if weights != "mixed":
            break
    if weights == "mixed":
        st = gx.State(dg, gx.GX_SSSP, source=source, pull_fraction=1e-9, phases=gx.GX_PHASES_LOCAL)
        follow(g, separate(st), st.values_numpy, *start(g, source), True, False, cap)


@pytest.mark.parametrize("V,degree", [(V0, 12), (V0 + 65, 12), (4 * V0 - 65, 1)])
def test_cc_sweep(gx, V, degree):
    import torch
    g = uniform(V, degree * V + V // 50, "zero", V)
    assert g.E >= degree * V
    dg = gx.DeviceGraph(g, gx.GX_NEED_SYM)
    lab, front = np.arange(V, dtype=np.uint32), np.zeros(V, bool)
    front[np.unique(np.r_[np.nonzero(np.diff(g.row_ptr))[0], g.col])] = True
    for frac in (1e-9, 0.0):
        st = gx.State(dg, gx.GX_CC, pull_fraction=frac)
        follow(g, lambda: st.superstep()[2], st.values_numpy, lab, front, False, True)
        st.close()
    st = gx.State(dg, gx.GX_CC, pull_fraction=1e-9, phases=gx.GX_PHASES_LOCAL)
    follow(g, separate(st), st.values_numpy, lab, front, False, True)
    st.close()
    # labels of another part before the first superstep: one neighbour no longer stands for a row
    pick = np.random.default_rng(1).choice(V, V // 3, replace=False)
    low = np.random.default_rng(2).integers(0, pick + 1).astype(np.uint32)
    st = gx.State(dg, gx.GX_CC, pull_fraction=1e-9)
    st.apply_delta(torch.tensor(pick.astype(np.int32), device="cuda:0"), torch.tensor(low.view(np.int32), device="cuda:0"))
    lab = lab.copy()
    lab[pick] = np.minimum(lab[pick], low)
    follow(g, lambda: st.superstep()[2], st.values_numpy, lab, front, False, True)
