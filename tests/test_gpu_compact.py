"""The compaction of 16 vertices per thread (CC and SSSP without snapshots by
slot: sparse graphs from 2^22 vertices on, all from 2^23): vertex counts that end
inside a thread's vertices, pulling, pushing and as the frontier decides.  Every
superstep against the oracle, bit for bit.  And the sparse graphs on which SSSP
pushes unless a pull fraction is named."""
import numpy as np
import pytest

from test_gpu_sweep import Csr, follow, gx, start, uniform  # noqa: F401  (gx: the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,E", [((1 << 22) + 17, 7_000_000), ((1 << 22) - 1, 7_000_000), ((1 << 23) + 5, 13_000_000)])
@pytest.mark.parametrize("frac", [1e-9, 0.05, 0.0])
def test_sparse_supersteps(gx, V, E, frac):  # noqa: F811
    g = uniform(V, E, "mixed", V)
    assert g.E < 2 * V
    source = int(np.argmax(np.diff(g.row_ptr)))
    dg = gx.DeviceGraph(g, gx.GX_NEED_OUT | gx.GX_NEED_SYM)
    st = gx.State(dg, gx.GX_SSSP, source=source, pull_fraction=frac)
    follow(g, lambda: st.superstep()[2], st.values_numpy, *start(g, source), True, False, 400)
    if frac == 0.05:
        return
    cc = gx.State(dg, gx.GX_CC, pull_fraction=frac)
    front = np.zeros(V, bool)
    front[np.unique(np.r_[np.nonzero(np.diff(g.row_ptr))[0], g.col])] = True
    follow(g, lambda: cc.superstep()[2], cc.values_numpy, np.arange(V, dtype=np.uint32), front, False, True, 400)


@pytest.mark.parametrize("V,E,hub_edges,pushes", [(1 << 20, 2_000_000, 0, True), (1 << 20, 2_000_000, 1_200_000, False),
                                                  ((1 << 20) - 1, 2_000_000, 0, False)])
def test_when_sssp_only_pushes(gx, V, E, hub_edges, pushes):  # noqa: F811
    rng = np.random.default_rng(V + hub_edges)
    src = rng.integers(0, V, E)
    src[:hub_edges] %= 2000
    g = Csr(V, src, rng.integers(0, V, E), rng.integers(1, 256, E).astype(np.uint32))
    top = np.sort(np.diff(g.row_ptr))[::-1][:1 << 17].sum()
    assert g.E < 3 * V and (top < 0.45 * g.E) == (hub_edges == 0)
    dg = gx.DeviceGraph(g, gx.GX_NEED_OUT)
    values = []
    for frac in (0.0, 0.02, 1.0):
        st = gx.State(dg, gx.GX_SSSP, source=int(np.argmax(np.diff(g.row_ptr))), pull_fraction=frac)
        rs, steps = st.run(1000, per_step=True, detail=True)
        values.append(st.values_numpy().copy())
        pulled = any(s["pulled"] for s in steps)
        assert pulled == (frac == 0.02 or (frac == 0.0 and not pushes and max(s["edges"] for s in steps) >= 0.3 * g.E))
    assert np.array_equal(values[0], values[1]) and np.array_equal(values[0], values[2])
