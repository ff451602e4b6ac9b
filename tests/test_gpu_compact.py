"""The compaction of 16 vertices per thread (sparse graphs from 2^22 vertices on,
all from 2^23): vertex counts that end inside a thread's vertices, SSSP (its
snapshots by slot) and CC (by vertex), pulling, pushing and as the frontier
decides.  Every superstep against the oracle, bit for bit."""
import numpy as np
import pytest

from test_gpu_sweep import follow, gx, start, uniform  # noqa: F401  (gx: the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,E", [((1 << 22) + 17, 7_000_000), ((1 << 22) - 1, 7_000_000), ((1 << 23) + 5, 13_000_000)])
@pytest.mark.parametrize("frac", [1e-9, 0.05, 1.0])
def test_sparse_supersteps(gx, V, E, frac):  # noqa: F811
    g = uniform(V, E, "mixed", V)
    assert g.E < 2 * V
    source = int(np.argmax(np.diff(g.row_ptr)))
    dg = gx.DeviceGraph(g, gx.GX_NEED_OUT | gx.GX_NEED_SYM)
    st = gx.State(dg, gx.GX_SSSP, source=source, pull_fraction=frac)
    follow(g, lambda: st.superstep()[2], st.values_numpy, *start(g, source), True, False, 400)
    if frac == 1.0:
        return
    cc = gx.State(dg, gx.GX_CC, pull_fraction=frac)
    front = np.zeros(V, bool)
    front[np.unique(np.r_[np.nonzero(np.diff(g.row_ptr))[0], g.col])] = True
    follow(g, lambda: cc.superstep()[2], cc.values_numpy, np.arange(V, dtype=np.uint32), front, False, True, 400)
