"""PageRank across parts that hold every vertex under its global id and name no
map (l2g NULL stands for the identity): merged sums, masters' ranks and sync
sets go by the ids themselves; ids out of range are ignored.  Against the whole
graph's float64 oracle: a rank and a contribution are each rounded once a
superstep, the start once more, (2 k + 1) 2^-24 relative after k."""
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


class Part:
    def __init__(self, g, mine, flags):
        p = gen.from_edges(g.V, g.src[mine], g.col[mine])
        self.V, self.E, self.row_ptr, self.col, self.w = p.V, p.E, p.row_ptr, p.col, p.w
        self.l2g, self.flags = None, flags


@pytest.mark.parametrize("V", [1, 2, 255, 256, 3000])
def test_parts_without_a_map(gx, V):
    import torch
    rng = np.random.default_rng(V)
    g = gen.from_edges(V, rng.integers(0, V, 6 * V), rng.integers(0, V, 6 * V))
    of = rng.integers(0, 2, g.E)
    first = rng.random(V) < 0.5  # whose master part 0 holds
    sts = []
    for p in (0, 1):
        flags = np.where(first == (p == 0), 1, 0).astype(np.uint8) | 6
        dg = gx.DeviceGraph(Part(g, of == p, flags), gx.GX_NEED_IN, V_global=V,
                            outdeg_global=np.diff(g.row_ptr).astype(np.int32))
        sts.append(gx.State(dg, gx.GX_PAGERANK, damping=0.85, phases=gx.GX_PHASES_MASTERS, delta_mode=gx.GX_DELTA_MASTERS))
    stray = torch.tensor([-1, V, V + 5], dtype=torch.int32, device="cuda:0")
    T = 6
    for _ in range(T):
        for st in sts:
            st.msg_gen()
            st.msg_merge()
        D = sum(st.dangling_get() for st in sts)
        sent = [st.partial_emit() for st in sts]
        for p, st in enumerate(sts):
            st.dangling_set(D)
            gid, val = sent[1 - p]
            st.partial_add(torch.cat([gid, stray]), torch.cat([val, torch.ones(3, dtype=torch.float64, device="cuda:0")]))
        for st in sts:
            st.msg_apply(stats=False)
        bc = [st.sync_delta(on_device=True) for st in sts]
        for p, st in enumerate(sts):
            st.apply_delta(torch.cat([bc[1 - p][0], stray]), torch.cat([bc[1 - p][1], stray]))
    ref = oracle.pagerank(g, T, float(np.float32(0.85)))
    for st in sts:
        assert np.max(np.abs(st.values_numpy() - ref) / ref) <= (2 * T + 1) * 2.0 ** -24
