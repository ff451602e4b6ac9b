"""The sync set and its merge at the sizes where their split changes: words and
blocks that are partly filled, graphs large enough for longer blocks, a
capacity below the count, and maps of local to global ids around the number of
samples that the search keeps.  Exact."""
import numpy as np
import pytest

import gen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2203_13005_amd as m
    return m


def sparse(V, seed):
    rng = np.random.default_rng(seed)
    E = max(1, V // 2)
    return gen.from_edges(V, rng.integers(0, V, E), rng.integers(0, V, E), np.ones(E, np.int64))


SIZES = [1, 31, 33, 1023, 1024, 1025, (1 << 20) - 1, (1 << 20) + 33, (1 << 21) + 1, (1 << 22) + 65]


@pytest.mark.parametrize("V", SIZES)
def test_changed_ranks(gx, V):
    import torch
    g = sparse(V, V)
    st = gx.State(gx.DeviceGraph(g, gx.GX_NEED_IN), gx.GX_PAGERANK, damping=0.85, delta_mode=gx.GX_DELTA_ALL)
    x0 = st.values_numpy().view(np.uint32).copy()
    st.run(1, allow_cap=True)
    x1 = st.values_numpy().view(np.uint32).copy()
    want = np.nonzero(x0 != x1)[0]
    if len(want) > 1:  # too little room: refused, and nothing counts as sent
        with pytest.raises(gx.GxError):
            st.sync_delta(cap=len(want) - 1)
    gid, val, skip = st.sync_delta()
    assert np.array_equal(gid, want) and np.array_equal(val, x1[want]) and skip == (len(want) == 0)
    gid, val, skip = st.sync_delta()
    assert len(gid) == 0 and skip
    st.run(1, allow_cap=True)
    x2 = st.values_numpy().view(np.uint32)
    want = np.nonzero(x2 != x1)[0]
    out = [torch.zeros(V, dtype=torch.int32, device="cuda") for _ in range(2)] + [torch.zeros(1, dtype=torch.int32, device="cuda")]
    st.sync_delta_noalloc(*out)
    n = int(out[2].item())
    assert n == len(want) and np.array_equal(out[0][:n].cpu().numpy(), want)
    assert np.array_equal(out[1][:n].cpu().numpy().view(np.uint32), x2[want])


@pytest.mark.parametrize("V", SIZES)
def test_changed_labels(gx, V):
    st = gx.State(gx.DeviceGraph(sparse(V, V + 1), gx.GX_NEED_SYM), gx.GX_CC, delta_mode=gx.GX_DELTA_ALL)
    st.run(10_000)
    labels = st.values_numpy()
    want = np.nonzero(labels != np.arange(V, dtype=np.uint32))[0]
    gid, val, _ = st.sync_delta()
    assert np.array_equal(gid, want) and np.array_equal(val, labels[want])
    gid, _, skip = st.sync_delta()
    assert len(gid) == 0 and skip


class Part:
    def __init__(self, l2g):
        self.V, self.E = len(l2g), 0
        self.row_ptr, self.col, self.w = np.zeros(self.V + 1, np.int32), np.zeros(0, np.int32), np.zeros(0, np.uint32)
        self.l2g, self.flags = l2g.astype(np.int32), None


@pytest.mark.parametrize("V", [1, 2, 255, 256, 257, 511, 1000, 4099])
def test_merge_by_global_id(gx, V):
    import torch
    rng = np.random.default_rng(V)
    G = 3 * V + 2
    l2g = np.sort(rng.choice(np.arange(1, G), V, replace=False))
    st = gx.State(gx.DeviceGraph(Part(l2g), gx.GX_NEED_OUT), gx.GX_SSSP, source=0)
    val = st.values_numpy().copy()
    gid = rng.permutation(G + 5).astype(np.int32)  # ids it holds, ids it does not, ids below and beyond its own
    new = rng.integers(1, 1 << 30, len(gid)).astype(np.int32)
    active = st.apply_delta(torch.from_numpy(gid).cuda(), torch.from_numpy(new).cuda())
    by_gid = np.empty(G + 5, np.uint32)
    by_gid[gid] = new
    want = np.minimum(val, by_gid[l2g])
    assert np.array_equal(st.values_numpy(), want)
    assert active == 1 + np.count_nonzero(want != val)  # the source was active
