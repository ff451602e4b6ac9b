"""PageRank pull at the sizes where its split changes: rows that end with a
lane's edges, a wave's tile or the last one, rows that cross one, some or many
tiles, tiles of nothing but one-edge rows, rows without in-edges, and graphs on
both sides of where the first contributions are kept in LDS.

Against the float64 oracle.  A rank and a contribution are each rounded once to
32 bits in a superstep (half an ulp, 2^-24 relative), and what a superstep
inherits is damped by d: at most 2 * 2^-24 / (1 - d) = 8e-7 at d = 0.85."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu

REL = 1e-6


@pytest.fixture(scope="module")
def gx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2203_13005_amd as m
    return m


def rows_graph(lengths, V, seed):
    """Vertex i has lengths[i] in-edges; the sources are drawn by a power law
    over the first 9/10 of the vertices, the rest only receive."""
    rng = np.random.default_rng(seed)
    E = int(np.sum(lengths))
    src = (rng.random(E) ** 3 * (V * 9 // 10)).astype(np.int64)
    dst = np.repeat(np.arange(len(lengths)), lengths)
    return gen.from_edges(V, src, dst, np.ones(E, np.int64))


def check(gx, g, tile, steps=6):
    st = gx.State(gx.DeviceGraph(g, gx.GX_NEED_IN, pr_tile_edges=tile), gx.GX_PAGERANK, damping=0.85)
    st.run(steps, allow_cap=True)
    x = st.values_numpy()
    ref = oracle.pagerank(g, steps, 0.85)
    assert np.max(np.abs(x - ref) / ref) <= REL
    st.reset()
    st.run(steps, allow_cap=True)
    assert np.array_equal(st.values_numpy().view(np.uint32), x.view(np.uint32))


@pytest.mark.parametrize("tile", [0, 256, 512, 1024, 2048])
@pytest.mark.parametrize("tail", [-1, 0, 1])
def test_row_and_tile_ends(gx, tile, tail):
    T = (tile or 2048) // 4
    lengths = [1, 7, 8, 9, 63, 64, 65, 0, T - 1, T, T + 1, 0, 2 * T, 4 * T + 1, 5 * T, 17 * T + 3, 66 * T + 5] + [1] * (2 * T + 3)
    lengths += [T - sum(lengths) % T + T + tail]  # the last tile is full, all but full, or holds one edge
    check(gx, rows_graph(lengths, 4000, 3), tile)


@pytest.mark.parametrize("E", [1, 63, 64, 511, 512, 513])
def test_one_tile(gx, E):
    check(gx, rows_graph([0, E], 700, E), 0)
    check(gx, rows_graph([1] * E, 700, E), 0)


@pytest.mark.parametrize("V,E,tile", [(30719, 1 << 22, 0), (30720, 1 << 22, 0), (30721, (1 << 22) - 1, 0),
                                      (40000, (1 << 22) + 513, 256), (40000, (1 << 22) + 513, 512),
                                      (40000, (1 << 22) + 513, 1024), (40000, (1 << 22) + 513, 2048)])
def test_contributions_in_lds(gx, V, E, tile):
    rng = np.random.default_rng(V + tile)
    lengths = np.bincount((rng.random(E - 70_000) ** 4 * (V * 3 // 4)).astype(np.int64), minlength=V * 3 // 4)
    lengths[11] += 70_000
    check(gx, rows_graph(lengths, V, 5), tile, 4)
