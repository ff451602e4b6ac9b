"""The limits in gx_limits.h, compiled as plain C++ (no GPU): widths of
counters and indexes at the largest graphs that a load accepts; and the graphs
whose load builds the sweep's image, by the arena bytes it asks for."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
E_MAX = (1 << 31) - 2048 - 1  # most edges of a graph


def run_cpp(tmp_path, body):
    """Compiles main() { body } against the header, with traps on signed overflow; its output's numbers."""
    src = tmp_path / "t.cpp"
    src.write_text('#include <cstdio>\n#include "gx_limits.h"\nusing namespace gx;\nint main() {\n' + body + "\n}\n")
    exe = str(tmp_path / "t")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-ftrapv", "-I",
                           os.path.join(ROOT, "paper_2203_13005_amd", "csrc"), "-o", exe, str(src)])
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout
    return [[int(x) for x in line.split()] for line in out.splitlines()]


EDGES = [0, 1, 1000, (1 << 29) - 513, (1 << 29) - 512, 1 << 29, 600_000_000, 613_566_171, 613_566_172, 715_827_199,
         715_827_200, 1 << 30, (1 << 30) + 1, 1_431_654_400, E_MAX]


@pytest.mark.parametrize("E", EDGES)
def test_batched_units_fit_32_bits(tmp_path, E):
    rows = run_cpp(tmp_path, f"""
        for (uint32_t w = 32; w <= 256; w += 32)
            std::printf("%u %u %u %lld\\n", w, bs_pass_width({E}ll, w), bs_groups_max({E}ll), (long long)BS_MAX_TILE);
    """)
    for width, got, groups, tile in rows:
        assert got % 32 == 0 and got > 0 and width % got == 0
        # every lane of every vertex active, rounded up to whole tiles, and no 32 ones (which say "never pulls")
        assert E * (got // 32) + tile <= (1 << 32) - 1
        assert E * groups + tile <= (1 << 32) - 1 and 2 <= groups <= 8
        if E * (width // 32) + tile <= (1 << 32) - 1:  # what fits is left alone
            assert got == width
        else:  # as wide as fits
            wider = [g for g in range(got + 32, width, 32) if width % g == 0]
            assert all(E * (g // 32) + tile > (1 << 32) - 1 for g in wider)


@pytest.mark.parametrize("chunk", [1, 1024])
def test_chunk_ends_at_the_last_entries(tmp_path, chunk):
    last = (1 << 31) - 513  # entries of the largest symmetric image
    cases = [(b, e) for e in (last, last - 1, 5000, 1, 0) for b in (e, e - 1, e - 511, e - 512, e - 1023, e - 1024, e - 1025)
             if 0 <= b]
    body = "".join(f'std::printf("%d\\n", chunk_end({b}, {e}, {chunk}));' for b, e in cases)
    assert [r[0] for r in run_cpp(tmp_path, body)] == [min(e, b + chunk) for b, e in cases]


V0 = 1 << 20  # smallest vertex count that sweeps with 12 edges per vertex


def arena_bytes(V, degree, hub_degree, need):
    """gx_graph_bytes of a CSR whose first 2^17 rows have hub_degree entries, the others `degree`."""
    from paper_2203_13005_amd import binding as b
    deg = np.full(V, degree)
    deg[:1 << 17] = hub_degree
    rp = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    col, w = np.zeros(rp[-1], np.int32), np.ones(rp[-1], np.uint32)
    d = b._GraphDesc(V, int(rp[-1]), b._np_ptr(rp), b._np_ptr(col), b._np_ptr(w), None, None, need)
    n = ctypes.c_size_t()
    assert b.lib.gx_graph_bytes(ctypes.byref(d), ctypes.byref(n)) == b.GX_OK
    return n.value, int(rp[-1])


def test_which_graphs_sweep():
    from paper_2203_13005_amd import binding as b

    def sssp(V, degree, hub_degree):  # 8 bytes an edge more (no others grow so)
        n, E = arena_bytes(V, degree, hub_degree, b.GX_NEED_OUT)
        return n > 18.5 * E + 24 * V

    assert sssp(V0, 12, 12) and not sssp(V0 - 1, 12, 12) and sssp(V0 // 2, 32, 32) and not sssp(V0 // 2 - 1, 32, 32)
    assert not sssp(V0, 11, 11) and not sssp(3 * V0 // 2 - 1, 11, 11)  # sparse: from 1.5 * 2^20 vertices on
    assert sssp(3 * V0 // 2, 3, 3) and not sssp(2 * V0, 2, 2)
    assert not sssp(V0, 12, 84)  # 2^17 vertices are the sources of half the edges
    assert sssp(2 * V0, 8, 40) and not sssp(2 * V0, 8, 100)  # of 0.25, of 0.45

    def cc(V, degree, hub_degree):  # 8 bytes an entry, two entries an edge
        n, E = arena_bytes(V, degree, hub_degree, b.GX_NEED_SYM)
        return n > 21 * E

    assert cc(V0, 12, 12) and not cc(V0 - 1, 12, 12) and not cc(V0, 11, 11)
    assert cc(3 * V0 // 2, 6, 6) and not cc(2 * V0, 5, 5)
    assert cc(4 * V0, 1, 2) and not cc(4 * V0, 1, 9) and not cc(6 * V0, 1, 1) and not cc(4 * V0, 2, 2)
    assert not cc(V0, 12, 84) and cc(2 * V0, 8, 40) and not cc(2 * V0, 8, 70)
