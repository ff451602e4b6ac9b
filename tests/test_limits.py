"""The limits in gx_limits.h, compiled as plain C++ (no GPU): widths of
counters and indexes at the largest graphs that a load accepts."""
import os
import subprocess

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
