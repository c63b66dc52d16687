"""LDS layout of the line-fused kernel (no GPU): the FP64 tables (trilinear coefficients, points, vertices) follow the
contraction arrays, whose length in FP32 can be an odd number of words, and have to start at a multiple of 8 bytes."""
import os
import subprocess

import pytest

from paper_2109_05072_amd.build import FLAGS, HIPCC

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2109_05072_amd", "csrc")
SRC = """
#include "apply_kernels.hpp"
using namespace mfhex;
// the tables are whole doubles, so the group's size is a multiple of 8 exactly where they start at one
template <int P, int Q, int S>
constexpr bool slot_ok()
{
    constexpr int G = kLineG[Q - 2][S];
    return line_lds<P, Q, float>(kDiff, G) % 8 == 0 && line_lds<P, Q, double>(kDiff, G) % 8 == 0 &&
           (P == Q || line_lds<P, Q, float>(kMass, G) % 8 == 0);
}
template <int P, int Q>
constexpr bool all_ok() { return slot_ok<P, Q, 0>() && slot_ok<P, Q, 1>() && slot_ok<P, Q, 2>() && slot_ok<P, Q, 3>() && slot_ok<P, Q, 4>(); }
"""
CHECK = 'static_assert(all_ok<{0}, {1}>(), "FP64 tables of a line-fused group at a multiple of 8 bytes");\n'


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not found")
@pytest.mark.parametrize("p", range(1, 9))
def test_fp64_tables_are_aligned(tmp_path, p):
    src = tmp_path / "layout.hip"
    src.write_text(SRC + CHECK.format(p + 1, p + 1) + CHECK.format(p + 1, p + 2))
    r = subprocess.run([HIPCC, *FLAGS, f"-I{CSRC}", "--offload-host-only", "-fsyntax-only", str(src)], capture_output=True,
                       text=True)
    assert r.returncode == 0, r.stderr[-3000:]
