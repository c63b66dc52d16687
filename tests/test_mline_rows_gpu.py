"""Several vectors of collocated diffusion: which kernel carries a chunk (k_mline's groups of elements along x, or the
element-at-a-time kernel) on short rows, small factors and partial chunks; results of both against the oracle or the
single-vector apply."""
import pytest
import torch

import oracle
import synth
from test_parity_gpu import TOL32, TOL64, build, dev, host, relerr

pytestmark = pytest.mark.gpu
F32, F64 = torch.float32, torch.float64


def check(op, pr, dtype, nvec):
    x = dev(synth.uniform_vector(pr.n_nodes, nvec))
    tol = TOL32 if dtype == F32 else TOL64
    one = [op.apply(x[:, v].contiguous()) for v in (0, nvec // 2, nvec - 1)]
    assert relerr(host(one[0]), oracle.apply(pr, host(x[:, 0].contiguous()))) <= TOL64
    scale = float(one[0].abs().max())
    y = op.apply(x.to(dtype))
    for c, v in enumerate((0, nvec // 2, nvec - 1)):
        assert float((y[:, v].double() - one[c]).abs().max()) <= tol * scale
    op.apply_add(x.to(dtype), y)
    assert float((y[:, 0].double() - 2 * one[0]).abs().max()) <= 2 * tol * scale


# (variant, elements per group): 5 .. 8 are chunks of 2, 4, 8, 16; the element-at-a-time kernel takes one element
@pytest.mark.parametrize("p,ne,dtype,nvec,launch", [
    # rows that leave k_mline's groups idle
    (1, (1, 5, 4), F64, 2, (5, 1)), (1, (2, 5, 4), F64, 4, (6, 1)), (2, (1, 3, 4), F64, 2, (5, 1)), (2, (1, 3, 4), F64, 8, (7, 1)),
    (2, (3, 3, 4), F64, 4, (6, 1)), (3, (1, 3, 2), F64, 8, (7, 1)), (3, (2, 3, 2), F64, 2, (5, 1)), (3, (5, 3, 2), F64, 2, (5, 1)),
    (4, (1, 2, 3), F64, 8, (7, 1)), (4, (3, 2, 3), F64, 12, (7, 1)), (1, (2, 5, 4), F32, 8, (7, 1)), (2, (1, 3, 4), F32, 4, (6, 1)),
    (4, (1, 2, 2), F32, 8, (7, 1)),
    # factors from the Infinity Cache
    (4, (5, 2, 3), F64, 8, (7, 1)), (4, (5, 2, 3), F64, 12, (7, 1)), (5, (3, 2, 2), F32, 2, (5, 1)), (6, (2, 2, 1), F32, 2, (5, 1)),
    # chunks of half a line: several of them with more than 256 elements
    (7, (3, 9, 10), F64, 10, (6, 1)), (7, (3, 9, 10), F64, 12, (6, 1)), (3, (5, 8, 8), F32, 22, (8, 1)),
    (2, (5, 8, 8), F32, 32, (8, 1)),
])
def test_element_kernel(gpu_lib, p, ne, dtype, nvec, launch):
    op, pr = build(gpu_lib, *ne, p, "diffusion", "gll", True, f32=True)
    print(p, ne, dtype, nvec, op.get_config(dtype, nvec), flush=True)
    assert op.get_config(dtype, nvec)[:2] == launch
    check(op, pr, dtype, nvec)


@pytest.mark.parametrize("p,ne,dtype,nvec,launch", [
    (1, (3, 5, 4), F64, 2, (6, 16)), (1, (2, 5, 4), F64, 3, (6, 16)), (2, (4, 3, 4), F64, 4, (6, 7)), (2, (2, 3, 4), F64, 8, (7, 3)),
    (3, (4, 3, 2), F64, 2, (6, 4)), (3, (2, 3, 2), F64, 12, (7, 2)), (3, (1, 3, 2), F64, 20, (7, 2)),
    (4, (5, 2, 3), F64, 7, (7, 2)), (4, (2, 2, 3), F64, 20, (7, 2)), (4, (5, 2, 3), F64, 16, (7, 2)), (4, (2, 2, 3), F64, 4, (6, 2)),
    (5, (1, 2, 2), F64, 8, (7, 1)), (7, (3, 9, 10), F64, 4, (6, 1)), (7, (2, 2, 2), F64, 10, (6, 1)),
    (1, (5, 8, 8), F32, 14, (7, 8)), (2, (5, 8, 8), F32, 20, (7, 3)), (3, (5, 8, 8), F32, 24, (7, 2)), (3, (2, 2, 2), F32, 22, (7, 2)),
    (6, (2, 2, 1), F32, 12, (7, 1)), (7, (3, 10, 9), F32, 17, (7, 1)),
])
def test_line_fused(gpu_lib, p, ne, dtype, nvec, launch):
    op, pr = build(gpu_lib, *ne, p, "diffusion", "gll", False, f32=True)
    print(p, ne, dtype, nvec, op.get_config(dtype, nvec), flush=True)
    assert op.get_config(dtype, nvec)[:2] == launch
    check(op, pr, dtype, nvec)
