"""The V-cycle's fused smoother steps at the degrees where their sequence changes (no product, one, several; the
coarsest level alone), on operators that scatter with atomics and from element values, in both precisions, with an output
that holds NaN on entry, twice in a row; against the oracle's V-cycle."""
import pytest
import torch

import synth
from test_parity_gpu import build, dev, host, interior_mask, relerr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("degree,coarse", [(1, 1), (1, 3), (2, 1), (2, 2), (4, 5)])
@pytest.mark.parametrize("p,ne,levels", [(1, (4, 3, 5), 0), (2, (3, 2, 4), 0), (5, (2, 3, 2), 0), (8, (2, 2, 3), 0)])
@pytest.mark.parametrize("det,dtype", [(False, torch.float64), (True, torch.float64), (False, torch.float32)])
def test_vcycle(gpu_lib, p, ne, levels, degree, coarse, det, dtype):
    from oracle import multigrid as omg
    f32 = dtype == torch.float32
    op, pr = build(gpu_lib, *ne, p, "diffusion", "gauss", True, f32=f32, det=det)
    op.mg_setup(degree=degree, coarse_degree=coarse, max_levels=levels, dtype=dtype)
    h = omg.Hierarchy(pr, degree=degree, coarse_degree=coarse)
    r = synth.uniform_vector(pr.n_nodes, seed=5) * interior_mask(pr)
    zo = h.vcycle(r)
    # FP64: the eigenvalue estimates agree to 1e-10, the cycle depends on them smoothly.  FP32: at most about 40
    # products and steps of 6e-8 each, amplified by the condition of the smoother (some tens).
    tol = 1e-4 if f32 else 1e-9
    z = torch.full((pr.n_nodes,), float("nan"), dtype=torch.float64, device="cuda")
    for _ in range(2):
        print(p, degree, coarse, det, dtype, flush=True)
        op.mg_apply(dev(r), z)
        assert relerr(host(z), zo) <= tol
