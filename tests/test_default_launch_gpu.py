"""The default launch of one vector follows the row length, in both precisions."""
import pytest
import torch

import oracle
import synth
from test_parity_gpu import TOL32, TOL64, build, dev, host, relerr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,quad", [("diffusion", "gauss"), ("diffusion", "gll"), ("mass", "gauss")])
@pytest.mark.parametrize("p", range(1, 9))
def test_short_rows_run_in_small_groups(gpu_lib, kind, quad, p):
    # a row of one element leaves all but one element's lanes of a group idle: groups of one wavefront, which takes its time
    # however many of its lanes idle, or of at most four elements, in FP32 as in FP64
    # (from 257 elements on: fewer take a launch's time in any group)
    op, pr = build(gpu_lib, 1, 19, 14, p, kind, quad, kind == "diffusion", f32=True)
    x = synth.uniform_vector(pr.n_nodes)
    yo = oracle.apply(pr, x) if p < 5 else host(op.apply(dev(x)))
    for dtype, tol in ((torch.float64, TOL64), (torch.float32, TOL32)):
        print(kind, quad, p, dtype, op.get_config(dtype), flush=True)
        _, elements, threads, _ = op.get_config(dtype)
        assert elements <= 4 or threads == 64
        assert relerr(host(op.apply(dev(x, dtype))), yo) <= tol
