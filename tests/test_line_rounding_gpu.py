"""Factors evaluated in the kernel against stored ones, on flat, stretched and sheared elements: the in-kernel launches are
as close to the oracle as the stored-factor one, in every slot and both precisions."""
import numpy as np
import pytest
import torch

import oracle
import synth
from test_parity_gpu import dev, host, relerr

pytestmark = pytest.mark.gpu


def _mesh(kind, a):
    vert = synth.mesh_vertices(5, 4, 4)
    if kind == "stretched":
        vert[:, 0] *= a
    elif kind == "flat":
        vert[:, 1] /= a
    else:
        vert[:, 0] += a * vert[:, 1]
    return vert


@pytest.mark.parametrize("kind,a", [("stretched", 200.0), ("stretched", 1e4), ("flat", 1e3), ("sheared", 20.0), ("sheared", 1e3)])
@pytest.mark.parametrize("p", [1, 3, 4, 6])
def test_in_kernel_factors_round_like_stored_ones(gpu_lib, p, kind, a):
    # both sides round the same map: 4 times the stored launch's own error, and a few units (8, 64 in FP32, where the
    # stored factors are rounded once more than the evaluated ones and the contractions bound both)
    vert = _mesh(kind, a)
    op = gpu_lib.Operator(5, 4, 4, p, vert, f32=True)
    pr = oracle.Problem(5, 4, 4, p, p + 2, oracle.GAUSS, oracle.DIFFUSION, 1, vert)
    x = synth.uniform_vector(pr.n_nodes)
    yo = oracle.apply(pr, x)
    for dtype, units in ((torch.float64, 8 * np.finfo(np.float64).eps), (torch.float32, 64 * np.finfo(np.float32).eps)):
        op.set_config(0, dtype)
        stored = relerr(host(op.apply(dev(x, dtype))), yo)
        for v in range(9, 14):
            op.set_config(v, dtype)
            err = relerr(host(op.apply(dev(x, dtype))), yo)
            print(kind, a, p, dtype, v, "stored", stored, "in kernel", err, flush=True)
            assert err <= 4 * stored + units
