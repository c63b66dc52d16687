"""CG's vector kernels, which form alpha and beta from the partial sums themselves: vector lengths around a block, the
grid and four grid strides, both preconditioners, scalars read back every iteration, every third and never; against the
same recurrence in torch on the same operator."""
import pytest
import torch

import synth
from test_parity_gpu import build, dev, interior_mask

pytestmark = pytest.mark.gpu


def torch_cg(op, b, dinv, iters):
    x, r = torch.zeros_like(b), b.clone()
    z = r * dinv if dinv is not None else r
    p, rz = z.clone(), r @ z
    for _ in range(iters):
        q = op.apply(p)
        a = rz / (p @ q)
        x += a * p
        r = r - a * q
        z = r * dinv if dinv is not None else r
        rz, old = r @ z, rz
        p = z + (rz / old) * p
    return x, r


@pytest.mark.parametrize("jacobi", [False, True])
@pytest.mark.parametrize("every", [1, 3, None])
@pytest.mark.parametrize("p,ne", [(1, (3, 3, 3)), (3, (2, 2, 2)), (4, (16, 16, 16)), (4, (23, 23, 23)), (4, (26, 25, 26))])
def test_iterates(gpu_lib, p, ne, every, jacobi):
    op, pr = build(gpu_lib, *ne, p)
    b = dev(synth.uniform_vector(pr.n_nodes, seed=3) * interior_mask(pr))
    iters = 4
    d = op.diagonal()
    dinv = torch.where(d > 0, 1 / d, torch.zeros_like(d)) if jacobi else None
    x, r = torch_cg(op, b, dinv, iters)
    print(p, ne, every, jacobi, flush=True)
    res = op.cg(b, maxit=iters, rtol=0.0, exact_iters=every is None, check_every=every or 1,
                precond="jacobi" if jacobi else "none")
    assert res.iters == iters
    # a few steps of a well-scaled system: reductions of up to 1.1e6 terms in another order, 1e-13 a step
    assert float((res.x - x).abs().max()) <= 4e-13 * float(x.abs().max())
    assert abs(float(res.history[-1]) - float(r.norm())) <= 4e-13 * float(b.norm())
