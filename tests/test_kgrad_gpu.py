"""The line-fused coefficient gradient where its bookkeeping can go wrong: every order and both rules, ragged element
groups, marches through several elements (also a shorter last one), masked and unmasked boundaries; against the
oracle."""
import pytest

import oracle
import synth
from test_parity_gpu import TOL64, build, dev, host, relerr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("quad", ["gauss", "gll"])
@pytest.mark.parametrize("dirichlet", [True, False])
@pytest.mark.parametrize("p,ne", [(1, (1, 1, 1)), (1, (61, 51, 43)), (2, (41, 37, 30)), (2, (3, 2, 1)), (3, (11, 2, 3)),
                                  (4, (7, 2, 3)), (4, (1, 3, 2)), (5, (4, 3, 2)), (6, (3, 2, 2)), (7, (2, 3, 1)),
                                  (8, (3, 1, 2))])
def test_coefficient_gradient(gpu_lib, p, ne, dirichlet, quad):
    op, pr = build(gpu_lib, *ne, p, "diffusion", quad, dirichlet, vark=True)
    u = synth.uniform_vector(pr.n_nodes, seed=1)
    r = synth.uniform_vector(pr.n_nodes, seed=2)
    print(p, ne, quad, dirichlet, flush=True)
    g = host(op.kappa_grad(dev(u), dev(r)))
    assert relerr(g, oracle.kappa_grad(pr, u, r)) <= TOL64
