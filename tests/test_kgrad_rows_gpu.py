"""The coefficient gradient on short rows, where a group's elements are stacked in z: ragged stacks, marches with a shorter
last one, masks; and what such a row costs."""
import pytest
import torch

import oracle
import synth
from test_parity_gpu import TOL64, build, dev, host, relerr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("quad", ["gauss", "gll"])
@pytest.mark.parametrize("dirichlet", [True, False])
@pytest.mark.parametrize("p,ne", [(1, (1, 401, 380)), (1, (1, 3, 2)), (1, (2, 3, 17)), (2, (1, 2, 8)), (2, (3, 2, 15)),
                                  (3, (1, 3, 6)), (3, (2, 1, 11)), (4, (1, 2, 5)), (4, (2, 3, 4)), (5, (1, 2, 7)),
                                  (5, (2, 2, 3))])
def test_stacked_groups(gpu_lib, p, ne, dirichlet, quad):
    op, pr = build(gpu_lib, *ne, p, "diffusion", quad, dirichlet, vark=True)
    u = synth.uniform_vector(pr.n_nodes, seed=1)
    r = synth.uniform_vector(pr.n_nodes, seed=2)
    print(p, ne, quad, dirichlet, flush=True)
    g = host(op.kappa_grad(dev(u), dev(r)))
    assert relerr(g, oracle.kappa_grad(pr, u, r)) <= TOL64


@pytest.mark.parametrize("p,quad", [(1, "gauss"), (1, "gll"), (2, "gll")])
def test_rows_of_one_cost_no_more_than_a_cube(gpu_lib, p, quad):
    # 4e5 elements (45 to 110 us) as a slab and as a cube: the same work.  Twice the time is far from both what the slab
    # took with its groups along x (3.5 to 4 times) and what it takes stacked (0.8)
    def us(ne):
        op, pr = build(gpu_lib, *ne, p, "diffusion", quad, True, vark=True)
        u = dev(synth.uniform_vector(pr.n_nodes, seed=1))
        times = []
        for _ in range(5):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            op.kappa_grad(u, u)
            e0.record()
            for _ in range(10):
                op.kappa_grad(u, u)
            e1.record()
            torch.cuda.synchronize()
            times.append(e0.elapsed_time(e1) * 100)
        return min(times)

    slab, cube = us((1, 650, 630)), us((75, 74, 74))
    print(p, quad, "slab", slab, "cube", cube, flush=True)
    assert slab <= 2 * cube
