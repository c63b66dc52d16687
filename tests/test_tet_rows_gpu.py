"""The tetrahedral apply on rows of one and two hexahedra, whose boxes of eight go along y: full and ragged boxes, several
steps of a set, masks at both ends; and what such a row costs."""
import pytest
import torch

import synth
from oracle import tet as otet
from test_tet_gpu import TOL64, build, dev, host, relerr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", range(1, 7))
@pytest.mark.parametrize("ne", [(1, 8, 1), (1, 9, 2), (2, 5, 3), (2, 17, 1), (1, 1, 1)])
@pytest.mark.parametrize("dirichlet", [True, False])
def test_boxes_along_y(gpu_lib, p, ne, dirichlet):
    op, pr = build(gpu_lib, ne, p, dirichlet=dirichlet)
    x = synth.uniform_vector(pr.n_nodes)
    y = host(op.apply(dev(x)))
    err = relerr(y, otet.apply(pr, x))
    print(p, ne, dirichlet, err, flush=True)
    assert err <= TOL64


def test_many_steps_of_a_set(gpu_lib):
    # more boxes than sets on the chip: A 1 = 0, and the middle column of nodes, which sees the slab's own elements only,
    # gets what it gets inside a wider mesh, whose boxes go along x
    wide, pw = build(gpu_lib, (5, 203, 300), 1, dirichlet=False, perturb=0.0)
    xw = synth.uniform_vector(pw.n_nodes).reshape(301, 204, 6)
    ref = host(wide.apply(dev(xw.reshape(-1)))).reshape(301, 204, 6)
    vert = synth.mesh_vertices(2, 203, 300, 0.0)
    vert[:, 0] *= 0.4
    op = gpu_lib.TetOperator(2, 203, 300, 1, vert, dirichlet=False)
    slab = xw[:, :, 2:5].copy()
    y = host(op.apply(dev(slab.reshape(-1)))).reshape(301, 204, 3)
    assert relerr(y[:, :, 1], ref[:, :, 3]) <= TOL64
    assert abs(host(op.apply(dev(0 * slab.reshape(-1) + 1)))).max() <= TOL64 * abs(y).max()


@pytest.mark.parametrize("p", [4, 6])
def test_rows_of_one_cost_no_more_than_a_cube(gpu_lib, p):
    # 2e4 hexahedra as a slab and as a cube.  Twice the time is far from both what the slab took with its boxes along x
    # (4 times and more) and what it takes with boxes along y
    def us(ne):
        op, pr = build(gpu_lib, ne, p)
        x = dev(synth.uniform_vector(pr.n_nodes))
        y = torch.empty_like(x)
        times = []
        for _ in range(5):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            op.apply(x, y)
            e0.record()
            for _ in range(10):
                op.apply(x, y)
            e1.record()
            torch.cuda.synchronize()
            times.append(e0.elapsed_time(e1) * 100)
        return min(times)

    slab, cube = us((1, 144, 144)), us((24, 29, 30))
    print(p, "slab", slab, "cube", cube, flush=True)
    assert slab <= 2 * cube
