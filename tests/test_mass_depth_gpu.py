"""Pipeline depths of the mass operator: each kernel's default is its own."""
import pytest
import torch

from test_parity_gpu import build

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", range(1, 8))
def test_several_vectors_take_the_depth_of_their_kernel(gpu_lib, p):
    # Gauss points with several vectors (or components) run on the kernel of the collocated mass operator with the
    # same points, one order up: same default depth
    coll, _ = build(gpu_lib, 2, 3, 2, p + 1, "mass", "gll", False)
    gauss, _ = build(gpu_lib, 2, 3, 2, p, "mass", "gauss", False, f32=True)
    three = gpu_lib.Operator(2, 3, 2, p, gauss._vert, kind="mass", ncomp=3, dirichlet=False)
    depth = coll.get_config()[3]
    for nrhs in (2, 3, 4, 8, 16):
        assert gauss.get_config(nrhs=nrhs)[3] == depth
        assert gauss.get_config(torch.float32, nrhs)[3] == depth
    assert three.get_config()[3] == depth


@pytest.mark.parametrize("p,ne,largest", [(1, (3, 2, 2), 1), (3, (40, 24, 24), 7), (3, (3, 70, 3), 1)])
def test_the_default_depth_is_automatic_when_it_is_set(gpu_lib, p, ne, largest):
    # meshes that leave a march fewer elements than the largest default: depth 0 is that same launch, and what is
    # reported is what runs (16384 wavefronts stay in flight)
    op, _ = build(gpu_lib, *ne, p, "mass", "gauss", False)
    default = op.get_config()
    assert 1 <= default[3] <= largest
    op.set_config(default[0], groups_per_block=0)
    assert op.get_config() == default
    op.set_config(default[0], groups_per_block=64)
    assert op.get_config()[3] == 64
