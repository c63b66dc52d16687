"""The line-fused kernel where its bookkeeping can go wrong: ragged element groups in x, marches that carry the
y-face (several elements per group, a shorter last march), masks at both ends of a march, y += A x, several
vectors in one launch, and the 64-bit node offsets of very large slabs; against the oracle or the single-vector
apply."""
import numpy as np
import pytest
import torch

import oracle
import synth
from test_parity_gpu import TOL32, TOL64, build, dev, host, relerr, valid_variants

pytestmark = pytest.mark.gpu


def line_variants(op, kind, quad, otf=False):
    vs = valid_variants(op)
    return [v for v in vs if (v < 5 if kind == "mass" or quad == "gll" or otf else 9 <= v <= 14)]


@pytest.mark.parametrize("kind,quad", [("diffusion", "gauss"), ("diffusion", "gll"), ("mass", "gauss")])
@pytest.mark.parametrize("p", [1, 2])
@pytest.mark.parametrize("dirichlet", [True, False])
def test_marches_and_ragged_groups(gpu_lib, kind, quad, p, dirichlet):
    # enough elements that one-wavefront groups march through two elements, and an odd count so that the last
    # march of a column is shorter; 41 is no multiple of any group size
    ne = (41, 37, 30) if p == 2 else (61, 51, 43)
    op, pr = build(gpu_lib, *ne, p, kind, quad, dirichlet)
    x = synth.uniform_vector(pr.n_nodes)
    yo = oracle.apply(pr, x)
    for v in line_variants(op, kind, quad):
        for depth in ((1, 2, 8, 64) if kind == "mass" else (0,)):
            op.set_config(v, groups_per_block=depth)
            print(kind, quad, p, dirichlet, v, depth, flush=True)
            assert relerr(host(op.apply(dev(x))), yo) <= TOL64
    y = dev(yo)
    op.apply_add(dev(x), y)
    assert relerr(host(y), 2 * yo) <= TOL64


@pytest.mark.parametrize("nex", [1, 2, 3, 4, 5, 6, 7, 8, 9, 11, 17])
@pytest.mark.parametrize("p", [3, 5, 7])
def test_default_launch_on_short_rows(gpu_lib, p, nex):
    # the default slot depends on the row length: every length near the group sizes, both precisions, OTF too
    op, pr = build(gpu_lib, nex, 2, 3, p, "diffusion", "gauss", True, f32=True)
    otf, _ = build(gpu_lib, nex, 2, 3, p, "diffusion", "gauss", True, otf=True)
    x = synth.uniform_vector(pr.n_nodes)
    yo = oracle.apply(pr, x)
    print(p, nex, op.get_config(), op.get_config(torch.float32), flush=True)
    assert relerr(host(op.apply(dev(x))), yo) <= TOL64
    assert relerr(host(otf.apply(dev(x))), yo) <= TOL64
    assert relerr(host(op.apply(dev(x, torch.float32))), yo) <= TOL32


def test_stretched_and_sheared_elements(gpu_lib):
    # factors from the trilinear coefficients of flat, skewed elements (aspect 200): as close to the oracle as the
    # stored-factor launch, within the conditioning of the element map (aspect^2 units of rounding)
    vert = synth.mesh_vertices(6, 5, 4)
    vert[:, 0] = 200.0 * vert[:, 0] + 30.0 * vert[:, 1]
    vert[:, 2] += 0.3 * vert[:, 1]
    op = gpu_lib.Operator(6, 5, 4, 4, vert)
    pr = oracle.Problem(6, 5, 4, 4, 6, oracle.GAUSS, oracle.DIFFUSION, 1, vert)
    x = synth.uniform_vector(pr.n_nodes)
    yo = oracle.apply(pr, x)
    tol = 4e4 * np.finfo(float).eps
    op.set_config(0)
    stored = relerr(host(op.apply(dev(x))), yo)
    for v in (9, 10):
        op.set_config(v)
        err = relerr(host(op.apply(dev(x))), yo)
        print("stretched: stored", stored, "in kernel", err, flush=True)
        assert err <= tol


def test_offsets_beyond_32_bits(gpu_lib):
    # 4096 vectors: a slab of P planes spans more than 2^31 bytes, so a lane's offset inside it needs 64 bits
    op, pr = build(gpu_lib, 181, 181, 1, 1, "diffusion", "gauss", False)
    nrhs = 4096
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    x = torch.rand(pr.n_nodes, nrhs, dtype=torch.float64, device="cuda", generator=gen)
    op.set_config(9, nrhs=nrhs)
    y = op.apply(x)
    for v in (0, 1777, 4095):
        ref = op.apply(x[:, v].contiguous())
        assert float((y[:, v] - ref).abs().max()) <= 1e-13 * float(ref.abs().max())
