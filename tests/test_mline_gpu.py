"""The line-fused multi-vector kernel of the collocated diffusion operator where its bookkeeping can go wrong: partial
chunks of vectors, ragged element groups, marches (also with a shorter last one), masks, both precisions, y += A x,
64-bit node offsets; against the oracle or the single-vector apply."""
import pytest
import torch

import oracle
import synth
from test_parity_gpu import TOL32, TOL64, build, dev, host, relerr, valid_variants

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nvec", [2, 3, 4, 5, 8, 9, 12])
@pytest.mark.parametrize("p,ne,dirichlet", [(1, (33, 40, 37), True), (2, (10, 33, 30), False), (3, (5, 41, 40), True),
                                            (4, (3, 2, 5), True), (5, (3, 2, 2), False), (6, (2, 3, 1), True),
                                            (7, (1, 2, 2), True), (8, (2, 1, 2), False)])
def test_chunks_groups_and_marches(gpu_lib, nvec, p, ne, dirichlet):
    op, pr = build(gpu_lib, *ne, p, "diffusion", "gll", dirichlet, f32=True)
    x = dev(synth.uniform_vector(pr.n_nodes, nvec))
    ref = oracle.apply(pr, host(x[:, nvec - 1].contiguous()))  # the last vector sits in the partial chunk
    one = [op.apply(x[:, v].contiguous()) for v in range(nvec)]
    scale = float(one[0].abs().max())
    for dtype, tol in ((torch.float64, TOL64), (torch.float32, TOL32)):
        xd = x.to(dtype)
        print(p, ne, nvec, dtype, "default", op.get_config(dtype, nvec), flush=True)
        assert relerr(host(op.apply(xd)[:, nvec - 1].contiguous()).astype("float64"), ref) <= tol
        for v in [v for v in valid_variants(op, dtype, nvec) if v in (6, 7)]:
            op.set_config(v, dtype, nvec)
            print(p, ne, nvec, dtype, v, op.get_config(dtype, nvec), flush=True)
            y = op.apply(xd)
            assert relerr(host(y[:, nvec - 1].contiguous()).astype("float64"), ref) <= tol
            for c in range(nvec):
                assert float((y[:, c].double() - one[c]).abs().max()) <= tol * scale
            op.apply_add(xd, y)
            assert float((y[:, 0].double() - 2 * one[0]).abs().max()) <= 2 * tol * scale


@pytest.mark.parametrize("v", [6, 7])
def test_offsets_beyond_32_bits(gpu_lib, v):
    # 4096 vectors: a slab of P planes spans more than 2^31 bytes, so a lane's offset inside it needs 64 bits
    op, pr = build(gpu_lib, 181, 181, 1, 1, "diffusion", "gll", False)
    nrhs = 4096
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    x = torch.rand(pr.n_nodes, nrhs, dtype=torch.float64, device="cuda", generator=gen)
    op.set_config(v, nrhs=nrhs)
    y = op.apply(x)
    for c in (0, 1777, 4095):
        ref = op.apply(x[:, c].contiguous())
        assert float((y[:, c] - ref).abs().max()) <= 1e-13 * float(ref.abs().max())


def test_grids_beyond_32_bits(gpu_lib):
    # 700 x 1 x 700 elements, 4096 vectors of p = 1: 8e9 lanes, more than one launch may have
    op, pr = build(gpu_lib, 700, 1, 700, 1, "diffusion", "gll", False, f32=True)
    nrhs = 4096
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    x = torch.rand(pr.n_nodes, nrhs, dtype=torch.float32, device="cuda", generator=gen)
    op.set_config(6, torch.float32, nrhs)
    y = op.apply(x)
    for c in (0, 2047, 4095):
        ref = op.apply(x[:, c].contiguous())
        assert float((y[:, c] - ref).abs().max()) <= TOL32 * float(ref.abs().max())
