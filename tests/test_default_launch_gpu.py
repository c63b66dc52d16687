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


F32, F64 = torch.float32, torch.float64


@pytest.mark.parametrize("p,quad,dtype,ne,variant", [
    (1, "gll", F64, (9, 11, 12), 3), (1, "gll", F64, (20, 9, 12), 3), (1, "gll", F32, (13, 9, 12), 3),
    (1, "gll", F32, (20, 9, 12), 3), (3, "gll", F32, (4, 9, 12), 2), (3, "gll", F32, (1, 20, 14), 2),
    (8, "gll", F32, (1, 19, 14), 4), (8, "gll", F64, (1, 2, 3), 4), (2, "gauss", F32, (4, 9, 12), 0),
    (2, "gauss", F32, (11, 9, 12), 0), (7, "gauss", F32, (1, 19, 14), 3), (8, "gauss", F32, (1, 19, 14), 3)])
@pytest.mark.parametrize("option", ["", "vark", "det"])
def test_stored_factors_where_they_are_faster(gpu_lib, p, quad, dtype, ne, variant, option):
    # short rows, and meshes whose stored factors stay in the Infinity Cache, run on the stored-factor kernel
    if option == "vark" and dtype == F32:
        pytest.skip("a coefficient is FP64 only")
    op, pr = build(gpu_lib, *ne, p, "diffusion", quad, True, f32=dtype == F32, vark=option == "vark", det=option == "det")
    print(p, quad, dtype, ne, option, op.get_config(dtype), flush=True)
    assert op.get_config(dtype)[0] == variant
    if option == "vark":
        kap = synth.kappa_field(host(op.qpoint_coords()))
        op.set_kappa(dev(kap))
        pr = pr.with_(kappa=kap)
    x = synth.uniform_vector(pr.n_nodes)
    yo = oracle.apply(pr, x) if p < 5 or len(set(ne)) == 3 and max(ne) < 5 else host(op.apply(dev(x)))
    xd = dev(x, dtype)
    y = op.apply(xd)
    tol = TOL32 if dtype == F32 else TOL64
    assert relerr(host(y), yo) <= tol
    op.apply_add(xd, y)
    assert relerr(host(y), 2 * yo) <= 2 * tol


@pytest.mark.parametrize("p,quad,dtype,ne", [(1, "gll", F64, (91, 91, 91)), (1, "gll", F32, (115, 115, 115)),
                                             (3, "gll", F32, (5, 9, 12)), (8, "gll", F32, (2, 14, 14)),
                                             (2, "gauss", F32, (71, 71, 71)), (7, "gauss", F32, (2, 14, 14)),
                                             (2, "gauss", F64, (4, 9, 12)), (3, "gll", F64, (4, 9, 12))])
def test_factors_in_the_kernel_elsewhere(gpu_lib, p, quad, dtype, ne):
    op, pr = build(gpu_lib, *ne, p, "diffusion", quad, True, f32=dtype == F32)
    v = op.get_config(dtype)[0]
    print(p, quad, dtype, ne, op.get_config(dtype), flush=True)
    assert 9 <= v <= 13 if quad == "gauss" else v < 5 and v != {1: 3, 3: 2, 8: 4}[p]


@pytest.mark.parametrize("p,option", [(8, ""), (8, "vark"), (8, "otf"), (8, "det"), (7, "det")])
@pytest.mark.parametrize("ne", [(2, 2, 2), (4, 4, 4), (6, 6, 7)])
def test_few_large_elements_run_alone(gpu_lib, p, option, ne):
    # at most 256 elements of 81 or 100 lines: groups of one element
    op, pr = build(gpu_lib, *ne, p, "diffusion", "gauss", True, vark=option == "vark", otf=option == "otf", det=option == "det")
    print(p, option, ne, op.get_config(), flush=True)
    assert op.get_config()[1] == 1
    if option == "vark":
        op.set_kappa(torch.ones(op.n_elem, op.q ** 3, dtype=torch.float64, device="cuda"))
    x = synth.uniform_vector(pr.n_nodes)
    if max(ne) < 5:
        assert relerr(host(op.apply(dev(x))), oracle.apply(pr, x)) <= TOL64
