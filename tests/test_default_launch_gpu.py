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


@pytest.mark.parametrize("p,ne,variant", [(1, (9, 11, 12), 3), (1, (20, 9, 12), 3), (8, (1, 2, 3), 4)])
@pytest.mark.parametrize("option", ["", "vark", "det"])
def test_stored_factors_where_they_are_faster(gpu_lib, p, ne, variant, option):
    # collocated, FP64: short rows, and meshes whose stored factors stay in the Infinity Cache
    op, pr = build(gpu_lib, *ne, p, "diffusion", "gll", True, vark=option == "vark", det=option == "det")
    print(p, ne, option, op.get_config(), flush=True)
    assert op.get_config()[0] == variant
    if option == "vark":
        kap = synth.kappa_field(host(op.qpoint_coords()))
        op.set_kappa(dev(kap))
        pr = pr.with_(kappa=kap)
    x = synth.uniform_vector(pr.n_nodes)
    yo = oracle.apply(pr, x)
    y = op.apply(dev(x))
    assert relerr(host(y), yo) <= TOL64
    op.apply_add(dev(x), y)
    assert relerr(host(y), 2 * yo) <= 2 * TOL64


@pytest.mark.parametrize("p,quad,dtype,ne", [(1, "gll", F64, (91, 91, 91)), (8, "gll", F64, (2, 3, 4)), (1, "gll", F32, (9, 11, 12)),
                                             (3, "gll", F32, (4, 9, 12)), (8, "gll", F32, (1, 19, 14)),
                                             (2, "gauss", F32, (4, 9, 12)), (7, "gauss", F32, (1, 19, 14)),
                                             (2, "gauss", F64, (4, 9, 12)), (3, "gll", F64, (4, 9, 12))])
def test_factors_in_the_kernel_elsewhere(gpu_lib, p, quad, dtype, ne):
    # and everywhere in FP32, where factors stored in FP32 would double the error
    op, pr = build(gpu_lib, *ne, p, "diffusion", quad, True, f32=dtype == F32)
    v = op.get_config(dtype)[0]
    print(p, quad, dtype, ne, op.get_config(dtype), flush=True)
    assert 9 <= v <= 13 if quad == "gauss" else v < 5 and v != {1: 3, 3: -1, 8: 4}[p]


@pytest.mark.parametrize("p,variant,elem,line", [(1, 3, 16, 64), (8, 4, 1, 3)])
def test_stored_factor_number_is_fp64_only(gpu_lib, p, variant, elem, line):
    # the number of the stored-factor kernel is a group of the line kernel in FP32 and with in-kernel factors
    op, pr = build(gpu_lib, 3, 2, 2, p, "diffusion", "gll", True, f32=True)
    x = synth.uniform_vector(pr.n_nodes)
    yo = oracle.apply(pr, x)
    for dtype, g, tol in ((F64, elem, TOL64), (F32, line, TOL32)):
        op.set_config(variant, dtype)
        assert op.get_config(dtype)[:2] == (variant, g)
        assert relerr(host(op.apply(dev(x, dtype))), yo) <= tol
    otf, _ = build(gpu_lib, 3, 2, 2, p, "diffusion", "gll", True, otf=True)
    otf.set_config(variant)
    assert otf.get_config()[:2] == (variant, line)
    assert relerr(host(otf.apply(dev(x))), yo) <= TOL64


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
