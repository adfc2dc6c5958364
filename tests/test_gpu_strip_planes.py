"""The explicit Bx/By solver on grids whose transforms use the wave and the
symmetric core and strip-ordered planes: one slice against the FP64 oracle
with a different family on each axis, and a box with launch budgets against
the same box launched kernel by kernel; and solves of FP32 rows of 2048
points (two a workgroup) with strip-ordered planes, and a slice of the loop with
them.  Bars as for the small
grids."""
import dataclasses

import numpy as np
import pytest

import workloads as W
from parity_util import DEPOSIT_NAMES, FIELD_NAMES, field_errors
from test_gpu_explicit import explicit
from test_gpu_graph import make_box, run, same
from test_gpu_parity import one_slice_case
from test_gpu_transforms import dense_solve, tolerance

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("nx,ny", [(32, 128), (128, 128), (128, 256), (256, 128), (512, 32), (32, 512),
                                   (1024, 32), (16, 1024)])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_one_slice(nx, ny, prec):
    # the cells of the square 32-node case, more of them along the long axes
    cfg, beam = W.small(n=32, nzeta=24, nb=1.0)
    hx, hy = cfg.hx, cfg.hy
    cfg = dataclasses.replace(cfg, nx=nx, ny=ny, x_lo=-hx * nx / 2, x_hi=hx * nx / 2,
                              y_lo=-hy * ny / 2, y_hi=hy * ny / 2)
    cfg = explicit(cfg, prec)
    print(f"explicit one slice {nx}x{ny} {prec}", flush=True)
    got, rec, _, _ = one_slice_case(cfg, beam, 6, prec)
    errs = field_errors({q: got[q] for q in FIELD_NAMES + DEPOSIT_NAMES},
                        {q: rec[q] for q in FIELD_NAMES + DEPOSIT_NAMES})
    print("  rel-L2", {q: f"{e:.1e}" for q, e in errs.items()})
    tol = 1e-9 if prec == "fp64" else 1e-4
    assert not {q: e for q, e in errs.items() if e > tol}, errs


@pytest.mark.parametrize("nx,ny", [(256, 256), (512, 256)])
@pytest.mark.parametrize("prec,tol", [("fp64", 1e-12), ("fp32", 1e-5)])
def test_budgeted_box(nx, ny, prec, tol):
    cfg, beam = W.small(n=64, nzeta=20, nb=1.0, pc_max_iter=8, pc_tol=1e-4)
    hx, hy = cfg.hx, cfg.hy
    cfg = dataclasses.replace(cfg, nx=nx, ny=ny, x_lo=-hx * nx / 2, x_hi=hx * nx / 2,
                              y_lo=-hy * ny / 2, y_hi=hy * ny / 2, bxby_solver="explicit")
    print(f"explicit budgets {nx}x{ny} {prec}", flush=True)
    eager = make_box(cfg, prec, graphs=False)
    eager.set_beam_gaussian(beam.amp, beam.sigma_x, beam.sigma_y)
    ref, ref_it, ref_st = run(eager, cfg)
    assert 1 <= ref_it.max() <= cfg.pc_max_iter and ref_it.min() < cfg.pc_max_iter
    box = make_box(cfg, prec, graphs=True)
    box.set_beam_gaussian(beam.amp, beam.sigma_x, beam.sigma_y)
    for rep in range(3):
        got, it, st = run(box, cfg)
        same(got, ref, tol)
        assert np.array_equal(it, ref_it)
        assert st["pc_iterations"] == ref_st["pc_iterations"]
    eager.close()
    box.close()


@pytest.mark.parametrize("nx,ny", [(2048, 256), (2048, 512), (2048, 1024)])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_solves_of_rows_of_2048_points_with_strips(nx, ny, prec):
    from paper_2109_10277_amd import qsp
    cfg = W.BoxConfig(nx=nx, ny=ny, x_lo=-3.0, x_hi=3.0, y_lo=-2.0, y_hi=2.5,
                      nzeta=2, zeta_hi=0.0, dzeta=0.1)
    print(f"solves {nx}x{ny} {prec}", flush=True)
    rng = np.random.default_rng(nx + 3 * ny)
    with qsp.Box(cfg, prec) as box:
        src = torch.tensor(rng.normal(size=(2, ny + 1, nx + 1)), dtype=box.fdtype, device="cuda")
        for shift in (0.0, 0.7):
            ref = dense_solve(cfg, src, shift)
            got = torch.full_like(src, float("nan"))
            box.solve_poisson(src, got, shift)
            torch.cuda.synchronize()
            err = float(torch.linalg.vector_norm(got.double() - ref) / torch.linalg.vector_norm(ref))
            print(f"  shift {shift}: {err:.2e} (tol {tolerance(prec, nx, ny):.1e})")
            assert err < tolerance(prec, nx, ny), (shift, err)


@pytest.mark.parametrize("prec,ny", [("fp32", 256), ("fp64", 128)])
def test_one_slice_of_rows_of_2048_points_with_strips(prec, ny):
    cfg, beam = W.small(n=32, nzeta=24, nb=1.0)
    hx, hy = cfg.hx, cfg.hy
    cfg = dataclasses.replace(cfg, nx=2048, ny=ny, x_lo=-hx * 1024, x_hi=hx * 1024,
                              y_lo=-hy * ny / 2, y_hi=hy * ny / 2)
    print(f"one slice 2048x{ny} {prec}", flush=True)
    got, rec, _, _ = one_slice_case(cfg, beam, 4, prec)
    errs = field_errors({q: got[q] for q in FIELD_NAMES + DEPOSIT_NAMES},
                        {q: rec[q] for q in FIELD_NAMES + DEPOSIT_NAMES})
    print("  rel-L2", {q: f"{e:.1e}" for q, e in errs.items()})
    tol = 1e-9 if prec == "fp64" else 1e-4
    assert not {q: e for q, e in errs.items() if e > tol}, errs
