"""The sine transforms at the edges of their families (matrix product for
n <= 64, wave for FP32 256 and 512, symmetric for the rest) and with a
different family on each axis: batched solves against a dense sine basis in
FP64, and one slice of the loop against the FP64 oracle on grids whose two
axes use different families and plane orders.

Solve tolerances: each of the four transform passes is a chain of at most
log2(2n) + 3 rounded levels of about 3 eps each, relative in L2, and the
round-off of the passes in front of the division by the eigenvalues is white
like the sources, so it is amplified like the source itself; a sum of up to 32
products rounds no worse."""
import dataclasses
import math

import numpy as np
import pytest

import workloads as W
from parity_util import DEPOSIT_NAMES, FIELD_NAMES, field_errors
from test_gpu_parity import one_slice_case

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def Q():
    from paper_2109_10277_amd import qsp
    return qsp


def sine(n):
    """S[k-1, i-1] = sin(pi i k / n), arguments reduced in whole numbers."""
    i = torch.arange(1, n, dtype=torch.int64, device="cuda")
    m = torch.outer(i, i) % (2 * n)
    return torch.sin(m.double() * (math.pi / n))


def dense_solve(cfg, src, shift):
    """-(Dxx + Dyy - shift) u = f inverted in the sine basis, interior nodes."""
    sx, sy = sine(cfg.nx), sine(cfg.ny)
    lam = []
    for n, h in ((cfg.nx, cfg.hx), (cfg.ny, cfg.hy)):
        k = torch.arange(1, n, dtype=torch.float64, device="cuda")
        lam.append(-(2.0 / h * torch.sin(math.pi * k / (2 * n))) ** 2)
    out = torch.zeros_like(src, dtype=torch.float64)
    scale = 4.0 / (cfg.nx * cfg.ny)
    for b in range(src.shape[0]):
        f = src[b, 1:-1, 1:-1].double()
        hat = sy @ f @ sx
        hat = hat * scale / (lam[1][:, None] + lam[0][None, :] - shift)
        out[b, 1:-1, 1:-1] = sy @ hat @ sx
    return out


def tolerance(prec, nx, ny):
    eps = 1.2e-7 if prec == "fp32" else 2.3e-16
    return eps * 4 * 3 * (math.log2(2 * max(nx, ny)) + 3)


@pytest.mark.parametrize("nx,ny", [(16, 16), (32, 64), (64, 32), (128, 16), (16, 128), (128, 128), (128, 256), (512, 128),
                                   (256, 1024), (1024, 256), (64, 512), (1024, 64), (2048, 128),
                                   (512, 2048), (2048, 16), (32, 2048)])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_solves_at_the_edges_of_the_transform_families(nx, ny, prec):
    cfg = W.BoxConfig(nx=nx, ny=ny, x_lo=-3.0, x_hi=3.0, y_lo=-2.0, y_hi=2.5,
                      nzeta=2, zeta_hi=0.0, dzeta=0.1)
    print(f"transforms {nx}x{ny} {prec}", flush=True)
    rng = np.random.default_rng(nx + 3 * ny)
    with Q().Box(cfg, prec) as box:
        src = torch.tensor(rng.normal(size=(2, ny + 1, nx + 1)), dtype=box.fdtype, device="cuda")
        for shift in (0.0, 0.7):
            ref = dense_solve(cfg, src, shift)   # boundary nodes of the source do not count
            outs = {"context": torch.full_like(src, float("nan")), "in place": src.clone(),
                    "no alloc": torch.full_like(src, float("nan"))}
            box.solve_poisson(src, outs["context"], shift)
            box.solve_poisson(outs["in place"], outs["in place"], shift)
            Q().solve_poisson_noalloc(cfg, src, outs["no alloc"], shift, prec)
            torch.cuda.synchronize()
            for name, got in outs.items():
                assert torch.isfinite(got).all(), name
                err = float(torch.linalg.vector_norm(got.double() - ref) /
                            torch.linalg.vector_norm(ref))
                print(f"  {name} shift {shift}: {err:.2e} (tol {tolerance(prec, nx, ny):.1e})")
                assert err < tolerance(prec, nx, ny), (name, shift, err)
                edge = got.clone()
                edge[:, 1:-1, 1:-1] = 0
                assert not edge.any(), name


@pytest.mark.parametrize("nx,ny", [(16, 32), (32, 64), (64, 32), (128, 16), (16, 128), (128, 256), (256, 128),
                                   (512, 32)])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_one_slice_with_two_transform_families(nx, ny, prec):
    # same cells as the square 32-node case, more of them along the long axes
    cfg, beam = W.small(n=32, nzeta=24, nb=1.0)
    hx, hy = cfg.hx, cfg.hy
    cfg = dataclasses.replace(cfg, nx=nx, ny=ny, x_lo=-hx * nx / 2, x_hi=hx * nx / 2,
                              y_lo=-hy * ny / 2, y_hi=hy * ny / 2)
    print(f"one slice {nx}x{ny} {prec}", flush=True)
    got, rec, _, _ = one_slice_case(cfg, beam, 6, prec)
    errs = field_errors({q: got[q] for q in FIELD_NAMES + DEPOSIT_NAMES},
                        {q: rec[q] for q in FIELD_NAMES + DEPOSIT_NAMES})
    print("  rel-L2", {q: f"{e:.1e}" for q, e in errs.items()})
    tol = 1e-9 if prec == "fp64" else 1e-4   # one slice, as for the square grids
    assert not {q: e for q, e in errs.items() if e > tol}, errs
