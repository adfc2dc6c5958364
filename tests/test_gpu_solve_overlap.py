"""Batched solves whose solutions overlap their sources: in place, shifted by
whole fields either way, or by a few values.  Every source counts as it was
before the call, whichever path a grid takes (one workgroup per field up to
64 x 64, three passes above).

Tolerance: the two paths sum in different orders, so the solutions differ by
the round-off of a solve, bounded as in the tests of the transforms by
4 passes of log2(2n) + 3 levels of 3 eps each, for both."""
import math

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nx,ny", [(16, 16), (32, 64), (64, 64), (64, 16), (128, 64)])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_sources_count_as_they_were(nx, ny, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2109_10277_amd import qsp
    cfg = W.BoxConfig(nx=nx, ny=ny, x_lo=-3.0, x_hi=3.0, y_lo=-2.0, y_hi=2.5,
                      nzeta=2, zeta_hi=0.0, dzeta=0.1)
    print(f"overlapping batches {nx}x{ny} {prec}", flush=True)
    tol = 2 * (1.2e-7 if prec == "fp32" else 2.3e-16) * 12 * (math.log2(2 * max(nx, ny)) + 3)
    rng = np.random.default_rng(nx + 5 * ny)
    field = (nx + 1) * (ny + 1)
    with qsp.Box(cfg, prec) as box:
        solves = {"context": box.solve_poisson,
                  "no alloc": lambda s, d, h: qsp.solve_poisson_noalloc(cfg, s, d, h, prec)}
        for nb in (1, 2, 4):
            values = torch.tensor(rng.normal(size=(nb, ny + 1, nx + 1)), dtype=box.fdtype, device="cuda")
            ref = torch.empty_like(values)
            box.solve_poisson(values, ref, 0.7)
            for off in (0, field, -field, 2 * field, nx + 1, -(nx + 1), 5, -3):
                if abs(off) >= nb * field:
                    continue
                for name, solve in solves.items():
                    pad = max(0, -off)
                    buf = torch.zeros(nb * field + abs(off), dtype=box.fdtype, device="cuda")
                    src = buf[pad:pad + nb * field].view_as(values)
                    dst = buf[pad + off:pad + off + nb * field].view_as(values)
                    src.copy_(values)
                    solve(src, dst, 0.7)
                    torch.cuda.synchronize()
                    err = float(torch.linalg.vector_norm((dst - ref).double()) /
                                torch.linalg.vector_norm(ref.double()))
                    assert err <= tol, (name, nb, off, err, tol)
