"""Solves with a shift so large that its product with nx ny / 4 overflows the
field precision, or nearly so: the exact solution is smaller than source /
shift, and comes out finite and near zero (every core of the sine transform,
and the solves in one workgroup)."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nx,ny", [(64, 64), (64, 128), (128, 256), (32, 512), (64, 1024), (32, 2048)])
@pytest.mark.parametrize("prec,shift", [("fp64", 1e307), ("fp32", 1e37), ("fp32", 1e300)])
def test_solution_is_finite(nx, ny, prec, shift):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2109_10277_amd import qsp
    cfg = W.BoxConfig(nx=nx, ny=ny, x_lo=-3.0, x_hi=3.0, y_lo=-2.0, y_hi=2.5,
                      nzeta=2, zeta_hi=0.0, dzeta=0.1)
    print(f"large shift {nx}x{ny} {prec} {shift}", flush=True)
    with qsp.Box(cfg, prec) as box:
        src = torch.ones(2, ny + 1, nx + 1, dtype=box.fdtype, device="cuda")
        outs = [torch.full_like(src, 7.0) for _ in range(2)]
        box.solve_poisson(src, outs[0], shift)
        qsp.solve_poisson_noalloc(cfg, src, outs[1], shift, prec)
        torch.cuda.synchronize()
        for name, u in zip(("context", "no alloc"), outs):
            assert torch.isfinite(u).all(), name
            assert float(u.abs().max()) < 1e-30, name
