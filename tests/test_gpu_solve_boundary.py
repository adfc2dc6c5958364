"""Boundary nodes of a solution are zero whatever the source holds: an
infinity or a NaN inside the grid reaches the inner nodes only (every core of
the sine transform, and the solves in one workgroup)."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nx,ny", [(16, 16), (32, 64), (64, 64), (128, 32), (32, 128), (128, 128),
                                   (256, 64), (16, 512), (1024, 32), (64, 2048)])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_boundary_stays_zero(nx, ny, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2109_10277_amd import qsp
    cfg = W.BoxConfig(nx=nx, ny=ny, x_lo=-3.0, x_hi=3.0, y_lo=-2.0, y_hi=2.5,
                      nzeta=2, zeta_hi=0.0, dzeta=0.1)
    print(f"boundary {nx}x{ny} {prec}", flush=True)
    with qsp.Box(cfg, prec) as box:
        src = torch.ones(2, ny + 1, nx + 1, dtype=box.fdtype, device="cuda")
        src[0, ny // 3, nx // 2] = float("nan")
        src[1, ny // 2, nx // 3] = float("inf")
        src[:, 0] = src[:, -1] = float("nan")      # boundary values do not count
        src[:, :, 0] = src[:, :, -1] = float("inf")
        outs = [torch.full_like(src, 7.0) for _ in range(2)]
        box.solve_poisson(src, outs[0], 0.3)
        qsp.solve_poisson_noalloc(cfg, src, outs[1], 0.3, prec)
        torch.cuda.synchronize()
        for name, u in zip(("context", "no alloc"), outs):
            inner = u[:, 1:-1, 1:-1]
            assert not torch.isfinite(inner).all(), name
            edge = u.clone()
            edge[:, 1:-1, 1:-1] = 0
            assert not edge.any(), (name, edge.nonzero()[:4].tolist())
