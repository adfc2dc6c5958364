"""The division by the eigenvalues of the shifted Laplacian in FP32 columns of
2048 points: the eigenvalue is summed in FP64, rounded once, and divided by.

Each source holds a few sine modes, one per column of the transform and all of
one size in the solution; a mode's amplitude, projected in FP64, shows what its
division lost.  Two classes of modes are taken: those whose eigenvalue a sum
of two terms rounded to FP32 would overestimate by 1.2 u or more (u = 2^-24),
and those it would underestimate as much, while the sum rounded once is within
0.25 u in both.  With such sums the mean amplitudes of the two classes lie
2.4 u or more apart; what else a mode goes through is common to both.
Tolerance 1 u: 0.5 u from the selection, and the scatter of a class of 40
modes or more with three independent roundings of up to u (the transform's
result, the quotient, the inverse), sqrt(3) 0.6 u / sqrt(40) = 0.16 u, for the
difference of two classes 0.23 u, twice."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

U = 2.0 ** -24


def eigenvalues(n, h):
    return -4.0 / (h * h) * np.sin(np.pi * np.arange(n) / (2 * n)) ** 2


def pick(cfg, sign, most):
    """[(source, x mode, y mode)] of the modes over- (sign 1) or underestimated
    (-1) by a sum of FP32 terms: up to `most` y modes for each x mode."""
    norm = 0.25 * cfg.nx * cfg.ny
    lx, ly = eigenvalues(cfg.nx, cfg.hx), eigenvalues(cfg.ny, cfg.hy)
    f32 = lambda v: np.asarray(v, dtype=np.float32).astype(np.float64)  # noqa: E731
    out = []
    for p in range(1, cfg.nx):
        d = (lx[p] + ly) * norm
        once = np.abs(f32(d) / d - 1) / U
        two = sign * (f32(f32(lx[p] * norm) + f32(ly * norm)) / d - 1) / U
        ok = (once < 0.25) & (np.abs(lx[p] + ly) > 5.0) & (np.arange(cfg.ny) > 0) & (two > 1.2)
        q = np.where(ok)[0]
        out += [(s, p, m) for s, m in enumerate(q[np.argsort(-two[q])][:most])]
    return out


@pytest.mark.parametrize("solve", ["context", "no alloc"])
def test_sum_in_fp64_and_one_rounding(solve):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2109_10277_amd import qsp
    cfg = W.BoxConfig(nx=64, ny=2048, x_lo=-3.0, x_hi=3.0, y_lo=-400.0, y_hi=400.0,
                      nzeta=2, zeta_hi=0.0, dzeta=0.1)
    print(f"eigenvalue division {solve}", flush=True)
    n_src = 16
    lx, ly = eigenvalues(cfg.nx, cfg.hx), eigenvalues(cfg.ny, cfg.hy)
    i, j = np.arange(cfg.nx + 1), np.arange(cfg.ny + 1)
    sx = np.sin(np.pi * np.outer(np.arange(cfg.nx), i) / cfg.nx)
    mean = {}
    with qsp.Box(cfg, "fp32") as box:
        for sign in (1, -1):
            modes = pick(cfg, sign, n_src)
            assert len(modes) >= 40
            src = np.zeros((n_src, cfg.ny + 1, cfg.nx + 1))
            for s, p, m in modes:
                src[s] += (lx[p] + ly[m]) * np.outer(np.sin(np.pi * m * j / cfg.ny), sx[p])
            src32 = torch.tensor(src, dtype=torch.float32, device="cuda")
            dst = torch.empty_like(src32)
            for s in range(0, n_src, 4):
                if solve == "context":
                    box.solve_poisson(src32[s:s + 4], dst[s:s + 4], 0.0)
                else:
                    qsp.solve_poisson_noalloc(cfg, src32[s:s + 4], dst[s:s + 4], 0.0, "fp32")
            torch.cuda.synchronize()
            f, u = src32.double().cpu().numpy(), dst.double().cpu().numpy()
            err = []
            for s, p, m in modes:
                sy = np.sin(np.pi * m * j[1:-1] / cfg.ny)
                fa = sy @ f[s, 1:-1, 1:-1] @ sx[p, 1:-1]
                ua = sy @ u[s, 1:-1, 1:-1] @ sx[p, 1:-1]
                err.append((ua * (lx[p] + ly[m]) / fa - 1) / U)
            mean[sign] = np.mean(err)
            print(f"  class {sign}: {len(err)} modes, mean {np.mean(err):.2f}, scatter {np.std(err):.2f}")
    assert abs(mean[1] - mean[-1]) < 1.0, mean
