"""The adjoint against the FP64 oracle for each way its reverse iterations
close a slice: one predictor-corrector iteration (the first trial push is also
the last), and four (steps of more than one later trial push in the ring).
Tolerances of the other comparisons with the oracle: 1e-9 (FP64), 1e-3
(FP32)."""
import numpy as np
import pytest

import workloads as W
from test_gpu_adjoint import Q, cotangents, gpu_grad, oracle_grad

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("iters", [1, 4])
@pytest.mark.parametrize("prec,tol", [("fp64", 1e-9), ("fp32", 1e-3)])
def test_adjoint_with_one_and_with_four_iterations(iters, order, prec, tol):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cfg, beam = W.small(n=32, nzeta=10, ppc=1, nb=0.9, sigma=0.8, pc_max_iter=iters, pc_tol=0.0,
                        extent=5.0)
    cfg.shape_order = order
    k_lo, k_hi = 4, cfg.nzeta - 1
    w = cotangents(cfg, k_lo, k_hi, seed=iters)
    ga_o, gs_o, L_o = oracle_grad(cfg, beam, k_lo, w)
    print(f"adjoint {iters} iterations order {order} {prec}", flush=True)
    with Q().Box(cfg, prec) as box:
        ga, gs, L = gpu_grad(box, cfg, beam, k_hi + 1, k_lo, w, ckpt_every=3)
    scale = np.abs(ga_o).max()
    assert scale > 0
    assert np.abs(ga - ga_o).max() <= tol * scale, (ga, ga_o)
    assert np.all(np.abs(gs - gs_o) <= tol * np.abs(gs_o)), (gs, gs_o)
    assert abs(L - L_o) <= tol * abs(L_o) + 1e-12, (L, L_o)
