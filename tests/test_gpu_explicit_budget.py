"""Launch budgets of the explicit Bx/By solver in whole boxes from HIP graphs:
boxes after the first launch only the iterations their slices needed, and a
box whose budgets are one short is run again with every iteration; both give
the results, iteration counts and counters of eager launches (differences:
the order of the deposits' atomic sums)."""
import numpy as np
import pytest

import workloads as W
from test_gpu_graph import make_box, run, same

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [32, 64])
@pytest.mark.parametrize("budget", [None, -1])
@pytest.mark.parametrize("prec,tol", [("fp64", 1e-12), ("fp32", 1e-5)])
def test_explicit_budgets_give_the_full_launch_results(n, budget, prec, tol):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cfg, beam = W.small(n=n, nzeta=30, nb=1.0, pc_max_iter=8, pc_tol=1e-4)
    cfg.bxby_solver = "explicit"
    print(f"explicit budgets {n} {budget} {prec}", flush=True)
    eager = make_box(cfg, prec, graphs=False)
    eager.set_beam_gaussian(beam.amp, beam.sigma_x, beam.sigma_y)
    ref, ref_it, ref_st = run(eager, cfg)
    assert 1 < ref_it.max() and ref_it.min() < cfg.pc_max_iter   # something to save, and to fall short of
    box = make_box(cfg, prec, graphs=True, budget=budget)
    box.set_beam_gaussian(beam.amp, beam.sigma_x, beam.sigma_y)
    for rep in range(3):
        got, it, st = run(box, cfg)
        same(got, ref, tol)
        assert np.array_equal(it, ref_it)
        for q in ("pc_iterations", "pc_not_converged"):
            assert st[q] == ref_st[q], q
        assert st["box_reruns"] == (1 if budget == -1 and rep > 0 else 0), rep
    eager.close()
    box.close()
