"""The solve count of an explicit box: psi, Ez and Bz of every slice, and one
preconditioner solve for Bx and By in every conjugate-gradient iteration that
ran, whether the box is launched kernel by kernel or from graphs with launch
budgets."""
import pytest

import workloads as W
from test_gpu_graph import make_box, run

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [32, 64])
def test_solves_of_an_explicit_box(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cfg, beam = W.small(n=n, nzeta=20, nb=1.0, pc_max_iter=8, pc_tol=1e-4)
    cfg.bxby_solver = "explicit"
    print(f"explicit solves {n}", flush=True)
    for graphs in (False, True):
        box = make_box(cfg, "fp64", graphs=graphs)
        box.set_beam_gaussian(beam.amp, beam.sigma_x, beam.sigma_y)
        for rep in range(3):
            _, it, st = run(box, cfg)
            assert 0 < it.sum() < cfg.nzeta * cfg.pc_max_iter
            assert st["dst_solves"] == 3 * cfg.nzeta + 2 * it.sum(), (graphs, rep)
        box.close()
