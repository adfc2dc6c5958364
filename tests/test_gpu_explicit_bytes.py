"""Device memory of a box grows by one iteration count a slice, with either
Bx/By solver."""
import dataclasses

import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("solver", ["pc", "explicit"])
def test_bytes_per_slice(solver):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2109_10277_amd import qsp
    cfg, _ = W.small(n=16, nzeta=1000)
    held = []
    for nzeta in (1000, 9000):
        with qsp.Box(dataclasses.replace(cfg, nzeta=nzeta, bxby_solver=solver), "fp32") as box:
            box.init_plasma()
            held.append(box.stats()["device_bytes"])
    assert held[1] - held[0] == 4 * 8000, held
