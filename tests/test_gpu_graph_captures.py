"""What a caller with a new drive for every box pays for: an explicit box
captures one graph when its drive is new, the graph with the launch budgets
when a second box of the same drive comes, and none from then on."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CODE = """
import sys
sys.path.insert(0, {root!r})
import torch
import workloads as W
from paper_2109_10277_amd import qsp
cfg, beam = W.small(n=32, nzeta=12, nb=1.0, pc_max_iter=8, pc_tol=1e-4)
cfg.bxby_solver = "explicit"
with qsp.Box(cfg, "fp32") as box:
    for drive in range(2):
        box.set_beam_gaussian((1.0 - 0.1 * drive) * beam.amp, beam.sigma_x, beam.sigma_y)
        for rep in range(4):
            box.init_plasma()
            box.run_box()
            torch.cuda.synchronize()
            print("@box", drive, rep, file=sys.stderr, flush=True)
"""


def test_one_capture_for_a_new_drive():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("graph captures of explicit boxes", flush=True)
    env = dict(os.environ, AMD_LOG_LEVEL="3")    # the HIP runtime logs its API calls
    r = subprocess.run([sys.executable, "-c", CODE.format(root=ROOT)], env=env, capture_output=True,
                       text=True, timeout=100, errors="replace")
    assert r.returncode == 0, r.stderr[-2000:]
    parts = r.stderr.split("@box")
    if "hipGraphLaunch" not in r.stderr:
        pytest.skip("the HIP runtime logs no API calls")
    made = [p.count("hipGraphInstantiate (") for p in parts[:8]]
    assert made == [1, 1, 0, 0] * 2, made
