"""Host memory of a state's upload.  set_state converts the populations on their
way to the device, through buffers of bounded size: the process's peak must not
grow by another array of them.  One process of its own, whose peak is that of the
inputs.  The transfers' pinned ring is 16 MiB and a kept buffer at most 8; an
array of 9 x 1024 x 1024 deviations would be 72 (FP64) and a converted one 36."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

CODE = """
import resource, sys
import numpy as np
from paper_1804_02883_amd import Simulation
from seeded_inputs import preset
peak = lambda: resource.getrusage(resource.RUSAGE_SELF).ru_maxrss / 1024
n, prec = 1024, int(sys.argv[1])
small = Simulation(preset("cfg1", precision=prec))
small.set_state(np.zeros((3, 32, 32)), np.full((3, 32, 32), 1 / 3), np.full((9, 32, 32), 1 / 9), np.zeros((2, 32, 32)))
small.step(1), small.sync()
sim = Simulation(preset("cfg1", nx=n, ny=n, precision=prec))
w, phi, f, u = np.full((3, n, n), 0.1), np.full((3, n, n), 1 / 3), np.full((9, n, n), 1 / 9), np.full((2, n, n), 0.01)
before = peak()
sim.set_state(w, phi, f, u)
print("grew", peak() - before)
got = sim.get_state()
assert np.all(np.abs(got[2] - f) <= 2.0 ** (-53 if prec == 0 else -24)) and np.all(np.abs(got[3] - u) <= 2.0 ** -30)
"""


@pytest.mark.parametrize("prec", [1, 0])
def test_set_state_needs_no_copy_of_the_populations(prec):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", CODE, str(prec)], capture_output=True, text=True, timeout=100, cwd=root)
    print(r.stdout, r.stderr[-500:])
    assert r.returncode == 0, r.stderr
    assert float(r.stdout.split("grew")[1]) < 32
