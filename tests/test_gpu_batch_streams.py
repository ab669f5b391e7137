"""A batch's groups run on streams of their own: more groups than hardware queues,
calls of odd and even step counts back to back, and one replica replaced between
calls without a synchronisation, each replica bit for bit as a run of its own."""
import numpy as np
import pytest

from seeded_inputs.presets import base_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grids", [[(32, 32)], [(32, 32), (32, 64), (64, 32), (64, 64), (128, 32), (256, 32), (32, 128)]])
@pytest.mark.parametrize("prec", [0, 1])
def test_groups_in_flight_equal_single_runs(grids, prec):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1804_02883_amd import Batch, Simulation
    print(f"[batch streams] {len(grids)} grids precision={prec}", flush=True)
    params = [base_params(nx, ny, 16, f, 0.1, "L", 1e-5 * (i + 1), precision=prec)
              for i, (nx, ny) in enumerate(grids) for f in (0.3, 0.5)]
    rng = np.random.default_rng(len(grids))
    fields = [1e-3 * rng.standard_normal((3, p["ny"], p["nx"])) for p in params]
    b = Batch(params)
    b.seed(list(range(len(params))), 1e-3)
    for r, w in enumerate(fields):
        b.set_fields(r, w)
    for n in (1, 2, 0, 3, 1):
        b.step(n)
    b.set_fields(len(params) - 1, fields[-1])
    b.step(5)
    for r, (p, w) in enumerate(zip(params, fields)):
        sim = Simulation(p)
        sim.set_fields(w)
        sim.step(7)
        if r == len(params) - 1:
            sim.set_fields(w)
        sim.step(5)
        assert np.array_equal(b.densities(r), sim.densities()), r
        assert np.array_equal(b.fields(r), sim.fields()), r
        assert b.diag(r)["Q_P"] == sim.diag()["Q_P"]
        sim.close()
    b.close()
