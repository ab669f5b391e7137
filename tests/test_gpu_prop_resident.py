"""Chain propagators resident on one CU: the grids at the edges of the rule that
selects them (narrowest, widest, most matrix work in either precision) and the
first ones past it, short and odd contours, junction segments, against the
FP64 oracle; and the field statistics a step leaves to them.

Bars: N steps of two convolutions, each a sum of nx or ny products whose
rounding errors add up at most coherently over the steps: 2 N (nx + ny) eps
relative to the largest density, eps = 2^-53, and in FP32 2 N * 16 * 2^-24 (the
kernel's weight sits on a few sites; its tails add rounding of their own size)."""
import numpy as np
import pytest

from oracle import epdlb_oracle as O
from seeded_inputs import preset

pytestmark = pytest.mark.gpu


def _sim(nx, ny, N, fA, prec, **kw):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1804_02883_amd import Simulation
    p = preset("cfg1", nx=nx, ny=ny, n_contour=N, f_A=fA, precision=prec, **kw)
    return p, Simulation(p)


@pytest.mark.parametrize("nx,ny,N,fA,prec", [
    (32, 16, 2, 0.5, 0), (64, 32, 17, 0.33, 0), (128, 16, 5, 0.71, 0), (64, 16, 3, 0.5, 0), (64, 64, 6, 0.45, 0),
    (32, 16, 5, 0.33, 1), (32, 64, 16, 0.5, 1), (64, 64, 33, 0.3, 1), (128, 32, 9, 0.62, 1), (128, 16, 2, 0.5, 1),
    (128, 64, 6, 0.45, 1), (256, 16, 4, 0.5, 1)])
def test_densities_vs_oracle(nx, ny, N, fA, prec):
    print(f"[resident] {nx}x{ny} N={N} f_A={fA} precision={prec}", flush=True)
    p, sim = _sim(nx, ny, N, fA, prec)
    w = 0.3 * np.random.default_rng(nx + ny + N).standard_normal((3, ny, nx))
    if prec:
        w = w.astype(np.float32).astype(float)
    ref = O.densities(w, p)
    sim.set_fields(w)
    phi, d = sim.densities(), sim.diag()
    sim.close()
    tol = 2 * N * ((nx + ny) * 2.0 ** -53 if prec == 0 else 16 * 2.0 ** -24)
    assert np.max(np.abs(phi - ref["phi"])) < tol * np.abs(ref["phi"]).max()
    for k in ("Q_P", "Q_P_bwd", "Q_S"):
        assert abs(d[k] / ref[k] - 1) < tol, k


@pytest.mark.parametrize("nx,ny,prec", [(32, 32, 0), (64, 64, 1), (128, 32, 1)])
def test_step_equals_its_stages(nx, ny, prec):
    """A step leaves the statistics of the new potentials to the propagators;
    stage by stage they are finished first.  Same potentials, densities and
    scalars, bit for bit (the velocity is not compared: the LB stage alone is
    another kernel than the step's fused one and rounds differently)."""
    from paper_1804_02883_amd import binding as B
    out = []
    for whole in (True, False):
        _, sim = _sim(nx, ny, 9, 0.3, prec, g=1e-4, g_units=1)
        sim.seed(5, 0.05)
        for _ in range(3):
            if whole:
                sim.step(1)
            else:
                for st in (B.EPDLB_STAGE_ADVECT_UPDATE, B.EPDLB_STAGE_DENSITIES, B.EPDLB_STAGE_FORCE, B.EPDLB_STAGE_LB):
                    sim.run_stage(st)
        sim.sync()
        d = sim.diag()
        d.pop("step")
        out.append((sim.get_state(), d))
        sim.close()
    assert out[0][1] == out[1][1]
    for a, b in zip(out[0][0][:2], out[1][0][:2]):
        assert np.array_equal(a, b)
