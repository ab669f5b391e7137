"""A surrogate context's propagator passes take the plain convolution at every
launch shape.  Of a line of equal values the plain convolution is the identity in
every bit: the butterflies add equal values and subtract them, the multiplier at
k = 0 is 1/L, a power of two.  (With the difference from 1 in the transforms a
value below 1/2 loses its last bits.)  So where the potentials vary along x only
the column passes change nothing, whatever their R and nf, and the densities agree
bit for bit over all their shapes; along y only, over the row passes' shapes.

The potentials keep q within exp(-3.6) to exp(3.6): the FP64 sums of Q_P are then
exact, whatever their order."""
import numpy as np
import pytest

from seeded_inputs import preset

pytestmark = pytest.mark.gpu

NX, NY = 128, 64
COLS = [(8, 4), (8, 8), (8, 16), (2, 4), (4, 4), (4, 16), (16, 4), (16, 16)]
ROWS = [(8, 4), (8, 3), (2, 1), (2, 4), (4, 1), (4, 5), (16, 2), (16, 8)]


def _sim(prec=1):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1804_02883_amd import Simulation
    return Simulation(preset("cfg1", nx=NX, ny=NY, n_contour=6, f_A=0.4, precision=prec, density_mode=1))


@pytest.mark.parametrize("family,shapes", [("prop_col", COLS), ("prop_row", ROWS)])
def test_lines_of_equal_values_pass_unchanged(family, shapes):
    sim = _sim()
    n = NX if family == "prop_col" else NY
    line = 0.6 * np.random.default_rng(n).uniform(-1, 1, (3, n))
    w = line[:, None, :] if family == "prop_col" else line[:, :, None]
    w = np.broadcast_to(w, (3, NY, NX)).astype(np.float32).astype(float)
    ref = None
    for R, nf in shapes:
        print(f"[surrogate shapes] {family} R={R} nf={nf}", flush=True)
        sim.set_shape(family, R, nf)
        sim.set_fields(w)
        out = sim.densities(), sim.diag()["Q_P"]
        ref = ref or out
        assert np.array_equal(out[0], ref[0]) and out[1] == ref[1], (R, nf)
    sim.close()


def test_fp64_tune_lines_are_their_own(tmp_path):
    from paper_1804_02883_amd import Simulation
    cache = tmp_path / "tune.txt"
    families = ("prop_row", "prop_col", "force_row", "force_col")
    lines = "".join(f"gfx950 {NX} {NY} 6 0 x1 {f} 4 4 1.000\n" for f in families)
    cache.write_text(lines)
    sim = _sim(0)
    sim.autotune(2, str(cache))
    assert all(R == 8 for R, _ in sim.shapes().values())
    sim.close()
    sim = Simulation(preset("cfg1", nx=NX, ny=NY, n_contour=6, f_A=0.4, precision=0))
    sim.autotune(2, str(cache))
    assert sim.shapes() == {f: (4, 4) for f in families}
    sim.close()
    assert cache.read_text().startswith(lines) and cache.read_text().count(" x1s ") == 4


def test_fp64_stays_at_eight():
    from paper_1804_02883_amd import EpdlbError
    sim = _sim(0)
    for family in ("prop_row", "prop_col", "force_row", "force_col"):
        with pytest.raises(EpdlbError):
            sim.set_shape(family, 4, 4)
    sim.autotune(2)
    assert all(R == 8 for R, _ in sim.shapes().values())
    sim.close()
