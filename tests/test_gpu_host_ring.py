"""Host transfers that go round the ring of pinned slots several times, and of
exactly the size from which it is taken.

A slot holds 1 MiB, the ring 16 of them: 4,194,304 FP32 or 2,097,152 FP64 values.
Bars as for smaller transfers: a population travels as f - w in the plane's
precision and comes back as w + that, off by at most the rounding of the two sums
and of the stored deviation; a plane of FP32 values comes back bit for bit."""
import threading

import numpy as np
import pytest

from seeded_inputs import preset

pytestmark = pytest.mark.gpu

W19 = np.array([1 / 3] + [1 / 18] * 6 + [1 / 36] * 12)[:, None, None, None]
# 19 planes: 13,934,752 values in FP32 (3.3 rings) and 7,268,184 in FP64 (3.5), the last chunk ragged
SHAPES = {1: (82, 86, 104), 0: (72, 77, 69)}


def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _round_trip(prec, seed, times=1):
    from paper_1804_02883_amd import Fluid3D
    nz, ny, nx = shape = SHAPES[prec]
    fl = Fluid3D(nx, ny, nz, 0.8, prec)
    ok = True
    for k in range(times):
        f = W19 * (1 + 0.2 * np.random.default_rng(seed + k).uniform(-1, 1, (19,) + shape))
        fl.set_populations(f)
        got = fl.populations()
        tol = 2.0 ** -53 * 2 + (np.abs(f - W19) * 2.0 ** -24 if prec else 0)
        ok = ok and bool(np.all(np.abs(got - f) <= tol))
    fl.close()
    return ok


@pytest.mark.parametrize("prec", [0, 1])
def test_three_times_round(prec):
    _gpu()
    per = 2 ** 20 // (4 if prec else 8)
    n = 19 * int(np.prod(SHAPES[prec]))
    assert n > 3 * 16 * per and n % per
    assert _round_trip(prec, 3 + prec, 2)


def test_two_threads_round():
    _gpu()
    ok = {}

    def work(k):
        ok[k] = _round_trip(k, 20 + k, 2)

    th = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    assert ok == {0: True, 1: True}


@pytest.mark.parametrize("prec", [0, 1])
def test_one_plane_of_the_smallest_size(prec):
    """1024 x 1024 sites: one plane is 2^20 values, two of the force 2^21."""
    _gpu()
    from paper_1804_02883_amd import EPDLB_AUX_FORCE, EPDLB_AUX_STILDE, Simulation
    sim = Simulation(preset("cfg1", nx=1024, ny=1024, precision=prec))
    rng = np.random.default_rng(prec)
    for which, planes in ((EPDLB_AUX_STILDE, 1), (EPDLB_AUX_FORCE, 2)):
        v = rng.standard_normal((planes, 1024, 1024)).astype(np.float32).astype(float)
        sim.write_aux(which, v if planes > 1 else v[0])
        assert np.array_equal(np.asarray(sim.aux(which)).reshape(v.shape), v)
    sim.close()
