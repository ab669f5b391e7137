"""Large host transfers (pinned slots, several threads) through the public
classes: sizes around the slot edges, values that survive the round trip, a
refused input, contexts in two threads at once.

Bars: a population travels as f - w in the plane's precision and comes back as
w + that, so it is off by at most the rounding of the two sums and of the
stored deviation."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

W19 = np.array([1 / 3] + [1 / 18] * 6 + [1 / 36] * 12)[:, None, None, None]


def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _round_trip(shape, prec, seed):
    from paper_1804_02883_amd import Fluid3D
    nz, ny, nx = shape
    f = W19 * (1 + 0.2 * np.random.default_rng(seed).uniform(-1, 1, (19,) + shape))
    fl = Fluid3D(nx, ny, nz, 0.8, prec)
    fl.set_populations(f)
    out = [fl.populations() for _ in range(2)]
    fl.close()
    tol = 2.0 ** -53 * 2 + (np.abs(f - W19) * 2.0 ** -24 if prec else 0)
    return all(bool(np.all(np.abs(o - f) <= tol)) for o in out)


# 19 planes of: just under 2^20 values, 2^20 and its neighbours, one slot more,
# many slots with a ragged last one
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("shape", [(1, 13, 4245), (1, 1, 4096), (4, 13, 1061 + 1), (5, 83, 133), (31, 37, 101)])
def test_round_trip(shape, prec):
    _gpu()
    if shape[2] > 4096:
        shape = (shape[0] * 5, shape[1], shape[2] // 5)
    assert _round_trip(shape, prec, sum(shape))


def test_two_threads():
    _gpu()
    ok = {}

    def work(k):
        ok[k] = all(_round_trip((20, 60, 70 + k), k % 2, 10 * k + i) for i in range(3))

    th = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    assert ok == {0: True, 1: True}


def test_refused_potentials_leave_the_context():
    _gpu()
    from paper_1804_02883_amd import Densities3D, EpdlbError
    d = Densities3D(128, 64, 64, 4, 0.3, 0.15)
    w = 0.1 * np.random.default_rng(1).standard_normal((3, 64, 64, 128))
    first = d.densities(w)
    bad = w.copy()
    bad[2, -1, -1, -1] = np.inf
    with pytest.raises(EpdlbError):
        d.densities(bad)
    d.time(1)  # evaluates the accepted potentials
    again = d.densities(w)
    assert np.array_equal(first[0], again[0]) and first[1:] == again[1:]
    d.close()
