"""The passes of the three-dimensional propagators at the grids where they can go
wrong: no axis, one axis (each place), two axes, the shortest and longest
lines, fewer lines than a block takes, an odd and an even number of contour
steps (the last pass then runs along different axes), against the FP64 oracle.

Bars: an evaluation is 2N convolutions per axis, each a pair of transforms of
log2 n radix-2 levels whose rounding errors add up at most coherently:
2 N * 2 log2(n) * eps relative to the largest density, eps = 2^-53 or 2^-24."""
import math

import numpy as np
import pytest

from oracle import epd3d_oracle as E3
from seeded_inputs import preset

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("shape,N,fA", [((1, 1, 1), 5, 0.3), ((1, 1, 2), 4, 0.5), ((1, 64, 1), 5, 0.45),
                                        ((512, 1, 1), 4, 0.3), ((1, 2, 512), 5, 0.7), ((512, 2, 1), 4, 0.3),
                                        ((2, 512, 4), 3, 0.5), ((16, 1, 256), 4, 0.45), ((4, 128, 32), 5, 0.3),
                                        ((64, 4, 16), 4, 0.62)])
def test_passes_vs_oracle(shape, N, fA, prec):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1804_02883_amd import Densities3D
    print(f"[epd3 passes] {shape} N={N} f_A={fA} precision={prec}", flush=True)
    nz, ny, nx = shape
    w = 0.3 * np.random.default_rng(N + sum(shape)).standard_normal((3,) + shape)
    ref = E3.densities3(w, preset("cfg1", n_contour=N, f_A=fA, phi_P=0.12))
    d = Densities3D(nx, ny, nz, N, fA, 0.12, 1.0, 1.0 / 3.0, prec)
    tol = 2 * N * 2 * max(1.0, math.log2(w[0].size)) * (2.0 ** -24 if prec else 2.0 ** -53)
    for _ in range(2):  # the second evaluation finds the planes of the first
        phi, QP, QS = d.densities(w)
        err = np.max(np.abs(phi - ref["phi"])) / np.max(np.abs(ref["phi"]))
        assert err < tol, (err, tol)
        assert abs(QP / ref["Q_P"] - 1) < tol and abs(QS / ref["Q_S"] - 1) < tol
    d.close()


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("shape,N,fA", [((64, 128, 128), 3, 0.5), ((4, 512, 512), 2, 0.3), ((512, 512, 2), 2, 0.5),
                                        ((32, 128, 128), 2, 0.3)])
def test_wide_and_narrow_blocks_vs_oracle(shape, N, fA, prec):
    """Grids on both sides of the block rule (two wide blocks per CU), each axis on its own side."""
    test_passes_vs_oracle(shape, N, fA, prec)
