"""Propagator passes over their launch shapes: values per lane, transforms per
block that do not divide the number of rows or columns, one and several waves
per transform, contours that end along x and along y, a junction segment first,
inside and last, against the FP64 oracle.

Bars: 2N convolutions, each a pair of transforms of at most log2(nx ny) radix-2
levels whose rounding errors add up at most coherently, two more for the
twiddles' products: 2 N * 4 log2(nx ny) * eps relative to the largest density,
eps = 2^-53 or 2^-24."""
import math

import numpy as np
import pytest

from oracle import epdlb_oracle as O
from seeded_inputs import preset

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,N,fA,prec,row,col", [
    (256, 128, 5, 0.33, 1, (4, 3), (4, 4)), (256, 128, 4, 0.05, 1, (2, 1), (2, 8)), (128, 256, 4, 0.97, 1, (16, 5), (16, 4)),
    (512, 64, 3, 0.5, 1, (8, 2), (8, 8)), (1024, 16, 4, 0.4, 1, (4, 1), (4, 16)), (32, 1024, 3, 0.4, 1, (4, 7), (8, 4)),
    (128, 128, 4, 0.33, 0, (4, 2), (4, 4)), (256, 512, 3, 0.6, 0, (8, 3), (8, 4)), (64, 256, 5, 0.1, 0, (4, 5), (4, 4))])
def test_densities_over_shapes(nx, ny, N, fA, prec, row, col):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1804_02883_amd import Simulation
    print(f"[shapes] {nx}x{ny} N={N} f_A={fA} precision={prec} row={row} col={col}", flush=True)
    p = preset("cfg1", nx=nx, ny=ny, n_contour=N, f_A=fA, precision=prec)
    w = 0.3 * np.random.default_rng(nx + ny + N).standard_normal((3, ny, nx))
    if prec:
        w = w.astype(np.float32).astype(float)
    ref = O.densities(w, p)
    tol = 2 * N * 4 * math.log2(nx * ny) * (2.0 ** -24 if prec else 2.0 ** -53)
    sim = Simulation(p)
    for shapes in (None, (row, col)):  # the default shapes, then these
        if shapes:
            sim.set_shape("prop_row", *row)
            sim.set_shape("prop_col", *col)
        sim.set_fields(w)
        phi, d = sim.densities(), sim.diag()
        assert np.max(np.abs(phi - ref["phi"])) < tol * np.abs(ref["phi"]).max(), shapes
        assert abs(d["Q_P"] / ref["Q_P"] - 1) < tol and abs(d["Q_P_bwd"] / ref["Q_P_bwd"] - 1) < tol, shapes
    sim.close()
