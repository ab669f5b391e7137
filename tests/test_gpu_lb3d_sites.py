"""The three-dimensional fluid's one-lane-per-site launch at the boxes where it
can go wrong: one site, one short of and one past a wave and a block, odd sides,
the longest side along each axis, both sides of the block rule (2^18 sites),
with both collisions, against the FP64 oracle.

Bars, as for the other boxes: FP64 to 1e-13 (rounding order only); FP32 storage
keeps the deviations f_i - w_i, of at most about 0.05 here, to a few ulps per
step: 5e-7 absolute."""
import numpy as np
import pytest

from oracle import lb3d_oracle as L
from test_gpu_lb3d import _fluid, _state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,tol", [(0, 1e-13), (1, 5e-7)])
@pytest.mark.parametrize("mrt", [0, 1])
@pytest.mark.parametrize("nx,ny,nz", [(1, 1, 1), (63, 1, 1), (13, 5, 1), (4, 8, 2), (3, 5, 17), (4096, 1, 2), (1, 4096, 2),
                                      (2, 1, 4096), (64, 64, 64), (67, 63, 63)])
def test_site_blocks_vs_oracle(nx, ny, nz, mrt, prec, tol):
    print(f"[lb3 sites] {nx}x{ny}x{nz} mrt={mrt} precision={prec}", flush=True)
    f, F = _state((nz, ny, nx), nx + 3 * ny + 7 * nz)
    fl = _fluid(nx, ny, nz, 0.8, prec)
    factors = (-0.25, 0.1, 0.2)
    if mrt:
        fl.set_collision(1, *factors)
    fl.set_populations(f)
    fl.set_force(F)
    if prec == 1:
        w = L.W19[:, None, None, None]
        f = w + (f - w).astype(np.float32).astype(np.float64)
        F = F.astype(np.float32).astype(np.float64)
    fl.step(2)
    for _ in range(2):
        f, rho, u = L.step_mrt(f, F, *factors) if mrt else L.step(f, F, 0.8)
    grho, gu = fl.velocity()
    assert np.max(np.abs(fl.populations() - f)) < tol
    assert np.max(np.abs(grho - rho)) < tol and np.max(np.abs(gu - u)) < tol
    fl.close()
