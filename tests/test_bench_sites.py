"""The bench's bytes per kernel family count the sites that its launches cover: the
propagator passes' leave out the grids whose chains run resident in one launch."""
import pytest

import bench
from seeded_inputs import replica_manifest



# the edges of the rule, as the library states it: cycles up to 5,120
@pytest.mark.parametrize("nx,ny,prec,expect", [
    (32, 16, 0, True), (32, 32, 0, True), (64, 32, 0, True), (32, 64, 0, False), (64, 64, 0, False), (128, 16, 0, True),
    (64, 64, 1, True), (128, 32, 1, True), (32, 64, 1, True), (128, 64, 1, False), (64, 128, 1, False), (256, 16, 1, False)])
def test_rule(nx, ny, prec, expect):
    p = dict(nx=nx, ny=ny, precision=prec)
    assert bench.resident(p) is expect
    assert bench.resident(dict(p, density_mode=1)) is False


def test_sites_of_the_manifest():
    plist = [m["params"] for m in replica_manifest()]
    every = sum(p["nx"] * p["ny"] for p in plist)
    small = sum(p["nx"] * p["ny"] for p in plist if (p["nx"], p["ny"]) == (64, 64))
    assert 0 < small < every
    for k in ("prop_row", "prop_col"):
        assert bench.family_sites(k, plist) == every - small
    for k in ("density", "advect_update", "force_inv_lb"):
        assert bench.family_sites(k, plist) == every
