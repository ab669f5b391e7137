"""Copies a context's creation makes, counted by torch's profiler: the constant
tables of a replica, and those of the 3D densities, go up in one piece each.  A
replica's scalars and guard words are two more."""
import pytest

from seeded_inputs import preset

pytestmark = pytest.mark.gpu


def _copies(make):
    """Host-to-device copies while make() runs, and its result."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from torch.profiler import ProfilerActivity, profile
    torch.zeros(4).cuda()
    with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as prof:
        marker = torch.zeros(4).cuda()
        torch.cuda.synchronize()
        made = make()
        torch.cuda.synchronize()
    del marker
    n = sum(1 for e in prof.events() if "memcpy" in e.name.lower() and "htod" in e.name.lower().replace(" ", ""))
    assert n >= 1, sorted({e.name for e in prof.events()})  # the marker's own
    return n - 1, made


@pytest.mark.parametrize("nx,ny,prec", [(32, 32, 0), (64, 64, 1), (128, 128, 1)])
def test_replica_tables_are_one_copy(nx, ny, prec):
    from paper_1804_02883_amd import Batch
    n, b = _copies(lambda: Batch([preset("cfg1", nx=nx, ny=ny, precision=prec)] * 24))
    b.close()
    print("copies", n)
    assert 24 <= n <= 3 * 24


def test_densities3d_tables_are_one_copy():
    from paper_1804_02883_amd import Densities3D
    n, d = _copies(lambda: Densities3D(64, 32, 16, 6, 0.3, 0.15))
    d.close()
    print("copies", n)
    assert n == 1
