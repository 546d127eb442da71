"""The reductions and the crossing search against plain sums over the fields read back, at the
sizes where their blocks and windows end: fewer nodes than one block, one block, one node more,
several domains of different sizes in a batch; rows one node wide, and rows around the crossing
kernel's windows of 64, 256 and 1024 nodes with the crossing in the first, the last and the
overlapping pair of a window, and none at all.  Sums of n terms of order one in FP64 differ by at
most n 2^-52 relative to the sum."""
import numpy as np
import pytest

from paper_1707_00198_amd import workloads as W

pytestmark = pytest.mark.gpu


def _box(nx, ny, cut):
    """Periodic box, red up to column `cut`, blue beyond."""
    solid = np.zeros((ny, nx), np.uint8)
    red = np.broadcast_to(np.arange(nx)[None, :] < cut, solid.shape)
    base = W.free_droplet(n=8, radius=2.0)
    return W.Setup(f"{nx}x{ny}", solid, np.where(red, 1.0, 0.0), np.where(red, 0.0, 1.0), dict(base.params))


@pytest.mark.parametrize("storage", ["f64", "c16"])
def test_masses_velocity_and_regions_match_the_fields(storage):
    from paper_1707_00198_amd.lbm import Lattice
    cases = [_box(*c) for c in ((1, 3, 1), (15, 17, 6), (16, 16, 5), (257, 1, 90), (300, 280, 100))]
    lat = Lattice(cases, storage=storage).step(3)
    before = [np.stack(lat.velocity(d)) for d in range(len(cases))]
    lat.velocity_stats(snapshot=True)
    lat.step(4)
    for turn in range(3):  # the snapshot and the current velocity change places
        mass, stats = lat.mass(), lat.velocity_stats(snapshot=True)
        after = [np.stack(lat.velocity(d)) for d in range(len(cases))]
        for d, s in enumerate(cases):
            n = s.solid.size
            rho = np.stack(lat.densities(d))
            assert np.abs(mass[d] - rho.sum(axis=(1, 2))).max() <= 4 * n * 2.0 ** -52 * n + (0.0 if storage == "f64" else 1e-6 * n)
            assert stats[d, 0] == np.sqrt((after[d] ** 2).sum(axis=0)).max()
            assert stats[d, 1] == np.abs(after[d] - before[d]).max()
            region = (np.arange(n).reshape(s.solid.shape) % 3 == 0).astype(np.uint8)
            r = lat.region_mass(d, region)
            want = [(rho[k] * (region == v)).sum() for k in (0, 1) for v in (1, 0)]
            assert np.abs(r - want).max() <= 4 * n * 2.0 ** -52 * n + (0.0 if storage == "f64" else 1e-6 * n)
        before = after
        lat.step(2)


@pytest.mark.parametrize("nx,cuts", [(1, (1,)), (2, (1,)), (63, (1, 62)), (64, (63,)), (65, (1, 64)), (256, (255,)), (257, (254, 255, 256)),
                                     (1024, (1023,)), (1025, (1022, 1023, 1024)), (2100, (1, 1022, 1023, 1024, 2045, 2046, 2047, 2099, 2100, 0))])
def test_crossing_windows(nx, cuts):
    from paper_1707_00198_amd.lbm import Lattice
    cases = [_box(nx, 2, c) for c in cuts]
    lat = Lattice(cases, storage="f64")
    for d, c in enumerate(cuts):
        got = [lat.crossings(d, [0, 1]), lat.crossings_noalloc(d, [1, 0])]
        want = c - 0.5 if 0 < c < nx else np.nan  # the sharp initial step, halfway between the nodes
        assert np.array_equal(np.concatenate(got), np.full(4, want), equal_nan=True), (nx, c, got)
