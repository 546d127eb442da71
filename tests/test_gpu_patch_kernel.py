"""The patch kernel (work items of 8 and 24 rows on blocks of 8) gives the march's results bit for
bit: widths around its 56-column strips and its window, heights around its 8 and 24 output rows,
domains narrower than the stencils, open and periodic x, curved walls, every wetting flag.  The
snapshot state's first step, later steps, the velocity of a diagnostic launch, the contact-line
list and the masses are compared.  (The march itself is held to the oracle by
test_gpu_instantiations and test_gpu_parity.)"""
import numpy as np
import pytest

from paper_1707_00198_amd import workloads as W

pytestmark = pytest.mark.gpu

FLAGS = [0, W.WET_SCHEME_B, W.WET_SURFACE_ENERGY, W.WET_SCHEME_B | W.WET_SURFACE_ENERGY]


def _cases(variants, many):
    out = []
    for nx, ny in ((1, 9), (3, 25), (55, 7), (56, 8), (57, 16), (64, 23), (65, 24), (112, 26), (113, 48), (121, 49)):
        s = W.droplet_flat(nx=nx, h=max(ny - 2, 1), radius=min(nx, ny) / 3.0 + 1.0, theta_deg=70.0,
                           xc=nx / 3.0 + 0.37, name=f"drop{nx}x{ny}")
        out.append(s)
    for nx, h in ((2, 6), (55, 5), (60, 22), (61, 23), (113, 30)):
        out.append(W.fingering_channel(nx=nx, h=h, x_interface=nx / 3.0, M=3.0, theta_deg=120.0, ca=0.2,
                                       sigma=0.05, name=f"open{nx}x{h + 2}"))
    out.append(W.cylinder_droplet(n=96, rc=20.0, rd=18.0, theta_deg=120.0, ccx=48.0, ccy=30.0, dcx_offset=0.37))
    out.append(W.droplet_box(theta_deg=150.0, M=10.0, nx=70, ny=50, radius=16.0, xc_offset=0.37))
    if many:  # over 256 work items of 8 rows: the 64-register build with FP64 arithmetic
        out.append(W.cylinder_droplet(n=452, rc=80.0, rd=60.0, theta_deg=60.0, ccx=220.0, ccy=150.0, dcx_offset=0.37))
    if variants:
        for k, s in enumerate(out):
            s.wetting = FLAGS[k % 4]
    return out


def _observe(lat, n):
    out = [lat.pops(d) for d in range(n)]
    out += [np.stack(lat.velocity(d)) for d in range(n)]
    out += [lat.contact_line(d) for d in range(n)]
    return out + [lat.mass(), lat.velocity_stats()]


@pytest.mark.parametrize("variants", [False, True], ids=["plain", "variants"])
@pytest.mark.parametrize("storage,chunk,many", [("f64", 8, False), ("f64", 8, True), ("f32", 8, False), ("f32", 24, False),
                                                ("f16", 8, False), ("f16", 24, True), ("c16", 8, True), ("c16", 24, False)])
def test_patch_kernel_equals_the_march(storage, chunk, many, variants):
    from paper_1707_00198_amd.lbm import Lattice
    cases = _cases(variants, many)
    ref, lat = Lattice(cases, storage=storage), Lattice(cases, storage=storage)
    ref.set_tile(16, 4, 1, 1)
    lat.set_tile(chunk, 8, 1, 1)
    assert (lat.tile["items"] > 256) == (many and chunk == 8)
    for steps in (1, 1, 10):
        print(f"{storage} chunk {chunk} many={many} variants={variants}: {steps} steps", flush=True)
        a, b = _observe(ref.step(steps), len(cases)), _observe(lat.step(steps), len(cases))
        for k, (x, y) in enumerate(zip(a, b)):
            assert np.array_equal(x, y, equal_nan=True), (steps, k)
