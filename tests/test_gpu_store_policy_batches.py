"""The patch kernel's store policies (test_gpu_store_policy) on batches with an open axis, curved
walls and ragged widths, with and without wetting variants: the march's results bit for bit."""
import numpy as np
import pytest

from paper_1707_00198_amd import workloads as W

pytestmark = pytest.mark.gpu

NODE_BYTES = {"f64": 192, "f32": 96, "f16": 60, "c16": 60}  # both copies of f, c and v


@pytest.mark.parametrize("variants", [False, True], ids=["plain", "variants"])
@pytest.mark.parametrize("storage,mib,chunk", [("f64", 180, 8), ("f64", 230, 8), ("f64", 320, 8), ("f32", 180, 8), ("f32", 180, 24),
                                               ("f32", 230, 8), ("f32", 230, 24), ("f16", 230, 24), ("c16", 230, 24)])
def test_store_policies_equal_the_march(storage, mib, chunk, variants):
    from paper_1707_00198_amd.lbm import Lattice
    cases = [W.cylinder_droplet(n=397, rc=80.0, rd=60.0, theta_deg=60.0, ccx=198.0, ccy=140.0, dcx_offset=0.37),
             W.droplet_box(theta_deg=150.0, M=10.0, nx=171, ny=107, radius=40.0, xc_offset=0.37)]
    # the rest of the state in one open channel
    nodes = mib * 2**20 // NODE_BYTES[storage] - sum(s.solid.size for s in cases)
    cases.append(W.fingering_channel(nx=2011, h=nodes // 2011, x_interface=700.0, M=3.0, theta_deg=120.0, ca=0.2, sigma=0.05))
    if variants:
        for s, f in zip(cases, (W.WET_SCHEME_B | W.WET_SURFACE_ENERGY, W.WET_SURFACE_ENERGY, W.WET_SCHEME_B)):
            s.wetting = f
    ref, lat = Lattice(cases, storage=storage), Lattice(cases, storage=storage)
    ref.set_tile(32, 4, 1, 1)
    lat.set_tile(chunk, 8, 1, 1)
    for steps in (1, 4):
        print(f"{storage} {mib} MiB chunk {chunk} variants={variants}: {steps} steps", flush=True)
        ref.step(steps), lat.step(steps)
        for d in range(len(cases)):
            assert np.array_equal(ref.pops(d), lat.pops(d))
            for a, b in zip(ref.velocity(d), lat.velocity(d)):
                assert np.array_equal(a, b, equal_nan=True)
