"""The patch kernel's store policies, chosen by the size of the state (both copies: up to 192 MiB,
above, and with FP64 from 300 MiB), give the march's results bit for bit."""
import numpy as np
import pytest

from paper_1707_00198_amd import workloads as W

pytestmark = pytest.mark.gpu

NODE_BYTES = {"f64": 192, "f32": 96, "f16": 60, "c16": 60}  # both copies of f, c and v


@pytest.mark.parametrize("storage,mib,chunk", [("f64", 180, 8), ("f64", 230, 8), ("f64", 320, 8), ("f32", 180, 24),
                                               ("f32", 230, 8), ("f16", 180, 24), ("f16", 230, 24), ("c16", 230, 8)])
def test_store_policies_equal_the_march(storage, mib, chunk):
    from paper_1707_00198_amd.lbm import Lattice
    nx = 1009
    h = mib * 2**20 // (NODE_BYTES[storage] * nx)
    cases = [W.droplet_flat(nx=nx, h=h, radius=90.0, theta_deg=70.0, xc=400.37)]
    ref, lat = Lattice(cases, storage=storage), Lattice(cases, storage=storage)
    ref.set_tile(32, 4, 1, 1)
    lat.set_tile(chunk, 8, 1, 1)
    for steps in (1, 4):
        print(f"{storage} {mib} MiB chunk {chunk}: {steps} steps", flush=True)
        ref.step(steps), lat.step(steps)
        assert np.array_equal(ref.pops(0), lat.pops(0))
        for a, b in zip(ref.velocity(0), lat.velocity(0)):
            assert np.array_equal(a, b, equal_nan=True)
