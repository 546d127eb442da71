"""The builds on blocks of 8 wavefronts, each at a height that pins its kernel: items of 16 rows are
marched through, items of 8 rows and, with FP32 arithmetic, of 24 rows are held whole (a height of 0
leaves the choice to the batch, which for the small one here is 8 rows).  Same batches, oracle and
tolerances as test_gpu_instantiations."""
import pytest

import test_gpu_instantiations as T

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variants", [False, True], ids=["plain", "variants"])
@pytest.mark.parametrize("chunk", [16, 8, 24])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16", "c16"])
def test_build_against_oracle(monkeypatch, storage, chunk, variants):
    from paper_1707_00198_amd.lbm import Lattice

    def lattice(setups, st, waves, cols, npl=1):
        lat = Lattice(setups, storage=st)
        lat.set_tile(chunk, waves, cols, npl)
        t = lat.tile
        assert (t["chunk_rows"], t["waves"], t["cols"], t["cols_per_lane"]) == (chunk, 8, 1, 1)
        return lat

    monkeypatch.setattr(T, "_lattice", lattice)
    if storage == "f64":
        T.test_fp64_build_against_oracle(8, 1, variants)
    else:
        T.test_fp32_arithmetic_build_one_step_from_gpu_state(storage, 8, 1, 1, variants)
