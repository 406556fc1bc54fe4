"""lbm_profile_end's wall time of d = 2 lattices whose passes take several steps: the
launch that forms their wall data counts there.  One launch is profiled, in two calls
of 16 steps: the first pass of a call follows the launch that forms its data, 16 modes
on 240 000 wall nodes, which takes far longer than the gap between two events (a few
microseconds) that a pass without it shows."""
import pytest

from paper_2410_13165_amd import inputs
from tests.pairs import gpu_lattice

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32_split"])
@pytest.mark.parametrize("bc", ["fullway", "halfway"])
def test_wall_data_count_as_wall_time(bc, precision):
    dims = (120000, 24)
    spec = inputs.random_cosines(2, [0.05, -0.1], 0.7, seed=86, kmax=1.0, n_modes=16)
    lat = gpu_lattice(2, dims, 1.0 / 119999, spec, bc=[bc] * 2, precision=precision)
    try:
        lat.step(16)
        for _ in range(2):
            lat.profile_begin(1)
            lat.step(16)
            prof = lat.profile_end()
            print(prof, flush=True)
            assert prof["launches"] == 1 and prof["steps"] > 1
            assert prof["bulk_ms"] > 0.0
            assert prof["wall_ms"] > 0.05
    finally:
        lat.close()
