"""Lattices near the library's limits of 2^31 - 1 nodes, one at a time on the GPU."""
import pytest

from paper_2410_13165_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(autouse=True)
def _memory():
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 240e9:
        pytest.skip("needs 240 GB of free device memory")
    yield
    torch.cuda.empty_cache()


def test_wall_data_of_a_long_lattice():
    """Walls of x_1 along 8.4 million rows: 64 steps of their data are more than 2^30
    values.  Passes of several steps give the phi of single steps, bit for bit."""
    from paper_2410_13165_amd import Lattice
    dims = (171, 8400000)
    spec = inputs.random_cosines(2, [0.05, -0.1], 0.7, seed=85, kmax=1.0)
    out = []
    for spp in (2, 1):
        with Lattice(2, dims, 0.5, dx=1 / 170, u=spec["u"], R=spec["R"],
                     bc=["fullway", "periodic"], precision="fp32", field=spec,
                     steps_per_pass=spp) as lat:
            print(f"[large] {dims} steps_per_pass={spp}", flush=True)
            lat.step(65)
            out.append(lat.phi().cpu())
        torch.cuda.empty_cache()
    assert torch.equal(out[0], out[1])
    assert bool(torch.isfinite(out[0]).all())
