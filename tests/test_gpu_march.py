"""Passes of several steps of d = 2 lattices: bitwise the states of single steps.

The single-step kernels are the reference (they are held to the oracle
elsewhere), so no tolerance enters.  Sizes sit at the edges of the passes' tiles:
output widths of 48 (8 steps) and 56 (2 and 4 steps) columns, one row, one
column, row chunks that end unevenly; step counts take every pass length and the
single-step remainder."""
import pytest

from paper_2410_13165_amd import inputs
from tests.pairs import gpu_lattice
from tests.test_zz_no_alloc import _node_state

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32_split"])
@pytest.mark.parametrize("dims,bc,wall_data", [
    ((1, 1), ["periodic"] * 2, "jets"),
    ((48, 7), ["periodic"] * 2, "jets"),
    ((57, 130), ["periodic"] * 2, "jets"),
    ((97, 300), ["periodic"] * 2, "jets"),
    ((2, 2), ["halfway"] * 2, "jets"),
    ((56, 33), ["fullway"] * 2, "jets"),
    ((113, 64), ["halfway"] * 2, "tangential"),
    ((64, 9), ["halfway", "periodic"], "jets"),
    ((65, 40), ["periodic", "halfway"], "jets"),
])
def test_march_passes_equal_single_steps_bitwise(dims, bc, wall_data, precision):
    from paper_2410_13165_amd import Lattice
    spec = inputs.random_cosines(2, [0.1, -0.15], 0.7, seed=73, kmax=1.0)
    dx = 1.0 / max(dims[0] - 1, 1)
    a = gpu_lattice(2, dims, dx, spec, bc=bc, precision=precision, wall_data=wall_data)
    b = Lattice(2, dims, 0.5, dx=dx, u=spec["u"], R=spec["R"], bc=bc, precision=precision,
                field=spec, wall_data=wall_data, steps_per_pass=1)
    try:
        print(f"[march] dims={dims} bc={bc} {wall_data} {precision}", flush=True)
        for n in (8, 15, 70):  # 8; 8 + 4 + 2 + 1; more steps than one wall-data launch holds
            a.step(n)
            b.step(n)
            assert torch.equal(_node_state(a), _node_state(b)), n
    finally:
        a.close()
        b.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32_split"])
def test_march_passes_stop_at_checkpoints(precision):
    """A tape with checkpoints every 5 steps: the passes end there, and the gradient
    is that of a tape recorded by single steps, bit for bit."""
    from paper_2410_13165_amd import Lattice
    out = []
    for spp in (2, 1):
        lat = Lattice(2, (61, 50), 0.7, dx=1 / 61, u=[0.1, -0.2], precision=precision,
                      steps_per_pass=spp)
        try:
            g = torch.Generator(device="cuda").manual_seed(11)
            lat.set_initial(torch.randn(50, 61, generator=g, dtype=torch.float64, device="cuda"))
            lat.step(3)
            lat.set_initial(torch.randn(50, 61, generator=g, dtype=torch.float64, device="cuda"))
            lat.tape_begin(5)
            lat.step(9)
            lat.step(8)
            phi = lat.phi()
            out.append((phi, lat.tape_gradient(phi)))
        finally:
            lat.close()
    assert torch.equal(out[0][0], out[1][0])
    assert torch.equal(out[0][1]["phi0"], out[1][1]["phi0"])
    assert out[0][1]["tau"] == out[1][1]["tau"]
