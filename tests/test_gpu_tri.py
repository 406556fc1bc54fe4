"""Three-step passes of d = 3 lattices: bitwise the states of single steps.

The single-step kernels are the reference, so no tolerance enters.  Sizes sit at
the edges of the passes' tiles (64 x 11, 64 x 7 and 32 x 10 columns), at the fewest
planes a march can have, and at walls two and three rows apart (lattices with walls
are as large as the passes take them, 1.4 million nodes; the thin ones go in pairs);
the step counts take 3, 3 + 1 as 2 + 2, 3 + 2, 3 + 3 + 1 as 3 + 2 + 2, and several
passes in a row."""
import pytest

from paper_2410_13165_amd import inputs
from tests.pairs import gpu_lattice
from tests.test_zz_no_alloc import _node_state

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32_split"])
@pytest.mark.parametrize("dims,bc,wall_data", [
    ((1, 1, 1), ["periodic"] * 3, "jets"),
    ((64, 11, 5), ["periodic"] * 3, "jets"),
    ((65, 12, 3), ["periodic"] * 3, "jets"),
    ((33, 29, 140), ["periodic"] * 3, "jets"),
    ((128, 121, 97), ["fullway"] * 3, "jets"),
    ((1601, 480, 2), ["fullway"] * 3, "jets"),
    ((1601, 313, 3), ["halfway"] * 3, "jets"),
    ((31, 2, 24500), ["halfway"] * 3, "jets"),
    ((2, 3, 250001), ["fullway"] * 3, "jets"),
    ((129, 99, 118), ["halfway", "periodic", "halfway"], "tangential"),
    ((160, 78, 121), ["periodic", "fullway", "periodic"], "jets"),
    ((45, 11, 3100), ["fullway", "periodic", "periodic"], "jets"),
    ((100, 150, 101), ["periodic", "periodic", "halfway"], "jets"),
])
def test_tri_passes_equal_single_steps_bitwise(dims, bc, wall_data, precision):
    from paper_2410_13165_amd import Lattice
    spec = inputs.random_cosines(3, [0.05, -0.1, 0.08], 0.7, seed=75, kmax=1.0)
    dx = 1.0 / max(dims[0] - 1, 1)
    a = gpu_lattice(3, dims, dx, spec, bc=bc, precision=precision, wall_data=wall_data)
    b = Lattice(3, dims, 0.5, dx=dx, u=spec["u"], R=spec["R"], bc=bc, precision=precision,
                field=spec, wall_data=wall_data, steps_per_pass=1)
    try:
        print(f"[tri] dims={dims} bc={bc} {wall_data} {precision}", flush=True)
        for n in (3, 4, 5, 7, 12):
            a.step(n)
            b.step(n)
            assert torch.equal(_node_state(a), _node_state(b)), n
    finally:
        a.close()
        b.close()


@pytest.mark.parametrize("bc", ["fullway", "halfway"])
def test_static_scratch_without_room_for_three_steps(bc):
    """lbm_step_static, whose fixed scratch holds one scratch state of this lattice
    but not two, gives the states of lbm_step."""
    spec = inputs.random_cosines(3, [0.05, -0.1, 0.08], 0.7, seed=76, kmax=1.0)
    lats = [gpu_lattice(3, (120, 113, 112), 1 / 119, spec, bc=[bc] * 3, precision="fp32")
            for _ in range(2)]
    try:
        lats[0].step(10)
        lats[1].step_static(10)
        assert torch.equal(_node_state(lats[0]), _node_state(lats[1]))
    finally:
        for lat in lats:
            lat.close()
