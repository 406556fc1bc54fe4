"""Which d = 3 lattices go three steps per pass, and the states of those that go in
pairs: bitwise those of single steps, on lattices on either side of the rule (thin
ones, small ones, columns that fill their tiles badly).  The launch counts show the
passes that a call takes."""
import pytest

from paper_2410_13165_amd import inputs
from tests.pairs import gpu_lattice
from tests.test_zz_no_alloc import _node_state

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# launches of calls of 3, 5, 6 and 7 steps
THREES, SMALL, PAIRS = (1, 2, 2, 3), (2, 3, 3, 3), (2, 3, 3, 4)


@pytest.mark.parametrize("dims,bc,precision,launches", [
    ((64, 64, 64), "periodic", "fp64", THREES), ((64, 64, 64), "periodic", "fp32", THREES),
    ((24, 24, 24), "periodic", "fp64", SMALL), ((48, 48, 48), "periodic", "fp32", SMALL),
    ((16, 16, 300), "periodic", "fp64", THREES), ((2, 2, 2), "periodic", "fp32", PAIRS), ((2000, 800, 2), "periodic", "fp64", PAIRS),
    ((300, 300, 8), "periodic", "fp64", PAIRS), ((300, 300, 8), "periodic", "fp32", PAIRS),
    ((2000, 800, 2), "fullway", "fp32", PAIRS), ((500, 400, 9), "halfway", "fp64", PAIRS),
    ((400, 300, 12), "fullway", "fp64", PAIRS), ((120, 120, 120), "fullway", "fp32", THREES),
    ((120, 120, 120), "halfway", "fp64", THREES), ((64, 64, 64), "fullway", "fp32", PAIRS),
    ((120, 120, 120), "fullway", "fp32_split", PAIRS),
])
def test_steps_per_pass_and_states(dims, bc, precision, launches):
    from paper_2410_13165_amd import Lattice
    spec = inputs.random_cosines(3, [0.05, -0.1, 0.08], 0.7, seed=77, kmax=1.0)
    dx = 1.0 / (dims[0] - 1)
    a = gpu_lattice(3, dims, dx, spec, bc=[bc] * 3, precision=precision)
    b = Lattice(3, dims, 0.5, dx=dx, u=spec["u"], R=spec["R"], bc=[bc] * 3, precision=precision,
                field=spec, steps_per_pass=1)
    try:
        print(f"[tri rule] dims={dims} bc={bc} {precision}", flush=True)
        for n, want in zip((3, 5, 6, 7), launches):
            a.profile_begin(16)
            a.step(n)
            prof = a.profile_end()
            b.step(n)
            assert prof["steps"] == n and prof["launches"] == want, (n, prof)
            assert torch.equal(_node_state(a), _node_state(b)), n
    finally:
        a.close()
        b.close()


@pytest.mark.parametrize("dims,precision,every,launches", [
    ((20, 20, 20), "fp32_split", 5, 12), ((20, 20, 20), "fp64", 5, 12),
    ((20, 20, 20), "fp32_split", 4, 6), ((90, 90, 90), "fp32_split", 5, 7),
    ((90, 90, 90), "fp64", 5, 5), ((90, 90, 90), "fp32", 5, 5),
])
def test_passes_between_odd_checkpoints(dims, precision, every, launches):
    """Twelve steps of a tape: small lattices go in single steps between odd checkpoints."""
    from paper_2410_13165_amd import Lattice
    lat = Lattice(3, dims, 0.7, dx=1.0 / dims[0], u=[0.05, -0.1, 0.08], precision=precision, K=1)
    try:
        lat.set_initial(torch.randn(*reversed(dims), dtype=torch.float64, device="cuda"))
        lat.tape_begin(every)
        lat.profile_begin(16)
        lat.step(12)
        prof = lat.profile_end()
        assert prof["steps"] == 12 and prof["launches"] == launches, prof
        lat.tape_end()
    finally:
        lat.close()
