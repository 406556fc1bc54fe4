"""lbm_step_static of walled d = 2 lattices whose state exceeds its fixed scratch: their
passes use none of it, so they are taken, and give bitwise the states of lbm_step."""
import pytest

from paper_2410_13165_amd import inputs
from tests.pairs import gpu_lattice
from tests.test_zz_no_alloc import _node_state

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("precision,bc", [("fp32", ["fullway"] * 2), ("fp64", ["halfway"] * 2),
                                          ("fp64", ["periodic", "fullway"]),
                                          ("fp32_split", ["fullway"] * 2)])
def test_large_walled_lattice(precision, bc):
    spec = inputs.random_cosines(2, [0.05, -0.1], 0.7, seed=84, kmax=1.0)
    a, b = (gpu_lattice(2, (2048, 2047), 1 / 2047, spec, bc=bc, precision=precision)
            for _ in range(2))
    try:
        assert a.state_bytes() > 128 << 20
        for n in (2, 7):
            a.step_static(n)
            b.step(n)
            assert torch.equal(_node_state(a), _node_state(b)), n
    finally:
        a.close()
        b.close()
