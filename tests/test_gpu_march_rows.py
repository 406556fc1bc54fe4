"""Passes of several steps of d = 2 lattices whose tiles have several rows: bitwise the
states of single steps.

The single-step kernels are the reference, so no tolerance enters.  The lattices are
large enough that a tile takes more than one row (with walls 5 to 32, periodic 8 to
over 100) and that the last chunk of rows and the last tile of columns are ragged;
the step counts take passes of 8 (4 with walls), 4, 2 and 1.  The periodic float32
and float64 ones from about a million nodes take their two-step passes in blocks of
256 columns.  The launch counts show the passes taken."""
import pytest

from paper_2410_13165_amd import inputs
from tests.pairs import gpu_lattice
from tests.test_zz_no_alloc import _node_state

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _check(dims, bc, wall_data, precision, counts, launches):
    from paper_2410_13165_amd import Lattice
    spec = inputs.random_cosines(2, [0.1, -0.15], 0.7, seed=83, kmax=1.0)
    dx = 1.0 / (dims[0] - 1)
    a = gpu_lattice(2, dims, dx, spec, bc=bc, precision=precision, wall_data=wall_data)
    b = Lattice(2, dims, 0.5, dx=dx, u=spec["u"], R=spec["R"], bc=bc, precision=precision,
                field=spec, wall_data=wall_data, steps_per_pass=1)
    try:
        print(f"[rows] dims={dims} bc={bc} {wall_data} {precision}", flush=True)
        for n, want in zip(counts, launches):
            a.profile_begin(64)
            a.step(n)
            prof = a.profile_end()
            b.step(n)
            assert prof["steps"] == n and prof["launches"] == want, (n, prof)
            assert torch.equal(_node_state(a), _node_state(b)), n
    finally:
        a.close()
        b.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32_split"])
@pytest.mark.parametrize("dims,bc,wall_data", [
    ((520, 701), ["halfway"] * 2, "jets"),
    ((777, 803), ["fullway"] * 2, "tangential"),
    ((1001, 1203), ["halfway"] * 2, "tangential"),
    ((777, 803), ["halfway", "periodic"], "jets"),
    ((777, 803), ["periodic", "fullway"], "jets"),
])
def test_walls_with_several_rows_per_tile(dims, bc, wall_data, precision):
    _check(dims, bc, wall_data, precision, (4, 2, 15), (1, 1, 5))


@pytest.mark.parametrize("dims,precision,launches", [
    ((1100, 1200), "fp64", (1, 1, 4)), ((1100, 1200), "fp32", (2, 1, 5)),
    ((1100, 1200), "fp32_split", (1, 1, 4)), ((2048, 2048), "fp32_split", (1, 1, 4)),
    ((2048, 2048), "fp64", (1, 1, 4)), ((2048, 2050), "fp32", (2, 1, 5)),
    ((4100, 1030), "fp32", (2, 1, 5)), ((1300, 1027), "fp64", (1, 1, 4)),
    ((1050, 2100), "fp32", (2, 1, 5)), ((300001, 11), "fp64", (1, 1, 4)),
    ((8000, 700), "fp32", (1, 1, 4)),
])
def test_periodic_with_several_rows_per_tile(dims, precision, launches):
    _check(dims, ["periodic"] * 2, "jets", precision, (8, 2, 15), launches)
