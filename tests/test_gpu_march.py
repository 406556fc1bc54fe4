"""Passes of several steps of d = 1 and 2 lattices: bitwise the states of single
steps.

The single-step kernels are the reference (they are held to the oracle
elsewhere), so no tolerance enters.  Sizes sit at the edges of the passes' tiles:
output widths of 48 (8 steps, taken in float64) and 56 (2 and 4 steps) columns, one
row, one column; at these sizes every tile has one row (test_gpu_march_rows.py has the
larger ones).  Step counts take several pass lengths and the single-step remainder.
d = 1: one node, the largest lattice held by one block (1024 nodes) and the first two
cut into windows."""
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


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32_split"])
@pytest.mark.parametrize("n,bc,wall_data", [
    (1, "periodic", "jets"), (255, "periodic", "jets"), (1024, "periodic", "jets"),
    (1025, "periodic", "jets"), (5000, "periodic", "jets"), (2, "fullway", "jets"),
    (1024, "halfway", "jets"), (1025, "fullway", "tangential"), (1930, "halfway", "jets"),
])
def test_line_passes_equal_single_steps_bitwise(n, bc, wall_data, precision):
    from paper_2410_13165_amd import Lattice
    spec = inputs.random_cosines(1, [0.15], 0.7, seed=74, kmax=1.0)
    kw = dict(dx=1.0 / max(n - 1, 1), u=spec["u"], R=spec["R"], bc=[bc], precision=precision,
              field=spec, wall_data=wall_data)
    a = Lattice(1, (n,), 0.5, **kw)
    b = Lattice(1, (n,), 0.5, steps_per_pass=1, **kw)
    try:
        print(f"[line] n={n} {bc} {wall_data} {precision}", flush=True)
        for steps in (1, 63, 1100):  # 1100: more than one launch of either form
            a.step(steps)
            b.step(steps)
            assert torch.equal(_node_state(a), _node_state(b)), steps
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


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("d", [1, 2, 3])
def test_batch_moments_and_initial_states_equal_per_instance(d, precision):
    """Whole-batch moments against lbm_moments of each instance, bit for bit, and
    whole-batch initialisation against lbm_set_initial of each lattice on its own:
    one node, one reduction block exactly, and more nodes than one pass of the
    reduction's blocks.  The two initialisations may fuse other products, one
    rounding each of at most eight sums of values up to 4 max |phi0|; in float32
    each stored deviation may then round the other way."""
    import numpy as np
    from paper_2410_13165_amd import Batch, Lattice
    dims = {1: [(1,), (256,), (300001,)], 2: [(1, 1), (16, 16), (37, 29), (600, 500)],
            3: [(1, 1, 1), (8, 8, 4), (9, 7, 5)]}[d]
    u = [0.05, -0.1, 0.08][:d]
    g = torch.Generator(device="cuda").manual_seed(12)
    phi0 = [torch.randn(*reversed(n), generator=g, dtype=torch.float64, device="cuda") for n in dims]
    specs = [{"dims": n, "tau": 0.6 + 0.1 * i, "dx": 1.0 / n[0], "u": u, "R": 0.3, "K": 3}
             for i, n in enumerate(dims)]
    eps = 2.0 ** -53 if precision == "fp64" else 2.0 ** -24
    with Batch(d, specs, precision=precision) as b:
        b.set_initial(torch.cat([p.reshape(-1) for p in phi0]))
        for i, sp in enumerate(specs):
            with Lattice(d, sp["dims"], sp["tau"], dx=sp["dx"], u=u, R=0.3, K=3,
                         precision=precision) as lat:
                lat.set_initial(phi0[i])
                bound = 32 * eps * float(phi0[i].abs().max() + 1.0)
                assert float((lat.phi() - b.instance(i).phi()).abs().max()) <= bound, i
        for n in (0, 5):
            b.step(n)
            m = b.moments()
            for i in range(len(specs)):
                want = np.array(list(b.instance(i).diagnostics().values()))
                assert np.array_equal(m[i], want, equal_nan=True), (n, i)
