"""Instances of a batch that are initialised by themselves (lbm_set_initial through
Batch.instance): the batch's moments and its later steps take their new states.

The instance's own lbm_moments and lattices of their own are the references, bit for
bit: the moments are the same reductions, and the passes those of single lattices."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("d,before", [(1, 0), (1, 3), (2, 0), (2, 2), (2, 4), (2, 7), (3, 1)])
def test_moments_and_steps_after_instance_initialisation(d, before, precision):
    from paper_2410_13165_amd import Batch, Lattice
    dims = {1: [(40,), (300,)], 2: [(21, 16), (50, 33)], 3: [(8, 7, 6), (9, 5, 4)]}[d]
    u = [0.05, -0.1, 0.08][:d]
    specs = [{"dims": n, "tau": 0.6, "dx": 1.0 / n[0], "u": u, "R": 0.3, "K": 3} for n in dims]
    g = torch.Generator(device="cuda").manual_seed(21)

    def field(n, mean):
        return mean + torch.randn(*reversed(n), generator=g, dtype=torch.float64, device="cuda")

    with Batch(d, specs, precision=precision) as b:
        b.set_initial(torch.cat([field(n, 1.0).reshape(-1) for n in dims]))
        b.step(before)
        phi0 = field(dims[1], 40.0)
        b.instance(1).set_initial(phi0)
        for n in (0, 4, 5):  # 0: not stepped since
            b.step(n)
            want = [list(b.instance(i).diagnostics().values()) for i in range(2)]
            assert np.array_equal(b.moments(), np.array(want), equal_nan=True), n
        with Lattice(d, dims[1], 0.6, dx=specs[1]["dx"], u=u, R=0.3, K=3,
                     precision=precision) as lat:
            lat.set_initial(phi0)
            lat.step(9)
            # phi of float32 adds R t, and the batch's clock ran before: the moving part
            # of the state is what has to agree
            own = lat.get_state().view(torch.float32 if precision == "fp32" else torch.float64)
            got = b.instance(1).get_state().view(own.dtype)
            info = lat.info()
            q, ps, nodes = info["q"], info["pstride"], info["nodes"]
            assert torch.equal(own.reshape(q, ps)[:, :nodes], got.reshape(q, ps)[:, :nodes])


@pytest.mark.parametrize("d", [1, 2, 3])
def test_initialisation_and_moments_allocate_nothing(d):
    """The first ones of a batch included."""
    from paper_2410_13165_amd import Batch
    dims = {1: [(40,), (300,)], 2: [(21, 16), (50, 33)], 3: [(8, 7, 6), (9, 5, 4)]}[d]
    specs = [{"dims": n, "tau": 0.6, "dx": 1.0 / n[0], "u": [0.05] * d} for n in dims]
    phi0 = torch.randn(sum(int(np.prod(n)) for n in dims), dtype=torch.float64, device="cuda")
    with Batch(d, specs, precision="fp32") as b:
        before = torch.cuda.memory_stats()["allocation.all.allocated"]
        b.set_initial(phi0)
        b.step(3)
        b.moments()
        assert torch.cuda.memory_stats()["allocation.all.allocated"] == before
