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


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("given", [False, True])
def test_initial_states_of_large_and_small_instances(given, precision):
    """A batch that mixes instances at the size (1024 blocks of 256 nodes), above and below
    it from which they are initialised by a launch of their own, with and without given
    gradients: phi of lattices of their own.  Bounds as for whole-batch initialisation."""
    from paper_2410_13165_amd import Batch, Lattice
    dims = [(20, 30), (512, 512), (513, 512), (700, 900)]
    u = [0.05, -0.1]
    specs = [{"dims": n, "tau": 0.6, "dx": 1.0 / n[0], "u": u, "R": 0.3, "K": 3} for n in dims]
    g = torch.Generator(device="cuda").manual_seed(22)
    phi0 = [torch.randn(*reversed(n), generator=g, dtype=torch.float64, device="cuda") for n in dims]
    grad = [torch.randn(2, *reversed(n), generator=g, dtype=torch.float64, device="cuda")
            for n in dims] if given else None
    eps = 2.0 ** -53 if precision == "fp64" else 2.0 ** -24
    with Batch(2, specs, precision=precision) as b:
        b.set_initial(torch.cat([p.reshape(-1) for p in phi0]),
                      torch.cat([p.reshape(-1) for p in grad]) if given else None)
        b.step(3)
        for i, sp in enumerate(specs):
            with Lattice(2, sp["dims"], 0.6, dx=sp["dx"], u=u, R=0.3, K=3,
                         precision=precision) as lat:
                lat.set_initial(phi0[i], grad[i] if given else None)
                lat.step(3)
                bound = 8 * 32 * eps * float(phi0[i].abs().max() + 1.0)
                assert float((lat.phi() - b.instance(i).phi()).abs().max()) <= bound, i


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_two_step_passes_of_large_and_small_instances(precision):
    """Two-step passes in blocks (large instances) and in wavefront tiles, alone and mixed in
    one batch: bitwise the states of single lattices in single steps."""
    from paper_2410_13165_amd import Batch, Lattice
    from tests.test_zz_no_alloc import _node_state
    for dims in ([(1500, 1401)], [(57, 9), (1500, 1401), (1, 1), (112, 300)], [(113, 17), (20, 300)]):
        specs = [{"dims": n, "tau": 0.6, "dx": 0.01, "u": [0.05, -0.1], "R": 0.3} for n in dims]
        g = torch.Generator(device="cuda").manual_seed(23)
        phi0 = [torch.randn(*reversed(n), generator=g, dtype=torch.float64, device="cuda")
                for n in dims]
        print(f"[two steps] {dims} {precision}", flush=True)
        with Batch(2, specs, precision=precision) as b:
            for i in range(len(dims)):
                b.instance(i).set_initial(phi0[i])
            for n in (2, 3, 6):
                b.step(n)
            for i, sp in enumerate(specs):
                with Lattice(2, sp["dims"], 0.6, dx=0.01, u=sp["u"], R=0.3, K=1,
                             precision=precision, steps_per_pass=1) as lat:
                    lat.set_initial(phi0[i])
                    lat.step(11)
                    assert torch.equal(_node_state(lat), _node_state(b.instance(i))), (dims, i)
