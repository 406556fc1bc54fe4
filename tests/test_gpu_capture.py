"""Calls captured into a HIP graph and replayed: where the call ends in the buffer that
it started from, replays go on from one another, and the state after r replays is that
of r calls, bit for bit.  That is so for an even number of pairs of steps (an odd last
step counts as one), or of steps where the storage mode has no pairs."""
import pytest

from paper_2410_13165_amd import inputs
from tests.test_zz_no_alloc import _node_state

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _state(lat, owner=None):
    with torch.cuda.stream((owner or lat).stream):
        state = _node_state(lat)
    torch.cuda.synchronize()
    return state


def _replay(stream, call, check):
    """Captures call() and checks after every replay, other work in between."""
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        call()
    with torch.cuda.stream(stream):
        for r in range(1, 5):
            graph.replay()
            torch.randn(1000, device="cuda").sum()
            torch.cuda.synchronize()
            with torch.cuda.stream(torch.cuda.default_stream()):
                check(r)


@pytest.mark.parametrize("d,dims,precision,counts", [
    (1, (300,), "fp64", (2, 8, 1500)), (1, (3000,), "fp32", (2, 130)),
    (2, (100, 70), "fp64", (3, 4, 7, 8, 12, 20)), (2, (100, 70), "fp32", (4, 8, 11)),
    (2, (1300, 900), "fp64", (4, 8)), (2, (100, 70), "fp32_split", (2, 4, 6, 8, 10)),
    (3, (40, 36, 50), "fp64", (3, 4, 7, 8, 12)), (3, (64, 64, 64), "fp32", (4, 7, 8, 11, 16)),
    (3, (40, 36, 50), "fp32_split", (4, 8)),
])
def test_replays_of_a_captured_call_go_on(d, dims, precision, counts):
    from paper_2410_13165_amd import Lattice
    u = [0.05, -0.1, 0.08][:d]
    stream = torch.cuda.Stream()
    phi0 = torch.randn(*reversed(dims), dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    for n in counts:
        print(f"[capture] {dims} {precision} n={n}", flush=True)
        with torch.cuda.stream(stream):
            lat = Lattice(d, dims, 0.7, dx=1.0 / dims[0], u=u, precision=precision, K=1)
            lat.set_initial(phi0)
        ref = Lattice(d, dims, 0.7, dx=1.0 / dims[0], u=u, precision=precision, K=1)
        ref.set_initial(phi0)
        try:
            def check(r):
                ref.step(n)
                assert torch.equal(_state(lat), _state(ref)), (n, r)

            _replay(stream, lambda: lat.step_static(n), check)
        finally:
            lat.close()
            ref.close()


@pytest.mark.parametrize("d,dims,bc,n", [(1, (200,), "fullway", 2), (1, (200,), "halfway", 64),
                                         (2, (60, 50), "fullway", 4), (2, (60, 50), "halfway", 8),
                                         (3, (60, 50, 40), "fullway", 4)])
def test_first_call_captured_with_steady_walls(d, dims, bc, n):
    """A lattice that has made no step before: its first call is captured.  The data of
    the walls do not change in time (u = 0 wave vectors), so replays go on too."""
    from paper_2410_13165_amd import Lattice
    spec = {"kind": "cos_sum", "u": [0.0] * d, "R": 0.0, "amps": [1.0],
            "kvecs": [[1.0, 0.5, 0.7][:d]], "phases": [0.3]}
    stream = torch.cuda.Stream()
    kw = dict(dx=1.0 / (dims[0] - 1), u=spec["u"], R=0.0, bc=[bc] * d, precision="fp64", field=spec)
    with torch.cuda.stream(stream):
        lat = Lattice(d, dims, 0.7, **kw)
    ref = Lattice(d, dims, 0.7, **kw)
    try:
        def check(r):
            ref.step(n)
            assert torch.equal(_state(lat), _state(ref)), r

        _replay(stream, lambda: lat.step_static(n), check)
    finally:
        lat.close()
        ref.close()


@pytest.mark.parametrize("form", ["per_pair", "resident"])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_replays_of_a_captured_batch_go_on(form, precision):
    from paper_2410_13165_amd import Batch
    specs = [{"dims": n, "tau": 0.6, "dx": 0.02, "u": [0.1, -0.05], "K": 1}
             for n in ((64, 64), (33, 50), (100, 20))]
    phi0 = torch.randn(sum(s["dims"][0] * s["dims"][1] for s in specs), dtype=torch.float64,
                       device="cuda")
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    for n in (3, 4, 7, 8, 12, 24):
        print(f"[capture] batch {form} {precision} n={n}", flush=True)
        with torch.cuda.stream(stream):
            b = Batch(2, specs, precision=precision)
            b.set_launch(form)
            b.set_initial(phi0)
        with b, Batch(2, specs, precision=precision) as ref:
            ref.set_initial(phi0)

            def check(r):
                ref.step(n)
                for i in range(len(specs)):
                    got, want = _state(b.instance(i), b), _state(ref.instance(i), ref)
                    assert torch.equal(got, want), (n, r)

            _replay(stream, lambda: b.step(n), check)
