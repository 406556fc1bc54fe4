"""Lattices whose memory runs short: a refused allocation that the library can do
without changes no result and leaves no error behind for the launches after it."""
import ctypes as C

import pytest

from paper_2410_13165_amd import inputs
from paper_2410_13165_amd import lbm as B
from tests.pairs import gpu_lattice
from tests.test_zz_no_alloc import _node_state

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _limited_lattice(limit, d, dims, spec, bc, precision, refuse_last=False):
    """A lattice whose allocator refuses what would exceed `limit(state_bytes)` bytes
    in all (or, refuse_last, the last allocation of lbm_create), and the list of the
    sizes it refused."""
    from paper_2410_13165_amd import Lattice
    kw = dict(dx=1.0 / (dims[0] - 1), u=spec["u"], R=spec["R"], bc=bc, precision=precision,
              field=spec)
    lat = Lattice(d, dims, 0.5, **kw)
    p, lib = lat._params, lat.lib
    state, count = lat.state_bytes(), len(lat._bufs)
    lib.lbm_destroy(lat._h)
    lat._h = None
    bufs, refused = {}, []

    def alloc(nbytes, ctx):
        if refuse_last:
            no = len(bufs) == count - 1
        else:
            no = sum(t.numel() for t in bufs.values()) + nbytes > limit(state)
        if no:
            refused.append(nbytes)
            return None
        t = torch.empty(int(nbytes), dtype=torch.uint8, device="cuda")
        bufs[t.data_ptr()] = t
        return t.data_ptr()

    def free(ptr, ctx):
        bufs.pop(ptr, None)

    lat._limited = (B._ALLOC(alloc), B._FREE(free), bufs)
    p.alloc, p.free_fn = lat._limited[0], lat._limited[1]
    h = C.c_void_p()
    dims_arr = (C.c_int64 * B.MAX_DIM)(*(list(dims) + [1] * (B.MAX_DIM - d)))
    rc = lib.lbm_create(d, dims_arr, 0.5, C.byref(p), C.byref(h))
    assert rc == B.OK, lib.lbm_last_error(None).decode()
    lat._h = h
    return lat, refused


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_second_scratch_state_refused(precision):
    """Walled d = 3 lattices without room for a fourth state: the states of a lattice
    with room, and the allocation is asked for once."""
    dims, bc = (120, 113, 112), ["fullway"] * 3
    spec = inputs.random_cosines(3, [0.05, -0.1, 0.08], 0.7, seed=81, kmax=1.0)
    lat, refused = _limited_lattice(lambda s: 3.5 * s, 3, dims, spec, bc, precision)
    ref = gpu_lattice(3, dims, 1.0 / 119, spec, bc=bc, precision=precision)
    try:
        for n in (6, 3, 4):
            lat.step(n)
            ref.step(n)
            assert torch.equal(_node_state(lat), _node_state(ref)), n
        assert refused == [lat.state_bytes()]
    finally:
        lat.close()
        ref.close()


def _default_allocator(p):
    p.alloc = C.cast(None, B._ALLOC)
    p.free_fn = C.cast(None, B._FREE)


def test_failed_device_allocation_leaves_no_error():
    """The library's own hipMalloc refuses a lattice larger than the memory of the
    device (2 states of 300 GB); the next lattice steps all the same."""
    lib = B.load_library()
    torch.zeros(1, device="cuda")
    p = B.LbmParams()
    lib.lbm_params_default(C.byref(p))
    _default_allocator(p)
    p.dx = 0.1
    h = C.c_void_p()
    dims = (C.c_int64 * B.MAX_DIM)(1024, 1024, 2000, 1)
    assert 19 * 8 * 1024 * 1024 * 2000 > torch.cuda.get_device_properties(0).total_memory
    assert lib.lbm_create(3, dims, 0.5, C.byref(p), C.byref(h)) == B.ENOMEM
    assert not h.value
    dims = (C.c_int64 * B.MAX_DIM)(16, 12, 8, 1)
    phi0 = torch.randn(8, 12, 16, dtype=torch.float64, device="cuda")
    p.init_order = 1
    assert lib.lbm_create(3, dims, 0.5, C.byref(p), C.byref(h)) == B.OK
    try:
        rc = lib.lbm_set_initial(h, C.c_void_p(phi0.data_ptr()), None)
        assert rc == B.OK, lib.lbm_last_error(h).decode()
        rc = lib.lbm_step(h, 6)
        assert rc == B.OK, lib.lbm_last_error(h).decode()
        torch.cuda.synchronize()
    finally:
        lib.lbm_destroy(h)


WALLED = [(1, (40,), ["fullway"], "fp64"), (1, (3000,), ["halfway"], "fp32"),
          (2, (41, 33), ["fullway"] * 2, "fp32_split"),
          (2, (41, 33), ["halfway", "periodic"], "fp64"),
          (2, (300, 41), ["halfway", "halfway"], "fp32"),
          (2, (20000, 3), ["periodic", "fullway"], "fp32")]


@pytest.mark.parametrize("d,dims,bc,precision", WALLED)
def test_stepping_walled_d1_and_d2_allocates_nothing(d, dims, bc, precision):
    """From the first call on, and the steps go several to a pass."""
    spec = inputs.random_cosines(d, [0.05, -0.1][:d], 0.7, seed=82, kmax=1.0)
    lat = gpu_lattice(d, dims, 1.0 / (dims[0] - 1), spec, bc=bc, precision=precision)
    try:
        before = torch.cuda.memory_stats()["allocation.all.allocated"]
        lat.profile_begin(64)
        lat.step(20)
        lat.step_static(7)
        torch.cuda.synchronize()
        assert torch.cuda.memory_stats()["allocation.all.allocated"] == before
        assert lat.profile_end()["launches"] < 27
    finally:
        lat.close()


@pytest.mark.parametrize("d,dims,bc,precision", WALLED)
def test_wall_data_workspace_refused(d, dims, bc, precision):
    """Without room for the wall data of several steps the lattice goes on in single
    steps: the states of a lattice with room."""
    spec = inputs.random_cosines(d, [0.05, -0.1][:d], 0.7, seed=82, kmax=1.0)
    lat, refused = _limited_lattice(None, d, dims, spec, bc, precision, refuse_last=True)
    ref = gpu_lattice(d, dims, 1.0 / (dims[0] - 1), spec, bc=bc, precision=precision)
    try:
        assert len(refused) == 1
        for n in (6, 3):
            lat.step(n)
            ref.step(n)
            assert torch.equal(_node_state(lat), _node_state(ref)), n
        lat.step_static(5)
        ref.step_static(5)
        assert torch.equal(_node_state(lat), _node_state(ref))
        assert len(refused) == 1
    finally:
        lat.close()
        ref.close()


def test_second_scratch_state_makes_room_for_a_gradient():
    """Two states, a scratch state, a checkpoint and the two adjoint buffers fit, a second
    scratch state besides does not: the gradient of a lattice with room."""
    dims, bc = (120, 113, 112), ["fullway"] * 3
    spec = inputs.random_cosines(3, [0.05, -0.1, 0.08], 0.7, seed=81, kmax=1.0)
    lat, refused = _limited_lattice(lambda s: 6.5 * s, 3, dims, spec, bc, "fp32")
    ref = gpu_lattice(3, dims, 1.0 / 119, spec, bc=bc, precision="fp32")
    try:
        out = []
        for one in (lat, ref):
            one.tape_begin(100)
            one.step(6)
            out.append(one.tape_gradient(one.phi(), want_tau=False)["phi0"])
            one.tape_end()
            one.step(6)
        assert refused
        assert torch.equal(out[0], out[1])
        assert torch.equal(_node_state(lat), _node_state(ref))
    finally:
        lat.close()
        ref.close()


def test_calls_of_two_steps_allocate_what_longer_ones_need():
    dims = (120, 113, 112)
    spec = inputs.random_cosines(3, [0.05, -0.1, 0.08], 0.7, seed=81, kmax=1.0)
    lat = gpu_lattice(3, dims, 1.0 / 119, spec, bc=["fullway"] * 3, precision="fp32")
    try:
        lat.step(2)
        before = torch.cuda.memory_stats()["allocation.all.allocated"]
        lat.step(9)
        assert torch.cuda.memory_stats()["allocation.all.allocated"] == before
    finally:
        lat.close()
