"""Stability maps at relaxation rates whose roots lie far out: the squares of their
distances overflow, and a reciprocal of infinity has to be 0, as a division gives it, for
the iteration to settle.  The oracle's dense eigenvalues are the reference."""
import numpy as np
import pytest

from oracle import lbm_oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("s", [1e70, 1e153])
def test_far_roots_settle(s):
    from paper_2410_13165_amd import stability_map
    out = stability_map(np.array([[0.3]]), s, m=8)
    want = O.spectral_radius_grid([0.3], s, 8)
    assert int(out["unconverged"][0]) == 0
    assert abs(float(out["rho"][0]) - want) <= 1e-12 * want


@pytest.mark.parametrize("d,count,m", [(1, 3, 200), (2, 1, 40), (2, 300, 8), (3, 2, 12)])
def test_outputs_in_the_memory_of_the_inputs(d, count, m):
    """rho written over s and, d = 1, the weights over sigma, as the C ABI lets a caller
    do: the values of separate arrays."""
    import ctypes as C
    from paper_2410_13165_amd import lbm as B
    lib = B.load_library()
    rng = np.random.default_rng(9)
    sigma = torch.tensor(rng.uniform(-0.4, 0.4, size=(count, d)), device="cuda")
    s = torch.tensor(rng.uniform(1.2, 2.0, size=count), device="cuda")
    want = B.stability_map(sigma, s, m=m)
    mw = sigma if d == 1 else torch.empty(count, dtype=torch.float64, device="cuda")
    unc = torch.empty(count, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    rc = lib.lbm_stability_map(d, count, C.c_void_p(sigma.data_ptr()), C.c_void_p(s.data_ptr()),
                               0.5, m, C.c_void_p(s.data_ptr()), C.c_void_p(mw.data_ptr()),
                               C.c_void_p(unc.data_ptr()), None)
    assert rc == B.OK
    torch.cuda.synchronize()
    assert torch.equal(s, want["rho"])
    assert torch.equal(mw.reshape(-1), want["min_omega"])
    assert torch.equal(unc, want["unconverged"])
