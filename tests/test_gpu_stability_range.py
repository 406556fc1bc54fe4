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
