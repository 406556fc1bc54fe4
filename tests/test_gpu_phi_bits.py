"""phi of float32 lattices to the last bit: the populations of the stored state summed in
their order in float64, each with its weight times the reference phi_mean + R t_{n+1},
which d = 3 and 4 round once."""
from fractions import Fraction

import numpy as np
import pytest

from paper_2410_13165_amd import inputs
from tests.pairs import gpu_lattice

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("d,dims", [(3, (11, 9, 7)), (4, (6, 5, 4, 3))])
def test_phi_rounds_the_reference_once(d, dims):
    u = [0.05, -0.1, 0.08, 0.03][:d]
    spec = inputs.random_cosines(d, u, 0.7, seed=87, kmax=1.0)
    lat = gpu_lattice(d, dims, 1.0 / (dims[0] - 1), spec, tau=0.7, precision="fp32")
    try:
        for _ in range(12):
            lat.step(1)
            info = lat.info()
            q, ps, nodes, dt = info["q"], info["pstride"], info["nodes"], info["dt"]
            f = lat.get_state().view(torch.float32).reshape(q, ps)[:, :nodes].double().cpu().numpy()
            t = np.float64(info["step"]) * np.float64(dt)
            ref = np.float64(float(Fraction(spec["R"]) * Fraction(float(t + dt))
                                   + Fraction(info["phi_ref"])))
            phi = np.zeros(nodes)
            for k in range(q):
                phi = phi + (f[k] + info["omega"][k] * ref)
            phi = phi - np.float64(dt) * np.float64(spec["R"])
            assert np.array_equal(lat.phi().reshape(-1).cpu().numpy(), phi), info["step"]
            assert lat.diagnostics(2)["max_abs_phi"] == np.abs(phi).max()
    finally:
        lat.close()
