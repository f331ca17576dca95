"""The exact stabiliser away from equilibrium, where Newton's first steps are
long and the next iterate's positivity is taken from max|dh / f*| or checked
population by population, against the oracle's bisection. With a relative
noise a on every population, |q| <= 2 a or so and the closed-form t is off by a
step D with |D| max|q| <= 0.5 for a <= 0.1; Newton squares (and halves) that
product: 0.125, 8e-3, 3e-5, 5e-10 after its four steps in FP64, relative to the
populations, which bounds the difference by 1e-9 of max|f - w|. In FP32 a = 0.02
leaves |D| max|q| <= 0.02 and rounding (30 * 2^-24) dominates."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu
mc = pytest.importorskip("paper_2608_23786_amd")


@pytest.mark.parametrize("q", [27, 19])
@pytest.mark.parametrize("precision,noise,tol", [("f64", 0.05, 1e-9), ("f64", 0.1, 1e-9), ("f32s", 0.02, 5e-6)])
def test_one_step_from_noise_matches_oracle(q, precision, noise, tol):
    n = 8
    rng = np.random.default_rng(900 + q)
    _, w = oracle.velocity_set(q)
    f = oracle.equilibrium_field(rng.uniform(-0.05, 0.05, (3, n, n, n)), q)
    f = np.ascontiguousarray(f * (1 + rng.uniform(-noise, noise, f.shape)))
    ens = mc.Ensemble([mc.Sample(n, 0.05, 100.0)], precision, lattice=q)
    ens.init(0, torch.zeros(1, 24, dtype=torch.float64))
    ens.set_stabiliser("exact")
    ens.set_state(0, torch.from_numpy(np.ascontiguousarray(f.T.reshape(q, n, n, n))).cuda())
    ens.step(1)
    fg = ens.get_state(0).cpu().numpy().reshape(q, n ** 3).T
    oracle.run(f, n, 1, oracle.omega_shear(oracle.lattice_viscosity(n, 0.05, 100.0)), mode=oracle.MODE_EXACT)
    assert float(np.max(np.abs(fg - f))) <= tol * float(np.max(np.abs(f - w)))
