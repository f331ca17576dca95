"""Spectrum and structure function of a random velocity at every resolution
(every split of a line into factors) against torch's transforms in FP64."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

mc = pytest.importorskip("paper_2608_23786_amd")

# A transform of n^3 values errs by a few log2(n^3) eps of its norm, either side; the
# sums over shells add about as much: 4 * 27 * 2.2e-16 * 4 < 1e-13, with a factor 4 to spare.
TOL = 4e-13


@pytest.mark.parametrize("n,m", [(8, 3), (16, 2), (32, 3), (64, 2), (128, 2), (256, 1), (512, 1)])
def test_random_velocity_matches_torch(n, m):
    gen = torch.Generator(device="cuda").manual_seed(n)
    u = torch.randn(m, 3, n, n, n, dtype=torch.float64, device="cuda", generator=gen)
    ens = mc.Ensemble([mc.Sample(n, 0.01, 100.0)] * m, "f32s")
    ens.two_step(False)
    s2, ek = ens.observables_velocity_range(0, m, u=u.view(-1))
    ens.synchronize()
    k = torch.fft.fftfreq(n, 1.0 / n, dtype=torch.float64, device="cuda")
    k2 = k[:, None, None] ** 2 + k[None, :, None] ** 2 + k[None, None, :] ** 2
    shell = torch.round(torch.sqrt(k2)).long().view(-1)
    count = torch.bincount(shell)[:n // 2 + 1].double()
    for s in range(m):
        psi = sum(torch.fft.fftn(u[s, c]).abs() ** 2 for c in range(3))
        sums = torch.bincount(shell, weights=(0.5 * k2 * psi).view(-1))[:n // 2 + 1]
        want_ek = 4.0 * math.pi * sums / count / float(n) ** 6
        r = torch.fft.ifftn(psi).real / float(n) ** 3
        r0 = float(r[0, 0, 0])
        want_s2 = torch.bincount(shell, weights=(2.0 * (r0 - r)).view(-1))[1:n // 2 + 1] / count[1:]
        assert float((ek[s].cuda() - want_ek).abs().max()) <= TOL * float(want_ek.max())
        assert float((s2[s].cuda() - want_s2).abs().max()) <= TOL * 2.0 * r0
