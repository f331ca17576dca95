"""Spectra and structure functions up to 64^3, whose shell sums take more threads
than the transforms of a block: against FP64 sums on the host, for several
samples per launch, and a field whose shells are known."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

mc = pytest.importorskip("paper_2608_23786_amd")


def _expected(u, n):
    """E[kappa] and S2[r] of u[3, n, n, n] (last axis x) by their definitions, on the host in float64."""
    f = torch.fft.fftn(u, dim=(1, 2, 3))
    psi = (f.real ** 2 + f.imag ** 2).sum(0)
    k = torch.fft.fftfreq(n, 1.0 / n, dtype=torch.float64)
    k[n // 2] = n // 2
    k2 = k[:, None, None] ** 2 + k[None, :, None] ** 2 + k[None, None, :] ** 2
    # round(sqrt(k2)) by whole numbers: no distance lies half way between two
    shell = torch.floor(torch.sqrt(k2) + 0.5).to(torch.int64)
    count = torch.bincount(shell.view(-1), minlength=n)[:n // 2 + 1].double()
    ek = torch.bincount(shell.view(-1), weights=(0.5 * k2 * psi).view(-1), minlength=n)[:n // 2 + 1]
    ek = 4.0 * math.pi / count * ek / float(n) ** 6
    r = torch.fft.ifftn(psi, dim=(0, 1, 2)).real / float(n) ** 3
    d = torch.bincount(shell.view(-1), weights=(2.0 * (r[0, 0, 0] - r)).view(-1), minlength=n)[:n // 2 + 1]
    return ek, (d / count)[1:]


@pytest.mark.parametrize("n,m", [(8, 1), (8, 5), (16, 3), (32, 1), (32, 3), (64, 2)])
def test_shell_sums(n, m):
    ens = mc.Ensemble([mc.Sample(n, 0.05, 25.0 * n)] * m, "f64")
    g = torch.Generator().manual_seed(n + m)
    u = torch.randn((m, 3, n, n, n), generator=g, dtype=torch.float64)
    s2, ek = ens.observables_velocity_range(0, m, u=u.cuda().view(-1))
    for s in range(m):
        e, d = _expected(u[s], n)
        # rounding of transforms and sums of n^3 terms of like size
        tol = 16 * math.log2(n) * 2.0 ** -53 * n
        assert torch.allclose(ek[s].cpu(), e, rtol=tol, atol=tol * float(e.max()) * 1e-3)
        assert torch.allclose(s2[s].cpu(), d, rtol=tol, atol=tol * float(d.max()))
