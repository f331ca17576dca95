"""Post-processing kernels at the sizes where their layouts change: the 1-point
Wasserstein distance around the sizes of its sorting networks, and both forms of
the dissipation rate around a block's samples."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

mc = pytest.importorskip("paper_2608_23786_amd")


@pytest.mark.parametrize("q", [1, 2])           # 3 and 24 columns: a part of a block, whole blocks
@pytest.mark.parametrize("m", [1, 2, 63, 64, 65, 128, 129, 256, 257, 512, 513, 1024, 1025, 4096])
def test_w1_sizes(m, q):
    rng = np.random.default_rng(m + q)
    a, b = rng.normal(size=(m, 3, q ** 3)), rng.normal(size=(m, 3, q ** 3)) * 1.3 + 0.2
    a[: m // 2, 0, 0] = 0.25                     # ties
    w = mc.w1_1pt(torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda(), q).cpu().numpy()
    ref = np.abs(np.sort(a, axis=0) - np.sort(b, axis=0)).mean(axis=0).mean(axis=1)
    assert np.max(np.abs(w - ref)) < 1e-13


@pytest.mark.parametrize("m", [5, 100, 1000])
def test_w1_of_a_nan_is_nan(m):
    a, b = torch.rand(m, 3, 8, dtype=torch.float64), torch.rand(m, 3, 8, dtype=torch.float64)
    a[m // 2, 1, 3] = float("nan")
    w = mc.w1_1pt(a.cuda(), b.cuda(), 2).cpu()
    assert torch.isnan(w[1]) and torch.isfinite(w[0]) and torch.isfinite(w[2])


@pytest.mark.parametrize("m", [1, 15, 16, 17, 256, 257])
@pytest.mark.parametrize("nrec", [2, 3, 9])
def test_dissipation_sizes(m, nrec):
    n, u0, re, every = 16, 0.05, 400.0, 7
    ens = mc.Ensemble([mc.Sample(n, u0, re)] * m, "f32s", lattice=19)
    g = torch.Generator(device="cpu").manual_seed(m * nrec)
    rec = torch.rand((nrec, m, 8), generator=g, dtype=torch.float64)
    rec[:, :, 4] = 1e-3 * (2.0 - torch.arange(nrec, dtype=torch.float64)[:, None] / nrec + 0.1 * rec[:, :, 4])
    ek = 1e-3 * torch.rand((nrec, m, n // 2 + 1), generator=g, dtype=torch.float64)
    ek += torch.linspace(1.0, 0.0, nrec, dtype=torch.float64)[:, None, None]
    t = torch.arange(nrec, dtype=torch.float64) * every * (2 * np.pi / n) * u0
    for energy, (d, eta) in ((rec[:, :, 4], ens.dissipation(rec.cuda(), 0, every)),
                             (ek.sum(2), ens.dissipation_spectra(0, ek.cuda(), 0, every))):
        lo = [max(k - 1, 0) for k in range(nrec)]
        hi = [min(k + 1, nrec - 1) for k in range(nrec)]
        ref = -(energy[hi] - energy[lo]) / u0 ** 2 / (t[hi] - t[lo])[:, None]
        # differences of energies of size 1/u0^2, each summed to a few roundings
        scale = float(energy.abs().max()) / u0 ** 2 / float(t[1])
        assert float((d.cpu() - ref).abs().max()) < 1e-14 * scale
        mean = ref.mean(1)
        want = ((1.0 / re) ** 3 / mean) ** 0.25
        ok = mean > 1e-3 * scale                 # a mean near zero is a difference of nearly equal sums
        assert torch.allclose(eta.cpu()[ok], want[ok], rtol=1e-10, atol=0.0)
