"""Launches over samples of very different sizes take the blocks they need: the
chunks of the records' first stage on the CPU (tests/c/group_check.hip), and on
the GPU the initial data, records and gradient of small samples beside large
ones, against ensembles of their own."""
import os
import shutil
import subprocess

import pytest
import torch

import mc_inputs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_chunks_on_the_host(tmp_path):
    hipcc = shutil.which("hipcc")
    if hipcc is None:
        pytest.skip("hipcc not found")
    exe = str(tmp_path / "group_check")
    src = os.path.join(ROOT, "tests", "c", "group_check.hip")
    subprocess.run([hipcc, "-std=c++17", "-O1", "--offload-host-only", "-x", "hip", "-I",
                    os.path.join(ROOT, "include"), "-o", exe, src], check=True, capture_output=True, text=True)
    p = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert p.returncode == 0 and "groups ok" in p.stdout, p.stderr[-2000:]


@pytest.mark.gpu
@pytest.mark.parametrize("sizes", [[16, 128, 32, 32, 128, 16], [8, 128, 8], [256, 16, 16, 64]], ids=str)
def test_small_beside_large(sizes):
    mc = pytest.importorskip("paper_2608_23786_amd")

    def sample(n):
        return mc.Sample(n, mc_inputs.diffusive_u0(n) if n >= 32 else 0.05, 25.0 * n, 0.05, True)

    m = len(sizes)
    y = torch.from_numpy(mc_inputs.draw_y(5, m))
    both = mc.Ensemble([sample(n) for n in sizes], "f64")
    both.init(0, y)
    initial = [both.get_state(s) for s in range(m)]
    records = both.step(3, record_every=1)
    both.init(0, y)
    grad, ke = both.backward(2, 1, both.forward_ckpt(2, 1))
    for s, n in enumerate(sizes):
        own = mc.Ensemble([sample(n)], "f64")
        own.init(0, y[s:s + 1])
        assert torch.equal(own.get_state(0), initial[s])
        # FP64 sums of one sample's nodes (mass, energy), and of its 24 parameters, in another order
        tol = n ** 3 * 2.0 ** -53
        r = own.step(3, record_every=1)
        assert torch.allclose(r[:, 0, [0, 4]], records[:, s, [0, 4]], rtol=tol, atol=0.0)
        assert torch.equal(r[:, 0, 5:7], records[:, s, 5:7])
        own.init(0, y[s:s + 1])
        g, k = own.backward(2, 1, own.forward_ckpt(2, 1))
        assert torch.allclose(k[0], ke[s], rtol=tol, atol=0.0)
        assert torch.allclose(g[0], grad[s] * m, rtol=0.0, atol=tol * float(g.abs().max()))
