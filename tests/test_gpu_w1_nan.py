"""A NaN among the values of a column makes the 1-point Wasserstein distance of its
component NaN, wherever it stands and however many samples are sorted, and leaves
the other components as they are."""
import pytest
import torch

pytestmark = pytest.mark.gpu

mc = pytest.importorskip("paper_2608_23786_amd")


@pytest.mark.parametrize("m", [3, 64, 1000, 1024, 1025, 2000, 4096])
def test_nan_in_a_column(m):
    q = 2
    g = torch.Generator().manual_seed(m)
    a, b = (torch.randn((m, 3, q ** 3), generator=g, dtype=torch.float64).cuda() for _ in range(2))
    clean = mc.w1_1pt(a, b, q)
    exact = (a.sort(dim=0).values - b.sort(dim=0).values).abs().mean(dim=(0, 2))
    # sums of m q^3 terms in another order
    assert torch.allclose(clean.view(-1)[:3], exact, rtol=m * q ** 3 * 2.0 ** -53, atol=0.0)
    for row in (0, m // 2, m - 1):
        for side in (0, 1):
            x = [a.clone(), b.clone()]
            x[side][row, 1, 5] = float("nan")
            d = mc.w1_1pt(x[0], x[1], q).view(-1)
            assert torch.isnan(d[1])
            assert torch.equal(d[[0, 2]], clean.view(-1)[[0, 2]])
