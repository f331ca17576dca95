"""Launches of fewer than 2^18 nodes take 128-thread blocks, and ensembles of
consecutive equal samples of one parity read their launch table from the kernel
arguments: every node's arithmetic is the same either way, so states and
gradients are compared bit for bit with a chosen 256-thread shape, with the
table in memory, and with launches on the other side of the rule."""
import pytest
import torch

import mc_inputs

pytestmark = pytest.mark.gpu

mc = pytest.importorskip("paper_2608_23786_amd")


def _sample(n, stride=1):
    return mc.Sample(n, mc_inputs.diffusive_u0(n) if n >= 32 else 0.05, 25.0 * n, 0.05, True, stride)


ENSEMBLES = {
    "one 8^3": [(8, 1)],
    "three 16^3": [(16, 1)] * 3,
    "seven 32^3, below the rule": [(32, 1)] * 7,
    "eight 32^3, above it": [(32, 1)] * 8,
    "mixed sizes": [(16, 1), (32, 1), (16, 1)],
    "mixed parities of one size": [(32, 1), (32, 2), (32, 1)],
    "strides below and above the rule": [(16, 4), (16, 4), (64, 1)],
}


@pytest.mark.parametrize("lattice", [27, 19])
@pytest.mark.parametrize("precision", ["f32s", "f64"])
@pytest.mark.parametrize("name", list(ENSEMBLES))
def test_states_equal_chosen_shape(name, precision, lattice):
    pair = []
    for chosen in (False, True):
        e = mc.Ensemble([_sample(n, stride) for n, stride in ENSEMBLES[name]], precision, lattice=lattice)
        e.two_step(False)
        if chosen:
            e.set_launch(256, 0, 1, 1)
        e.init(11)
        pair.append(e)
    a, b = pair
    for ticks in (1, 4, 3):
        a.step(ticks)
        b.step(ticks)
        for s in range(a.m):
            assert a.steps(s) == b.steps(s)
            assert torch.equal(a.get_state(s), b.get_state(s)), s
    # sums of one sample in another order of blocks: rounding of FP64 sums of up to 2^18 terms
    ra, rb = a.reduce(), b.reduce()
    assert torch.allclose(ra[:, [0, 4]], rb[:, [0, 4]], rtol=2.0 ** 18 * 2.0 ** -53, atol=0.0)


@pytest.mark.parametrize("precision", ["f32s", "f64"])
@pytest.mark.parametrize("sizes", [[32] * 8, [32, 32, 32, 16]], ids=["256-thread blocks", "table in memory"])
def test_gradients_equal_small_uniform_launch(precision, sizes):
    y = torch.from_numpy(mc_inputs.draw_y(5, 8))

    def grad(ns):
        e = mc.Ensemble([_sample(n) for n in ns], precision)
        v = y[:len(ns)].cuda().requires_grad_()
        return torch.autograd.grad(mc.EnsembleKE.apply(v, e, 7, 3), v)[0] * len(ns)   # the mean's 1 / M, a power of two

    small, other = grad([32] * 4), grad(sizes)
    assert torch.equal(small[:3], other[:3])
