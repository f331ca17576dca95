"""Ensembles in which only some runs take passes of two: the other samples step
in launches of their own, replayed from graphs in stretches long enough, and
every sample's populations are those of single steps of the whole ensemble."""
import pytest
import torch

import mc_inputs

pytestmark = pytest.mark.gpu

mc = pytest.importorskip("paper_2608_23786_amd")


def _sample(n, stride):
    return mc.Sample(n, mc_inputs.diffusive_u0(n) if n >= 32 else 0.05, 25.0 * n, 0.05, True, stride)


ENSEMBLES = {
    # (n, samples, stride): a run in passes beside smaller ones
    "one run beside two": [(64, 9, 1), (16, 5, 1), (32, 3, 2)],
    "below the line of a run with others": [(64, 4, 1), (8, 2, 1)],
    "two runs in passes": [(16, 2, 4), (64, 9, 2), (128, 1, 1), (8, 3, 1)],
}


@pytest.mark.parametrize("graphs", [True, False])
@pytest.mark.parametrize("precision,lattice", [("f32s", 27), ("f32s", 19), ("f64", 27)])
@pytest.mark.parametrize("name", list(ENSEMBLES))
def test_states_equal_single_steps(name, precision, lattice, graphs):
    pair = []
    for two in (True, False):
        ens = mc.Ensemble([_sample(n, stride) for n, m, stride in ENSEMBLES[name] for _ in range(m)], precision,
                          lattice=lattice)
        assert ens.two_step(two) == two
        ens.use_graphs(two and graphs)
        ens.init(11)
        pair.append(ens)
    a, b = pair
    # replays from several phases, with read-outs, records and short stretches between them
    for ticks, every in ((80, 0), (7, 0), (1, 0), (120, 40), (80, 0)):
        ra, rb = a.step(ticks, record_every=every), b.step(ticks, record_every=every)
        if every:
            # sums of one sample in another order of blocks
            assert torch.allclose(ra[..., [0, 4]], rb[..., [0, 4]], rtol=2.0 ** 21 * 2.0 ** -53, atol=0.0)
        for s in range(a.m):
            assert a.steps(s) == b.steps(s)
            assert torch.equal(a.get_state(s), b.get_state(s)), (ticks, s)
