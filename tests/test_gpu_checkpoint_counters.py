"""A checkpoint holds the step counter of every sample: ensembles on both sides
of the 507 counters that fit the smallest header continue from one as if they
had not been interrupted, and its populations lie behind the counters."""
import pytest
import torch

import mc_inputs

pytestmark = pytest.mark.gpu

mc = pytest.importorskip("paper_2608_23786_amd")


@pytest.mark.parametrize("m", [507, 508, 2051])
def test_counters_of_every_sample(m):
    ens = mc.Ensemble([mc.Sample(8, 0.05, 200.0, 0.05, True, 1 if s % 3 else 2) for s in range(m)], "f32s")
    state_bytes = m * 27 * 8 ** 3 * 4
    assert ens.checkpoint_bytes() >= state_bytes + 8 * (5 + m)
    ens.init(0, torch.from_numpy(mc_inputs.draw_y(7, m)))
    ens.step(6)
    saved = ens.checkpoint()
    ens.step(5)
    expected = [(ens.steps(s), ens.get_state(s)) for s in (0, 1, m // 2, m - 1)]
    ens.restore(saved)
    assert [ens.steps(s) for s in range(m)] == [6 if s % 3 else 3 for s in range(m)]
    ens.step(5)
    for s, (steps, f) in zip((0, 1, m // 2, m - 1), expected):
        assert ens.steps(s) == steps and torch.equal(ens.get_state(s), f), s
