"""A sample's populations do not depend on how its steps are cut into calls,
records and passes of two, or on the ensemble it is part of: bit for bit, in
both precisions and on both lattices, against the same steps taken one by one."""
import pytest
import torch

import mc_inputs

pytestmark = pytest.mark.gpu

mc = pytest.importorskip("paper_2608_23786_amd")

STEPS = 21


def _ensemble(n, m, precision, lattice, two=True):
    u0 = mc_inputs.diffusive_u0(n) if n >= 32 else 0.05
    ens = mc.Ensemble([mc.Sample(n, u0, 25.0 * n, 0.05, True)] * m, precision, lattice=lattice)
    ens.two_step(two)
    ens.init(0, torch.from_numpy(mc_inputs.draw_y(5, m)))
    return ens


def _at_once(ens):
    ens.step(STEPS)


def _in_calls(ens):
    for ticks in (1, 9, 3, 8):
        ens.step(ticks)


def _with_records(ens):
    ens.step(STEPS, record_every=10)


def _timed(ens):
    ens.time_launches(True)
    ens.step(STEPS)
    ens.time_launches(False)


def _resumed(ens):
    ens.step(10)
    saved = ens.checkpoint()
    ens.step(4)
    ens.restore(saved)
    ens.step(STEPS - 10)


# every tile of the passes: whole planes, bands of rows, rows with rim columns, several trips through
# the scratch with a shorter last one (77 x 64^3 in FP32: 39 and 38 samples)
@pytest.mark.parametrize("n,m,precision,lattice", [
    (n, m, p, q) for p in ("f32s", "f64") for q in (27, 19)
    for n, m in ((8, 2051), (16, 259), (32, 33), (64, 5), (128, 2), (256, 1))] + [(64, 77, "f32s", 27)])
def test_states_do_not_depend_on_the_cut(n, m, precision, lattice):
    single = _ensemble(n, m, precision, lattice, two=False)
    for _ in range(STEPS):
        single.step(1)
    samples = sorted({0, m // 2, m - 1})
    expected = [single.get_state(s) for s in samples]
    for cut in (_at_once, _in_calls, _with_records, _timed, _resumed):
        ens = _ensemble(n, m, precision, lattice)
        cut(ens)
        for s, f in zip(samples, expected):
            assert torch.equal(ens.get_state(s), f), (cut.__name__, s)


@pytest.mark.parametrize("precision", ["f32s", "f64"])
def test_states_do_not_depend_on_the_ensemble(precision):
    """One 64^3 sample by itself, which takes single steps, and the same one among five, which take passes."""
    y = torch.from_numpy(mc_inputs.draw_y(5, 5))
    states = []
    for m in (1, 5):
        ens = mc.Ensemble([mc.Sample(64, 0.025, 1600.0, 0.05, True)] * m, precision)
        ens.init(0, y[:m])
        ens.step(STEPS)
        states.append(ens.get_state(0))
    assert torch.equal(*states)
