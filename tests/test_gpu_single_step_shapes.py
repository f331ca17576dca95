"""Single steps at every launch shape: with the passes of two steps off, the
ensembles of the launch-shape tests take every step, odd and even, in the
single-step kernel (256^3 with block 128 is addressed directly, with longer
blocks it exchanges rows over up to 4 waves), and launches on both sides of the
lines from which their waves are held back round alike."""
import pytest
import torch

import mc_inputs

pytestmark = pytest.mark.gpu

mc = pytest.importorskip("paper_2608_23786_amd")


def _states(precision, lattice, shape, graphs):
    ens = mc.Ensemble([mc.Sample(128, 0.0125, 1600.0, 0.3, True, 4), mc.Sample(256, 0.00625, 3200.0, 0.3, True, 1),
                       mc.Sample(16, 0.05, 100.0, 0.2, True, 4)], precision, lattice=lattice)
    ens.init(0, torch.from_numpy(mc_inputs.draw_y(9, 3)))
    ens.two_step(False)
    if shape:
        ens.set_launch(*shape)
    ens.use_graphs(graphs)
    ens.step(9)
    return [ens.get_state(s) for s in range(3)]


@pytest.mark.parametrize("lattice", [27, 19])
@pytest.mark.parametrize("precision", ["f32s", "f64"])
def test_states_do_not_depend_on_the_shape(precision, lattice):
    ref = _states(precision, lattice, (128, 0, 0, 0), False)
    shapes = [(None, True), ((256, 0, 1, 1), True), ((128, 1, 1, 1), False), ((512, 0, 1, 0), False)]
    if precision == "f32s":
        shapes.append(((1024, 0, 1, 1), True))
    for shape, graphs in shapes:
        for s, (a, b) in enumerate(zip(ref, _states(precision, lattice, shape, graphs))):
            assert torch.equal(a, b), (shape, graphs, s)


@pytest.mark.parametrize("lattice", [27, 19])
def test_held_launches_round_as_free_ones(lattice):
    """The same 64^3 sample among 15 (a launch below 2^22 nodes), 16 and 17, and in one 512-thread shape."""
    y = torch.from_numpy(mc_inputs.draw_y(5, 17))
    states = []
    for m, shape in ((15, None), (16, None), (17, None), (16, (512, 0, 1, 1))):
        ens = mc.Ensemble([mc.Sample(64, 0.025, 1600.0, 0.05, True)] * m, "f32s", lattice=lattice)
        ens.two_step(False)
        if shape:
            ens.set_launch(*shape)
        ens.init(0, y[:m])
        rec = ens.step(5, record_every=2)
        states.append((ens.get_state(0), ens.get_state(14), rec[:, :15, 5:7]))
    for other in states[1:]:
        for a, b in zip(states[0], other):
            assert torch.equal(a, b)
