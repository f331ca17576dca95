"""The scratch buffer of the two-step passes: taken by the first step that can
use it and by nothing else, only out of plenty, and given back to a later call
of the ensemble that runs out of memory."""
import pytest
import torch

import mc_inputs

pytestmark = pytest.mark.gpu

mc = pytest.importorskip("paper_2608_23786_amd")

SAMPLE = mc.Sample(64, 0.025, 1600.0, 0.05, True)


def _ensemble(samples=None, precision="f32s"):
    ens = mc.Ensemble(samples or [SAMPLE] * 5, precision)
    ens.init(0, torch.from_numpy(mc_inputs.draw_y(5, ens.m)))
    return ens


def test_taken_by_the_first_step_that_can_use_it():
    ens = _ensemble()
    need = int(mc.lib().mclbm_step_scratch_bytes(ens._ctx))
    ens.step(3)                       # no pass fits
    ens.step(9, record_every=4)       # nor between these records
    ens.reduce(), ens.point_values(8)
    assert ens._scratch is None
    ens.step(5)
    assert ens._scratch is not None and ens._scratch.numel() >= need
    held = ens._scratch
    ens.step(50, record_every=10)
    assert ens._scratch is held


def test_not_taken_by_what_cannot_use_it():
    exact = _ensemble()
    exact.set_stabiliser("exact")
    exact.step(8)
    assert exact._scratch is None
    gradient = _ensemble()
    y = torch.from_numpy(mc_inputs.draw_y(3, 5)).cuda().requires_grad_()
    mc.EnsembleKE.apply(y, gradient, 10, 5).backward()
    assert gradient._scratch is None
    strided = _ensemble([mc.Sample(64, 0.025, 1600.0, 0.05, True, 4)] * 5)
    strided.step(12)
    assert strided._scratch is None
    off = _ensemble()
    assert not off.two_step(False)
    off.step(20)
    assert off._scratch is None


@pytest.mark.parametrize("times,taken", [(3.9, False), (4.1, True)])
def test_taken_out_of_plenty(monkeypatch, times, taken):
    torch.cuda.empty_cache()
    ens = _ensemble()
    need = int(mc.lib().mclbm_step_scratch_bytes(ens._ctx))
    idle = torch.cuda.memory_reserved() - torch.cuda.memory_allocated()
    monkeypatch.setattr(torch.cuda, "mem_get_info", lambda device=None: (int(times * need) - idle, 1 << 40))
    ens.step(8)
    assert (ens._scratch is not None) == taken


def test_given_back_when_memory_runs_out():
    ens, plain = _ensemble(), _ensemble()
    plain.two_step(False)
    ens.step(8)
    plain.step(8)
    expected = plain.get_state(4)
    del plain
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(0).total_memory
    torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + (32 << 20)) / total)
    try:
        saved = ens.checkpoint()      # five samples' populations, as the scratch holds
        assert ens._scratch is None
        ens.step(8)                   # single steps from here on
        assert ens._scratch is None
        ens.restore(saved)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert torch.equal(ens.get_state(4), expected)
