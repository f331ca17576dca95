"""Memory that an ensemble takes from the caching allocator may still be in use
by work queued on the caller's stream: the library's first write waits for it."""
import pytest
import torch

import mc_inputs

pytestmark = pytest.mark.gpu

mc = pytest.importorskip("paper_2608_23786_amd")

BUSY_CYCLES = 20_000_000   # some ten milliseconds


def _queue_copy(bytes_):
    """A copy queued behind a wait on the current stream, of a tensor that is freed at once: (its address, the copy)."""
    held = torch.full((bytes_,), 7, dtype=torch.uint8, device="cuda")
    torch.cuda._sleep(BUSY_CYCLES)
    copy = held.clone()
    return held.data_ptr(), copy


def _overlaps(address, bytes_, tensor):
    return address < tensor.data_ptr() + tensor.numel() and tensor.data_ptr() < address + bytes_


@pytest.mark.parametrize("side", [False, True])
def test_scratch_waits_for_the_caller(side):
    samples = [mc.Sample(64, 0.025, 1600.0, 0.05, True)] * 5
    with torch.cuda.stream(torch.cuda.Stream() if side else torch.cuda.current_stream()):
        ens = mc.Ensemble(samples, "f32s")
        ens.init(0, torch.from_numpy(mc_inputs.draw_y(5, 5)))
        ens.step(1)
        assert not ens.two_step(False)
        ens.synchronize()
        torch.cuda.empty_cache()
        bytes_ = int(mc.lib().mclbm_step_scratch_bytes(ens._ctx)) + 256
        address, copy = _queue_copy(bytes_)
        assert ens.two_step(True)
        assert _overlaps(address, bytes_, ens._scratch)
        ens.step(8)
        ens.synchronize()
        torch.cuda.synchronize()
        assert int(copy.min()) == 7 and int(copy.max()) == 7


@pytest.mark.parametrize("side", [False, True])
def test_workspace_waits_for_the_caller(side):
    samples = [mc.Sample(64, 0.025, 1600.0, 0.05, True)]
    with torch.cuda.stream(torch.cuda.Stream() if side else torch.cuda.current_stream()):
        bytes_ = mc.Ensemble(samples, "f32s").workspace.numel()
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        address, copy = _queue_copy(bytes_)
        ens = mc.Ensemble(samples, "f32s")
        assert _overlaps(address, bytes_, ens.workspace)
        ens.init(3)
        ens.step(2)
        torch.cuda.synchronize()
        assert int(copy.min()) == 7 and int(copy.max()) == 7
