"""Passes that take two steps (mclbm_set_step_scratch) against single steps, in
FP64 bit for bit, in FP32 to the rounding of both: every tile shape (whole
planes, bands of rows with a rim, 64-node tiles with rim columns, 64-bit
addresses), both lattices and precisions, odd starts and remainders of the step
count, records, mixed strides, the checkpointed forward run (which stays with
single steps), and the instability flags."""
import pytest
import torch

import mc_inputs

pytestmark = pytest.mark.gpu

mc = pytest.importorskip("paper_2608_23786_amd")


def _ensemble(n, m, precision, lattice, two):
    u0 = mc_inputs.diffusive_u0(n) if n >= 32 else 0.05
    ens = mc.Ensemble([mc.Sample(n, u0, 25.0 * n, 0.05, True)] * m, precision, lattice=lattice)
    # 32^3 of D3Q27 in FP64 keeps single steps
    assert ens.two_step(two) == (two and (n, precision, lattice) != (32, "f64", 27))
    ens.init(5)
    return ens


# FP32: either path's step is within 2e-6 of max |f - w| of the exact one (the
# bound of the single-step tests), so after k steps the two are within 4e-6 k.
FP32_STEP = 4e-6


def _same_state(a, b, samples):
    for s in samples:
        fa, fb = a.get_state(s), b.get_state(s)
        if a.precision == "f64":
            assert torch.equal(fa, fb), s
        else:
            scale = float((fb - fb.mean(dim=(1, 2, 3), keepdim=True)).abs().max())
            assert float((fa - fb).abs().max()) <= FP32_STEP * b.steps(s) * scale, s


def _same_records(ra, rb, steps):
    """Records [..., 8] of FP32 runs: mass and momentum per node, kinetic energy and gamma."""
    assert ra.shape == rb.shape
    assert torch.allclose(ra[..., 0], rb[..., 0], rtol=FP32_STEP * steps, atol=0.0)
    assert torch.allclose(ra[..., 4], rb[..., 4], rtol=FP32_STEP * steps, atol=0.0)
    assert torch.allclose(ra[..., 7], rb[..., 7], rtol=1e-3, atol=0.0)


# one run of each resolution at the smallest ensemble that takes two-step passes
@pytest.mark.parametrize("lattice", [27, 19])
@pytest.mark.parametrize("precision", ["f32s", "f64"])
@pytest.mark.parametrize("n,m", [(8, 2051), (16, 259), (32, 33), (64, 5), (128, 2), (256, 1)])
def test_states_equal_single_steps(n, m, precision, lattice):
    a, b = (_ensemble(n, m, precision, lattice, two) for two in (True, False))
    last = sorted({0, m // 2, m - 1})
    for ticks in (1, 5, 5, 10):     # starts at odd and even parity, with and without remainder, one and two trips
        a.step(ticks)
        b.step(ticks)
        _same_state(a, b, last)
    assert a.steps(m - 1) == b.steps(m - 1) == 21 and a.ticks == b.ticks == 21


def test_512_takes_64_bit_addresses():
    states = []
    for two in (True, False):
        a = _ensemble(512, 1, "f32s", 27, two)
        a.step(5)
        g = torch.Generator(device="cpu").manual_seed(3)
        cells = torch.cat([torch.randint(0, 512 ** 3, (4096,), generator=g), torch.tensor([0, 512 ** 3 - 1])])
        states.append((a.get_cells(0, cells), a.reduce()))
        del a
        torch.cuda.empty_cache()
    (fa, ra), (fb, rb) = states
    scale = float((fb - fb.mean(dim=0)).abs().max())
    assert float((fa - fb).abs().max()) <= FP32_STEP * 5 * scale
    _same_records(ra, rb, 5)


def test_records_between_passes():
    a, b = (_ensemble(64, 7, "f32s", 27, two) for two in (True, False))
    ra, rb = a.step(23, record_every=10), b.step(23, record_every=10)
    _same_records(ra, rb, 23)
    _same_state(a, b, [0, 6])


def test_mixed_strides():
    def ens(two):
        e = mc.Ensemble([mc.Sample(32, 0.05, 800.0, 0.05, True, 16)] * 3 + [mc.Sample(64, 0.025, 1600.0, 0.05, True, 4)] * 5
                        + [mc.Sample(128, 0.0125, 3200.0, 0.05, True, 1)], "f32s")
        assert e.two_step(two) == two
        e.init(9)
        return e

    a, b = ens(True), ens(False)
    for ticks, every in ((48, 16), (21, 0), (11, 0)):
        ra, rb = a.step(ticks, record_every=every), b.step(ticks, record_every=every)
        if every:
            _same_records(ra, rb, a.ticks)
        assert [a.steps(s) for s in range(a.m)] == [b.steps(s) for s in range(b.m)]
        _same_state(a, b, range(a.m))


def test_checkpointed_forward_keeps_single_steps():
    grads = []
    for two in (True, False):
        e = _ensemble(64, 4, "f32s", 27, two)
        y = torch.from_numpy(mc_inputs.draw_y(3, 4)).cuda().requires_grad_()
        j = mc.EnsembleKE.apply(y, e, 13, 6)
        grads.append((j.detach(), torch.autograd.grad(j, y)[0]))
    assert torch.equal(grads[0][0], grads[1][0]) and torch.equal(grads[0][1], grads[1][1])


def test_instability_is_flagged():
    a = _ensemble(64, 6, "f32s", 27, True)
    a.step(2)
    a.poison(4, 12345, 7)
    a.step(5)
    assert a.check() == 4


def test_scratch_arguments():
    a = _ensemble(64, 5, "f32s", 27, True)
    nb = int(mc.lib().mclbm_step_scratch_bytes(a._ctx))
    assert nb >= 5 * 27 * 64 ** 3 * 4
    import ctypes

    from paper_2608_23786_amd import _lib
    assert mc.lib().mclbm_set_step_scratch(a._ctx, ctypes.c_void_p(256), nb - 1) == _lib.ERR_OOM
    assert mc.lib().mclbm_set_step_scratch(a._ctx, ctypes.c_void_p(100), nb) == _lib.ERR_ARG
    small = mc.Ensemble([mc.Sample(16, 0.05, 100.0)], "f64")
    assert int(mc.lib().mclbm_step_scratch_bytes(small._ctx)) == 0 and not small.two_step(True)
