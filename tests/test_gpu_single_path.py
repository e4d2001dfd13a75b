"""Maps of a width that the fusion switch does not offer (160, 192, 16) have one set of bits:
whichever way the library runs the x transforms there (160 columns inside the stencil kernel,
unless the switch or the tuner turns that off), the iterations give the bits of the separate
sweeps that the recorded forward of the reverse mode runs, in every instance of the kernel."""
import numpy as np
import pytest
import torch

from oracle import spg_ref as O
from paper_1905_13408_amd import spg, synth

from gpu_util import announce, oracle_problem, rel_l2, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["compensated", "fp32"])
@pytest.mark.parametrize("shape,gamma,weights,accel", [
    ((32, 16, 160), 0.0, True, True), ((8, 160, 160), 0.3, True, True), ((64, 4, 160), 0.3, False, True),
    ((192, 32, 160), 0.0, False, False), ((512, 512, 160), 0.0, True, True), ((16, 8, 192), 0.3, True, True),
    ((16, 16, 16), 0.0, True, True)])
def test_widths_without_a_choice_have_one_set_of_bits(shape, gamma, weights, accel, storage):
    announce(f"one set of bits shape={shape} gamma={gamma} weights={weights} accel={accel} {storage}")
    big = np.prod(shape) > 1 << 24
    gen = torch.Generator(device="cuda").manual_seed(107)
    w = torch.rand(shape, device="cuda", generator=gen) + 0.1
    b = torch.view_as_complex(torch.randn(*shape, 2, device="cuda", generator=gen) * 0.3)
    u, v = (torch.rand(shape, device="cuda", generator=gen) * 1.5 + 0.5 for _ in range(2))
    x0, xp = (torch.randn(shape, device="cuda", generator=gen) * 0.1 for _ in range(2))
    K = 4 if big else 12

    def solver(**kw):
        s = spg.SPGSolver(shape, 0.02, 0.05, 1e-2, storage=storage, accel=accel, **kw)
        s.set_data(w, b)
        if weights:
            s.set_penalty_weights(u, v)
        if gamma:
            s.set_prior(gamma, xp)
        s.set_map(x0)
        return s

    r = solver()
    r.run_checkpointed(K, K if big else 5)
    x = r.get_map()
    s = solver()
    s.run(K)
    assert torch.equal(s.get_map(), x)
    off = solver()
    off.set_fusion(False)
    off.run(K)
    assert torch.equal(off.get_map(), x)
    # monitored, where the z pass has another instance (on 512 planes with another rounding)
    mon, rec = solver(monitor_every=3), solver(monitor_every=3)
    mon.run(K)
    rec.run_checkpointed(K, K if big else 5)
    assert torch.equal(mon.get_map(), rec.get_map())
    if big:
        return
    # a tuned solver, and one set to what the tuned one reports
    g = solver()
    g.autotune(2)
    g.set_map(x0)
    g.run(K)
    h = solver()
    h.set_fusion(g.fusion)
    h.run(K)
    assert torch.equal(g.get_map(), x) and torch.equal(h.get_map(), x)
    # the switch turned off: the separate sweeps run, an inverse and a forward one per iteration
    off.profile_begin(None, 64)
    off.run(2)
    prof = off.profile_end()
    assert not off.fusion and prof["c2r_x"][1] == 2 and prof["r2c_x"][1] == 2


@pytest.mark.parametrize("storage", ["compensated", "fp32"])
def test_160_columns_match_the_oracle(storage):
    shape, K = (16, 16, 160), 15
    announce(f"160 columns against the oracle {storage}")
    rng = np.random.default_rng([109, *shape])
    w = synth.fourier_weights(shape).astype(np.float32)
    b = (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).astype(np.complex64) * 0.3
    s = spg.SPGSolver(shape, 0.02, 0.05, 1e-2, storage=storage)
    s.set_data(w, b)
    s.set_map(None)
    s.run(K)
    assert rel_l2(to_np(s.get_map()), O.spg_solve(oracle_problem(w, b, 0.02, 0.05, 1e-2), K)) < 1e-5
