"""Maps of a width that the fused x transforms do not support (160, 192, 16) run the separate x
sweeps, in every call: the iterations give the bits of the recorded forward of the reverse mode,
which always runs them, and those of a tuned solver, whatever the tuner timed; the fusion
switch reports what runs."""
import numpy as np
import pytest
import torch

from paper_1905_13408_amd import spg, synth

from gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["compensated", "fp32"])
@pytest.mark.parametrize("shape", [(32, 16, 160), (8, 160, 160), (16, 8, 192), (16, 16, 16)])
def test_unsupported_widths_have_one_path(shape, storage):
    announce(f"one path shape={shape} {storage}")
    rng = np.random.default_rng([107, *shape])
    w = synth.fourier_weights(shape).astype(np.float32)
    b = (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).astype(np.complex64) * 0.3
    u, v = (rng.uniform(0.5, 2.0, size=shape).astype(np.float32) for _ in range(2))
    K = 12

    def solver():
        s = spg.SPGSolver(shape, 0.02, 0.05, 1e-2, storage=storage)
        s.set_data(w, b)
        s.set_penalty_weights(u, v)
        s.set_map(None)
        return s

    s = solver()
    s.run(K)
    x = s.get_map()
    r = solver()
    r.run_checkpointed(K, 5)
    assert torch.equal(r.get_map(), x)
    g = solver()
    g.autotune(2)
    g.run(K)
    h = solver()
    h.set_fusion(g.fusion)
    h.run(K)
    assert torch.equal(g.get_map(), x) and torch.equal(h.get_map(), x)
    # the recorded launches of an iteration: the sweeps show whether the reported path ran
    h.profile_begin(None, 64)
    h.run(2)
    prof = h.profile_end()
    assert not h.fusion and prof["c2r_x"][1] == 2
