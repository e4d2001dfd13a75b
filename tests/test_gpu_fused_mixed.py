"""The fused stencil kernel on 160-wide maps, whose row transforms are mixed radix:
against the oracle, and against the separate x sweeps that the recorded forward of the reverse
mode runs (the same operations, to rounding), with slabs that do not divide the depth, a
single tile of four rows, explicit weights and the prior map; launch shapes give the same
bits.  The fusion switch has no say on this width."""
import numpy as np
import pytest
import torch

from oracle import spg_ref as O
from paper_1905_13408_amd import spg, synth

from gpu_util import announce, oracle_problem, rel_l2, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["compensated", "fp32"])
@pytest.mark.parametrize("shape,zc,gamma", [((8, 4, 160), 5, 0.0), ((32, 8, 160), 7, 0.3), ((16, 160, 160), 16, 0.3),
                                            ((64, 32, 160), 64, 0.0)])
def test_mixed_widths_match_oracle_and_separate_sweeps(shape, zc, gamma, storage):
    announce(f"fused mixed widths shape={shape} zc={zc} gamma={gamma} {storage}")
    rng = np.random.default_rng([91, *shape])
    w = synth.fourier_weights(shape).astype(np.float32)
    b = (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).astype(np.complex64) * 0.3
    u, v = (rng.uniform(0.5, 2.0, size=shape).astype(np.float32) for _ in range(2))
    x0, xp = (rng.standard_normal(shape).astype(np.float32) * 0.1 for _ in range(2))
    K = 15

    def solver(z):
        s = spg.SPGSolver(shape, 0.02, 0.05, 1e-2, storage=storage)
        if z:
            s.set_launch_shape(16, 16, z)
        assert not s.fusion
        with pytest.raises(RuntimeError):
            s.set_fusion(True)
        s.set_fusion(False)
        s.set_data(w, b)
        s.set_penalty_weights(u, v)
        if gamma:
            s.set_prior(gamma, xp)
        s.set_map(x0)
        return s

    s = solver(zc)
    s.run(K)
    x = s.get_map()
    p = oracle_problem(w, b, 0.02, 0.05, 1e-2, u=u, v=v)
    if gamma:
        p.gamma, p.x_prev = gamma, xp.astype(np.float64)
    assert rel_l2(to_np(x), O.spg_solve(p, K, x0=x0.astype(np.float64))) < 1e-5
    t = solver(zc)
    t.run_checkpointed(K, K)
    assert rel_l2(to_np(x), to_np(t.get_map())) < 1e-6
    for z in (32, None):
        r = solver(z)
        r.run(K)
        assert torch.equal(r.get_map(), x)
