"""The packed kx = 0 / kx = nx/2 plane of the z pass on every way it is run (paired rows inside
the pass, leading blocks of its launch, a launch of its own) against the fp64 oracle: the
iterates, the objective's data term and the Hessian product of the reverse mode, on boxes of
few columns (rows of 2, 4 and 8 packed values, so that the plane is half or more of the
spectrum) and few rows (ky = 0 and ny/2, their own partners, among them)."""
import numpy as np
import pytest
import torch

from oracle import adjoint_ref as A
from oracle import spg_ref as O
from paper_1905_13408_amd import spg

from gpu_util import announce, oracle_problem, rel_l2, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(128, 4, 4), (64, 128, 16), (160, 8, 4), (192, 4, 64), (256, 4, 4), (256, 8, 64),
                                   (256, 128, 16), (512, 4, 4), (512, 8, 32)])
def test_packed_plane_matches_oracle(shape):
    announce(f"packed plane shape={shape}")
    rng = np.random.default_rng([83, *shape])
    w = rng.uniform(0.1, 1.0, size=shape).astype(np.float32)
    b = (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).astype(np.complex64)
    b[..., 0] *= 3.0                    # kx = 0 and kx = nx/2 carry most of the data
    b[..., shape[2] // 2] *= 3.0
    lam, mu, eps, K = 0.02, 0.05, 1e-1, 6
    s = spg.SPGSolver(shape, lam, mu, eps)
    s.set_data(w, b)
    s.set_map(None)
    s.run(K)
    p = oracle_problem(w, b, lam, mu, eps)
    x = to_np(s.get_map())
    assert rel_l2(x, O.spg_solve(p, K)) < 1e-5
    fe, _, _ = s.final_check()
    assert abs(fe - O.objective(x, p)) <= 1e-6 * abs(O.objective(x, p))
    s.set_map(None)
    s.run_checkpointed(K, 4)
    xt = rng.standard_normal(shape)
    lb, mb, bb = s.vjp(w, 2.0 * (s.get_map() - torch.from_numpy(xt.astype(np.float32)).cuda()))
    _, olb, omb, obb = A.loss_and_grad(p, K, xt.astype(np.float32).astype(np.float64))
    # the bounds of the reverse-mode parity tests
    assert abs(lb - olb) <= 1e-3 * abs(olb) and abs(mb - omb) <= 1e-3 * abs(omb)
    assert rel_l2(bb.cpu().numpy().view(np.float32).astype(np.float64), obb.view(np.float64)) < 1e-3
