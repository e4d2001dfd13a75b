"""The reverse mode at the edges of its kernels against the fp64 reference gradient: rows that
are no multiple of a 64-column tile, boxes lower than a tile's 8 rows, depths that leave a
short slab, explicit weights, and more steps than are held between two reads of their sums."""
import numpy as np
import pytest
import torch

from oracle import adjoint_ref as A
from paper_1905_13408_amd import spg, synth

from gpu_util import announce, oracle_problem, rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,K,C,weighted", [((8, 4, 160), 5, 2, True),
                                                ((64, 8, 192), 4, 3, True), ((8, 8, 16), 165, 40, False)])
def test_reverse_edges_match_reference(shape, K, C, weighted):
    announce(f"reverse mode edges shape={shape} K={K} C={C}")
    rng = np.random.default_rng([97, K, *shape])
    w = synth.fourier_weights(shape).astype(np.float32)
    b = ((rng.standard_normal(shape) + 1j * rng.standard_normal(shape)) * 0.5).astype(np.complex64)
    u, v = ((rng.uniform(0.5, 2.0, size=shape).astype(np.float32) for _ in range(2)) if weighted else (None, None))
    xt = rng.standard_normal(shape).astype(np.float32)
    lam, mu, eps = 0.01, 0.05, 1e-1
    s = spg.SPGSolver(shape, lam, mu, eps)
    s.set_data(w, b)
    if weighted:
        s.set_penalty_weights(u, v)
    s.set_map(None)
    s.run_checkpointed(K, C)
    lb, mb, bb = s.vjp(w, 2.0 * (s.get_map() - torch.from_numpy(xt).cuda()))
    p = oracle_problem(w, b, lam, mu, eps, u=u, v=v)
    _, olb, omb, obb = A.loss_and_grad(p, K, xt.astype(np.float64))
    # the bounds of the reverse-mode parity tests
    assert abs(lb - olb) <= 1e-3 * abs(olb) and abs(mb - omb) <= 1e-3 * abs(omb)
    assert rel_l2(bb.cpu().numpy().view(np.float32).astype(np.float64), obb.view(np.float64)) < 1e-3
