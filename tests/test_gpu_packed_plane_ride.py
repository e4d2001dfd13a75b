"""The packed kx = 0 / kx = nx/2 plane where it rides as leading blocks of the z pass (256 planes
and more tiles than CUs): the iterates, the objective and the Hessian product of the reverse mode
against the fp64 oracle, with 16 and 8 columns per tile, and, where the passes run in four column
ranges of which only the first has the plane, a step against fp64 transforms."""
import numpy as np
import pytest
import torch

from oracle import adjoint_ref as A
from oracle import spg_ref as O
from paper_1905_13408_amd import spg

from gpu_util import announce, oracle_problem, rel_l2, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,nt_z", [((256, 512, 4), 16), ((256, 192, 64), 16), ((256, 192, 64), 8)])
def test_riding_plane_matches_oracle(shape, nt_z):
    announce(f"riding packed plane shape={shape} columns={nt_z}")
    rng = np.random.default_rng([149, *shape])
    w = rng.uniform(0.1, 1.0, size=shape).astype(np.float32)
    b = (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).astype(np.complex64)
    b[..., 0] *= 3.0                    # kx = 0 and kx = nx/2 carry most of the data
    b[..., shape[2] // 2] *= 3.0
    lam, mu, eps, K = 0.02, 0.05, 1e-1, 6
    s = spg.SPGSolver(shape, lam, mu, eps)
    s.set_launch_shape(16, nt_z, 32)
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
    xt = rng.standard_normal(shape).astype(np.float32)
    lb, mb, bb = s.vjp(w, 2.0 * (s.get_map() - torch.from_numpy(xt).cuda()))
    _, olb, omb, obb = A.loss_and_grad(p, K, xt.astype(np.float64))
    # the bounds of the reverse-mode parity tests
    assert abs(lb - olb) <= 1e-3 * abs(olb) and abs(mb - omb) <= 1e-3 * abs(omb)
    assert rel_l2(bb.cpu().numpy().view(np.float32).astype(np.float64), obb.view(np.float64)) < 1e-3


def test_riding_plane_with_column_ranges():
    shape = (256, 512, 512)
    announce(f"riding packed plane with column ranges {shape}")
    gen = torch.Generator(device="cuda").manual_seed(151)
    w = torch.rand(shape, device="cuda", generator=gen) + 0.1
    b = torch.view_as_complex(torch.randn(*shape, 2, device="cuda", generator=gen) * 0.3)
    b[..., 0] *= 8.0
    b[..., 256] *= 8.0
    x0 = torch.randn(shape, device="cuda", generator=gen) * 0.1
    lam = mu = 1e-9                     # leaves the data term's gradient step
    s = spg.SPGSolver(shape, lam, mu, 1e-2)
    s.set_data(w, b)
    s.set_map(x0)
    lr = s.run(1).lr
    step = (s.get_map() - x0).double()
    grad = torch.fft.ifftn(w.double() * (torch.fft.fftn(x0.double(), norm="ortho") - b.to(torch.complex128)),
                           norm="ortho").real
    # float32 transforms of 2^26 points: 1e-6 of the gradient, as in the parity tests
    assert float((step + lr * grad).norm() / (lr * grad).norm()) < 1e-5
    del grad, step
    s.run(4)
    x = s.get_map()
    for nt_y, nt_z in ((16, 8), (8, 16)):
        t = spg.SPGSolver(shape, lam, mu, 1e-2)
        t.set_launch_shape(nt_y, nt_z, 32)
        t.set_data(w, b)
        t.set_map(x0)
        t.run(5)
        assert torch.equal(t.get_map(), x)
        del t
