"""Backprojection by volume tiles with so many images that every tile fills its pixel queue many
times over and all its waves meet the limit at once: against the fp64 oracle, and the same
bits from every run and every order of the images."""
import numpy as np
import pytest
import torch

from oracle import backproject_ref as BR
from paper_1905_13408_amd import spg

from gpu_util import announce, rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,m,n_img", [((16, 24, 32), 32, 500), ((64, 64, 72), 48, 400), ((16, 16, 16), 5, 9000)])
def test_full_queues_match_oracle(shape, m, n_img):
    announce(f"backprojection queues shape={shape} m={m} n_img={n_img}")
    rng = np.random.default_rng([113, m, n_img])
    imgs = (rng.standard_normal((n_img, m, m)) + 1j * rng.standard_normal((n_img, m, m))).astype(np.complex64)
    rots = BR.random_rotations(n_img, rng)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    w, b = spg.backproject(shape, dev(imgs), dev(rots))
    ow, ob = BR.backproject(shape, imgs.astype(np.complex128), rots)
    # the bounds of the other tests of the tiles
    assert rel_l2(w.cpu().numpy(), ow) < 1e-6
    assert rel_l2(b.cpu().numpy().view(np.float32).astype(np.float64), ob.view(np.float64)) < 1e-5
    for _ in range(4):
        perm = rng.permutation(n_img)
        w2, b2 = spg.backproject(shape, dev(imgs[perm]), dev(rots[perm]))
        assert torch.equal(w2, w) and torch.equal(b2, b)
