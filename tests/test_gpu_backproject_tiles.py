"""Backprojection by volume tiles at the edges of its range, against the fp64 oracle: both tile
sizes, boxes that are no multiple of a tile, images wider than the box (several periodic
copies of a tile), fewer pixels than the fast rounding needs, narrow and wide kernels,
matrices that are no rotations (the atomic path, also beside rotations), and pixels that are
not numbers.  The sums are integers, so a permuted stack has to give the same bits."""
import numpy as np
import pytest
import torch

from oracle import backproject_ref as BR
from paper_1905_13408_amd import spg

from gpu_util import announce, rel_l2

pytestmark = pytest.mark.gpu


def _inputs(m, n_img, seed):
    rng = np.random.default_rng([73, m, n_img, seed])
    imgs = (rng.standard_normal((n_img, m, m)) + 1j * rng.standard_normal((n_img, m, m))).astype(np.complex64)
    ctf = (rng.uniform(0.1, 1.0, size=(n_img, m, m)) * rng.choice([-1.0, 1.0], size=(n_img, m, m))).astype(np.float32)
    return imgs, BR.random_rotations(n_img, rng), ctf, rng.uniform(0.2, 1.0, size=n_img).astype(np.float32), rng


def _check(shape, imgs, rots, ctf, wts, h, perm=None):
    dev = lambda a: None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    w, b = spg.backproject(shape, dev(imgs), dev(rots), dev(ctf), dev(wts), h=h)
    clean = np.where(np.isfinite(imgs), imgs, 0).astype(np.complex128)
    ow, ob = BR.backproject(shape, clean, rots, None if ctf is None else ctf.astype(np.float64),
                            None if wts is None else wts.astype(np.float64), h=h)
    # float32 outputs of sums held to 2^-35 of the largest term or better
    assert rel_l2(w.cpu().numpy(), ow) < 1e-6
    assert rel_l2(b.cpu().numpy().view(np.float32).astype(np.float64), ob.view(np.float64)) < 1e-5
    assert np.array_equal(w.cpu().numpy() > 0, ow.astype(np.float32) > 0)
    if perm is not None:
        w2, b2 = spg.backproject(shape, dev(imgs[perm]), dev(rots[perm]), dev(ctf[perm]), dev(wts[perm]), h=h)
        assert torch.equal(w2, w) and torch.equal(b2, b)


@pytest.mark.parametrize("shape,m,n_img,h", [
    ((64, 64, 64), 64, 30, 2.0),      # 8^3 tiles
    ((72, 61, 70), 60, 12, 2.0),      # 8^3 tiles, ragged, an odd image
    ((20, 33, 17), 31, 25, 2.0),      # 4^3 tiles, ragged
    ((16, 24, 32), 32, 20, 2.0),      # images twice the shortest axis: copies of each tile
    ((128, 64, 96), 127, 5, 0.7),
    ((32, 32, 32), 8, 2, 2.0),        # 128 pixels: the plain conversion
    ((32, 32, 32), 13, 1, 6.0),
    ((12, 40, 40), 24, 10, 2.0),      # below the tiles' range
    ((16, 16, 16), 33, 4, 2.0),       # beyond twice the box
])
def test_backprojection_tiles_match_oracle(shape, m, n_img, h):
    announce(f"backprojection tiles shape={shape} m={m} n_img={n_img} h={h}")
    imgs, rots, ctf, wts, rng = _inputs(m, n_img, 1)
    _check(shape, imgs, rots, ctf, wts, h, rng.permutation(n_img))
    _check(shape, imgs, rots, None, None, h)


def test_other_matrices_and_non_numbers():
    announce("backprojection: sheared and scaled matrices beside rotations, NaN pixels")
    shape, m, n_img = (32, 40, 32), 32, 16
    imgs, rots, ctf, wts, rng = _inputs(m, n_img, 2)
    rots[3] *= 1.7
    rots[7] = rng.standard_normal((3, 3))
    rots[11, :, 1] = rots[11, :, 0]
    rots[12] = 0.0
    imgs[5, 3, 4] = np.nan + 1j * np.nan
    imgs[7, 0, 1] = np.nan + 1j * np.nan
    _check(shape, imgs, rots, ctf, wts, 2.0, rng.permutation(n_img))
