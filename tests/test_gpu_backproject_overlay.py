"""Backprojection whose outputs overlay its inputs: the outputs are written after the last read of
an input, so that a program may give the image stack's memory for b, or the contrast transfer
functions' for w (the calls that would otherwise run by volume tiles among them), and gets
the results of a call with memory of its own.  The two kernels form K from different
exponentials, an error of 1e-14 in a term; the float32 results differ by one rounding at most."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import backproject_ref as BR
from paper_1905_13408_amd import spg

from gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m,n_img,off", [(16, 16, 16, 0), (32, 32, 40, 0), (64, 64, 70, 4096)])
def test_outputs_over_inputs(n, m, n_img, off):
    announce(f"backprojection outputs over inputs n={n} m={m} n_img={n_img} offset={off}")
    rng = np.random.default_rng([127, n, m, n_img])
    imgs = torch.from_numpy((rng.standard_normal((n_img, m, m, 2))).astype(np.float32)).cuda()
    ctf = torch.from_numpy(rng.uniform(0.1, 1.0, size=(n_img, m, m)).astype(np.float32)).cuda()
    rots = torch.from_numpy(BR.random_rotations(n_img, rng)).cuda()
    L = spg.lib()
    size = ctypes.c_size_t(0)
    assert L.spg_backproject_workspace_size(n, n, n, ctypes.byref(size)) == 0
    ws = torch.empty(size.value, dtype=torch.uint8, device="cuda")
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731

    def call(images, c, w, b):
        assert L.spg_backproject(n, n, n, n_img, m, ptr(images), ptr(rots), ptr(c), None, 2.0, ptr(ws), size,
                                 ctypes.c_void_p(torch.cuda.current_stream().cuda_stream), ptr(w), ptr(b)) == 0
        torch.cuda.synchronize()
        return w.clone(), b.clone()

    nv = n ** 3
    w0, b0 = call(imgs, ctf, torch.empty(nv, device="cuda"), torch.empty(2 * nv, device="cuda"))
    i1 = imgs.clone()
    w1, b1 = call(i1, ctf, torch.empty(nv, device="cuda"), i1.view(-1)[off:off + 2 * nv])
    c2 = ctf.clone()
    w2, b2 = call(imgs, c2, c2.view(-1)[off:off + nv], torch.empty(2 * nv, device="cuda"))
    for w, b in ((w1, b1), (w2, b2)):
        assert float((w - w0).abs().max()) <= 2.0 ** -23 * float(w0.abs().max())
        assert float((b - b0).abs().max()) <= 2.0 ** -23 * float(b0.abs().max())
