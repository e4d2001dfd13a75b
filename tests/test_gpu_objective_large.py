"""The objective's data term (final check, monitor) on grids whose objective z pass has the packed
kx = 0 / nx/2 plane in a launch of its own, and on the next smaller ones, against fp64
transforms; monitored iterates are those of an unmonitored run."""
import numpy as np
import pytest
import torch

from paper_1905_13408_amd import spg

from gpu_util import announce

pytestmark = pytest.mark.gpu


def _data_term(x, w, b):
    """1/2 sum w |A x - b|^2 with the unitary transform, in fp64."""
    n = float(np.prod(x.shape))
    y = torch.fft.fftn(x.double()) / np.sqrt(n)
    return float(0.5 * (w.double() * (y - b.to(torch.complex128)).abs() ** 2).sum())


# tiles of 16 columns: 1280 and 1536 at 256 planes, 1024 and 1152 at 160, 2048 and 4096 at 128; 192 planes
@pytest.mark.parametrize("shape", [(256, 160, 256), (256, 192, 256), (160, 128, 256), (160, 192, 192), (128, 256, 256),
                                   (128, 256, 512), (192, 256, 256), (256, 512, 128)])
@pytest.mark.parametrize("storage", ["compensated", "bf16"])
def test_large_objective_passes(shape, storage):
    announce(f"large objective passes {shape} {storage}")
    gen = torch.Generator(device="cuda").manual_seed(137)
    w = torch.rand(shape, device="cuda", generator=gen) + 0.1
    b = torch.view_as_complex(torch.randn(*shape, 2, device="cuda", generator=gen) * 0.3)
    b[..., 0] *= 8.0                  # kx = 0 and kx = nx/2 carry a good part of the term
    b[..., shape[2] // 2] *= 8.0
    x0 = torch.randn(shape, device="cuda", generator=gen) * 0.1
    lam, mu = 1e-9, 1e-9              # leaves the data term
    s = spg.SPGSolver(shape, lam, mu, 1e-2, storage=storage)
    s.set_data(w, b)
    s.set_map(x0)
    s.run(5)
    x = s.get_map()
    fe, _, _ = s.final_check()
    want = _data_term(x, w, b)
    # float32 transforms: 1e-6 relative in the spectrum, and the penalties' 1e-9 sums
    assert abs(fe - want) <= 2e-6 * want
    m = spg.SPGSolver(shape, lam, mu, 1e-2, storage=storage, monitor_every=2)
    m.set_data(w, b)
    m.set_map(x0)
    m.run(5)
    assert torch.equal(m.get_map(), x)
    m.set_map(x0)
    m.run(2)                          # F_eps at y_2 = x_1 (no momentum yet at the second iteration)
    s.set_map(x0)
    s.run(1)
    x1 = s.get_map()
    if storage == "bf16" and not s.fusion:   # the separate sweeps read the rounded map buffer
        x1 = x1.bfloat16().float()
    assert abs(m.objective_history()[1][-1] - _data_term(x1, w, b)) <= 2e-6 * want
