"""FSC curves with more shells than the box has frequencies: the same values as the curve of the
occupied shells, against the fp64 oracle, and zeros past the corner frequency."""
import numpy as np
import pytest
import torch

from oracle import fsc_ref as F
from paper_1905_13408_amd import spg

from gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(4, 4, 4), (64, 128, 4), (8, 32, 16), (160, 16, 64), (192, 192, 192)])
@pytest.mark.parametrize("nshells", [1, 1024])
def test_shells_past_the_corner(shape, nshells):
    announce(f"fsc shells shape={shape} nshells={nshells}")
    rng = np.random.default_rng([139, *shape])
    a = rng.standard_normal(shape).astype(np.float32)
    b = (0.6 * a + 0.8 * rng.standard_normal(shape)).astype(np.float32)
    got = np.asarray(spg.fsc(torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda(), nshells))
    want = F.fsc(a.astype(np.float64), b.astype(np.float64), nshells)
    assert got.shape == (nshells,)
    # the bound of the FSC parity test
    assert np.max(np.abs(got - want)) < 1e-5
    corner = int(np.floor(0.5 * min(shape) * np.sqrt(3.0) + 0.5))
    assert np.all(got[corner + 1:] == 0.0)
    if nshells > corner:
        assert got[0] != 0.0 and abs(got[corner] - want[corner]) < 1e-5
