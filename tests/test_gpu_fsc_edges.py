"""Shell sums at the edges of their work split: rows shorter than a wave, a last piece of 16
or 32 columns, axes whose +k and -k coincide, more shells than the spectrum has, and shell
counts that leave 8, 4 and 2 waves per block."""
import numpy as np
import pytest
import torch

from oracle import fsc_ref as FR
from paper_1905_13408_amd import spg

from gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,nsh", [((4, 4, 4), 3), ((8, 32, 8), 5), ((16, 192, 160), 9), ((32, 8, 512), 200),
                                       ((64, 16, 192), 600), ((4, 128, 128), 1024)])
def test_fsc_edges_match_oracle(shape, nsh):
    announce(f"FSC edges shape={shape} nshells={nsh}")
    rng = np.random.default_rng([37, nsh, *shape])
    x = rng.standard_normal(shape)
    a = (x + 0.5 * rng.standard_normal(shape)).astype(np.float32)
    b = (x + 0.5 * rng.standard_normal(shape)).astype(np.float32)
    ta, tb = torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()
    got = spg.fsc(ta, tb, nsh)
    ref = FR.fsc(a.astype(np.float64), b.astype(np.float64), nsh)
    # fp32 transforms: an error of about 1e-6 of each shell's root power, as in the parity tests
    assert np.max(np.abs(got - ref)) < 1e-5
    assert np.array_equal(got, spg.fsc(ta, tb, nsh))
