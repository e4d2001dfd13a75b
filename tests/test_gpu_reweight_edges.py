"""Reweighting (eq 11) four voxels to a thread: the narrowest rows, whose left neighbours all
wrap, rows that no whole number of threads' groups fills, the widest; every voxel against eq 11
in fp64 on the same float32 map."""
import numpy as np
import pytest
import torch

from oracle import spg_ref as O
from paper_1905_13408_amd import spg, synth

from gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["compensated", "fp32", "bf16"])
@pytest.mark.parametrize("shape", [(4, 4, 4), (8, 4, 16), (4, 32, 160), (16, 8, 192), (8, 4, 512), (64, 160, 32)])
def test_reweight_matches_eq_11(shape, storage):
    announce(f"reweight shape={shape} {storage}")
    rng = np.random.default_rng([107, *shape])
    x = rng.standard_normal(shape).astype(np.float32)
    x[rng.uniform(size=shape) < 0.3] = 0.0
    s = spg.SPGSolver(shape, 0.02, 0.05, 1e-2, storage=storage)
    s.set_data(synth.fourier_weights(shape).astype(np.float32), torch.zeros(shape, dtype=torch.complex64))
    s.set_map(torch.from_numpy(x))
    s.reweight(0.02, 0.05)
    want = O.reweight(x.astype(np.float64), 0.02, 0.05)
    # a float32 map is held exactly, so only the stored weight rounds: half an ulp in float32,
    # and in bf16 storage exactly that float32 rounded once more
    for got, ref in zip(s.get_penalty_weights(), want):
        if storage == "bf16":
            assert torch.equal(got.cpu(), torch.from_numpy(ref.astype(np.float32)).bfloat16().float())
        else:
            got = got.cpu().numpy().astype(np.float64)
            assert np.max(np.abs(got - ref) / ref) <= 2.0**-24 * (1 + 2.0**-6)
