"""Members of a batch graph that share the GPU agree bitwise with their own eager runs on the
separate x-sweep path, run after run: concurrent branches shift the waves of a block against
each other, which a missing barrier in the stencil kernel would show."""
import numpy as np
import pytest
import torch

from paper_1905_13408_amd import spg, synth

from gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shapes", [[(160, 160, 128), (192, 192, 192), (256, 160, 16), (128, 128, 128)]])
def test_separate_path_members_equal_eager_runs(shapes):
    solvers, refs = [], []
    for i, shape in enumerate(shapes):
        rng = np.random.default_rng([5, i, *shape])
        w = torch.from_numpy(synth.fourier_weights(shape).astype(np.float32)).cuda()
        b = torch.from_numpy((rng.standard_normal((*shape, 2), dtype=np.float32) * 0.3).view(np.complex64)[..., 0]).cuda()
        for lst in (solvers, refs):
            s = spg.SPGSolver(shape, 0.01, 0.05, 1e-3)
            s.set_fusion(False)
            s.set_data(w, b)
            lst.append(s)
    announce(f"batch of separate-path members {shapes} against eager runs")
    batch = spg.SPGBatch(solvers)
    for r in refs:
        r.set_map(None)
        r.run(10)
    for _ in range(3):
        for s in solvers:
            s.set_map(None)
        batch.run(10)
        for s, r in zip(solvers, refs):
            assert torch.equal(s.get_map(), r.get_map())
    batch.close()
