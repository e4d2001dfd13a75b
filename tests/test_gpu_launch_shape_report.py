"""The launch shape that a solver reports is the one that runs: set on another solver it gives
the same launches, which the monitored objective shows (an fp64 sum of one partial per block, so
that another slab depth sums it in another order), for the depths that the path picks itself
as for tuned ones, on both x-transform paths."""
import numpy as np
import pytest
import torch

from paper_1905_13408_amd import spg

from gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(64, 64, 64), (128, 128, 128), (32, 128, 256), (192, 64, 32), (64, 192, 192), (16, 32, 512),
                                   (128, 64, 16)])
@pytest.mark.parametrize("fused", [True, False])
def test_reported_shape_gives_the_same_launches(shape, fused):
    announce(f"reported launch shape {shape} fused={fused}")
    gen = torch.Generator(device="cuda").manual_seed(131)
    w = torch.rand(shape, device="cuda", generator=gen) + 0.1
    b = torch.view_as_complex(torch.randn(*shape, 2, device="cuda", generator=gen) * 0.3)

    def solver():
        s = spg.SPGSolver(shape, 0.02, 0.05, 1e-2, monitor_every=1)
        if not fused:
            s.set_fusion(False)
        s.set_data(w, b)
        s.set_map(None)
        return s

    def objectives(s):
        s.set_map(None)
        s.run(8)
        return s.objective_history()[1][-8:]

    for tune in (False, True):
        g = solver()
        shape_g = g.autotune(2) if tune else g.launch_shape()
        assert shape_g == g.launch_shape() and 4 <= shape_g[2] <= 512
        h = solver()
        h.set_fusion(g.fusion)
        h.set_launch_shape(*shape_g)
        assert h.launch_shape() == shape_g
        assert np.array_equal(np.asarray(objectives(g)), np.asarray(objectives(h)))
