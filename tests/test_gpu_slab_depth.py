"""The fused path's own slab depth (one plane on small maps, whole halves of the map on the
widest) gives the bits of any other: every width, depths that the slabs do not divide, in the
three storage modes and with the objective monitor."""
import numpy as np
import pytest
import torch

from paper_1905_13408_amd import spg, synth

from gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["compensated", "fp32", "bf16"])
@pytest.mark.parametrize("shape", [(8, 8, 32), (64, 64, 64), (16, 128, 128), (192, 32, 128), (16, 128, 160), (160, 16, 256),
                                   (8, 32, 512), (160, 512, 32)])
def test_own_depth_gives_the_same_bits(shape, storage):
    announce(f"own slab depth shape={shape} {storage}")
    rng = np.random.default_rng([101, *shape])
    w = synth.fourier_weights(shape).astype(np.float32)
    b = torch.from_numpy((rng.standard_normal((*shape, 2), dtype=np.float32) * 0.3).view(np.complex64)[..., 0])
    u, v = (rng.uniform(0.5, 2.0, size=shape).astype(np.float32) for _ in range(2))
    out = []
    for zc in (None, 32, 5):
        s = spg.SPGSolver(shape, 0.02, 0.05, 1e-2, storage=storage, monitor_every=4)
        if zc:
            s.set_launch_shape(16, 16, zc)
        s.set_data(w, b)
        s.set_penalty_weights(u, v)
        s.set_map(None)
        stats = s.run(9)
        out.append((s.get_map(), stats.obj_smoothed))
    for x, f in out[1:]:
        assert torch.equal(x, out[0][0])
        # the same terms, summed by other blocks in fp64
        assert abs(f - out[0][1]) <= 1e-12 * abs(f)
