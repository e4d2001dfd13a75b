"""The slab depth that a solver picks for its stencil kernel, by the size of the grid: one round
of as many blocks as a CU holds of each width, and no deeper than the depth that measured faster
where one round of blocks would march through more planes (host query, no GPU)."""
import ctypes

import pytest

from paper_1905_13408_amd import spg


def _depth(shape, storage):
    L = spg.lib()
    p = spg.make_params(shape, 0.01, 0.05, 1e-3, storage=storage)
    need = ctypes.c_size_t(0)
    assert L.spg_workspace_size(ctypes.byref(p), ctypes.byref(need)) == 0
    h = ctypes.c_void_p()
    assert L.spg_create(ctypes.byref(p), ctypes.c_void_p(1 << 20), need, None, ctypes.byref(h)) == 0
    zc = ctypes.c_int32()
    assert L.spg_get_launch_shape(h, None, None, ctypes.byref(zc)) == 0
    assert L.spg_destroy(h) == 0
    return zc.value


@pytest.mark.parametrize("shape,storage,depth", [
    # narrow maps with many rows: 16 and 8 blocks per CU
    ((512, 512, 32), "compensated", 16), ((512, 512, 32), "bf16", 16), ((512, 512, 64), "compensated", 32),
    ((512, 512, 64), "fp32", 32), ((512, 512, 128), "compensated", 32),
    # the widths whose one round is the best
    ((128, 128, 128), "compensated", 4), ((160, 160, 160), "fp32", 14), ((256, 256, 256), "compensated", 32),
    ((512, 512, 512), "compensated", 256), ((32, 32, 32), "compensated", 4),
    # the separate path: deep slabs cost more in compensated storage
    ((512, 512, 192), "compensated", 32), ((512, 512, 192), "fp32", 103), ((192, 192, 192), "compensated", 14),
    ((512, 512, 160), "bf16", 103), ((8, 8, 16), "compensated", 4)])
def test_depth_follows_the_rule(shape, storage, depth):
    assert _depth(shape, storage) == depth
