"""The binless rasterizer's merge with 1 to 64 lanes a triangle (few large
triangles to many small ones, images a box exceeds, odd widths, two views)
selects the layers of the tile rasterizer, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2204_01386_amd import binding as Bd
from paper_2204_01386_amd import scenes
from test_gpu_parity import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sub", [0, 2, 4, 6])
@pytest.mark.parametrize("H,W", [(1, 1), (5, 3), (33, 17), (70, 129), (200, 333)])
@pytest.mark.parametrize("cull", [0, 1])
def test_direct_lanes(sub, H, W, cull):
    p, tris = scenes.noisy_sphere(sub, 7)
    mvp = scenes.view_proj(scenes.camera_ring(2, 3, radius=1.6))
    pc = Bd.dressi_transform(dev(p.astype(np.float32)), dev(mvp.astype(np.float32)))
    ctx = Bd.context(torch.cuda.current_device())
    out = []
    try:
        for strategy in (0, 3):
            ctx.tune(Bd.TUNE_HARD_RASTER, strategy)
            for _ in range(2):   # the keys are left cleared
                r = Bd.dressi_rasterize(pc, dev(tris.astype(np.int32)), H, W, cull=cull)
            out.append([host(r[0]), host(r[1])])
    finally:
        ctx.tune(Bd.TUNE_HARD_RASTER, 0)
    assert np.array_equal(out[0][0], out[1][0])
    hit = out[0][0] >= 0
    assert H * W < 100 or hit.any()
    assert np.array_equal(out[0][1][hit], out[1][1][hit])
