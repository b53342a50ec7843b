"""The rasterization operator's bins that hold every triangle: no status read
and no overflow where they are small enough, the checked form (grown and run
again after an overflow) where they are not, the layers of the binless
strategy in both, and the plain call under capture."""
import numpy as np
import pytest
import torch

from helpers import screen_to_clip
from paper_2204_01386_amd import binding as B
from test_gpu_parity import dev, host

pytestmark = pytest.mark.gpu


def crowd(T, H, W, seed=3):
    """T small triangles in one corner of the image."""
    rng = np.random.default_rng(seed)
    xy = (rng.uniform(2.0, 14.0, (T, 1, 2)) + rng.uniform(-1.5, 1.5, (T, 3, 2))).reshape(-1, 2)
    pc = screen_to_clip(xy, H, W, z=np.repeat(rng.uniform(0.1, 0.9, T), 3))
    return dev(pc[None].astype(np.float32)), dev(np.arange(3 * T, dtype=np.int32).reshape(T, 3))


def flag(ctx, pc, tris, H, W, K, r):
    T = tris.shape[0]
    out = [torch.empty((1, K, H, W) + c, dtype=d, device="cuda")
           for c, d in (((), torch.int32), ((2,), torch.float32), ((), torch.float32))]
    full = B.C.c_int(7)
    rc = B._lib.dressi_rasterize_full_bins(ctx.handle, B._ptr(pc), B._ptr(tris), 1, 3 * T, T, H, W, K, r, 0,
                                           *[B._ptr(t) for t in out], B.C.byref(full), B._stream())
    ctx.check(rc, "full bins")
    return full.value, ctx.check_status(), host(out[0])


@pytest.mark.parametrize("H,W,T,full", [(64, 64, 9000, 1), (16, 16, 1, 1), (64, 64, 0, 1), (2048, 2048, 9000, 0)])
@pytest.mark.parametrize("r", [0.0, 0.001])
def test_full_bins(H, W, T, full, r):
    pc, tris = crowd(max(T, 1), H, W)
    if T == 0:
        tris = tris[:0].contiguous()
    saved, dv = B._ctxs.get(torch.cuda.current_device()), torch.cuda.current_device()
    B._ctxs[dv] = B.Context(dv)
    try:
        c = B._ctxs[dv]
        got = flag(c, pc, tris, H, W, 1, r) if T else (1, 0, None)
        assert got[0] == full
        assert (got[1] == 0) == bool(full)          # only bins that may overflow report it
        tid = host(B.dressi_rasterize(pc, tris, H, W, 1, r)[0])
        assert c.check_status() == 0
        if r == 0.0:
            c.tune(B.TUNE_HARD_RASTER, 3)
            assert np.array_equal(tid, host(B.dressi_rasterize(pc, tris, H, W, 1, r)[0]))
        elif T:
            c.reserve(0, T)
            assert np.array_equal(tid, host(B.dressi_rasterize(pc, tris, H, W, 1, r)[0]))
        if full and T:
            assert np.array_equal(tid, got[2])
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g):
                t2 = B.dressi_rasterize(pc, tris, H, W, 1, r)[0]
            g.replay()
            assert np.array_equal(tid, host(t2))
    finally:
        if saved is not None:
            B._ctxs[dv] = saved
