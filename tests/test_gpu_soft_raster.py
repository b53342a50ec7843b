"""Soft rasterization (quadrant workgroups, near and far bin ends, gap rings)
against the oracle where its cases change: images smaller than a quadrant,
more near triangles than one staged batch holds, reaches beyond the gap
histogram, triangles beyond the 32-bit products, clusters that most pixels see
only through the far rings.  Bars as in test_gpu_parity: ids and hard flags
bit-exact, barycentrics 1e-5 max(1, |ref|), distances 1e-5."""
import numpy as np
import pytest
import torch

import oracle
from helpers import screen_to_clip
from test_gpu_parity import assert_vals_close, check_raster, dev, host
from paper_2204_01386_amd import binding as B

pytestmark = pytest.mark.gpu


def cloud(seed, T, H, W, lo, hi, side, views=1):
    """T random triangles of about `side` pixels with centres in the
    rectangle lo..hi (fractions of the image)."""
    out = []
    for v in range(views):
        rng = np.random.default_rng([seed, v])
        c = rng.uniform(lo, hi, (T, 1, 2)) * (W, H)
        xy = (c + rng.uniform(-0.5, 0.5, (T, 3, 2)) * side).reshape(-1, 2)
        out.append(screen_to_clip(xy, H, W, z=rng.uniform(0.05, 0.95, 3 * T), w=rng.uniform(0.5, 2.0, 3 * T)))
    return np.stack(out), np.arange(3 * T, dtype=np.int32).reshape(T, 3)


CASES = [
    # H, W, T, centres, side in pixels, r, K, views
    (5, 7, 40, (0.0, 1.0), 2.0, 0.3, 3, 1),          # smaller than a quadrant
    (1, 1, 9, (0.0, 1.0), 2.0, 1.0, 2, 2),
    (40, 33, 6000, (0.3, 0.7), 1.5, 0.05, 3, 1),     # several staged batches in a quadrant
    (24, 40, 900, (0.0, 1.0), 4.0, 0.08, 5, 2),
    (50, 100, 30, (0.0, 1.0), 60.0, 1.0, 2, 1),      # the reach is the whole image
    (150, 210, 12, (0.2, 0.8), 300.0, 0.1, 4, 1),    # double-precision products
    (64, 160, 500, (0.05, 0.15), 2.0, 0.9, 4, 1),    # seen through the far rings
    (64, 160, 2, (0.05, 0.15), 3.0, 0.9, 3, 1),      # fewer triangles than layers
    (97, 65, 300, (0.0, 1.0), 9.0, 0.004, 1, 3),     # a reach below one pixel
]


@pytest.mark.parametrize("H,W,T,box,side,r,K,views", CASES)
def test_soft_raster(H, W, T, box, side, r, K, views):
    pc, tris = cloud(T + K, T, H, W, *box, side, views)
    check_raster(B, pc, tris, H, W, K, r, bwd=False)
    # a second call finds the bins' counters back at zero
    check_raster(B, pc, tris, H, W, K, r, bwd=False)


@pytest.mark.parametrize("H,W,T,box,side,r,K,views", CASES)
@pytest.mark.parametrize("mode", [B.BLEND_HSR, B.BLEND_AA, B.BLEND_HARD])
def test_soft_raster_banded(H, W, T, box, side, r, K, views, mode):
    pc, tris = cloud(T + K, T, H, W, *box, side, views)
    delta = min(r, 3.5 / W)
    ref = oracle.rasterize(pc, tris, H, W, K=K, r=r)
    tid_o, hard_o, bary_o, dist_o = oracle.band_layers(*ref, delta, mode)
    for _ in range(2):
        tid, bary, dist = B.dressi_rasterize_banded(dev(pc), dev(tris), H, W, K, r, delta, mode)
        assert np.array_equal(host(tid), tid_o)
        assert_vals_close(host(bary), bary_o, what="bary", scale_by_ref=True)
        d = host(dist)
        assert_vals_close(d, dist_o, what="dist")
        m = tid_o >= 0
        assert np.array_equal(np.signbit(d[m]), hard_o[m] == 0)


def test_soft_overflow_counts_both_ends():
    """The near and far ends of a bin share its capacity: the need that is
    reported is their sum, and a context sized to it gives the layers."""
    H, W, T, r, K = 64, 256, 3000, 0.02, 2
    pc, tris = cloud(5, T, H, W, 0.06, 0.13, 2.0)
    tid_o = oracle.rasterize(pc, tris, H, W, K=K, r=r)[0]
    c = B.Context(torch.cuda.current_device())
    pt, tt = dev(pc), dev(tris)
    tid = torch.empty((1, K, H, W), dtype=torch.int32, device="cuda")
    bary = torch.empty((1, K, H, W, 2), device="cuda")
    dist = torch.empty((1, K, H, W), device="cuda")
    p = lambda t: B.C.c_void_p(t.data_ptr())

    def go():
        c.check(B._lib.dressi_rasterize(c.handle, p(pt), p(tt), 1, 3 * T, T, H, W, K, r, 0, p(tid), p(bary), p(dist),
                                        None), "rasterize")
        torch.cuda.synchronize()
        return c.check_status()

    need = go()       # the automatic capacity at these sizes is 2048
    assert 2048 < need <= T
    c.reserve(0, need)
    assert go() == 0
    assert np.array_equal(host(tid), tid_o)
