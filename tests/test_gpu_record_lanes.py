"""Per-tile records summed by one lane, by 8 and by 16 lanes: tiles of as many
triangles as the edges of that choice, one to three layers, channel counts
below, at and above the lanes, against sums in double (every record is a sum of
at most 768 float products) and, through whole steps, against the oracle's
rasterization adjoint."""
import numpy as np
import pytest

import oracle
from paper_2204_01386_amd import binding as B
from test_gpu_parity import assert_grad_close, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 2, 15, 16, 17, 31, 32, 33, 64, 128, 256])
@pytest.mark.parametrize("C", [1, 2, 6, 9, 20])
@pytest.mark.parametrize("K", [1, 3])
def test_interp_records(T, C, K):
    rng = np.random.default_rng(T * 64 + C)
    H, W = 16, 31     # a whole tile and one of 15 columns
    tris = np.arange(3 * T, dtype=np.int32).reshape(T, 3)
    tid = rng.integers(-1 if T > 1 else 0, T, (1, K, H, W)).astype(np.int32)
    bary = rng.uniform(0, 1, (1, K, H, W, 2)).astype(np.float32)
    attr = rng.standard_normal((3 * T, C)).astype(np.float32)
    g = rng.standard_normal((1, K, H, W, C)).astype(np.float32)
    ga, _ = B.dressi_interpolate_bwd(dev(attr), dev(tris), dev(tid), dev(bary), dev(g))
    hit = tid >= 0
    w = bary[hit].astype(np.float64)
    w = np.stack([w[:, 0], w[:, 1], 1.0 - w[:, 0] - w[:, 1]], 1)
    terms = w[:, :, None] * g[hit].astype(np.float64)[:, None, :]
    ref, mag = np.zeros((T, 3, C)), np.zeros((T, 3, C))
    np.add.at(ref, tid[hit], terms)
    np.add.at(mag, tid[hit], np.abs(terms) + np.abs(g[hit])[:, None, :])
    err = np.abs(host(ga).reshape(T, 3, C) - ref)
    assert (err <= 768 * 2.0 ** -24 * mag + 1e-30).all(), (err / (mag + 1e-30)).max()


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 6, 9])
def test_rast_records(n):
    # a 16 x 16 image of 2 n^2 triangles: 2 to 162 records in its tile
    u = np.linspace(-0.9, 0.9, n + 1)
    p = np.array([[x + 0.01 * y, y - 0.02 * x, 0.1 * x, 1.0] for y in u for x in u], np.float32)
    tris = []
    for r in range(n):
        for c in range(n):
            a = r * (n + 1) + c
            tris += [[a, a + 1, a + n + 2], [a, a + n + 2, a + n + 1]]
    tris = np.array(tris, np.int32)
    pc = p[None]
    tid_o, hard_o, _, _ = oracle.rasterize(pc, tris, 16, 16, K=1)
    tid, _, _ = B.dressi_rasterize(dev(pc), dev(tris), 16, 16)
    assert np.array_equal(host(tid), tid_o) and (tid_o >= 0).any()
    gb = np.random.default_rng(n).standard_normal((1, 1, 16, 16, 2)).astype(np.float32)
    gp = B.dressi_rasterize_bwd(dev(pc), dev(tris), tid, dev(gb))
    gp_o = oracle.rasterize_bwd(pc, tris, tid_o, hard_o, gb.astype(np.float64), None)
    assert_grad_close(host(gp), gp_o, what=f"{n}")
