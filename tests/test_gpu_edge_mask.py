"""The blend's edge mask on words of bits against the oracle's loop over
pixels: rows of one 8-bit word, of one 64-bit word and of several, their
remainders, rows too long for a workgroup's LDS, and dilations within a word,
of whole words, across words and of the whole row.  Exact."""
import numpy as np
import pytest

import oracle
from paper_2204_01386_amd import binding as B
from test_gpu_parity import dev, host

pytestmark = pytest.mark.gpu


def layers(seed, Bv, K, H, W, p):
    rng = np.random.default_rng(seed)
    tid = np.where(rng.random((Bv, K, H, W)) < p, 3, -1).astype(np.int32)
    dist = (rng.random((Bv, K, H, W)) * rng.choice([-0.01, 0.01], (Bv, K, H, W))).astype(np.float32)
    return tid, dist


SIZES = [(1, 1, 1), (2, 5, 3), (1, 40, 8), (3, 7, 9), (1, 33, 63), (2, 70, 64), (1, 30, 65), (2, 200, 130),
         (1, 3, 300), (1, 2, 17000), (1, 2, 33000), (300, 3, 5), (40, 20, 17)]


@pytest.mark.parametrize("Bv,H,W", SIZES)
@pytest.mark.parametrize("p", [0.0, 0.002, 0.5, 1.0])
def test_edge_mask(Bv, H, W, p):
    tid, dist = layers(H + W, Bv, 2, H, W, p)
    col = np.ones(tid.shape + (1,), np.float32)
    for rho in sorted({0, 1, 2, 7, 8, 31, 63, 64, 65, 130, W - 1, 2 * W}):
        if W > 4096 and rho > 130:
            continue                    # the oracle's loop is quadratic in it
        delta = (rho + 0.5) / W
        E_o = oracle.edge_mask(tid, dist, delta, oracle.BLEND_HSR)
        for with_dist in (True, False):
            ref = E_o if with_dist else oracle.edge_mask(tid, None, delta, oracle.BLEND_HSR)
            E = B.dressi_softras(dev(col), dev(dist) if with_dist else None, dev(tid), 0.01, delta)[2]
            assert np.array_equal(host(E), ref), (rho, with_dist)
    E = B.dressi_softras(dev(col), dev(dist), dev(tid), 0.01, 0.0, B.BLEND_AA)[2]
    assert np.array_equal(host(E), oracle.edge_mask(tid, dist, 0.0, oracle.BLEND_AA))


def test_views_of_few_pixels():
    # views that begin and end within a workgroup: every view blends as alone
    tid, dist = layers(5, 70, 3, 9, 11, 0.5)
    rng = np.random.default_rng(6)
    col = rng.random(tid.shape + (4,), dtype=np.float32)
    gc, gs = (rng.random((70, 9, 11) + c, dtype=np.float32) for c in ((4,), ()))

    def run(v):
        out = B.dressi_softras(dev(col[v]), dev(dist[v]), dev(tid[v]), 0.01, 0.2)
        return out + B.dressi_softras_bwd(dev(col[v]), dev(dist[v]), dev(tid[v]), 0.01, out[2], dev(gc[v]),
                                          dev(gs[v]))

    both = [host(a) for a in run(slice(None))]
    for v in (0, 1, 2, 33, 68, 69):
        for a, b in zip(both, run(slice(v, v + 1))):
            assert np.array_equal(a[v], host(b)[0])
