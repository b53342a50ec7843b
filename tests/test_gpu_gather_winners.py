"""The inverse-UV gather packs each slice's winners onto a wavefront's first
lanes: slices whose texel blocks hold none, one, a wavefront's worth or a
winner in every cell of the halo (more than a wavefront), in textures that end
inside a block, against the oracle (the tolerance of the texture tests)."""
import numpy as np
import pytest

import oracle
from paper_2204_01386_amd import binding as B
from test_gpu_parity import assert_grad_close, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Ht,Wt", [(3, 3), (4, 16), (5, 17), (9, 33), (35, 50)])
@pytest.mark.parametrize("Ct", [1, 3, 4, 8])
@pytest.mark.parametrize("wrap", [(0, 1), (1, 0)])
def test_gather_winners(Ht, Wt, Ct, wrap):
    rng = np.random.default_rng(Ht * 100 + Ct)
    covered = [0.0, 1.0, 0.01, 0.6, 0.0, 1.0, 0.3]        # of each slice's pixels
    S = len(covered)
    ys, xs = np.meshgrid(np.arange(Ht) + 0.5, np.arange(Wt) + 0.5, indexing="ij")
    uv = np.stack([xs / Wt, ys / Ht], -1)[None] + rng.uniform(-0.4, 0.4, (S, Ht, Wt, 2)) / [Wt, Ht]
    uv = uv.astype(np.float32)                            # one winner in each covered pixel's cell
    tid = np.where(rng.random((S, Ht, Wt)) < np.reshape(covered, (S, 1, 1)), 0, -1).astype(np.int32)
    tex = rng.random((Ht, Wt, Ct)).astype(np.float32)
    g = rng.standard_normal((S, Ht, Wt, Ct)).astype(np.float32)
    ref = oracle.texture_bwd_tex(tex.shape, uv, tid, g, wrap_u=wrap[0], wrap_v=wrap[1])
    ctx = B.context(0)
    sums = []
    try:
        for rows in (0, 1, 2, 4):
            ctx.tune(B.TUNE_IV_ROWS, rows)
            gt, _ = B.dressi_texture_bwd(dev(tex), dev(uv), dev(tid), dev(g), 0, wrap[0], wrap[1])
            sums.append(host(gt))
    finally:
        ctx.tune(B.TUNE_IV_ROWS, 0)
    assert_grad_close(sums[0], ref, what="grad_tex")
    for s in sums[1:]:
        assert np.array_equal(s, sums[0])
