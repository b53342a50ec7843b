"""The environment filters' contraction where its launch changes: fewer rows
than a wavefront's block and fewer columns than a workgroup's step, remainders
of both, one, two and four rows a lane (filter and adjoint), and values that
are not finite, which may reach only the outputs that their texel lights.
Bars as in test_gpu_pbs: maps 1e-5, gradients 1e-4 relative."""
import numpy as np
import pytest
import torch

from oracle import pbs as OP
from paper_2204_01386_amd import binding as B
from test_gpu_parity import assert_grad_close, assert_vals_close, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,Si,Sp,L", [
    (1, 1, 1, 2), (3, 2, 1, 3), (5, 3, 2, 3),
    (4, 30, 3, 2),      # two rows a lane in the filter
    (4, 37, 3, 2),      # four
    (38, 2, 1, 2),      # four in the adjoint
    (53, 2, 2, 2),      # two
])
def test_filter_and_adjoint(S, Si, Sp, L):
    rng = np.random.default_rng(S * 100 + Si)
    env = rng.random((6, S, S, 3)).astype(np.float32)
    irr, pref, norm = B.dressi_ibl_filter(dev(env), Si, Sp, L)
    irr_o, pref_o = OP.ibl_filter(env, Si, Sp, L)
    assert_vals_close(host(irr), irr_o, what="irradiance")
    assert_vals_close(host(pref), pref_o, what="prefiltered")
    gi = rng.standard_normal(irr_o.shape).astype(np.float32)
    gp = rng.standard_normal(pref_o.shape).astype(np.float32)
    ge = B.dressi_ibl_filter_bwd(S, norm, dev(gi), dev(gp))
    assert_grad_close(host(ge), OP.ibl_filter_bwd(S, Si, Sp, L, gi, gp), what="environment gradient")


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_a_value_that_is_not_finite_stays_in_its_hemisphere(bad):
    S, Si, Sp, L = 8, 6, 5, 3
    rng = np.random.default_rng(3)
    env = rng.random((6, S, S, 3)).astype(np.float32)
    env[2, 3, 4] = 0.0
    at = 2 * S * S + 3 * S + 4
    w = OP.cube_texels(S)[0][at]
    hit = {n: (OP.cube_texels(n)[0] @ w).reshape(6, n, n) for n in (Si, Sp)}
    ref = [host(t) for t in B.dressi_ibl_filter(dev(env), Si, Sp, L)[:2]]
    env[2, 3, 4] = bad
    out = [host(t) for t in B.dressi_ibl_filter(dev(env), Si, Sp, L)[:2]]
    for r, o, n in zip(ref, out, (Si, Sp)):
        dark = np.broadcast_to((hit[n] < -1e-9)[..., None], o.shape)
        lit = np.broadcast_to((hit[n] > 1e-9)[..., None], o.shape)
        assert dark.any() and lit.any()
        assert np.abs(o[dark] - r[dark]).max() < 1e-6
        assert not np.isfinite(o[lit]).any()
    # the adjoint: an output's gradient reaches only the texels that light it
    norm = B.dressi_ibl_filter(dev(np.abs(rng.random((6, S, S, 3))).astype(np.float32)), Si, Sp, L)[2]
    gi = rng.standard_normal((6, Si, Si, 3)).astype(np.float32)
    gp = rng.standard_normal((L, 6, Sp, Sp, 3)).astype(np.float32)
    gi[1, 2, 3] = 0.0
    ref = host(B.dressi_ibl_filter_bwd(S, norm, dev(gi), dev(gp)))
    gi[1, 2, 3] = bad
    out = host(B.dressi_ibl_filter_bwd(S, norm, dev(gi), dev(gp)))
    c = (OP.cube_texels(S)[0] @ OP.cube_texels(Si)[0][Si * Si + 2 * Si + 3]).reshape(6, S, S)
    dark, lit = (np.broadcast_to(m[..., None], out.shape) for m in (c < -1e-9, c > 1e-9))
    assert np.abs(out[dark] - ref[dark]).max() <= 1e-6 * np.abs(ref).max()
    assert not np.isfinite(out[lit]).any()
