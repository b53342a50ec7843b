"""The packed PBS pass gives the separate stages' image, loss and gradients bit
for bit: one to three layers, odd images and views smaller than a workgroup,
map sizes from one texel, the ends of the level range and roughness outside
it, and an albedo that it leaves to the stages."""
import numpy as np
import pytest
import torch

from paper_2204_01386_amd import scenes
from paper_2204_01386_amd.pipeline import PbsStep
from test_gpu_parity import host

pytestmark = pytest.mark.gpu


def scene(views, H, W, K):
    s = scenes.fit_scene(subdiv=3, H=64, tex_size=32, n_views=views, K=K, r=0.03)
    s.H, s.W = H, W
    return s


def run(s, env, material, Si, Sp, L, fused, params=None):
    ps = PbsStep(s, env, material, Si, Sp, L, 16, 64, params=params)
    ps.st.target.copy_(torch.linspace(0, 1, ps.st.target.numel(), device=ps.dev).reshape(ps.st.target.shape))
    ps.fuse_layers = fused
    assert params is not None or (ps._layers() is not None) == fused
    for _ in range(2):
        ps.run()
    torch.cuda.synchronize()
    cov = ps.st.tri_id >= 0
    out = {k: host(v) for k, v in ps.grads().items()}
    out.update(loss=host(ps.st.loss), color=host(ps.st.color), g_irr=host(ps.g_irr), g_pref=host(ps.g_pref),
               samp=host(ps.st.samp[cov]), layer=host(ps.st.layer_color[cov]), g_samp=host(ps.st.g_samp[cov]))
    return out


@pytest.mark.parametrize("views,H,W,K", [(1, 64, 64, 1), (3, 45, 61, 2), (7, 9, 5, 3)])
@pytest.mark.parametrize("S,Si,Sp,L,material", [(8, 4, 8, 5, (0.5, 0.4)), (4, 1, 1, 2, (0.0, 0.0)),
                                                (8, 3, 17, 3, (1.0, 1.0)), (4, 2, 4, 4, (0.3, 1.5)),
                                                (4, 2, 4, 4, (0.3, -0.5))])
def test_pbs_layers_equal_stages(views, H, W, K, S, Si, Sp, L, material):
    s = scene(views, H, W, K)
    env = np.random.default_rng(3).uniform(0.1, 2.0, (6, S, S, 3)).astype(np.float32)
    a, b = (run(s, env, material, Si, Sp, L, f) for f in (True, False))
    assert (a["layer"] != 0).any()
    for k in b:
        assert np.array_equal(a[k], b[k], equal_nan=True), k


def test_unaligned_albedo_keeps_the_stages():
    s = scene(2, 40, 40, 1)
    env = np.random.default_rng(3).uniform(0.1, 2.0, (6, 4, 4, 3)).astype(np.float32)
    ref = run(s, env, (0.2, 0.7), 2, 4, 3, True)
    raw = torch.empty(s.tex.size + 1, device="cuda")
    tex = raw[1:].view(s.tex.shape)
    tex.copy_(torch.from_numpy(s.tex))
    got = run(s, env, (0.2, 0.7), 2, 4, 3, True, params={"tex": tex})
    for k in ref:
        assert np.array_equal(got[k], ref[k]), k
