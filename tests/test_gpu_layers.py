"""The packed pass over a soft image's layers gives the separate stages'
values bit for bit: every mode, one to five layers, images that end inside a
workgroup and views smaller than one, with and without the empty slots
written, and the forms that it leaves to the separate stages."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2204_01386_amd import binding as B
from paper_2204_01386_amd import pipeline, scenes
from test_gpu_parity import dev, host

pytestmark = pytest.mark.gpu

BUFS = ["gbuf", "uvbuf", "samp", "dir", "env_s", "layer_color", "color", "sil", "E", "loss", "g_gbuf", "g_samp",
        "g_env_s", "g_bary_uv", "g_bary", "g_vattr", "g_pos", "g_tex", "g_envtex"]


def scene(shading, views, H, W, K, r):
    s = scenes.config3(n_views=views, subdiv=3, H=64, tex_size=48, env_size=8)
    s.H, s.W, s.K, s.r, s.shading = H, W, K, r, shading
    s.extra.pop("band", None)
    if shading == "lambert":
        s.color = np.random.default_rng(1).random((len(s.pos), 3)).astype(np.float32)
    if shading != "phong_env":
        s.nmap = None
    return s


def step(s, **kw):
    st = pipeline.Step(s, **kw)
    # (a step without a target step has its target uninitialised)
    st.target.copy_(torch.linspace(0, 1, st.target.numel(), device=st.dev).reshape(st.target.shape))
    return st


def state(st, covered):
    out = {}
    for b in BUFS:
        t = getattr(st, b)
        if t is None:
            continue
        if covered and tuple(t.shape[:4]) == tuple(st.tri_id.shape):
            t = t[st.tri_id >= 0]
        out[b] = host(t)
    return out


@pytest.mark.parametrize("shading", ["lambert", "phong", "phong_env"])
@pytest.mark.parametrize("views,H,W,K,r", [(1, 64, 64, 1, 0.03), (3, 61, 45, 3, 0.05), (5, 9, 7, 2, 0.2),
                                           (2, 33, 128, 5, 0.04)])
@pytest.mark.parametrize("skip", [True, False])
def test_layers_equal_stages(shading, views, H, W, K, r, skip):
    s = scene(shading, views, H, W, K, r)
    out = []
    for fused in (True, False):
        st = step(s)
        st.skip_empty = skip
        st.fuse_layers = fused
        assert (st._layer_scene() is not None) == fused
        for _ in range(2):
            st.run()
        out.append(state(st, skip))
    assert (out[0]["layer_color"] != 0).any()
    for k in out[1]:
        assert np.array_equal(out[0][k], out[1][k], equal_nan=True), k


def test_forms_left_to_the_stages():
    s = scene("phong", 2, 40, 48, 2, 0.05)
    ref = step(s)
    ref.run()
    # texels that float4 loads are not aligned for
    raw = torch.empty(ref.tex.numel() + 1, device=ref.dev)
    tex = raw[1:].view(ref.tex.shape)
    tex.copy_(ref.tex)
    st = step(s, params={"tex": tex})
    assert st._layer_scene() is None
    st.run()
    assert np.array_equal(host(st.color), host(ref.color))
    assert np.array_equal(host(st.g_tex), host(ref.g_tex)) and np.array_equal(host(st.g_pos), host(ref.g_pos))
    # the jitter and the texel branch keep their own backward
    for kw in ({"frame": 3}, {"concurrent": "texel"}):
        a, b = step(s), step(s)
        b.fuse_layers = False
        for x in (a, b):
            for k, v in kw.items():
                setattr(x, k, v)
            x.run()
        assert np.array_equal(host(a.g_tex), host(b.g_tex)) and np.array_equal(host(a.g_pos), host(b.g_pos)), kw


def test_refusals():
    s = scene("phong", 1, 16, 16, 1, 0.1)
    st = pipeline.Step(s)
    p, ls = pipeline._p, st._layer_scene()

    def fwd(ls, samp=st.samp):
        return B._lib.dressi_layers_forward(st.ctx.handle, C.byref(ls), p(st.tri_id), p(st.bary), 1, 1, 16, 16,
                                            p(st.gbuf), p(st.uvbuf), p(samp), None, None, p(st.layer_color), st._s())

    assert fwd(ls) == 0
    for field, value in (("Cv", 9), ("mode", 7), ("tri_eye", p(st.tri_id)), ("vattr", None), ("uv", None)):
        bad = st._layer_scene()
        setattr(bad.s, field, value)
        assert fwd(bad) != 0, field
    bad = st._layer_scene()
    bad.s.td.Ct = 3
    assert fwd(bad) != 0
    assert fwd(ls, None) != 0
