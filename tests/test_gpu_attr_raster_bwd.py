"""The per-tile adjoints of several hard views in one pass give the two calls'
gradients bit for bit: one to five views, images that end inside a tile, both
shadings, with and without empty slots skipped, and a capture on an arena that
the two calls sized."""
import numpy as np
import pytest
import torch

from paper_2204_01386_amd import binding as Bd
from paper_2204_01386_amd import scenes
from paper_2204_01386_amd.pipeline import Step
from test_gpu_parity import host

pytestmark = pytest.mark.gpu


def scene(shading, views, H, W, sub=3):
    s = scenes.config3(n_views=views, subdiv=sub, H=64, tex_size=32, env_size=4)
    s.H, s.W, s.K, s.r, s.shading, s.nmap = H, W, 1, 0.0, shading, None
    s.extra.pop("band", None)
    if shading == "lambert":
        s.color = np.random.default_rng(1).random((len(s.pos), 3)).astype(np.float32)
    return s


def step(s, fused, skip=True):
    st = Step(s)
    st.target.fill_(0.5)
    st.fuse_tiles, st.skip_empty, st.packed_geo = fused, skip, False
    st.whole_step = False
    return st


def grads(st):
    torch.cuda.synchronize()
    out = {k: host(v).copy() for k, v in st.grads().items()}
    out.update(vattr=host(st.g_vattr).copy(), clip=host(st.g_clip).copy(),
               bary=host(st.g_bary[st.tri_id >= 0]).copy())
    return out


@pytest.mark.parametrize("shading", ["lambert", "phong"])
@pytest.mark.parametrize("views,H,W", [(1, 33, 50), (2, 16, 16), (3, 61, 45), (5, 9, 7), (2, 130, 97)])
@pytest.mark.parametrize("skip", [True, False])
@pytest.mark.parametrize("sub", [1, 3])
def test_fused_tiles(shading, views, H, W, skip, sub):
    s = scene(shading, views, H, W, sub)
    out = []
    for fused in (True, False):
        st = step(s, fused, skip)
        for _ in range(2):
            st.run()
        out.append(grads(st))
    for k in out[1]:
        assert np.array_equal(out[0][k], out[1][k], equal_nan=True), k


def test_capture_on_the_calls_arena():
    s = scene("lambert", 3, 512, 512, 4)
    st = step(s, False)
    st.ctx = Bd.Context(torch.cuda.current_device())
    st.run()
    ref = grads(st)
    st.fuse_tiles = True
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        st.run()
    for _ in range(2):
        for v in st.grads().values():
            v.zero_()
        g.replay()
        got = grads(st)
        for k in ref:
            assert np.array_equal(got[k], ref[k]), k
