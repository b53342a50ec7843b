"""A small scene's whole step (one scan job in the packed forward, the fill in
the packed backward, the ranking beside the texel gather or the geometry
adjoint, the Lambert loss's sum beside the latter) gives the separate calls'
results bit for bit at the edges of the scan's chunks and of its small form,
eagerly, captured, and captured on an arena that only the separate calls
sized."""
import numpy as np
import pytest
import torch

from paper_2204_01386_amd import binding as Bd
from paper_2204_01386_amd import scenes
from paper_2204_01386_amd.pipeline import Step
from test_gpu_parity import host

pytestmark = pytest.mark.gpu


def scene(T, shading):
    s = scenes.config2(H=80, subdiv=5, tex_size=32)
    s.tris, s.uv_tris = s.tris[:T], s.uv_tris[:T]
    if shading == "lambert":
        s.shading = "lambert"
        s.color = np.random.default_rng(T).random((len(s.pos), 3)).astype(np.float32)
    return s


def results(st):
    torch.cuda.synchronize()
    out = {k: host(v).copy() for k, v in st.grads().items()}
    out["loss"], out["color"] = host(st.loss).copy(), host(st.color).copy()
    return out


@pytest.mark.parametrize("T", [1, 20, 1023, 1024, 1025, 5000, 16384, 16385])
@pytest.mark.parametrize("shading", ["lambert", "phong"])
def test_small_step_jobs(T, shading):
    s = scene(T, shading)
    st = Step(s)
    st.target.fill_(0.5)
    st.hard_raster = 3
    st.whole_step = False
    st.run()
    ref = results(st)
    st.whole_step = True
    g = torch.cuda.CUDAGraph()
    for rep in range(4):
        if rep == 2:
            with torch.cuda.graph(g):
                st.run()
        for v in list(st.grads().values()) + [st.loss, st.color]:
            v.zero_()
        (g.replay if rep >= 2 else st.run)()
        got = results(st)
        for k in ref:
            assert np.array_equal(got[k], ref[k], equal_nan=True), (rep, k)
    if T > 16384:
        return   # (a capture of the larger form needs dressi_reserve_limits first)
    # the separate calls' arena, then a capture of the whole step
    st.ctx = Bd.Context(torch.cuda.current_device())
    st.whole_step = False
    st.run()
    st.whole_step = True
    torch.cuda.synchronize()
    g2 = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g2):
        st.run()
    g2.replay()
    got = results(st)
    for k in ref:
        assert np.array_equal(got[k], ref[k], equal_nan=True), k
