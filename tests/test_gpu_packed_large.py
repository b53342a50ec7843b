"""The packed backward of an image with more pixels than its grid has lanes
(65,536 workgroups of 256): the grid-stride form gives the separate stages'
gradients bit for bit, and their loss up to the grouping of its sum."""
import numpy as np
import pytest

from paper_2204_01386_amd import scenes
from paper_2204_01386_amd.pipeline import Step
from test_gpu_parity import host

pytestmark = pytest.mark.gpu


def test_packed_backward_grid_stride():
    s = scenes.config2(H=4099, subdiv=3, tex_size=64)
    out = []
    for packed in (True, False):
        s.extra["packed"] = packed
        st = Step(s)
        assert st.B * st.H * st.W > 65536 * 256 and st.packed == packed
        st.target.fill_(0.25)
        st.run()
        out.append([host(t) for t in (st.g_pos, st.g_tex, st.loss)])
        del st
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
    # float sums of 16.8 million equal-signed terms in groups of at most 4,096: 2^-24 a step
    assert abs(out[0][2] - out[1][2]) <= 1e-4 * abs(out[1][2])
