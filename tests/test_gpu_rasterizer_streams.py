"""GaussianRasterizer and streams (needs an MI355X)."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


def setup(n=4000, W=401, H=267):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2608_15785_amd as rgs
    from paper_2608_15785_amd.autograd import GaussianRasterizer
    sc = wl.make_scene(n, 1.0, -2.5, 0.5, 9)
    cam = wl.config_camera("small", width=W, height=H)
    leaves = [torch.from_numpy(np.array(a)).cuda().requires_grad_() for a in
              (sc.means, sc.scales, sc.quats, sc.opacity, sc.sh)]
    return torch, rgs, GaussianRasterizer(rgs.Renderer(0)), cam, leaves


@pytest.mark.parametrize("own", ["default", "side"])
def test_workspace_is_the_context_streams(own):
    """Whatever stream is current when a workspace is made, it is memory of the context's stream,
    so that it is not handed out again before that stream's frames are done with it."""
    torch, rgs, rast, cam, leaves = setup()
    side = torch.cuda.Stream()
    if own == "side":
        rast.R.ctx.set_stream(side.cuda_stream)
    torch.cuda.synchronize()
    with torch.cuda.stream(torch.cuda.Stream()), torch.no_grad():
        rast(*leaves, cam)
    ptr = rast.workspace(cam).data_ptr()
    segment = [s for s in torch.cuda.memory_snapshot() if s["address"] <= ptr < s["address"] + s["total_size"]]
    assert len(segment) == 1 and segment[0]["stream"] == rast.R.ctx.stream
