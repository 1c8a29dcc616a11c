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


def test_another_stream_is_waited_for_and_waits():
    """On a stream that is not the context's and whose queue still computes the parameters and
    dL/d(image), image and gradients are those of a run on the context's own stream."""
    torch, rgs, rast, cam, leaves = setup()
    dimg = torch.randn((3, cam.height, cam.width), device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    img = rast(*leaves, cam)
    want = [img.detach().clone(), *torch.autograd.grad(img, leaves, dimg)]
    late = [torch.zeros_like(p).requires_grad_() for p in leaves]
    with torch.no_grad():
        late[1] += 1.0
        late[2] += 0.5
        late[3] += 0.5
    late_dimg = torch.zeros_like(dimg)
    torch.cuda.synchronize()
    with torch.cuda.stream(torch.cuda.Stream()):
        torch.cuda._sleep(20_000_000)           # some ten milliseconds
        with torch.no_grad():
            for a, b in zip(late, leaves):
                a.copy_(b)
        img = rast(*late, cam)
        torch.cuda._sleep(20_000_000)
        late_dimg.copy_(dimg)
        got = [img.detach().clone(), *torch.autograd.grad(img, late, late_dimg)]
        got = [g.clone() for g in got]          # on that stream, after the call
    torch.cuda.synchronize()
    for a, b in zip(got, want):
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))
