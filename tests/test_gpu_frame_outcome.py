"""The outcome of a plain frame before the whole frame has finished (needs an MI355X): it is what the
workspace's header says afterwards, overflow included; the rasterizer under autograd grows its
workspace by it; and a backward call on another stream than the frame's waits for the frame."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


def setup(n=4000, log_scale=-2.5, W=401, H=267):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2608_15785_amd as rgs
    from paper_2608_15785_amd import _binding as B
    sc = wl.make_scene(n, 1.0, log_scale, 0.5, 9)
    cam = wl.config_camera("small", width=W, height=H)
    return torch, rgs, B, sc, cam


@pytest.mark.parametrize("path", ["plain", "plain/hw-exp2"])
@pytest.mark.parametrize("entries", [1000, 400000])
def test_outcome_is_the_headers(path, entries):
    torch, rgs, B, sc, cam = setup()
    R = rgs.Renderer(0)
    ds = R.upload(sc, ("plain", "fast"))
    ws = rgs.new_workspace(sc.n, cam.width, cam.height, path, entries)
    rgs.render(R.ctx, ds, cam, path, ws)
    if entries == 1000:
        with pytest.raises(rgs.RGSError) as e:
            B.frame_outcome(R.ctx, ws, sc.n)
        assert e.value.status == B.RGS_E_CAPACITY
        assert B.workspace_stats(R.ctx, ws, sc.n)["overflow"]
    else:
        assert B.frame_outcome(R.ctx, ws, sc.n) == rgs.workspace_check(R.ctx, ws, sc.n)
    # a fast frame leaves no outcome of a plain one
    rgs.render(R.ctx, ds, cam, "fast", ws)
    with pytest.raises(rgs.RGSError) as e:
        B.frame_outcome(R.ctx, ws, sc.n)
    assert e.value.status == B.RGS_E_INVALID
    torch.cuda.synchronize()
    ds.release()


@pytest.mark.parametrize("other_stream", [False, True])
def test_autograd_grows_and_matches(other_stream):
    """Large splats: the first workspace is too small.  Image and gradients are those of a
    synchronising render and backward, also when the caller's stream is not the context's."""
    torch, rgs, B, sc, cam = setup(n=3000, log_scale=-0.8)
    from paper_2608_15785_amd.autograd import GaussianRasterizer
    rast = GaussianRasterizer(rgs.Renderer(0))
    leaves = [torch.from_numpy(np.array(a)).cuda().requires_grad_() for a in
              (sc.means, sc.scales, sc.quats, sc.opacity, sc.sh)]
    dimg = torch.from_numpy(np.random.default_rng(1).standard_normal((3, cam.height, cam.width)).astype(np.float32)).cuda()
    torch.cuda.synchronize()
    with torch.cuda.stream(torch.cuda.Stream() if other_stream else torch.cuda.current_stream()):
        img = rast(*leaves, cam)
        got = [img.detach().clone(), *torch.autograd.grad(img, leaves, dimg)]
    torch.cuda.synchronize()
    R = rgs.Renderer(0)
    ds = R.upload(sc, ("plain",))
    want, st = R.render(ds, cam, "plain")
    assert st["n_entries"] > max(4 * sc.n, 1 << 16)
    ws = R.workspace(sc.n, cam.width, cam.height, "plain")
    R.ctx.set_stream(torch.cuda.Stream().cuda_stream)
    g = rgs.render_backward(R.ctx, ds, cam, ws, dimg)
    torch.cuda.synchronize()
    for a, b in zip(got, [want, g["means"], g["scales"], g["quats"], g["opacity"], g["sh"]]):
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))
    ds.release()
