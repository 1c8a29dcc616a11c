"""The rasterizer with a pixel per lane (frames of up to 3072 tiles) against the dual pixel, and the
schedules without, and by, buckets against that by tile (needs an MI355X): a render takes the
first of each, a counting render of the same frame the other, and images, and gradients computed
from the final T and pair counts that the render left, are the same bit for bit."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2608_15785_amd as rgs
    return rgs.Renderer(0)


@pytest.mark.parametrize("path", ["fast", "fast/hw-exp2", "fast/no-fastexp", "plain", "plain/hw-exp2"])
@pytest.mark.parametrize("W,H,n", [(16, 16, 257), (21, 30, 1), (37, 61, 3000), (401, 267, 20000), (1024, 768, 60000),
                                   (1025, 768, 60000), (1300, 900, 3000), (1300, 900, 60000), (2064, 2048, 5000)])
def test_single_pixel_is_the_dual_pixel(R, path, W, H, n):
    import torch
    import paper_2608_15785_amd as rgs
    print(f"[single] {path} n={n} {W}x{H}", flush=True)
    sc = wl.make_scene(n, 1.0, -3.0, 0.6, n + W)
    cam = wl.config_camera("small", width=W, height=H)
    cam.bg = np.array([0.2, 0.5, 0.1], np.float32)
    ds = R.upload(sc, ("plain", "fast"))
    dual = R.render_debug(ds, cam, path)
    train = path.startswith("plain")
    dimg = torch.from_numpy(np.random.default_rng(n).standard_normal((3, H, W)).astype(np.float32)).cuda()

    def grads():
        ws = R.workspace(n, W, H, path)
        g = rgs.render_backward(R.ctx, ds, cam, ws, dimg, screen=True)
        torch.cuda.synchronize()
        return {k: v.cpu().numpy() for k, v in g.items()}

    want = grads() if train else {}
    img = torch.full((3, H, W), float("nan"), device="cuda")
    R.render(ds, cam, path, out=img)
    torch.cuda.synchronize()
    assert np.array_equal(img.cpu().numpy().view(np.uint32), dual["image"].view(np.uint32))
    got = grads() if train else {}
    for k in want:
        assert np.array_equal(got[k].view(np.uint32), want[k].view(np.uint32)), k
    ds.release()
