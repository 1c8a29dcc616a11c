"""rgs_render_backward on another stream than its frame's (needs an MI355X): the frame's outcome is
known before its pixels are blended, so the call waits for the frame's stream.  The frame is queued
behind others that take some milliseconds, and the backward call follows at once."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("path", ["plain", "plain/hw-exp2"])
def test_waits_for_the_frames_stream(path):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2608_15785_amd as rgs
    sc, big = wl.make_scene(4000, 1.0, -2.5, 0.5, 9), wl.make_scene(400_000, 1.0, -3.5, 0.5, 2)
    cam, wide = wl.config_camera("small", width=401, height=267), wl.config_camera("small", width=1024, height=768)
    dimg = torch.from_numpy(np.random.default_rng(1).standard_normal((3, 267, 401)).astype(np.float32)).cuda()
    R = rgs.Renderer(0)
    ds, db = R.upload(sc, ("plain",)), R.upload(big, ("plain",))
    R.render(db, wide, "plain")
    want_img, _ = R.render(ds, cam, path)
    ws = R.workspace(sc.n, 401, 267, path)
    want = rgs.render_backward(R.ctx, ds, cam, ws, dimg)
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    scratch = torch.empty(rgs.backward_scratch_size(sc.n, 401, 267, ws.numel()), dtype=torch.uint8, device="cuda")
    for _ in range(3):
        R.render(ds, wl.orbit_camera(3, 8, 4.0, 20.0, 60.0, 401, 267, 1.0), path)      # another frame's pixels
        torch.cuda.synchronize()
        R.ctx.set_stream(a.cuda_stream)
        images = [R.render(db, wide, "plain", check=False)[0] for _ in range(6)]
        img, _ = R.render(ds, cam, path, check=False)
        R.ctx.set_stream(b.cuda_stream)
        got = rgs.render_backward(R.ctx, ds, cam, ws, dimg, scratch=scratch)
        torch.cuda.synchronize()
        assert torch.equal(img.view(torch.int32), want_img.view(torch.int32))
        for k in want:
            assert torch.equal(got[k].view(torch.int32), want[k].view(torch.int32)), k
        del images
    ds.release()
    db.release()
