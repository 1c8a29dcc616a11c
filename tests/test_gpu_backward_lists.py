"""The backward kernels' lists and rows of sums at their edges (needs an MI355X): tiles of no, one,
a batch's and more entries, entries that reach all sixteen regions of a tile, so that a batch's
rows hold fewer entries than it stages (on frames that take a pixel per lane and, 800x800, on
ones that take two), and Gaussians of more partials than a workgroup of the
per-Gaussian pass stages.  The image-space sums against the float64 adjoint, to 1e-3 of
the sum of their terms' magnitudes and the slack of near-threshold decisions, as in the backward
pass's other tests; a second run is the same bit for bit."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import workloads as wl
from oracle import backward as OB
from test_gpu_backward import MARGINS, PATHS, gpu_backward

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2608_15785_amd as rgs
    return rgs.Renderer(0)


@pytest.mark.parametrize("path", PATHS)
@pytest.mark.parametrize("W,H,n,log_scale", [(W, H, n, s) for W, H in ((16, 16), (50, 35))
                                             for n, s in ((1, -3.0), (65, -0.5), (400, -0.7), (900, -4.5))]
                         + [(401, 267, 1, 0.4), (401, 267, 65, 0.2), (800, 800, 1, -0.5), (800, 800, 65, 0.0),
                            (800, 800, 300, -2.5)])
def test_lists(R, W, H, n, log_scale, path):
    sc = wl.make_scene(n, 1.0, log_scale, 0.3, 100 + n)
    if n > 1:
        sc.opacity[:] = np.clip(sc.opacity * 0.08, 0.006, 1.0)     # few pixels stop: long lists
    cam = wl.config_camera("small", width=W, height=H)
    cam.bg = np.array([0.3, 0.1, 0.2], np.float32)
    rng = np.random.Generator(np.random.PCG64(n))
    dimg = rng.standard_normal((3, H, W)).astype(np.float32)
    g = gpu_backward(R, sc, cam, dimg, path)
    adj = OB.render_adjoint(oracle.prepare_plain(sc), cam, dimg.astype(np.float64), margins=MARGINS[path],
                            decisions=g["decisions"])
    assert adj.unexplained == 0
    assert np.all(g["screen"][~adj.touched] == 0.0)
    err = np.abs(g["screen"][adj.touched] - adj.screen[adj.touched])
    bound = 1e-3 * adj.screen_abs[adj.touched] + adj.slack[adj.touched] + 1e-7
    print(f"[bwd lists] n={n} {W}x{H} {path}: touched {int(adj.touched.sum())}, "
          f"longest pixel {int(g['decisions'][0].max())}, worst err/bound {np.max(err / bound, initial=0.0):.3g}", flush=True)
    assert np.all(err <= bound)
    again = gpu_backward(R, sc, cam, dimg, path)
    for k in ("means", "scales", "quats", "opacity", "sh", "screen"):
        assert np.array_equal(g[k], again[k]), k


def test_sh_gradients_at_an_odd_address(R):
    """The SH gradients leave in 16-byte stores where the caller's buffer allows them."""
    import ctypes as C
    import torch
    import paper_2608_15785_amd as rgs
    from paper_2608_15785_amd import _binding as B
    sc = wl.make_scene(131, 1.0, -2.0, 0.4, 7)
    cam = wl.config_camera("small", width=64, height=48)
    dimg = torch.ones((3, 48, 64), device="cuda")
    ds = R.upload(sc, ("plain",))
    R.render(ds, cam, "plain")
    ws = R.workspace(sc.n, 64, 48, "plain")
    want = rgs.render_backward(R.ctx, ds, cam, ws, dimg)
    g = {k: torch.empty_like(v) for k, v in want.items()}
    sh = torch.full((sc.n * 48 + 2,), float("nan"), device="cuda")
    scratch = torch.empty(rgs.backward_scratch_size(sc.n, 64, 48, ws.numel()), dtype=torch.uint8, device="cuda")
    gr = B.Grads(d_means=g["means"].data_ptr(), d_scales=g["scales"].data_ptr(), d_quats=g["quats"].data_ptr(),
                 d_opacity=g["opacity"].data_ptr(), d_sh=sh.data_ptr() + 4, d_screen=None, scratch=scratch.data_ptr(),
                 scratch_bytes=scratch.numel())
    cc = rgs.camera_struct(cam)
    assert B.lib.rgs_render_backward(R.ctx.handle, ds.handle, C.byref(cc), 64, 48, dimg.data_ptr(), ws.data_ptr(),
                                     ws.numel(), C.byref(gr)) == 0
    torch.cuda.synchronize()
    assert torch.equal(sh[1:-1], want["sh"].reshape(-1))
    assert torch.isnan(sh[0]) and torch.isnan(sh[-1])
    ds.release()
