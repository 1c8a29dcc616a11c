"""The backward kernel's lists and rows of sums at their edges (needs an MI355X): tiles of no, one,
a batch's and more entries, and entries that reach all sixteen regions of a tile, so that a batch's
rows hold fewer entries than it stages.  The image-space sums against the float64 adjoint, to 1e-3 of
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
@pytest.mark.parametrize("n,log_scale", [(1, -3.0), (65, -0.5), (400, -0.7), (900, -4.5)])
@pytest.mark.parametrize("W,H", [(16, 16), (50, 35)])
def test_lists(R, n, log_scale, W, H, path):
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
