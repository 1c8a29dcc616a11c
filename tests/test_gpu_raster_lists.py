"""The rasterizer's batches, groups and region lists at their edges (needs an MI355X).

One tile's list of 1 to 257 entries, around whole groups of four entries and whole batches
of 64, on frames of one and of 2x2 ragged tiles, against the oracle on every pixel."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as wl
from parity import compare_entries, compare_front_end, compare_image, oracle_frame

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2608_15785_amd as rgs
    return rgs.Renderer(0)


@pytest.mark.parametrize("path", ["fast", "plain", "plain/hw-exp2"])
@pytest.mark.parametrize("n", [1, 3, 4, 5, 63, 64, 65, 128, 257])
@pytest.mark.parametrize("W,H", [(16, 16), (21, 30)])
def test_list_lengths(R, path, n, W, H):
    print(f"[lists] {path} n={n} {W}x{H}", flush=True)
    r = np.random.default_rng(100 * n + W)
    sc = wl.make_scene(n, 0.35, -2.6, 0.6, n)
    sc.opacity = r.uniform(0.02, 0.3, n).astype(np.float32)          # long lists without many stops
    cam = wl.config_camera("small", width=W, height=H)
    ds = R.upload(sc, ("plain", "fast"))
    g = R.render_debug(ds, cam, path)
    ds.release()
    fr = oracle_frame(sc, cam, path)
    compare_front_end(g, fr)
    compare_entries(g, fr)
    compare_image(g["image"], fr, "plain" if path.startswith("plain") else path)
    mask = ~fr.flagged & ~(fr.mode_slack > 0) & ~np.isnan(fr.T_final)
    assert np.array_equal(g["n_proc"][mask], fr.n_proc[mask].astype(np.uint32))
    assert np.array_equal(g["n_blend"][mask], fr.n_blend[mask].astype(np.uint32))


def test_plain_non_finite_colour_stays_with_its_pixels(R):
    """A Gaussian whose colour is not finite reaches only the pixels where its pair is blended:
    everywhere else the plain image is the one without it, bit for bit."""
    import paper_2608_15785_amd as rgs
    import torch
    n = 300
    sc = wl.make_scene(n, 0.5, -3.2, 0.4, 5)
    cam = wl.config_camera("small", width=40, height=40)
    images = []
    for colour in (0.3, np.inf):
        sc.sh[7] = 0.0
        ds = R.upload(sc, ("plain",))
        t = [torch.from_numpy(np.array(a)).cuda() for a in (sc.means, sc.scales, sc.quats, sc.opacity, sc.sh)]
        t[4][7, 0, :] = colour
        rgs.scene_update_plain(R.ctx, ds, *t)
        images.append(R.render(ds, cam, "plain")[0].cpu().numpy())
        ds.release()
    a, b = images
    touched = ~np.isfinite(b)
    assert touched.any() and not touched.all()
    # a pixel without the pair differs from the other image by nothing
    same = a.view(np.uint32) == b.view(np.uint32)
    assert np.all(same | touched)
