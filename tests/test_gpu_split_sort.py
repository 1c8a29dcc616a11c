"""The split sort at its edges (needs an MI355X): buckets of one LDS run, of two and of more, for
both key widths and with few and many entries (one bucket size rule each), and depth intervals
that fit the 64-bit keys' local key and that do not.  Every key, index and range bit-exact."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
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


def check(R, scene, cam, path, n_tiles=None):
    plan = oracle.frame_plan(cam.width, cam.height)
    print(f"[split] {path} n={scene.n} {cam.width}x{cam.height} b_t={plan.b_t}", flush=True)
    tiles = None if n_tiles is None else np.random.default_rng(scene.n).choice(plan.n_tiles, n_tiles, replace=False)
    ds = R.upload(scene, (path,))
    g = R.render_debug(ds, cam, path)
    ds.release()
    fr = oracle_frame(scene, cam, path, tiles=tiles)
    compare_front_end(g, fr)
    compare_entries(g, fr)
    compare_image(g["image"], fr, path)
    return int((g["ranges"][:, 1].astype(np.int64) - g["ranges"][:, 0]).max())


@pytest.mark.parametrize("path", ["fast", "plain"])
@pytest.mark.parametrize("copies,least", [(1200, 4608), (2400, 9216)])
def test_busy_buckets_of_a_sparse_workspace(R, path, copies, least):
    """Copies of 40 Gaussians at 256x256 (one tile a bucket), in the smallest bucket workgroup: the
    busiest tile is sorted as two runs and merged, or in chunks through global memory."""
    base = wl.config_scene("small", n=40)
    sc = base.subset(np.tile(np.arange(40), copies))
    assert check(R, sc, wl.config_camera("small", width=256, height=256), path, 6) > least


@pytest.mark.parametrize("path", ["fast", "plain"])
@pytest.mark.parametrize("W,H", [(256, 256), (257, 256), (512, 496), (513, 512)])
@pytest.mark.parametrize("n", [3000, 70000])
def test_tile_bits_and_capacities(R, path, W, H, n):
    """b_t = 8, 9 and 10 (992 and 1056 tiles), with workspaces on both sides of the entry count
    that takes 1024 buckets."""
    check(R, wl.config_scene("small", n=n), wl.config_camera("small", width=W, height=H), path,
          None if n < 10000 else 12)


@pytest.mark.parametrize("near,far", [(0.2, 5.0), (1e-30, 6.0), (0.01, 1e30), (1e-30, 1e38), (1e-42, 1e39)])
@pytest.mark.parametrize("W,H", [(256, 256), (700, 500), (1024, 768)])
def test_depth_intervals(R, near, far, W, H):
    """The plain key's depth bits relative to z_near fit the local key beside its 0, 1 or 2 tile
    bits, or (31 depth bits and 2 tile bits, or a subnormal z_near) the frame takes the LSD passes."""
    cam = wl.config_camera("small", width=W, height=H)
    cam.z_near, cam.z_far = near, far
    check(R, wl.config_scene("small", n=4000), cam, "plain")


@pytest.mark.parametrize("W,H,wide,graphs", [(700, 500, (0.01, 1e30), [1, 1, 1, 1, 1, 1]),
                                             (1024, 768, (1e-30, 1e30), [1, 0, 1, 1, 0, 1])])
def test_served_frames_follow_their_own_depth_interval(R, W, H, wide, graphs):
    """Requests of one class whose cameras sort differently: a graph is replayed only for the sort it
    was captured with, and every image is rgs_render's, bit for bit."""
    import paper_2608_15785_amd as rgs
    import torch
    sc = wl.config_scene("small", n=4000)
    ds = R.upload(sc, ("plain",))
    cams = []
    for i in range(6):
        cam = wl.config_camera("small", width=W, height=H)
        cam.z_near, cam.z_far = ((0.2, 5.0), wide, (1.0, 6.0))[i % 3]
        cams.append(cam)
    ref = [R.render(ds, c, "plain")[0].clone() for c in cams]
    outs = [torch.zeros((3, H, W), dtype=torch.float32, device="cuda") for _ in cams]
    server = rgs.Server(0, n_streams=1)
    torch.cuda.synchronize()
    for _ in range(2):
        resp, _ = server.serve([(ds, c, "plain", 0.0, o) for c, o in zip(cams, outs)])
        assert all(r["status"] == 0 for r in resp)
        assert [r["graph"] for r in resp] == graphs
        for a, b in zip(ref, outs):
            assert torch.equal(a.view(torch.int32), b.view(torch.int32))
            b.zero_()
    server.close()
    ds.release()
