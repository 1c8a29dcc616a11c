"""Buckets of the split sort beyond one workgroup (needs an MI355X): views whose entries crowd into
few tiles, for every bucket workgroup and both key widths.  The sorted keys and indices are the
stable sort of the frame's unsorted ones, bit for bit, and the ranges theirs; frames in which every
bucket has its own workgroup and crowded ones follow each other through one workspace and one graph."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu

# what the bucket workgroups hold, by the workspace's entries per bucket: up to 4608, 12288, and more
SHAPES = {4608: 600_000, 8192: 2_000_000, 16384: 4_000_000}


@pytest.fixture(scope="module")
def R():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2608_15785_amd as rgs
    return rgs.Renderer(0)


def check(R, scene, cam, path, min_entries):
    """Renders and compares; returns the busiest tile's and the busiest bucket's entries."""
    import paper_2608_15785_amd as rgs
    from paper_2608_15785_amd import _binding as B
    W, H = cam.width, cam.height
    plan = rgs.frame_plan(W, H)
    need = R.render(R.upload(scene, (path,)), cam, path)[1]["n_entries"]
    ws = rgs.new_workspace(scene.n, W, H, path, max(min_entries, need))
    ds = R.upload(scene, (path,))
    g = B.render_debug(R.ctx, ds, cam, path, ws, need)
    ds.release()
    keys, vals = g["keys_unsorted"], g["vals_unsorted"]
    order = np.argsort(keys, kind="stable")
    assert np.array_equal(g["keys_sorted"], keys[order]), "sorted keys differ"
    assert np.array_equal(g["vals_sorted"], vals[order]), "sorted indices differ"
    tile = (keys[order] >> np.uint64(32 if path == "plain" else plan["b_d"])).astype(np.int64)
    n = np.bincount(tile, minlength=plan["n_tiles"])
    first = np.concatenate([[0], np.cumsum(n)])[:-1]
    want = np.where(n[:, None] > 0, np.stack([first, first + n], 1), 0)
    assert np.array_equal(g["ranges"].astype(np.int64), want), "tile ranges differ"
    bits = 10 if plan["b_t"] >= 10 and (path == "plain" or max(min_entries, need) >= 1 << 18) else 8
    bucket = np.bincount(tile >> (plan["b_t"] - bits), minlength=1 << bits)
    print(f"[divided] {path} n={scene.n} {W}x{H} entries={need} busiest tile {n.max()} bucket {bucket.max()}", flush=True)
    return int(n.max()), int(bucket.max())


def copies_of(n, times):
    base = wl.config_scene("small", n=n)
    return base.subset(np.tile(np.arange(n), times))


def far(distance, W, H, half=1.0):
    return wl.orbit_camera(5, 64, distance, 20.0, 60.0, W, H, half)


@pytest.mark.parametrize("path", ["fast", "plain"])
@pytest.mark.parametrize("cap", list(SHAPES))
@pytest.mark.parametrize("runs", [2, 3, 9])
def test_every_workgroup(R, path, cap, runs):
    """Buckets of just over one and two of what a workgroup holds, and of many, with long runs of equal
    keys: merged as two runs in LDS, streamed, or divided."""
    cam = wl.config_camera("small", width=256, height=256)
    times = int({2: 1.5, 3: 2.6, 9: 9.0}[runs] * cap / 5)          # the busiest tile has about 5 entries a copy
    sc = copies_of(40, times)
    _, busiest = check(R, sc, cam, path, SHAPES[cap])
    assert {2: cap < busiest <= 2 * cap, 3: 2 * cap < busiest, 9: 7 * cap < busiest}[runs], busiest


@pytest.mark.parametrize("path", ["fast", "plain"])
@pytest.mark.parametrize("W,H", [(256, 256), (401, 267), (700, 500), (1024, 768)])
@pytest.mark.parametrize("distance,order", [(8.0, "drawn"), (40.0, "drawn"), (40.0, "by depth"), (400.0, "by tile")])
def test_views_from_afar(R, path, W, H, distance, order):
    """Distinct depths, several tiles a bucket: parts begin and end inside tiles, and the entries'
    order makes the radix tiles' runs alike, or far apart in depth or in tiles."""
    sc = wl.make_scene(60_000, 1.0, -3.5, 0.5, 3)
    cam = far(distance, W, H)
    if order != "drawn":
        p = sc.means.astype(np.float64) @ np.asarray(cam.R).T + np.asarray(cam.t)
        sc = sc.subset(np.argsort(p[:, 2] if order == "by depth" else p[:, 1]))
    _, busiest = check(R, sc, cam, path, 1 << 16)
    assert distance < 40.0 or busiest > 2 * 4608, busiest


@pytest.mark.parametrize("path", ["fast", "plain"])
@pytest.mark.parametrize("n", [9217, 18432, 60_001])
def test_equal_keys_only(R, path, n):
    """One Gaussian copied: every key of a tile is equal, and the cuts between parts go by entry order."""
    sc = wl.make_scene(1, 0.0, -5.0, 0.0, 1).subset(np.zeros(n, np.int64))
    _, busiest = check(R, sc, wl.config_camera("small", width=256, height=256), path, 1 << 16)
    assert busiest == n


@pytest.mark.parametrize("path", ["fast", "plain"])
def test_two_depths_far_apart(R, path):
    sc = wl.make_scene(30_000, 0.01, -6.0, 0.2, 4)
    sc.means[::3, 2] += 60.0
    cam = wl.config_camera("small", width=512, height=496)
    cam.z_near, cam.z_far = 0.01, 1000.0
    _, busiest = check(R, sc, cam, path, 1 << 16)
    assert busiest > 2 * 4608


@pytest.mark.parametrize("path", ["fast", "plain"])
def test_workspace_beyond_the_bucket_sort(R, path):
    """More entries a bucket than the split sort takes: the frame takes the LSD passes."""
    check(R, copies_of(40, 500), wl.config_camera("small", width=256, height=256), path, (57345 << 8) + 4096)


@pytest.mark.parametrize("path", ["fast", "plain"])
def test_overflow_of_a_crowded_frame(R, path):
    import paper_2608_15785_amd as rgs
    sc = wl.make_scene(60_000, 1.0, -3.5, 0.5, 3)
    cam = far(400.0, 700, 500)
    ds = R.upload(sc, (path,))
    ws = rgs.new_workspace(sc.n, 700, 500, path, 30_000)
    with pytest.raises(rgs.RGSError) as e:
        rgs.render(R.ctx, ds, cam, path, ws, stats=True)
    assert e.value.status == -4
    ds.release()


@pytest.mark.parametrize("path", ["fast", "plain"])
def test_crowded_and_other_frames_take_turns(R, path):
    """Served through one captured graph, each image is the renderer's, bit for bit; and a crowded frame
    leaves nothing in its workspace that another one would read."""
    import paper_2608_15785_amd as rgs
    import torch
    W, H = 700, 500
    sc = wl.make_scene(60_000, 1.0, -3.5, 0.5, 3)
    ds = R.upload(sc, (path,))
    cams = [far(d, W, H) for d in (3.0, 400.0, 3.0, 40.0, 8.0, 400.0)]
    fresh = [rgs.render(R.ctx, ds, c, path, rgs.new_workspace(sc.n, W, H, path, 1 << 21), stats=True)[0] for c in cams]
    again = [R.render(ds, c, path)[0].clone() for c in cams]
    outs = [torch.zeros((3, H, W), dtype=torch.float32, device="cuda") for _ in cams]
    server = rgs.Server(0, n_streams=1)
    torch.cuda.synchronize()
    for _ in range(3):
        resp, _ = server.serve([(ds, c, path, 0.0, o) for c, o in zip(cams, outs)])
        assert all(r["status"] == 0 for r in resp)
        for a, b, c in zip(fresh, again, outs):
            assert torch.equal(a.view(torch.int32), b.view(torch.int32))
            assert torch.equal(a.view(torch.int32), c.view(torch.int32))
            c.zero_()
    server.close()
    ds.release()
