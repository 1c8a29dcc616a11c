"""How the front end spreads small scenes over workgroups, at the edges of the rule (needs an
MI355X): one and two workgroups of 256 Gaussians, and 256 of them with one Gaussian more."""
import pytest

import workloads as wl
from test_gpu_parity import R, run_parity  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("path", ["plain", "fast"])
@pytest.mark.parametrize("n", [256, 257, 65536, 65537])
def test_small_scenes(R, path, n):  # noqa: F811
    tiles = None if n < 10_000 else [0, 37, 136, 255]
    run_parity(R, wl.config_scene("small", n=n), wl.config_camera("small"), path, tiles=tiles)
