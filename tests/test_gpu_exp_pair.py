"""The plain path's exponential on the device (needs an MI355X): against e^p in float64 and the device
library's expf.  One unit in the last place is half a unit of the hardware's 2^x and half of its
argument's rounding; expf takes the same steps behind its range checks."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def probe(p):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2608_15785_amd as rgs
    from paper_2608_15785_amd import _binding as B
    out = B.probe_exp(rgs.Context(0), torch.from_numpy(p).cuda())
    torch.cuda.synchronize()
    return [o.cpu().numpy() for o in out]


@pytest.mark.parametrize("lo,hi", [(-1e-6, 0.0), (-0.01, 0.0), (-1.0, 0.0), (-6.0, -1.0), (-87.0, -6.0)])
def test_within_an_ulp_and_no_further_off_than_expf(lo, hi):
    p = np.random.default_rng(1).uniform(lo, hi, 1 << 20).astype(np.float32)
    pair, libm = probe(p)
    want = np.exp(p.astype(np.float64))
    ulp = np.spacing(want.astype(np.float32)).astype(np.float64)
    off, off_libm = np.abs(pair - want) / ulp, np.abs(libm - want) / ulp
    assert off.max() <= 1.0
    assert off.max() <= off_libm.max() + 1e-2 and abs(off.mean() - off_libm.mean()) <= 1e-4
    assert np.count_nonzero(pair.view(np.int32) != libm.view(np.int32)) <= 20


def test_far_below_and_not_a_number():
    p = np.array([-87.5, -104.0, -200.0, -201.0, -1e5, -1e9, -3e9, -1e12, -3e38, -np.inf, np.nan], np.float32)
    pair, _ = probe(p)
    assert np.all(pair[:-1] >= 0.0) and np.all(pair[:-1] < 1e-37) and np.isnan(pair[-1])
