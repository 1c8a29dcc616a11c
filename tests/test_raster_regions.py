"""The rasterizer's region lists drop only pairs that fail the skip test.

A float32 replica (numpy, every operation rounded as the kernel's) of the span
rule that decides which 4x4 regions of a half-tile a Gaussian is listed for,
against the exact quadratic form in float64: a region holding a pixel with
q <= tau, the pairs with alpha >= 1/255, must always be listed.  The rule's
margin on tau is 1e-3 of it plus 0.02, its margin on the spans 0.05 pixel."""
from __future__ import annotations

import numpy as np
import pytest

F = np.float32


def spans(u, v, A, B, C, tau, bx, by, top):
    """left, right [2] per Gaussian, and whether the closed form (not the box) was used."""
    u, v, A, B, C, tau = (np.asarray(a, F) for a in (u, v, A, B, C, tau))
    with np.errstate(all="ignore"):
        qlim = tau * F(1.001) + F(0.02)
        AC = A * C
        det = AC - B * B
        iA, iC, iD = F(1) / A, F(1) / C, F(1) / det
        hx, hy = np.sqrt(qlim * C * iD), np.sqrt(qlim * A * iD)
        slope, peak, qA = -B * iA, -B * iC * hx, qlim * A
        closed = (det * F(2048) > AC) & (hx < F(1e4)) & (hy < F(1e4))
        left, right = [], []
        for b in range(2):
            y0 = F(top + 4 * b) - v
            lo, hi = np.fmax(y0, -hy), np.fmin(y0 + F(3), hy)
            dr, dl = np.fmin(np.fmax(peak, lo), hi), np.fmin(np.fmax(-peak, lo), hi)
            sr = np.sqrt(np.fmax(qA - det * dr * dr, F(0)))
            sl = np.sqrt(np.fmax(qA - det * dl * dl, F(0)))
            out = lo > hi + F(0.05)
            r = np.where(out, F(-1e30), sr * iA + (slope * dr + u) + F(0.05))
            le = -sl * iA + (slope * dl + u) - F(0.05)
            bxw, byw = bx * F(1.001) + F(0.05), by * F(1.001) + F(0.05)
            t = F(top + 4 * b)
            bout = (v - byw > t + F(3)) | (v + byw < t)
            right.append(np.where(closed, r, np.where(bout, F(-1e30), u + bxw)))
            left.append(np.where(closed, le, u - bxw))
        none = qlim < 0
    return [np.where(none, F(1), x) for x in left], [np.where(none, F(-1e30), x) for x in right], closed


def hits(left, right):
    out = []
    for k in range(8):
        x0 = F(4 * (k % 4)) - F(7.5)
        out.append(~(left[k // 4] > x0 + F(3)) & ~(right[k // 4] < x0))
    return np.stack(out, 1)


def gaussians(n, seed, s_lo, s_hi):
    """Random 2D covariances (+ 0.3 I) with standard deviations in [s_lo, s_hi] px, near the half-tile."""
    r = np.random.default_rng(seed)
    s = np.exp(r.uniform(np.log(s_lo), np.log(s_hi), (n, 2)))
    th = r.uniform(0, np.pi, n)
    c, d = np.cos(th), np.sin(th)
    c00 = c * c * s[:, 0] ** 2 + d * d * s[:, 1] ** 2 + 0.3
    c11 = d * d * s[:, 0] ** 2 + c * c * s[:, 1] ** 2 + 0.3
    c01 = c * d * (s[:, 0] ** 2 - s[:, 1] ** 2)
    det = c00 * c11 - c01 * c01
    lno = np.log(1.0 / (1.0 + np.exp(-r.normal(0, 2.5, n))))
    tau = 2 * (np.log(255.0) + lno)
    reach = np.sqrt(np.maximum(tau, 0) * np.maximum(c00, c11)) + 10
    u, v = r.uniform(-1, 1, n) * reach, r.uniform(-1, 1, n) * reach
    f = [a.astype(F) for a in (u, v, c11 / det, -c01 / det, c00 / det, tau)]
    box = [np.nextafter(np.sqrt(np.maximum(tau * c, 0)).astype(np.float16), np.float16(np.inf)).astype(F) for c in (c00, c11)]
    return f, box


@pytest.mark.parametrize("top", [-7.5, 0.5])
@pytest.mark.parametrize("s_lo,s_hi", [(0.01, 1.0), (0.3, 6.0), (0.05, 400.0), (20.0, 3000.0)])
@pytest.mark.parametrize("boxed", [True, False])
def test_listed_regions_hold_every_passing_pixel(top, s_lo, s_hi, boxed):
    (u, v, A, B, C, tau), box = gaussians(200_000, 17, s_lo, s_hi)
    if not boxed:                                   # the plain path's records store no box
        box = [np.full_like(u, 1e30)] * 2
    left, right, closed = spans(u, v, A, B, C, tau, box[0], box[1], top)
    listed = hits(left, right)
    # q from the float32 record, in float64
    u, v, A, B, C, tau = (a.astype(np.float64) for a in (u, v, A, B, C, tau))
    missed = 0
    for k in range(8):
        need = np.zeros(u.size, bool)
        for j in range(16):
            dx = 4 * (k % 4) + j % 4 - 7.5 - u
            dy = top + 4 * (k // 4) + j // 4 - v
            need |= A * dx * dx + 2 * B * dx * dy + C * dy * dy <= tau
        if boxed:                                   # an ill-conditioned record's own q is not the ellipse its box bounds
            need &= closed
        missed += int((need & ~listed[:, k]).sum())
    assert missed == 0
    if s_hi <= 6.0:
        assert closed[tau >= 0].all()


def test_nan_is_kept_and_transparent_is_dropped():
    """A conic or opacity that is NaN keeps every region (a visible Gaussian's mean is never NaN:
    its depth would be)."""
    one = np.ones(1, F)
    for bad in range(2, 6):
        args = [0 * one, 0 * one, one, 0 * one, one, 4 * one]
        args[bad] = np.full(1, np.nan, F)
        left, right, _ = spans(*args, 1e30 * one, 1e30 * one, -7.5)
        assert hits(left, right).all()
    left, right, _ = spans(0 * one, 0 * one, one, 0 * one, one, -one, one, one, -7.5)
    assert not hits(left, right).any()
