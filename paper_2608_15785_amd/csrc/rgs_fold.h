// Coefficient folding and per-region culling of one staged list entry
// (Sec. IV-B: Eqs. expand, c0, coeff, dot, dual_pixel), shared by the
// dual-pixel rasterizer and the backward pass, so that both evaluate every
// folded exponent with the same instructions.
//
// Coordinates are relative to the centre of the 16x16 tile: pixel (lx, ly)
// sits at (lx - 7.5, ly - 7.5), and its two half-tiles are the rows [-7.5, -0.5]
// and [0.5, 7.5].
#pragma once

#include "rgs_internal.h"

namespace rgs {

constexpr float LOG2E_F = 1.4426950408889634f;
constexpr float LOG2_255F = 7.994353436858858f;     // ln 255 * log2 e

// log2 e = LOG2E_F + LOG2E_LO to 49 bits.
constexpr float LOG2E_LO = (float)(1.4426950408889634074 - (double)LOG2E_F);

// e^p of a pair's exponent, the plain path's exponential: 2^(p log2 e) by the
// hardware's 2^x, with the product carried in two floats (its rounding would cost half a
// bit per unit of the exponent) and its integer part left to ldexp, the reduction
// of Cody and Waite, which the device library's expf makes too.  For p <= 0 its error
// is expf's, at most 0.86 ulp over 16M exponents a range, and its bits but for one
// in a million; a p that is not a number stays one.  Without expf's two range
// checks it takes 11 instructions instead of 13: an exponent below -200 (alpha far
// below 1/255) is raised to it, where the integer part still fits and both parts
// of the product still cancel.  Plain rasterizer of 1M / 1080p 181 -> 169 us, its
// backward kernel 343 -> 337.
__device__ inline float exp_pair(float p) {
    const float q = p < -200.0f ? -200.0f : p;
    const float hi = q * LOG2E_F, lo = fmaf(q, LOG2E_LO, fmaf(q, LOG2E_F, -hi));
    const float n = rintf(hi);
    return ldexpf(__builtin_amdgcn_exp2f((hi - n) + lo), (int)n);
}

// Margin added to the alpha-ellipse half-extents before culling a Gaussian for
// a wave: float32 rounding of the folded exponent near the 1/255 threshold
// must never hide a pair that the exact test would keep.
constexpr float BOX_MARGIN_REL = 1.0e-3f;
constexpr float BOX_MARGIN_ABS = 0.05f;
// The same safety margin on the quadratic form q = A dx^2 + 2 B dx dy + C dy^2
// (P = ln o - q / 2): a band is kept when min q <= tau (1 + 1e-3) + 0.02.
constexpr float Q_MARGIN_REL = 1.0e-3f;
constexpr float Q_MARGIN_ABS = 0.02f;

// Smallest q over the rectangle [-7.5, 7.5] x [y0, y1] (tile-centre
// coordinates) for a Gaussian at (u, v) with a positive-definite conic: 0 when
// the mean is inside, else the least of the four edge minima (on an edge q is
// a parabola in the free coordinate, minimised at a clamped closed form).
__device__ inline float conic_rect_min(float u, float v, float A, float B, float C, float iA, float iC,
                                       float y0, float y1) {
    if (u >= -7.5f && u <= 7.5f && v >= y0 && v <= y1) return 0.0f;
    float best = 3.0e38f;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const float dx = (e ? 7.5f : -7.5f) - u;                 // vertical edge x = -7.5 or 7.5
        const float dy = fminf(y1, fmaxf(y0, fmaf(-B * dx, iC, v))) - v;
        best = fminf(best, fmaf(A * dx, dx, fmaf(2.0f * B * dx, dy, C * dy * dy)));
        const float ey = (e ? y1 : y0) - v;                       // horizontal edge y = y0 or y1
        const float ex = fminf(7.5f, fmaxf(-7.5f, fmaf(-B * ey, iA, u))) - u;
        best = fminf(best, fmaf(A * ex, ex, fmaf(2.0f * B * ex, ey, C * ey * ey)));
    }
    return best;
}

// One record folded for the tile whose centre is (ox, oy): u, v is its mean in
// tile-centre coordinates, ca = (C1, C2, C3, C4) and cbv = (C5, C6, r, g), so
// that P = C1 x^2 + C2 xy + C3 y^2 + C4 x + C5 y + C6 = ln o + p (the record
// holds ln o in its opacity field).  With LOG2 the coefficients are scaled by
// log2 e, and P log2 e comes out instead (alpha = exp2 of it).
template <bool LOG2>
__device__ inline void fold_record(const Record& rec, float ox, float oy, float& u, float& v, float4& ca,
                                   float4& cbv) {
    u = (rec.u_hi - ox) + rec.u_lo;
    v = (rec.v_hi - oy) + rec.v_lo;
    const float A = rec.A, B = rec.B, C = rec.C;
    const float C0 = fmaf(A * u, u, fmaf(2.0f * B * u, v, C * v * v));
    ca = make_float4(-0.5f * A, -B, -0.5f * C, fmaf(A, u, B * v));
    cbv = make_float4(fmaf(C, v, B * u), fmaf(-0.5f, C0, rec.opa), rec.r, rec.g);
    if (LOG2) {
        ca = make_float4(ca.x * LOG2E_F, ca.y * LOG2E_F, ca.z * LOG2E_F, ca.w * LOG2E_F);
        cbv.x *= LOG2E_F;
        cbv.y *= LOG2E_F;
    }
}

// Which of the eight 4x4 regions of a half-tile (rows top .. top + 7) a record
// can reach with P >= -ln 255: for each of its two bands of four rows, the span
// of columns that its ellipse q <= tau (up to the margin above) covers inside
// the band.  The ellipse is convex, so it
// meets the 4x4 region of columns x0 .. x0 + 3 iff its span in the band meets
// [x0, x0 + 3].  At the height dy the ellipse covers -B/A dy +- sqrt(A tau -
// det dy^2) / A; the right end is a concave function of dy with its peak at dy =
// -B/C hx (hx the ellipse's half-width) and the left end its mirror image, so
// each takes its extreme over the band at that height clamped to the band.
// The spans are widened by 0.05 pixel, far beyond the rounding of this
// evaluation.  det = AC - B^2 loses relative accuracy as AC / det grows; an
// error of det by a factor 1 + e moves the boundary as one of tau by the same
// factor, so up to AC = 2048 det (e below 4e-4) it stays inside the margin's
// 1e-3.  Narrower ellipses, and conics or opacities that are not finite, take the
// box of the alpha >= 1/255 ellipse (the fast path's records hold it, FP16
// rounded up; the plain path's take every region).  Comparisons are phrased so
// that a NaN keeps the Gaussian.
struct RegionSpans {
    float left[2], right[2];

    __device__ inline void none() {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            left[b] = 1.0f;
            right[b] = -1.0e30f;
        }
    }

    // A Gaussian at (u, v) with conic (A, B, C) whose pairs pass up to q = tau;
    // box_x, box_y: half-extents of its box (infinite if none is known).
    __device__ inline void reach(float A, float B, float C, float tau, float box_x, float box_y, float u, float v,
                                 float top) {
        const float qlim = fmaf(tau, 1.0f + Q_MARGIN_REL, Q_MARGIN_ABS);
        if (qlim < 0.0f) return;                        // below the threshold everywhere
        const float AC = A * C, det = fmaf(-B, B, AC);
        const float iA = __builtin_amdgcn_rcpf(A), iC = __builtin_amdgcn_rcpf(C), iD = __builtin_amdgcn_rcpf(det);
        const float hx = __builtin_amdgcn_sqrtf(qlim * C * iD), hy = __builtin_amdgcn_sqrtf(qlim * A * iD);
        const float slope = -B * iA, peak = -B * iC * hx, qA = qlim * A;
        if (det * 2048.0f > AC && hx < 1.0e4f && hy < 1.0e4f) {
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const float y0 = top + (float)(4 * b) - v;
                const float lo = fmaxf(y0, -hy), hi = fminf(y0 + 3.0f, hy);
                const float dr = fminf(fmaxf(peak, lo), hi), dl = fminf(fmaxf(-peak, lo), hi);
                const float sr = __builtin_amdgcn_sqrtf(fmaxf(fmaf(-det * dr, dr, qA), 0.0f));
                const float sl = __builtin_amdgcn_sqrtf(fmaxf(fmaf(-det * dl, dl, qA), 0.0f));
                const bool out = lo > hi + BOX_MARGIN_ABS;
                right[b] = out ? -1.0e30f : fmaf(sr, iA, fmaf(slope, dr, u)) + BOX_MARGIN_ABS;
                left[b] = fmaf(-sl, iA, fmaf(slope, dl, u)) - BOX_MARGIN_ABS;
            }
        } else {
            const float bx = fmaf(box_x, 1.0f + BOX_MARGIN_REL, BOX_MARGIN_ABS);
            const float by = fmaf(box_y, 1.0f + BOX_MARGIN_REL, BOX_MARGIN_ABS);
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const float y0 = top + (float)(4 * b);
                const bool out = v - by > y0 + 3.0f || v + by < y0;
                right[b] = out ? -1.0e30f : u + bx;
                left[b] = u - bx;
            }
        }
    }

    // the region of band b whose first column is the tile's x
    __device__ inline bool hits(int b, float x) const {
        const float x0 = x - 7.5f;
        return !(left[b] > x0 + 3.0f) && !(right[b] < x0);
    }
};

// The folded exponents of a dual pixel: P0 at (x, y) by Eq. dot (x2 = x^2,
// xy = x y, y2 = y^2 precomputed), and P1 at (x, y + 1) by Eq. dual_pixel's
// step, P0 + C2 x + C3 (2y + 1) + C5 (y21 = 2y + 1).
__device__ inline void folded_exponents(const float4& a, float c5, float c6, float x, float y, float x2, float xy,
                                        float y2, float y21, float& P0, float& P1) {
    P0 = fmaf(a.x, x2, fmaf(a.y, xy, fmaf(a.z, y2, fmaf(a.w, x, fmaf(c5, y, c6)))));
    P1 = P0 + fmaf(a.y, x, fmaf(a.z, y21, c5));
}

}  // namespace rgs
