// Reverse mode of the plain render (differentiation of Sec. II-A / III-D's
// image definition with its discrete decisions held fixed), and the device
// update of plain attributes that a training step needs.
//
// raster_backward: two waves per 16x16 tile, the tile's sorted list walked back
// to front in batches staged in LDS.  A pixel starts after its last blended
// pair (the forward pass left its final T, the number of pairs it visited and
// whether it stopped); T before each blended pair is recovered as T_after /
// (1 - alpha).  With S' the colour accumulated behind the pair plus the
// background's share (it starts at T_final bg),
//   dC/dc_j = alpha_j T_j,   dC/dalpha_j = c_j T_j - S'_j / (1 - alpha_j),
// and of S' only its product with dL/dC is carried along.  The nine image-space
// derivatives of a pair (u, v, A, B, C, o, r, g, b) are summed over 4x4-pixel
// regions, then over the tile, and each entry receives one 48-byte partial at
// its position in emission order: no atomics.  Ordered allocation emitted a
// Gaussian's entries contiguously, one per tile of its rectangle in row-major
// order, from the offset the duplication kernel recorded, so that position is
// known from the tile.
//
// grad_gaussian: one thread per Gaussian sums its contiguous partials and
// applies the chain rule through the EWA projection and the SH colour in
// double precision; the SH gradients leave through LDS in coalesced rows.
#include "rgs_fold.h"

namespace rgs {


// ---------------------------------------------------------------------------
// Plain attributes from [n][...] rows.  A block takes 256 Gaussians.  Their
// SH rows (48 floats each, 48 KB together) are read as one contiguous span of
// 16-byte loads into LDS, each row padded to 49 floats so that the plane-wise
// reads below hit distinct banks; each thread then writes its Gaussian's 48
// coefficients into the 48 SH planes, consecutive threads at consecutive
// addresses.  Reading the rows directly, each load instruction of a wave would
// touch 64 rows 192 bytes apart.

constexpr int UPD_THREADS = 256;
constexpr int UPD_SH = 48;
constexpr int UPD_ROW = UPD_SH + 1;

__global__ __launch_bounds__(UPD_THREADS) void k_update_plain(float* __restrict__ planes, uint64_t n_pad, int64_t n,
                                                              const float* __restrict__ means,
                                                              const float* __restrict__ scales,
                                                              const float* __restrict__ quats,
                                                              const float* __restrict__ opacity,
                                                              const float* __restrict__ sh) {
    __shared__ float s_sh[UPD_THREADS * UPD_ROW];
    const int64_t first = (int64_t)blockIdx.x * UPD_THREADS;
    const int64_t rows = n - first < UPD_THREADS ? n - first : UPD_THREADS;
    const int64_t words = rows * UPD_SH;
    const float* src = sh + first * UPD_SH;
    if (rows == UPD_THREADS && (reinterpret_cast<uintptr_t>(src) % 16) == 0) {
        const float4* src4 = reinterpret_cast<const float4*>(src);
        for (int q = threadIdx.x; q < UPD_THREADS * UPD_SH / 4; q += UPD_THREADS) {
            const float4 v = src4[q];
            const float vals[4] = {v.x, v.y, v.z, v.w};
            const int w = 4 * q;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int we = w + e;
                s_sh[(we / UPD_SH) * UPD_ROW + we % UPD_SH] = vals[e];
            }
        }
    } else {
        for (int64_t w = threadIdx.x; w < words; w += UPD_THREADS)
            s_sh[(w / UPD_SH) * UPD_ROW + w % UPD_SH] = src[w];
    }
    __syncthreads();
    const int64_t i = first + threadIdx.x;
    if (i >= n) return;
#pragma unroll
    for (int k = 0; k < 3; ++k) planes[(P_MX + k) * n_pad + i] = means[3 * i + k];
#pragma unroll
    for (int k = 0; k < 3; ++k) planes[(P_SX + k) * n_pad + i] = scales[3 * i + k];
#pragma unroll
    for (int k = 0; k < 4; ++k) planes[(P_QW + k) * n_pad + i] = quats[4 * i + k];
    planes[P_OPA * n_pad + i] = opacity[i];
    planes[P_LNO * n_pad + i] = (float)log((double)opacity[i]);
    const float* row = s_sh + threadIdx.x * UPD_ROW;
#pragma unroll 8
    for (int k = 0; k < UPD_SH; ++k) planes[(P_SH0 + k) * n_pad + i] = row[k];
}

void launch_update_plain(hipStream_t s, float* planes, uint64_t n_pad, int64_t n, const float* means,
                         const float* scales, const float* quats, const float* opacity, const float* sh) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_update_plain, dim3((uint32_t)((n + UPD_THREADS - 1) / UPD_THREADS)), dim3(UPD_THREADS), 0,
                       s, planes, n_pad, n, means, scales, quats, opacity, sh);
}

// ---------------------------------------------------------------------------
// Sums over the eight lanes of each group of the wave, nine values at once:
// lane 8 q + i (i < 4) receives the sums of g[0..3] of group q in o[0..3], lane
// 8 q + 4 + i those of g[4..7], and every lane that of g[8] in o[4].  A mirror
// within the group adds lane i to lane 7 - i; the masked second half of it
// (bank_mask 0xa: lanes 4..7 of each group) puts g[4..7] into the same registers,
// so the two additions within the quad are shared: 19 instructions for 27
// additions.  One block, since the compiler does not know DPP operands inside
// it: the leading s_nop covers the wait states of a DPP read after the last
// write of g or of EXEC, and every DPP operand written inside is written at
// least three instructions before it is read.  EXEC must be full.
__device__ inline void group_sums(const float (&g)[9], float (&o)[5]) {
    asm volatile(
        "s_nop 4\n\t"
        "v_add_f32_dpp %4, %13, %13 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %0, %5, %5 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %1, %6, %6 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %2, %7, %7 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %3, %8, %8 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %0, %9, %9 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
        "v_add_f32_dpp %1, %10, %10 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
        "v_add_f32_dpp %2, %11, %11 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
        "v_add_f32_dpp %3, %12, %12 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
        "v_add_f32_dpp %4, %4, %4 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %1, %1, %1 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %2, %2, %2 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %3, %3, %3 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %4, %4, %4 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %1, %1, %1 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %2, %2, %2 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %3, %3, %3 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        : "=&v"(o[0]), "=&v"(o[1]), "=&v"(o[2]), "=&v"(o[3]), "=&v"(o[4])
        : "v"(g[0]), "v"(g[1]), "v"(g[2]), "v"(g[3]), "v"(g[4]), "v"(g[5]), "v"(g[6]), "v"(g[7]), "v"(g[8]));
}

// The same over the sixteen lanes of each row of the wave: lanes 16 q .. 16 q + 7
// receive the sums of g[0..3] of row q, lanes 16 q + 8 .. 16 q + 15 those of g[4..7].
__device__ inline void row_sums(const float (&g)[9], float (&o)[5]) {
    asm volatile(
        "s_nop 4\n\t"
        "v_add_f32_dpp %4, %13, %13 row_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %0, %5, %5 row_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %1, %6, %6 row_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %2, %7, %7 row_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %3, %8, %8 row_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %0, %9, %9 row_mirror row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %1, %10, %10 row_mirror row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %2, %11, %11 row_mirror row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %3, %12, %12 row_mirror row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %4, %4, %4 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %1, %1, %1 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %2, %2, %2 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %3, %3, %3 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %4, %4, %4 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %1, %1, %1 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %2, %2, %2 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %3, %3, %3 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %4, %4, %4 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %1, %1, %1 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %2, %2, %2 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %3, %3, %3 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        : "=&v"(o[0]), "=&v"(o[1]), "=&v"(o[2]), "=&v"(o[3]), "=&v"(o[4])
        : "v"(g[0]), "v"(g[1]), "v"(g[2]), "v"(g[3]), "v"(g[4]), "v"(g[5]), "v"(g[6]), "v"(g[7]), "v"(g[8]));
}

// Position, in emission order, of Gaussian g's entry for tile (tx, ty).
__device__ inline uint64_t emission_pos(const WsDev& ws, uint32_t g, uint32_t tx, uint32_t ty) {
    const uint64_t rc = ws.rects[g];
    const uint32_t x0 = rc & 0xffff, x1 = (rc >> 16) & 0xffff, y0 = (rc >> 32) & 0xffff;
    return (uint64_t)ws.offsets[g] + (uint64_t)(ty - y0) * (x1 - x0 + 1) + (tx - x0);
}

// Whether the workspace still holds the frame the caller asked for; if not,
// the first workgroup flags it in the header and every workgroup leaves.
__device__ inline bool frame_matches(const WsDev& ws, FrameKey key) {
    const FrameParams* prm = ws.params;
    if (prm->scene_tag == key.scene_tag && prm->cam_hash == key.cam_hash) return true;
    if (blockIdx.x == 0 && threadIdx.x == 0) atomicOr(&ws.header->error, 8u);
    return false;
}

// Adds one blended pair's terms at one pixel to g[9] and steps the pixel's
// state back over the pair.  dx, dy: pixel minus mean; a = (u, v, A, B), m = (C,
// o, r, g), cb: b; d: dL/dC at the pixel; DS = d . S, S the colour behind the
// pair plus the background's share, so that dL/dalpha = Tb (d . col) -
// DS / (1 - alpha), Tb = T / (1 - alpha) the transmittance in front of the pair; the
// difference is taken of T (d . col) and DS, before the division, whose rounding
// would otherwise enter both sides of it.  raw = o e.
__device__ inline void pair_adjoint_plain(float e, float raw, float dx, float dy, const float4& a, const float4& m,
                                          float cb, const float (&d)[3], float& T, float& DS, float (&g)[9]) {
    const float alpha = fminf(ALPHA_MAX, raw);
    const float inv = __builtin_amdgcn_rcpf(1.0f - alpha);
    const float Tb = T * inv;
    const float w = alpha * Tb;
    g[6] = fmaf(w, d[0], g[6]);
    g[7] = fmaf(w, d[1], g[7]);
    g[8] = fmaf(w, d[2], g[8]);
    const float dcol = fmaf(d[0], m.z, fmaf(d[1], m.w, d[2] * cb));
    const float dA = inv * fmaf(T, dcol, -DS);
    DS = fmaf(w, dcol, DS);
    T = Tb;
    const float dRaw = raw <= ALPHA_MAX ? dA : 0.0f;   // a clamped alpha is constant
    g[5] = fmaf(dRaw, e, g[5]);
    const float dP = dRaw * raw;
    g[0] = fmaf(dP, fmaf(a.z, dx, a.w * dy), g[0]);    // dp/du = A dx + B dy
    g[1] = fmaf(dP, fmaf(m.x, dy, a.w * dx), g[1]);    // dp/dv = C dy + B dx
    g[2] = fmaf(-0.5f * dP, dx * dx, g[2]);
    g[3] = fmaf(-dP, dx * dy, g[3]);
    g[4] = fmaf(-0.5f * dP, dy * dy, g[4]);
}

// The same for the training variant, P the pair's exponent in log2 units.  The conic
// terms are left as moments of dL/dP: g[0] += dP dx, g[1] += dP dy, g[2] += dP
// dx^2, g[3] += dP dx dy, g[4] += dP dy^2; an entry's sums of them are turned
// into dL/d(u, v, A, B, C) once (the conic is constant over its pixels).
__device__ inline void pair_adjoint(float P, float dx, float dy, float cr, float cg, float cb, const float (&d)[3],
                                    float& T, float& DS, float (&g)[9]) {
    const float raw = __builtin_amdgcn_exp2f(P);
    const float alpha = fminf(ALPHA_MAX, raw);
    const float inv = __builtin_amdgcn_rcpf(1.0f - alpha);
    const float Tb = T * inv;
    const float w = alpha * Tb;
    g[6] = fmaf(w, d[0], g[6]);
    g[7] = fmaf(w, d[1], g[7]);
    g[8] = fmaf(w, d[2], g[8]);
    const float dcol = fmaf(d[0], cr, fmaf(d[1], cg, d[2] * cb));
    const float dA = inv * fmaf(T, dcol, -DS);
    DS = fmaf(w, dcol, DS);
    T = Tb;
    const float dP = raw <= ALPHA_MAX ? dA * raw : 0.0f;     // a clamped alpha is constant
    g[5] += dP;                                               // dL/d(ln o)
    const float ex = dP * dx, ey = dP * dy;
    g[0] += ex;
    g[1] += ey;
    g[2] = fmaf(ex, dx, g[2]);
    g[3] = fmaf(ex, dy, g[3]);
    g[4] = fmaf(ey, dy, g[4]);
}

// The backward pass in the forward pass's layout: wave w owns the half-tile of
// rows 8 w .. 8 w + 7, the eight lanes of a group own a 4x4 region, a dual pixel
// each (with PIX = 1 four waves of four rows, sixteen lanes a region, a pixel
// each), and walk the region's own list, so that up to eight entries are
// evaluated at once and about 2.3 pixels per blended one (a wave per tile with
// four pixels per lane and skipped bands of four rows: about 3.5; half-tile
// lists: 4.8).  Staging, folding and culling are the forward's (rgs_fold.h), and
// every exponent, alpha and skip decision is the forward's, bit for bit.
//
// An entry's nine sums over a region take 19 DPP additions for eight regions at
// a time and go to a row of LDS of their own; the staging lane of an entry
// adds its rows and writes the partial, so the result does not depend on the
// order in which waves run.  The rows of a batch are those of its lists, one
// list after the other, so no row is written for a region that an entry does
// not reach.  A batch whose rows do not fit BWD_ROWS keeps the entries that do
// (304 rows are a batch of the usual four to five regions an entry, and leave
// LDS for ten workgroups a CU).  The two waves take turns: one adds the rows of a
// batch while the other stages the next.
//
// Bound by VALU issue, about 0.31 instructions per SIMD and cycle with four
// transcendentals in each 150, and at a tile a CU or two by the latency of the
// entry loop; two entries in flight (BWD_UNROLL) shorten it, four take
// registers that cost a wave per SIMD.  Measured, plain at 1M / 1080p, 401x267
// with 20K Gaussians, and the training variant at 1M / 1080p (us): 689, 349, 520
// with the layouts named above; 379, 129, 301 with lists of regions in
// two passes over the ballots; 318, 112, 267 as it stands (one entry at a
// time: 335, 119, 265; four: 348, 108, 291; the next batch's records loaded
// ahead: no change).
constexpr int BWD_BATCH = 64;              // entries staged at once, one per lane of the staging wave
constexpr int BWD_UNROLL = 2;              // entries of a list taken at once; divides 4
constexpr int BWD_REGIONS = 16;            // 4x4 pixels each
constexpr uint32_t BWD_ROWS = 304;         // (entry, region) sums of a batch; at least 16, one entry's

// PIX: pixels per lane, 2 (wave w: rows 8 w .. 8 w + 7) or 1 (four waves, wave w rows 4 w .. 4 w + 3).
template <bool TRAIN, int PIX>
__global__ __launch_bounds__(256 / PIX, 4) void k_raster_backward(FrameDev f, WsDev ws,
                                                                 const uint32_t* __restrict__ vals,
                                                                 const float* __restrict__ dimg,
                                                                 float4* __restrict__ partial, FrameKey key) {
    constexpr uint32_t THREADS = 256 / PIX, REGION_LANES = 16 / PIX, WAVE_REGIONS = 4 * PIX;
    // the batch's entries: (u, v, A, B), (C, o, r, g), (b); TRAIN: (C1, C2, C3, C4), (C5, C6, r, g), (b, u, v)
    __shared__ float4 s_a[BWD_BATCH], s_b[BWD_BATCH], s_c[BWD_BATCH];
    // per region, the slots of the entries that reach it, back to front, and the rows of their sums
    __shared__ uint32_t s_list4[BWD_REGIONS][BWD_BATCH / 4];
    __shared__ uint32_t s_count[BWD_REGIONS], s_base[2][BWD_REGIONS];     // (s_base: by staging wave)
    __shared__ uint32_t s_last[BWD_REGIONS];     // end of the entries that a pixel of the region may have blended
    __shared__ uint32_t s_kept, s_longest[THREADS / 64];
    __shared__ float4 s_row[BWD_ROWS][2];        // sums of one entry over one region
    __shared__ float s_row8[BWD_ROWS];
    if (!frame_matches(ws, key)) return;
    if (blockIdx.x >= (uint32_t)f.n_tiles) return;
    const uint32_t tile = f.ordered ? ws.order[blockIdx.x] : blockIdx.x;   // the rasterizers' schedule
    const uint32_t tx = tile % (uint32_t)f.tiles_x, ty = tile / (uint32_t)f.tiles_x;
    const uint32_t tid = threadIdx.x;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64;
    const uint32_t region = tid / REGION_LANES;
    const uint32_t lx = (region % 4) * 4 + lane % 4;
    const uint32_t ly = (region / 4) * 4 + (PIX == 1 ? lane / 4 % 4 : lane / 4 % 2 * 2);
    const uint32_t px = tx * TILE + lx, py = ty * TILE + ly;
    const uint32_t start = ws.ranges[2 * tile], end = ws.ranges[2 * tile + 1];
    // as the forward pass: tile-centre coordinates, or relative to the tile's corner
    constexpr float CENTRE = TRAIN ? 7.5f : 0.0f;
    const float ox = (float)(tx * TILE) + CENTRE, oy = (float)(ty * TILE) + CENTRE;
    // the dual pixel's rows; with one pixel per lane it is the first or (odd) the second of them
    const bool odd = PIX == 1 && ly % 2 != 0;
    const float x = (float)lx - CENTRE, y = (float)(ly / 2 * 2) - CENTRE, y1 = y + 1.0f;
    const float x2 = x * x, xy = x * y, y2 = y * y, y21 = fmaf(2.0f, y, 1.0f);
    const uint64_t plane = (uint64_t)f.width * f.height;
    const float bg0 = ws.params->cam.bg[0], bg1 = ws.params->cam.bg[1], bg2 = ws.params->cam.bg[2];

    // per pixel: T after the pairs behind, dL/dC, DS = dL/dC . (colour behind + T_final
    // bg), and the end of the pairs [start, last) that may have been blended
    float T[PIX], d[PIX][3], DS[PIX];
    uint32_t last[PIX], rlast = start;
#pragma unroll
    for (int k = 0; k < PIX; ++k) {
        T[k] = 1.0f;
        last[k] = start;
        d[k][0] = d[k][1] = d[k][2] = 0.0f;
        if (px < (uint32_t)f.width && py + k < (uint32_t)f.height) {
            const uint64_t o = (uint64_t)(py + k) * f.width + px;
            T[k] = ws.t_final[o];
            const uint32_t word = ws.n_proc[o];
            last[k] = start + (word & ~N_PROC_STOPPED) - ((word & N_PROC_STOPPED) ? 1u : 0u);
            d[k][0] = dimg[o];
            d[k][1] = dimg[plane + o];
            d[k][2] = dimg[2 * plane + o];
        }
        DS[k] = T[k] * fmaf(d[k][0], bg0, fmaf(d[k][1], bg1, d[k][2] * bg2));
        rlast = max(rlast, last[k]);
    }
#pragma unroll
    for (uint32_t off = 1; off < REGION_LANES; off <<= 1) rlast = max(rlast, (uint32_t)__shfl_xor((int)rlast, off));
    if (lane % REGION_LANES == 0) s_last[region] = rlast;
    __syncthreads();
    uint32_t tile_last = start;
#pragma unroll
    for (int r = 0; r < BWD_REGIONS; ++r) tile_last = max(tile_last, s_last[r]);
    tile_last = __builtin_amdgcn_readfirstlane(tile_last);

    // the staging wave's lane: its entry's position in emission order, the regions it is listed
    // in and its place in each of their lists (a byte each)
    uint64_t my_pos = 0;
    uint32_t my_mask = 0, my_place[4] = {0, 0, 0, 0};
    float eA = 0.0f, eB = 0.0f, eC = 0.0f;     // TRAIN: its conic

    auto list_of = [&](int r) { return reinterpret_cast<uint8_t*>(s_list4[r]); };
    // One wave stages the entries before b_end, lane l the l-th from the back,
    // and lists them in the regions whose pixels they can reach; the last ones,
    // from the first whose rows of sums do not fit, are left to the next batch.
    auto stage = [&](uint32_t b_end) {
        const uint32_t cnt = min(b_end - start, (uint32_t)BWD_BATCH);
        RegionSpans lo, hi;
        lo.none();
        hi.none();
        uint32_t idx = 0xffffffffu;
        if (lane < cnt) {
            idx = b_end - 1 - lane;
            const uint32_t g0 = vals[idx];
            const uint32_t g = g0 < f.n_gaussians ? g0 : 0u;
            const Record rec = ws.records[g];
            my_pos = emission_pos(ws, g, tx, ty);
            float u, v, tau, bx = 1.0e30f, by = 1.0e30f;
            if (TRAIN) {
                float4 ca, cb;
                fold_record<true>(rec, ox, oy, u, v, ca, cb);
                s_a[lane] = ca;
                s_b[lane] = cb;
                s_c[lane] = make_float4(rec.b, u, v, 0.0f);
                eA = rec.A;
                eB = rec.B;
                eC = rec.C;
                tau = 2.0f * (LN255F + rec.opa);
                bx = half_lo(rec.extra);
                by = half_hi(rec.extra);
            } else {
                u = (rec.u_hi - ox) + rec.u_lo;
                v = (rec.v_hi - oy) + rec.v_lo;
                s_a[lane] = make_float4(u, v, rec.A, rec.B);
                s_b[lane] = make_float4(rec.C, rec.opa, rec.r, rec.g);
                s_c[lane].x = rec.b;
                u -= 7.5f;
                v -= 7.5f;
                tau = 2.0f * logf(255.0f * rec.opa);
            }
            lo.reach(rec.A, rec.B, rec.C, tau, bx, by, u, v, -7.5f);
            hi.reach(rec.A, rec.B, rec.C, tau, bx, by, u, v, 0.5f);
        }
        uint32_t mask = 0, below = 0;
        uint64_t m[BWD_REGIONS];
#pragma unroll
        for (int r = 0; r < BWD_REGIONS; ++r) {
            const bool hit = (r < 8 ? lo : hi).hits(r / 4 % 2, (float)(r % 4 * 4)) && idx < s_last[r];
            m[r] = __ballot(hit);
            const uint32_t p = __builtin_amdgcn_mbcnt_hi((uint32_t)(m[r] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m[r], 0u));
            if (hit) list_of(r)[p] = (uint8_t)lane;
            mask |= hit ? 1u << r : 0u;
            my_place[r / 4] = r % 4 ? my_place[r / 4] | p << (8 * (r % 4)) : p;
            below += p;
        }
        my_mask = mask;
        const uint64_t kept = __ballot(below + (uint32_t)__popc(mask) <= BWD_ROWS);
        uint32_t base = 0, longest[THREADS / 64];
#pragma unroll
        for (uint32_t w = 0; w < THREADS / 64; ++w) longest[w] = 0;
#pragma unroll
        for (int r = 0; r < BWD_REGIONS; ++r) {
            const uint32_t n = (uint32_t)__popcll(m[r] & kept);
            if (lane == 0) {
                s_count[r] = n;
                s_base[wave][r] = base;
            }
            base += n;
            longest[r / WAVE_REGIONS] = max(longest[r / WAVE_REGIONS], n);
        }
        if (lane == 0) {
            s_kept = min(cnt, (uint32_t)__popcll(kept));
#pragma unroll
            for (uint32_t w = 0; w < THREADS / 64; ++w) s_longest[w] = longest[w];
        }
    };

    uint32_t stager = 0;
    if (tile_last > start && wave == 0) stage(tile_last);
    for (uint32_t b_end = tile_last; b_end > start;) {
        __syncthreads();                         // the batch is staged, and the last one's rows are read
        const uint32_t kept = __builtin_amdgcn_readfirstlane(s_kept);
        const uint32_t longest = __builtin_amdgcn_readfirstlane(s_longest[wave]);
        const uint32_t n = s_count[region], row0 = s_base[stager][region];
        // slots from which each pixel may have blended
        int lim[PIX];
#pragma unroll
        for (int i = 0; i < PIX; ++i) lim[i] = (int)(b_end - last[i]);
        for (uint32_t k0 = 0; k0 < longest; k0 += BWD_UNROLL) {
            const uint32_t word = s_list4[region][k0 / 4] >> (8 * (k0 % 4));
            uint32_t slot[BWD_UNROLL];
            float4 a[BWD_UNROLL], m[BWD_UNROLL];
            float P[BWD_UNROLL][PIX];          // exponents; plain: e^p
            bool pass[BWD_UNROLL][PIX];
#pragma unroll
            for (int u = 0; u < BWD_UNROLL; ++u) {
                slot[u] = (word >> (8 * u)) % BWD_BATCH;
                a[u] = s_a[slot[u]];
                m[u] = s_b[slot[u]];
            }
            auto row_of = [&](int i) { return i == 1 || odd ? y1 : y; };
#pragma unroll
            for (int u = 0; u < BWD_UNROLL; ++u) {
                const int at = k0 + u < n ? (int)slot[u] : -0x7fffffff;
                if (TRAIN) {
                    float P0, P1;
                    folded_exponents(a[u], m[u].x, m[u].y, x, y, x2, xy, y2, y21, P0, P1);
                    P[u][0] = odd ? P1 : P0;
                    if (PIX == 2) P[u][PIX - 1] = P1;
#pragma unroll
                    for (int i = 0; i < PIX; ++i) pass[u][i] = at >= lim[i] && P[u][i] >= -LOG2_255F;
                } else {
                    const float dx = x - a[u].x;
#pragma unroll
                    for (int i = 0; i < PIX; ++i) {
                        const float dy = row_of(i) - a[u].y;
                        P[u][i] = exp_pair(fmaf(-0.5f, fmaf(a[u].z * dx, dx, m[u].x * dy * dy), -a[u].w * dx * dy));
                        pass[u][i] = at >= lim[i] && fminf(ALPHA_MAX, m[u].y * P[u][i]) >= ALPHA_MIN;
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < BWD_UNROLL; ++u) {
                float g[9];
#pragma unroll
                for (int c = 0; c < 9; ++c) g[c] = 0.0f;
                if (TRAIN) {
                    const float4 c = s_c[slot[u]];
                    const float dx = x - c.y;
#pragma unroll
                    for (int i = 0; i < PIX; ++i)
                        if (pass[u][i])
                            pair_adjoint(P[u][i], dx, row_of(i) - c.z, m[u].z, m[u].w, c.x, d[i], T[i], DS[i], g);
                } else {
                    const float cb = s_c[slot[u]].x;
                    const float dx = x - a[u].x;
#pragma unroll
                    for (int i = 0; i < PIX; ++i)
                        if (pass[u][i])
                            pair_adjoint_plain(P[u][i], m[u].y * P[u][i], dx, row_of(i) - a[u].y, a[u], m[u], cb, d[i],
                                               T[i], DS[i], g);
                }
                float o[5];
                if (PIX == 1) row_sums(g, o);
                else group_sums(g, o);
                if (k0 + u < n && lane % (REGION_LANES / 2) == 0) {
                    const uint32_t row = row0 + k0 + u;
                    s_row[row][lane / (REGION_LANES / 2) % 2] = make_float4(o[0], o[1], o[2], o[3]);
                    if (lane % REGION_LANES == 0) s_row8[row] = o[4];
                }
            }
        }
        __syncthreads();                         // the rows are complete, and the batch's lists are read
        if (wave == stager && lane < kept) {
            float sum[9];            // of the upper half-tile's regions, then the lower's, then both
#pragma unroll
            for (int c = 0; c < 9; ++c) sum[c] = 0.0f;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                float half[9];
#pragma unroll
                for (int c = 0; c < 9; ++c) half[c] = 0.0f;
#pragma unroll
                for (int r = 8 * h; r < 8 * h + 8; ++r) {
                    if (!((my_mask >> r) & 1u)) continue;
                    const uint32_t q = s_base[wave][r] + ((my_place[r / 4] >> (8 * (r % 4))) & 0xffu);
                    const float4 s0 = s_row[q][0], s1 = s_row[q][1];
                    half[0] += s0.x; half[1] += s0.y; half[2] += s0.z; half[3] += s0.w;
                    half[4] += s1.x; half[5] += s1.y; half[6] += s1.z; half[7] += s1.w;
                    half[8] += s_row8[q];
                }
#pragma unroll
                for (int c = 0; c < 9; ++c) sum[c] += half[c];
            }
            if (TRAIN) {
                // moments of dL/dP -> dL/d(u, v, A, B, C) with the entry's conic
                const float m1 = sum[0], m2 = sum[1];
                sum[0] = fmaf(eA, m1, eB * m2);      // dp/du = A dx + B dy
                sum[1] = fmaf(eC, m2, eB * m1);      // dp/dv = C dy + B dx
                sum[2] *= -0.5f;
                sum[3] = -sum[3];
                sum[4] *= -0.5f;
            }
            float4* dst = partial + 3ull * my_pos;
            dst[0] = make_float4(sum[0], sum[1], sum[2], sum[3]);
            dst[1] = make_float4(sum[4], sum[5], sum[6], sum[7]);
            dst[2] = make_float4(sum[8], 0.0f, 0.0f, 0.0f);
        }
        b_end -= kept;
        stager ^= 1u;
        if (wave == stager && b_end > start) stage(b_end);
    }
    // entries no pixel of the tile reached
    for (uint32_t idx = tile_last + tid; idx < end; idx += THREADS) {
        const uint32_t g = vals[idx];
        float4* dst = partial + 3ull * emission_pos(ws, g < f.n_gaussians ? g : 0u, tx, ty);
        dst[0] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        dst[1] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        dst[2] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
}

// With few tiles the longest tile's chain of batches and entries is what takes
// time, and four waves of a pixel per lane shorten it for more instructions in
// all.  Both passes of the backward call with dual and single pixels (us): 20K Gaussians at
// 401x267 (442 tiles) 149 and 127, 640x480 166 and 151, 960x540 (2040) 252 and 245,
// 1024x768 (3072) 301 and 314; 1M at 640x480 561 and 507, 960x540 405 and 371,
// 1024x768 413 and 439, 1080p 468 and 527; training variant, 1M, 379 and 368 at
// 960x540, 377 and 428 at 1024x768.
constexpr int32_t BWD_SINGLE_MAX_TILES = 2048;

void launch_raster_backward(hipStream_t s, const FrameDev& f, const WsDev& ws, const uint32_t* vals,
                            const float* dimg, float4* partial, FrameKey key, bool train) {
    const dim3 grid((uint32_t)f.n_tiles);
    auto launch = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, s, f, ws, vals, dimg, partial, key);
    };
    if (f.n_tiles > BWD_SINGLE_MAX_TILES) {
        if (train) launch(k_raster_backward<true, 2>, 128);
        else launch(k_raster_backward<false, 2>, 128);
    } else {
        if (train) launch(k_raster_backward<true, 1>, 256);
        else launch(k_raster_backward<false, 1>, 256);
    }
}

// ---------------------------------------------------------------------------
// Per-Gaussian gather and chain rule.

// sum_k gY_k dY_k/d(x, y, z) for the degree-3 basis written as polynomials in
// (x, y, z) (the forward basis, in double).
__device__ inline void sh_basis_backward(double x, double y, double z, const double* gY, double& gx,
                                         double& gy, double& gz) {
    const double pi = 3.14159265358979323846;
    const double c1 = sqrt(3.0 / (4.0 * pi));
    const double c2a = 0.5 * sqrt(15.0 / pi), c2b = 0.25 * sqrt(5.0 / pi), c2c = 0.25 * sqrt(15.0 / pi);
    const double c3a = 0.25 * sqrt(35.0 / (2.0 * pi)), c3b = 0.5 * sqrt(105.0 / pi);
    const double c3c = 0.25 * sqrt(21.0 / (2.0 * pi)), c3d = 0.25 * sqrt(7.0 / pi);
    const double c3e = 0.25 * sqrt(105.0 / pi);
    const double xx = x * x, yy = y * y, zz = z * z;
    gx = -c1 * gY[3] + c2a * y * gY[4] - 2.0 * c2b * x * gY[6] - c2a * z * gY[7] + 2.0 * c2c * x * gY[8] -
         c3a * 6.0 * x * y * gY[9] + c3b * y * z * gY[10] + c3c * 2.0 * x * y * gY[11] -
         c3d * 6.0 * x * z * gY[12] - c3c * (4.0 * zz - 3.0 * xx - yy) * gY[13] + c3e * 2.0 * x * z * gY[14] -
         c3a * (3.0 * xx - 3.0 * yy) * gY[15];
    gy = -c1 * gY[1] + c2a * x * gY[4] - c2a * z * gY[5] - 2.0 * c2b * y * gY[6] - 2.0 * c2c * y * gY[8] -
         c3a * (3.0 * xx - 3.0 * yy) * gY[9] + c3b * x * z * gY[10] - c3c * (4.0 * zz - xx - 3.0 * yy) * gY[11] -
         c3d * 6.0 * y * z * gY[12] + c3c * 2.0 * x * y * gY[13] - c3e * 2.0 * y * z * gY[14] +
         c3a * 6.0 * x * y * gY[15];
    gz = c1 * gY[2] - c2a * y * gY[5] + 4.0 * c2b * z * gY[6] - c2a * x * gY[7] + c3b * x * y * gY[10] -
         c3c * 8.0 * y * z * gY[11] + c3d * (6.0 * zz - 3.0 * xx - 3.0 * yy) * gY[12] - c3c * 8.0 * x * z * gY[13] +
         c3e * (xx - yy) * gY[14];
}

__device__ inline void sh_basis_double(double x, double y, double z, double* Y) {
    const double pi = 3.14159265358979323846;
    const double c1 = sqrt(3.0 / (4.0 * pi));
    const double c2a = 0.5 * sqrt(15.0 / pi), c2b = 0.25 * sqrt(5.0 / pi), c2c = 0.25 * sqrt(15.0 / pi);
    const double c3a = 0.25 * sqrt(35.0 / (2.0 * pi)), c3b = 0.5 * sqrt(105.0 / pi);
    const double c3c = 0.25 * sqrt(21.0 / (2.0 * pi)), c3d = 0.25 * sqrt(7.0 / pi);
    const double c3e = 0.25 * sqrt(105.0 / pi);
    const double xx = x * x, yy = y * y, zz = z * z;
    Y[0] = 0.5 / sqrt(pi);
    Y[1] = -c1 * y;
    Y[2] = c1 * z;
    Y[3] = -c1 * x;
    Y[4] = c2a * x * y;
    Y[5] = -c2a * y * z;
    Y[6] = c2b * (2.0 * zz - xx - yy);
    Y[7] = -c2a * x * z;
    Y[8] = c2c * (xx - yy);
    Y[9] = -c3a * y * (3.0 * xx - yy);
    Y[10] = c3b * x * y * z;
    Y[11] = -c3c * y * (4.0 * zz - xx - yy);
    Y[12] = c3d * z * (2.0 * zz - 3.0 * xx - 3.0 * yy);
    Y[13] = -c3c * x * (4.0 * zz - xx - yy);
    Y[14] = c3e * z * (xx - yy);
    Y[15] = -c3a * x * (xx - 3.0 * yy);
}

constexpr int GRAD_THREADS = 64;

// Gradients of Gaussian i from the sum of its count partials by the chain rule.
// The SH gradients go to dsh (48 floats, LDS), the rest straight to global memory.
__device__ inline void grad_one(const PlainSceneDev& sc, const CamDev& cam, const WsDev& ws, const float (&acc)[9],
                                uint32_t count, const GradOut& go, int64_t i, float4* dsh, bool lno_opacity) {
    double gs[9];
#pragma unroll
    for (int c = 0; c < 9; ++c) gs[c] = 0.0;
    if (count) {
#pragma unroll
        for (int c = 0; c < 9; ++c) gs[c] = acc[c];
        if (lno_opacity) {      // dL/do = dL/d(ln o) / o
            const double o = sc.base[P_OPA * sc.n_pad + i];
            gs[5] = o > 0.0 ? gs[5] / o : 0.0;
        }
    }
    if (go.screen) {
#pragma unroll
        for (int c = 0; c < 9; ++c) go.screen[9 * i + c] = (float)gs[c];
    }
    float* dm = go.means + 3 * i;
    float* ds = go.scales + 3 * i;
    float* dq = go.quats + 4 * i;
    if (!count) {
#pragma unroll
        for (int k = 0; k < 3; ++k) dm[k] = 0.0f, ds[k] = 0.0f;
#pragma unroll
        for (int k = 0; k < 4; ++k) dq[k] = 0.0f;
        go.opacity[i] = 0.0f;
        for (int k = 0; k < 12; ++k) dsh[k] = make_float4(0.f, 0.f, 0.f, 0.f);
        return;
    }
    const float* P = sc.base;
    const uint64_t np = sc.n_pad;
    const double mx = P[P_MX * np + i], my = P[P_MY * np + i], mz = P[P_MZ * np + i];
    const double s[3] = {P[P_SX * np + i], P[P_SY * np + i], P[P_SZ * np + i]};
    const double qw0 = P[P_QW * np + i], qx0 = P[P_QX * np + i], qy0 = P[P_QY * np + i], qz0 = P[P_QZ * np + i];
    const double* r = cam.r;
    const double g_u = gs[0], g_v = gs[1], g_A = gs[2], g_B = gs[3], g_C = gs[4];

    // forward quantities (the forward pass's expressions)
    const double tx = r[0] * mx + r[1] * my + r[2] * mz + cam.t[0];
    const double ty = r[3] * mx + r[4] * my + r[5] * mz + cam.t[1];
    const double d = r[6] * mx + r[7] * my + r[8] * mz + cam.t[2];
    const double nq = sqrt(qw0 * qw0 + qx0 * qx0 + qy0 * qy0 + qz0 * qz0);
    const double w = qw0 / nq, x = qx0 / nq, y = qy0 / nq, z = qz0 / nq;
    double R[3][3];
    R[0][0] = 1.0 - 2.0 * (y * y + z * z);
    R[0][1] = 2.0 * (x * y - w * z);
    R[0][2] = 2.0 * (x * z + w * y);
    R[1][0] = 2.0 * (x * y + w * z);
    R[1][1] = 1.0 - 2.0 * (x * x + z * z);
    R[1][2] = 2.0 * (y * z - w * x);
    R[2][0] = 2.0 * (x * z - w * y);
    R[2][1] = 2.0 * (y * z + w * x);
    R[2][2] = 1.0 - 2.0 * (x * x + y * y);
    double M[3][3], S[3][3];
    for (int a = 0; a < 3; ++a)
        for (int k = 0; k < 3; ++k) M[a][k] = R[a][k] * s[k];
    for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b) S[a][b] = M[a][0] * M[b][0] + M[a][1] * M[b][1] + M[a][2] * M[b][2];
    const double limx = J_CLAMP * cam.tanx, limy = J_CLAMP * cam.tany;
    const double rx = tx / d, ry = ty / d;
    const bool inx = rx > -limx && rx < limx, iny = ry > -limy && ry < limy;
    const double xc = fmin(limx, fmax(-limx, rx)) * d;
    const double yc = fmin(limy, fmax(-limy, ry)) * d;
    const double dd = d * d;
    const double j00 = cam.fx / d, j02 = -(cam.fx * xc) / dd;
    const double j11 = cam.fy / d, j12 = -(cam.fy * yc) / dd;
    double T0[3], T1[3];
    for (int k = 0; k < 3; ++k) {
        T0[k] = j00 * r[k] + j02 * r[6 + k];
        T1[k] = j11 * r[3 + k] + j12 * r[6 + k];
    }
    double ST0[3], ST1[3];
    for (int a = 0; a < 3; ++a) {
        ST0[a] = S[a][0] * T0[0] + S[a][1] * T0[1] + S[a][2] * T0[2];
        ST1[a] = S[a][0] * T1[0] + S[a][1] * T1[1] + S[a][2] * T1[2];
    }
    const double c00 = T0[0] * ST0[0] + T0[1] * ST0[1] + T0[2] * ST0[2] + DILATION;
    const double c01 = T0[0] * ST1[0] + T0[1] * ST1[1] + T0[2] * ST1[2];
    const double c11 = T1[0] * ST1[0] + T1[1] * ST1[1] + T1[2] * ST1[2] + DILATION;
    const double det = c00 * c11 - c01 * c01;
    const double id = 1.0 / det, id2 = id * id;

    // conic (A, B, C) = (c11, -c01, c00) / det  ->  Sigma' entries
    const double g00 = g_A * (-c11 * c11 * id2) + g_B * (c01 * c11 * id2) + g_C * (id - c00 * c11 * id2);
    const double g11 = g_A * (id - c11 * c00 * id2) + g_B * (c01 * c00 * id2) + g_C * (-c00 * c00 * id2);
    const double g01 = g_A * (2.0 * c01 * c11 * id2) + g_B * (-id - 2.0 * c01 * c01 * id2) +
                       g_C * (2.0 * c00 * c01 * id2);
    // Sigma' = T Sigma T^T
    double gT0[3], gT1[3];
    for (int a = 0; a < 3; ++a) {
        gT0[a] = 2.0 * g00 * ST0[a] + g01 * ST1[a];
        gT1[a] = 2.0 * g11 * ST1[a] + g01 * ST0[a];
    }
    // symmetrised dL/dSigma: GS + GS^T with GS = g00 T0 T0^T + g01 T0 T1^T + g11 T1 T1^T
    double GSs[3][3];
    for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b)
            GSs[a][b] = 2.0 * g00 * T0[a] * T0[b] + g01 * (T0[a] * T1[b] + T0[b] * T1[a]) +
                        2.0 * g11 * T1[a] * T1[b];
    // T = J R_w
    const double g_j00 = gT0[0] * r[0] + gT0[1] * r[1] + gT0[2] * r[2];
    const double g_j02 = gT0[0] * r[6] + gT0[1] * r[7] + gT0[2] * r[8];
    const double g_j11 = gT1[0] * r[3] + gT1[1] * r[4] + gT1[2] * r[5];
    const double g_j12 = gT1[0] * r[6] + gT1[1] * r[7] + gT1[2] * r[8];
    // J and (u, v) -> camera-space t
    const double g_tx = g_u * cam.fx / d + (inx ? g_j02 * (-cam.fx / dd) : 0.0);
    const double g_ty = g_v * cam.fy / d + (iny ? g_j12 * (-cam.fy / dd) : 0.0);
    const double sgx = rx > 0.0 ? 1.0 : -1.0, sgy = ry > 0.0 ? 1.0 : -1.0;
    const double g_d = g_u * (-cam.fx * tx / dd) + g_v * (-cam.fy * ty / dd) + g_j00 * (-cam.fx / dd) +
                       g_j11 * (-cam.fy / dd) +
                       g_j02 * (inx ? 2.0 * cam.fx * tx / (dd * d) : cam.fx * sgx * limx / dd) +
                       g_j12 * (iny ? 2.0 * cam.fy * ty / (dd * d) : cam.fy * sgy * limy / dd);
    double gmu[3];
    for (int k = 0; k < 3; ++k) gmu[k] = r[k] * g_tx + r[3 + k] * g_ty + r[6 + k] * g_d;
    // Sigma = M M^T, M = R diag(s)
    double gM[3][3], gR[3][3];
    for (int a = 0; a < 3; ++a)
        for (int k = 0; k < 3; ++k) gM[a][k] = GSs[a][0] * M[0][k] + GSs[a][1] * M[1][k] + GSs[a][2] * M[2][k];
    for (int k = 0; k < 3; ++k) ds[k] = (float)(gM[0][k] * R[0][k] + gM[1][k] * R[1][k] + gM[2][k] * R[2][k]);
    for (int a = 0; a < 3; ++a)
        for (int k = 0; k < 3; ++k) gR[a][k] = gM[a][k] * s[k];
    // rotation of the unit quaternion (w, x, y, z)
    const double gw = 2.0 * (-z * gR[0][1] + y * gR[0][2] + z * gR[1][0] - x * gR[1][2] - y * gR[2][0] + x * gR[2][1]);
    const double gx = 2.0 * (y * gR[0][1] + z * gR[0][2] + y * gR[1][0] - 2.0 * x * gR[1][1] - w * gR[1][2] +
                             z * gR[2][0] + w * gR[2][1] - 2.0 * x * gR[2][2]);
    const double gy = 2.0 * (-2.0 * y * gR[0][0] + x * gR[0][1] + w * gR[0][2] + x * gR[1][0] + z * gR[1][2] -
                             w * gR[2][0] + z * gR[2][1] - 2.0 * y * gR[2][2]);
    const double gz = 2.0 * (-2.0 * z * gR[0][0] - w * gR[0][1] + x * gR[0][2] + w * gR[1][0] - 2.0 * z * gR[1][1] +
                             y * gR[1][2] + x * gR[2][0] + y * gR[2][1]);
    const double qdot = w * gw + x * gx + y * gy + z * gz;
    dq[0] = (float)((gw - w * qdot) / nq);
    dq[1] = (float)((gx - x * qdot) / nq);
    dq[2] = (float)((gy - y * qdot) / nq);
    dq[3] = (float)((gz - z * qdot) / nq);
    go.opacity[i] = (float)gs[5];

    // colour: a channel clamped at 0 in the forward pass has no gradient
    const Record rec = ws.records[i];
    const double ga[3] = {rec.r > 0.0f ? gs[6] : 0.0, rec.g > 0.0f ? gs[7] : 0.0, rec.b > 0.0f ? gs[8] : 0.0};
    double cp[3];
    for (int k = 0; k < 3; ++k) cp[k] = -(r[k] * cam.t[0] + r[3 + k] * cam.t[1] + r[6 + k] * cam.t[2]);
    const double vx = mx - cp[0], vy = my - cp[1], vz = mz - cp[2];
    const double vlen = sqrt(vx * vx + vy * vy + vz * vz);
    const double ux = vx / vlen, uy = vy / vlen, uz = vz / vlen;
    double Y[16], gY[16];
    sh_basis_double(ux, uy, uz, Y);
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        double dot = 0.0;
#pragma unroll
        for (int c = 0; c < 3; ++c) dot += (double)P[(P_SH0 + 3 * k + c) * np + i] * ga[c];
        gY[k] = dot;
    }
#pragma unroll
    for (int q = 0; q < 12; ++q)
        dsh[q] = make_float4((float)(Y[4 * q / 3] * ga[4 * q % 3]), (float)(Y[(4 * q + 1) / 3] * ga[(4 * q + 1) % 3]),
                             (float)(Y[(4 * q + 2) / 3] * ga[(4 * q + 2) % 3]),
                             (float)(Y[(4 * q + 3) / 3] * ga[(4 * q + 3) % 3]));
    double gdx, gdy, gdz;
    sh_basis_backward(ux, uy, uz, gY, gdx, gdy, gdz);
    const double dot = ux * gdx + uy * gdy + uz * gdz;
    gmu[0] += (gdx - ux * dot) / vlen;
    gmu[1] += (gdy - uy * dot) / vlen;
    gmu[2] += (gdz - uz * dot) / vlen;
    for (int k = 0; k < 3; ++k) dm[k] = (float)gmu[k];
}

// The partials of a workgroup's Gaussians follow one another in emission order.
// They pass through LDS in spans of GRAD_STAGE, read as one run of 16-byte loads
// while the span before is added, and each thread adds its Gaussian's in order,
// four rows' LDS reads in flight.  Bound by HBM at 1M Gaussians (planes, records,
// partials and gradients: 620 MB, 120 us as a copy) and on small scenes by the
// latency of the partials.  Measured, 1M / 1080p and 20K at 401x267 (us): each
// thread reading its own rows from global memory, and SH rows of 48 floats in LDS
// (16-way bank conflicts), 165 and 47; through LDS 138 and 44; four rows at a
// time 135 and 33; the next span's loads ahead 123 and 24; workgroups of 64
// threads instead of 128 124 and 22.
constexpr int GRAD_ROW4 = 13;                  // a Gaussian's SH gradients in LDS: 48 floats and a pad of 4
constexpr uint32_t GRAD_STAGE = GRAD_THREADS * GRAD_ROW4 / 3;

template <bool LNO>
__global__ __launch_bounds__(GRAD_THREADS) void k_grad_gaussian(PlainSceneDev sc, CamDev cam, WsDev ws,
                                                                const float4* __restrict__ partial,
                                                                GradOut go, FrameKey key) {
    __shared__ float4 s_buf[GRAD_THREADS * GRAD_ROW4];
    __shared__ uint32_t s_lo[GRAD_THREADS / 64], s_hi[GRAD_THREADS / 64];
    const int64_t first = (int64_t)blockIdx.x * GRAD_THREADS;
    const int64_t i = first + threadIdx.x;
    // the workspace holds another frame than the caller's: all gradients are zero
    const bool refused = ws.params->scene_tag != key.scene_tag || ws.params->cam_hash != key.cam_hash;
    const uint32_t count = i < sc.n && !refused ? ws.counts[i] : 0u;
    const uint32_t begin = count ? ws.offsets[i] : 0u, end = begin + count;
    uint32_t lo = count ? begin : 0xffffffffu, hi = end;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        lo = min(lo, (uint32_t)__shfl_xor((int)lo, off));
        hi = max(hi, (uint32_t)__shfl_xor((int)hi, off));
    }
    if (lane_id() == 0) {
        s_lo[threadIdx.x / 64] = lo;
        s_hi[threadIdx.x / 64] = hi;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < GRAD_THREADS / 64; ++w) {
        lo = min(lo, s_lo[w]);
        hi = max(hi, s_hi[w]);
    }
    float acc[9];
#pragma unroll
    for (int c = 0; c < 9; ++c) acc[c] = 0.0f;
    // the next span's loads are in flight while this one is added
    float4 next[GRAD_ROW4];
    auto fetch = [&](uint32_t c0) {
        const uint32_t words = c0 < hi ? 3 * min(GRAD_STAGE, hi - c0) : 0;
        const float4* src = partial + 3ull * c0;
#pragma unroll
        for (uint32_t k = 0; k < GRAD_ROW4; ++k) {
            const uint32_t q = k * GRAD_THREADS + threadIdx.x;
            next[k] = q < words ? src[q] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    };
    fetch(lo);
    for (uint32_t c0 = lo; c0 < hi; c0 += GRAD_STAGE) {
#pragma unroll
        for (uint32_t k = 0; k < GRAD_ROW4; ++k) s_buf[k * GRAD_THREADS + threadIdx.x] = next[k];
        __syncthreads();
        if (c0 + GRAD_STAGE < hi) fetch(c0 + GRAD_STAGE);
        const uint32_t e1 = min(end, c0 + GRAD_STAGE);
        uint32_t e = max(begin, c0);
        for (; e + 4 <= e1; e += 4) {
            const float4* p = s_buf + 3 * (e - c0);
            float4 p0[4], p1[4];
            float p2[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                p0[u] = p[3 * u];
                p1[u] = p[3 * u + 1];
                p2[u] = p[3 * u + 2].x;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                acc[0] += p0[u].x; acc[1] += p0[u].y; acc[2] += p0[u].z; acc[3] += p0[u].w;
                acc[4] += p1[u].x; acc[5] += p1[u].y; acc[6] += p1[u].z; acc[7] += p1[u].w;
                acc[8] += p2[u];
            }
        }
        for (; e < e1; ++e) {
            const float4* p = s_buf + 3 * (e - c0);
            const float4 p0 = p[0], p1 = p[1];
            acc[0] += p0.x; acc[1] += p0.y; acc[2] += p0.z; acc[3] += p0.w;
            acc[4] += p1.x; acc[5] += p1.y; acc[6] += p1.z; acc[7] += p1.w;
            acc[8] += p[2].x;
        }
        __syncthreads();
    }
    if (i < sc.n) grad_one(sc, cam, ws, acc, count, go, i, s_buf + GRAD_ROW4 * threadIdx.x, LNO);
    __syncthreads();
    const int64_t rows = sc.n - first < GRAD_THREADS ? sc.n - first : GRAD_THREADS;
    float* dst = go.sh + 48 * first;
    if (reinterpret_cast<uintptr_t>(dst) % 16 == 0) {
        float4* dst4 = reinterpret_cast<float4*>(dst);
        for (int k = threadIdx.x; k < (int)rows * 12; k += GRAD_THREADS) dst4[k] = s_buf[k / 12 * GRAD_ROW4 + k % 12];
    } else {
        const float* buf = reinterpret_cast<const float*>(s_buf);
        for (int k = threadIdx.x; k < (int)rows * 48; k += GRAD_THREADS) dst[k] = buf[k / 48 * 4 * GRAD_ROW4 + k % 48];
    }
}

void launch_grad_gaussian(hipStream_t s, const PlainSceneDev& sc, const CamDev& cam, const WsDev& ws,
                          const float4* partial, const GradOut& go, bool lno_opacity, FrameKey key) {
    if (sc.n <= 0) return;
    const dim3 grid((uint32_t)((sc.n + GRAD_THREADS - 1) / GRAD_THREADS)), block(GRAD_THREADS);
    if (lno_opacity) hipLaunchKernelGGL(k_grad_gaussian<true>, grid, block, 0, s, sc, cam, ws, partial, go, key);
    else hipLaunchKernelGGL(k_grad_gaussian<false>, grid, block, 0, s, sc, cam, ws, partial, go, key);
}

}  // namespace rgs
