// Tile rasterizers (Sec. III-D, Sec. IV-B).
//
// A tile (16x16 pixels) is blended front to back over its sorted list, the
// Gaussian records of each batch staged in LDS; every thread owns fixed pixels
// and keeps their transmittance T and colour in registers.  A pair is skipped
// when its opacity is below 1/255, blending of a pixel stops at the first pair
// that would take T below 1e-4, and alpha is clamped at 0.99
// (Eq. opacity_clamped).  A workgroup leaves as soon as all its pixels have
// stopped (checked at every batch).
//
// `k_raster` serves every path: a workgroup is one wave and blends one
// half-tile, a dual pixel (x, y), (x, y + 1) per lane, each of the half-tile's
// eight 4x4 regions walking a list of its own (in frames of few tiles a quarter
// of a tile, a pixel per lane, in four regions).  What a pair's alpha is
// computed from is its template argument:
//   * EXP_PLAIN, the 3DGS baseline: the exponent of Eq. power from (x - u,
//     y - v) and an accurate exponential (exp_pair);
//   * EXP_BITS, the paper's Sec. IV-B: coefficient folding (Eqs. expand, c0,
//     coeff, dot): while a batch is staged the conic, mean and ln o are folded
//     into C1..C6 so that the folded exponent P = p + ln o (Eq.
//     folded_exponent) is C1 x^2 + C2 xy + C3 y^2 + C4 x + C5 y + C6, five FMAs
//     per pixel with x^2, xy, y^2, x, y hoisted.  The paper's b is the doubled
//     off-diagonal of the conic, so C2 = -B and the 0.5 b terms become B.
//     Coordinates are taken relative to the tile centre, which keeps |x|, |y|
//     <= 7.5 and the folded terms small enough for float32 at any image size;
//     dual-pixel evaluation (Eq. dual_pixel): the second exponent is P(x,y) +
//     C2 x + C3 (2y + 1) + C5, and both pixels reuse one LDS read of the
//     coefficients; the range-aware bit-level exponential (Eq. fma_exp): for P
//     in [-ln 255, 0] the bits of exp(P) are built as the integer
//     floor(P 2^23 log2 e + 2^23 (127 - sigma)), sigma = 0.045677, one FMA and
//     one float-to-int conversion.  The skip test is made on P itself;
//   * EXP_HW2: the same with log2 e folded into C1..C6 and alpha = min(0.99,
//     exp2(P)) from the hardware exp2, over the fast path's records or, as the
//     training variant of the plain path, over the plain path's float32 records
//     (which then carry ln o and the box); EXP_LIBM: an ablation.
// With TRAIN it also leaves each pixel's final T and visited-pair count; the
// backward pass recomputes every alpha from them bit for bit.
//
// The lists.  A lane costs the same whether its pair passes the skip test or
// not, so what bounds the kernel (VALU issue: 0.29 wave instructions per SIMD
// and cycle over the launch at 1M / 1080p, of the 0.40 that eight waves of
// independent FMA chains reach) is how many pairs it evaluates for each one it blends: at 1M /
// 1080p 5.1 with one list per 16x8 half-tile, 3.4 with one per 8x8, 2.64 with one per
// 4x4 (eight lists walked side by side, to the length of the longest of each
// batch), 2.1 with one per 4x2, whose lists would cost twice the staging.
// While a batch is staged, one entry per lane, each entry finds the columns
// that its alpha >= 1/255 ellipse covers in each band of four rows (RegionSpans
// in rgs_fold.h), and the eight lists take its index in depth order from eight
// ballots.  A culled pair would have failed the skip test, so no result
// changes.  The stop test is made once per group of four entries: T never
// grows, so a pixel stops inside a group iff it is below the limit at its end,
// and such a group is blended again entry by entry.
// Measured, kernel alone (1M / 1080p orbit frame, 3M / 4K orbit frame): fast
// 115 -> 87 and 322 -> 242 us, plain 612 -> 172 us at 1080p, against one list
// per half-tile (plain: none) and two waves per workgroup.  Batches of 64, 128
// and 192 entries differ by less than 3 % at 1080p (192: less occupancy, +7 % at
// 4K); two waves per workgroup with barriers 96 and 285 us; a whole tile per
// wave with four pixels per lane 103 and 264 us; the exponents and colours on
// v_mfma_f32_4x4x1 (bit for bit the same FMAs) 129 us against 115: a float32
// matrix instruction occupies the vector ALUs (16 of them and 64 FMAs take 530
// cycles, 165 and 166 alone).
//
// Workgroups b, b + 8, .. blend the parts of tile ws.order[..] (longest
// lists first, so that the grid does not end on a few long tiles; see the
// tile-order kernel) in frames that take the schedule, else of tiles in
// row-major order.  Workgroups are dispatched to the 8 XCDs round-robin, so
// all parts of a tile share an L2, and the tiles' uneven work spreads evenly
// over the XCDs.
#include "rgs_fold.h"

namespace rgs {

// 2^23 log2(e) = 12102203.16 and 2^23 (127 - 0.045677) = 1064970049.55,
// rounded to the nearest float32 (spacing 1 and 64 at these magnitudes).
constexpr float FEXP_A = 12102203.0f;
constexpr float FEXP_B = 1064970048.0f;

// ---------------------------------------------------------------------------

constexpr int LIST_UNROLL = 4;
// What a pair's alpha is computed from.  The first three take it from the
// folded exponent P = p + ln o; EXP_PLAIN is the 3DGS baseline.
enum ExpMode : int {
    EXP_BITS = 0,   // Eq. fma_exp: the bit-level exponential (the paper's fast path)
    EXP_LIBM = 1,   // min(0.99, expf(P)): the exponential's ablation
    EXP_HW2 = 2,    // min(0.99, v_exp_f32(P log2 e)) with log2 e folded into C1..C6
    EXP_PLAIN = 3,  // min(0.99, o expf(p)), p by Eq. power from (x - u, y - v)
};

// Alpha of a pair that passes the skip test, from its folded exponent P.
template <int EXPM>
__device__ inline float kept_alpha(float P) {
    if (EXPM == EXP_LIBM) return fminf(ALPHA_MAX, expf(P));      // the exponential's ablation
    if (EXPM == EXP_HW2) return fminf(ALPHA_MAX, __builtin_amdgcn_exp2f(P));
    // min(0.99, exp_hat(P)) without the minimum, which cannot bind here: P = ln o - q/2 with
    // ln o <= 0 and q >= 0, and for a kept pair every term of its float32 evaluation is below
    // ~1600 in magnitude (conic entries <= 1/0.3, coordinates within a tile), so P < 1e-3 and
    // exp_hat(P) < 0.978
    return __int_as_float((int)fmaf(P, FEXP_A, FEXP_B));
}

// Alpha of a pair, 0 when P is below the threshold thr (the skip threshold, or NaN
// for a pixel that has stopped or lies outside the image: no P passes).
template <int EXPM>
__device__ inline float alpha_of(float P, float thr) {
    const float al = kept_alpha<EXPM>(P);
    return P >= thr ? al : 0.0f;
}

// A lane's pixels: a dual pixel (x, y), (x, y + 1), or with PIX = 1 one of the two
// (odd: the second); in tile-centre coordinates with the monomials of Eq. dot,
// or for EXP_PLAIN relative to the tile's corner.
struct LanePixels {
    float x, y, x2, xy, y2, y21;
    bool odd;
};

// The pixels' alphas of a staged entry; thr: the thresholds of alpha_of, for
// EXP_PLAIN on alpha itself.  A single pixel's alpha is that of the dual pixel, bit
// for bit.
template <int EXPM, int PIX>
__device__ inline void pair_alphas(const float4& a, const float2& c, const LanePixels& d, const float (&thr)[PIX],
                                   float (&al)[PIX]) {
    if (EXPM == EXP_PLAIN) {
        // a = (u, v, A, B), c = (C, o)
        const float dx = d.x - a.x;
#pragma unroll
        for (int i = 0; i < PIX; ++i) {
            const float row = PIX == 1 ? d.y + (d.odd ? 1.0f : 0.0f) : d.y + (float)i;
            const float dy = row - a.y;
            const float p = fmaf(-0.5f, fmaf(a.z * dx, dx, c.x * dy * dy), -a.w * dx * dy);
            al[i] = fminf(ALPHA_MAX, c.y * exp_pair(p));
            al[i] = al[i] >= thr[i] ? al[i] : 0.0f;
        }
    } else {
        float P0, P1;
        folded_exponents(a, c.x, c.y, d.x, d.y, d.x2, d.xy, d.y2, d.y21, P0, P1);
        if (PIX == 1) {
            al[0] = alpha_of<EXPM>(d.odd ? P1 : P0, thr[0]);
        } else {
            al[0] = alpha_of<EXPM>(P0, thr[0]);
            al[PIX - 1] = alpha_of<EXPM>(P1, thr[PIX - 1]);
        }
    }
}

// T behind a pair of opacity al and weight w = al T.
template <int EXPM>
__device__ inline float behind(float T, float al, float w) {
    return EXPM == EXP_PLAIN ? T * (1.0f - al) : T - w;
}

// A workgroup is one wave and blends one half-tile (16x8 pixels), a dual pixel
// per lane, in eight regions of 4x4 pixels, or with PIX = 1 a quarter (8x8), a
// pixel per lane, in four: the lanes of a region walk the region's own list.
constexpr int REGION = 4;
constexpr int FAST_BATCH = 64;                    // entries staged at once, one per lane
constexpr int FAST_LIST = FAST_BATCH + LIST_UNROLL;
constexpr uint32_t XCDS = 8;                      // workgroups go to the XCDs round-robin

// The outcome of the frame, decided by now, to the host (FrameStamp).
__device__ void export_stamp(const WsDev& ws) {
    const FrameParams* prm = ws.params;
    FrameStamp* dst = prm->stamp;
    if (!dst) return;
    const WsHeader* h = ws.header;
    dst->n_entries = h->n_entries;
    dst->n_visible = h->n_visible;
    dst->capacity = h->capacity;
    dst->path = h->path;
    dst->passes = h->passes;
    dst->overflow = h->overflow;
    dst->error = h->error;
    dst->scene_tag = prm->scene_tag;
    dst->cam_hash = prm->cam_hash;
    __threadfence_system();
    __hip_atomic_store(&dst->seq, prm->stamp_seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The workgroup that exports the stamp: among the first that the grid starts (the
// kernels that export it run 6 to 8 waves a SIMD, so 256 CUs hold 6144 or more), but not
// one of the longest tiles'.
constexpr uint32_t STAMP_BLOCK = 4096;

// TRAIN: a path with a backward pass (EXP_PLAIN, and its training variant:
// EXP_HW2 over the plain path's records, which then hold ln o and the
// alpha-ellipse box): every render also leaves each pixel's final T and
// visited-pair count for it.
template <bool COUNT, int EXPM, bool TRAIN, int PIX>
__global__ __launch_bounds__(64) void k_raster(FrameDev f, WsDev ws, const uint32_t* __restrict__ vals) {
    constexpr uint32_t PARTS = 4 / PIX;               // of a tile
    constexpr int REGIONS = 4 * PIX;                  // of a part
    constexpr uint32_t REGION_LANES = 16 / PIX;
    // the batch's folded entries, and at FAST_BATCH an inert one (P = -1e30, or o = 0: always
    // skipped), in three arrays of 16 bytes an entry, so that one address serves all three:
    // (C1, C2, C3, C4), (C5, C6, r, g), b; EXP_PLAIN: (u, v, A, B), (C, o, r, g), b
    constexpr uint32_t PART = (FAST_BATCH + 1) * 16;
    __shared__ __align__(16) char s_ent[3 * PART];
    auto coef = [&](uint32_t at) { return *reinterpret_cast<const float4*>(s_ent + at); };
    auto tail = [&](uint32_t at) { return *reinterpret_cast<const float2*>(s_ent + at + PART); };
    auto red_green = [&](uint32_t at) { return *reinterpret_cast<const float2*>(s_ent + at + PART + 8); };
    auto blue = [&](uint32_t at) { return *reinterpret_cast<const float*>(s_ent + at + 2 * PART); };
    auto put_entry = [&](uint32_t e, const float4& a, const float4& b, float c) {
        *reinterpret_cast<float4*>(s_ent + e * 16) = a;
        *reinterpret_cast<float4*>(s_ent + e * 16 + PART) = b;
        *reinterpret_cast<float*>(s_ent + e * 16 + 2 * PART) = c;
    };
    // per region, the batch's entries that can reach it, in depth order
    __shared__ uint32_t s_list4[REGIONS * FAST_LIST / 4];
    uint8_t* s_list = reinterpret_cast<uint8_t*>(s_list4);
    if (TRAIN && blockIdx.x == min(gridDim.x - 1, STAMP_BLOCK) && threadIdx.x == 0) export_stamp(ws);
    // all parts of a tile on one XCD, whose L2 then serves the records to all
    const uint32_t slot_t = blockIdx.x / (PARTS * XCDS) * XCDS + blockIdx.x % XCDS, part = blockIdx.x / XCDS % PARTS;
    if (slot_t >= (uint32_t)f.n_tiles) return;
    const uint32_t tile = f.ordered ? ws.order[slot_t] : slot_t;
    const uint32_t tx = tile % (uint32_t)f.tiles_x, ty = tile / (uint32_t)f.tiles_x;
    const uint32_t lane = threadIdx.x;
    const uint32_t region = lane / REGION_LANES;
    // the part's first column and row of the tile, and the lane's first row
    const uint32_t left = PIX == 1 ? part % 2 * 8 : 0, top_row = PIX == 1 ? part / 2 * 8 : part * 8;
    constexpr uint32_t ACROSS = 2 * PIX;              // regions of a band of four rows
    const uint32_t lx = left + (region % ACROSS) * REGION + lane % REGION;
    const uint32_t band_row = PIX == 1 ? lane / REGION % REGION : lane / REGION % 2 * 2;
    const uint32_t ly = top_row + (region / ACROSS) * REGION + band_row;
    const uint32_t px = tx * TILE + lx, py = ty * TILE + ly;
    bool in[PIX];
#pragma unroll
    for (int i = 0; i < PIX; ++i) in[i] = px < (uint32_t)f.width && py + i < (uint32_t)f.height;
    const uint32_t start = ws.ranges[2 * tile], end = ws.ranges[2 * tile + 1];
    // tile-centre coordinates (EXP_PLAIN: relative to the tile's corner)
    constexpr float CENTRE = EXPM == EXP_PLAIN ? 0.0f : 7.5f;
    const float ox = (float)(tx * TILE) + CENTRE, oy = (float)(ty * TILE) + CENTRE;
    LanePixels dp;
    dp.odd = ly % 2 != 0;
    dp.x = (float)lx - CENTRE;
    dp.y = (float)(ly / 2 * 2) - CENTRE;
    dp.x2 = dp.x * dp.x;
    dp.xy = dp.x * dp.y;
    dp.y2 = dp.y * dp.y;
    dp.y21 = fmaf(2.0f, dp.y, 1.0f);
    const float top = (float)top_row - 7.5f;

    constexpr float SKIP = EXPM == EXP_PLAIN ? ALPHA_MIN : EXPM == EXP_HW2 ? -LOG2_255F : -LN255F;
    const float NEVER = __uint_as_float(0x7fc00000u);
    // the exponents (EXP_PLAIN: alphas) that pass at each pixel: >= thr, none once it has stopped
    float T[PIX], r[PIX], g[PIX], b[PIX], thr[PIX];
    uint32_t stop[PIX], nbl[PIX];
#pragma unroll
    for (int i = 0; i < PIX; ++i) {
        T[i] = 1.0f;
        r[i] = g[i] = b[i] = 0.0f;
        thr[i] = in[i] ? SKIP : NEVER;
        stop[i] = 0xffffffffu;
        nbl[i] = 0;
    }
    auto all_stopped = [&] {
        bool live = false;
#pragma unroll
        for (int i = 0; i < PIX; ++i) live = live || thr[i] == thr[i];
        return __ballot(live) == 0;
    };
    uint32_t steps = 0;         // counting renders: list entries this wave evaluated
    if (lane == 0)
        put_entry(FAST_BATCH, make_float4(0.f, 0.f, 0.f, 0.f),
                  make_float4(0.f, EXPM == EXP_PLAIN ? 0.f : -1.0e30f, 0.f, 0.f), 0.f);

    uint32_t ahead = start + lane < end ? vals[start + lane] : 0u;      // this lane's Gaussian of the next batch
    for (uint32_t base = start; base < end; base += FAST_BATCH) {
        if (all_stopped()) break;
        // ---- stage: fold, and list each entry in the regions it can reach ----
        __syncthreads();                 // (one wave: orders its LDS accesses for the compiler)
#pragma unroll
        for (uint32_t i = 0; i < REGIONS * FAST_LIST / 4; i += 64)
            if (i + 64 <= REGIONS * FAST_LIST / 4 || i + lane < REGIONS * FAST_LIST / 4)
                s_list4[i + lane] = FAST_BATCH * 0x01010101u;
        __syncthreads();
        // EXP_PLAIN leaves a skipped pair out altogether: with a colour that is
        // not finite, a blend by zero would not, and the batch goes entry by entry
        bool careful = false;
        RegionSpans sp;
        sp.none();
        if (base + lane < end) {
            const Record rec = ws.records[ahead < f.n_gaussians ? ahead : 0u];
            float u, v;
            if (EXPM == EXP_PLAIN) {
                u = (rec.u_hi - ox) + rec.u_lo;
                v = (rec.v_hi - oy) + rec.v_lo;
                put_entry(lane, make_float4(u, v, rec.A, rec.B), make_float4(rec.C, rec.opa, rec.r, rec.g), rec.b);
                careful = !(fabsf(rec.r) + fabsf(rec.g) + fabsf(rec.b) < 1.0e30f);
                // o e^p >= 1/255 iff q <= 2 ln(255 o); the record stores no box
                sp.reach(rec.A, rec.B, rec.C, 2.0f * logf(255.0f * rec.opa), 1.0e30f, 1.0e30f, u - 7.5f, v - 7.5f, top);
            } else {
                float4 ca, cbv;
                fold_record<EXPM == EXP_HW2>(rec, ox, oy, u, v, ca, cbv);
                put_entry(lane, ca, cbv, rec.b);
                sp.reach(rec.A, rec.B, rec.C, 2.0f * (LN255F + rec.opa), half_lo(rec.extra), half_hi(rec.extra), u, v,
                         top);
            }
        }
        uint32_t n = 0;                  // the longest list
#pragma unroll
        for (int k = 0; k < REGIONS; ++k) {
            const bool hit = sp.hits(k / (int)ACROSS, (float)left + (float)(k % (int)ACROSS * REGION));
            const uint64_t m = __ballot(hit);
            const uint32_t p = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            if (hit) s_list[k * FAST_LIST + p] = (uint8_t)lane;
            n = max(n, (uint32_t)__popcll(m));
        }
        n = __builtin_amdgcn_readfirstlane(n);
        const bool one_by_one = EXPM == EXP_PLAIN && __ballot(careful) != 0;
        const uint32_t next = base + FAST_BATCH + lane;
        ahead = next < end ? vals[next] : 0u;
        __syncthreads();

        // ---- blend: every region's lanes walk the region's list ----
        const uint8_t* list = s_list + region * FAST_LIST;
        uint32_t k0 = 0;
        while (true) {
            // whole groups, until one in which some pixel stops
            for (; k0 < n; k0 += LIST_UNROLL) {
                const uint32_t word = *reinterpret_cast<const uint32_t*>(list + k0);
                float al[LIST_UNROLL][PIX], w[LIST_UNROLL][PIX];
                uint32_t at[LIST_UNROLL];
                float4 a[LIST_UNROLL];
                float2 c[LIST_UNROLL];
#pragma unroll
                for (int u = 0; u < LIST_UNROLL; ++u) {
                    at[u] = ((word >> (8 * u)) & 0xffu) * 16;
                    a[u] = coef(at[u]);
                    c[u] = tail(at[u]);
                }
#pragma unroll
                for (int u = 0; u < LIST_UNROLL; ++u) pair_alphas<EXPM, PIX>(a[u], c[u], dp, thr, al[u]);
                float Tn[PIX];
                uint32_t pass[PIX];
#pragma unroll
                for (int i = 0; i < PIX; ++i) {
                    Tn[i] = T[i];
                    pass[i] = 0;
                }
                float2 rg[LIST_UNROLL];
                float bl[LIST_UNROLL];
#pragma unroll
                for (int u = 0; u < LIST_UNROLL; ++u) {
                    rg[u] = red_green(at[u]);
                    bl[u] = blue(at[u]);
                }
#pragma unroll
                for (int u = 0; u < LIST_UNROLL; ++u) {
#pragma unroll
                    for (int i = 0; i < PIX; ++i) {
                        w[u][i] = al[u][i] * Tn[i];
                        Tn[i] = behind<EXPM>(Tn[i], al[u][i], w[u][i]);
                        if (COUNT) pass[i] += al[u][i] > 0.0f ? 1u : 0u;
                    }
                }
                // T never grows: a pixel stops in this group iff T falls below the limit at its end
                bool stops = false;
#pragma unroll
                for (int i = 0; i < PIX; ++i) stops = stops || Tn[i] < T_MIN;
                if (one_by_one || __ballot(stops) != 0) break;
#pragma unroll
                for (int i = 0; i < PIX; ++i) {
                    T[i] = Tn[i];
#pragma unroll
                    for (int u = 0; u < LIST_UNROLL; ++u) {
                        r[i] = fmaf(w[u][i], rg[u].x, r[i]);
                        g[i] = fmaf(w[u][i], rg[u].y, g[i]);
                        b[i] = fmaf(w[u][i], bl[u], b[i]);
                    }
                    if (COUNT) nbl[i] += pass[i];
                }
                if (COUNT) steps += LIST_UNROLL;
            }
            if (k0 >= n) break;
            // that group entry by entry: the pair that would take a pixel below the limit
            // is not blended
#pragma unroll 1
            for (uint32_t u = k0; u < k0 + LIST_UNROLL; ++u) {
                const uint32_t e = list[u];
                float al[PIX];
                pair_alphas<EXPM, PIX>(coef(e * 16), tail(e * 16), dp, thr, al);
                const float2 col = red_green(e * 16);
                const float bl = blue(e * 16);
#pragma unroll
                for (int i = 0; i < PIX; ++i) {
                    if (EXPM == EXP_PLAIN && al[i] == 0.0f) continue;
                    const float w = al[i] * T[i];
                    const float Tn = behind<EXPM>(T[i], al[i], w);
                    if (Tn < T_MIN) {
                        thr[i] = NEVER;
                        stop[i] = base + e;
                    } else {
                        T[i] = Tn;
                        r[i] = fmaf(w, col.x, r[i]);
                        g[i] = fmaf(w, col.y, g[i]);
                        b[i] = fmaf(w, bl, b[i]);
                        if (COUNT) nbl[i] += al[i] > 0.0f ? 1u : 0u;
                    }
                }
            }
            if (COUNT) steps += LIST_UNROLL;
            if (all_stopped()) break;
            k0 += LIST_UNROLL;
        }
    }
    if (COUNT && EXPM != EXP_PLAIN && lane == 0 && steps)
        atomicAdd(reinterpret_cast<unsigned long long*>(&ws.header->list_steps), (unsigned long long)steps);
    const uint64_t plane = (uint64_t)f.width * f.height;
    float* __restrict__ out = ws.params->out;
    const float bg0 = ws.params->cam.bg[0], bg1 = ws.params->cam.bg[1], bg2 = ws.params->cam.bg[2];
#pragma unroll
    for (int i = 0; i < PIX; ++i) {
        if (!in[i]) continue;
        const uint64_t o = (uint64_t)(py + i) * f.width + px;
        out[o] = fmaf(T[i], bg0, r[i]);
        out[plane + o] = fmaf(T[i], bg1, g[i]);
        out[2 * plane + o] = fmaf(T[i], bg2, b[i]);
        if (COUNT || TRAIN) {       // the debug render's and the training variant's per-pixel outputs
            ws.t_final[o] = T[i];
            ws.n_proc[o] = stop[i] != 0xffffffffu ? (stop[i] - start + 1) | N_PROC_STOPPED : end - start;
        }
        if (COUNT) ws.n_blend[o] = nbl[i];
    }
}

// One, or four, pixels per lane: the dual-pixel ablation (one pixel per
// thread, four waves of 16x4 rows) and its extension along the column (four
// pixels per lane, Eq. dual_pixel applied three times, one wave per tile).  A
// tile's workgroup has one wave per band of 4 PIX rows: the 64 lanes of a wave
// form four row groups of 16 columns, group j owning PIX consecutive rows and
// each lane PIX pixels of one column.  The per-pair decisions are those of the
// dual-pixel kernel above, written for any PIX; a wave has one list, of the entries
// that reach its band of rows, so against the dual pixel's eight lists it evaluates more pairs.
template <int PIX>
struct FastShape {
    static constexpr int ROWS = 4 * PIX;            // rows of a wave's band
    static constexpr int WAVES = TILE / ROWS;       // waves per tile
    static constexpr int THREADS = 64 * WAVES;
    static constexpr int BATCH = THREADS;           // entries staged at once, one per thread
    static constexpr int CAP = BATCH + LIST_UNROLL;
};

template <bool COUNT, int EXPM, int PIX>
__global__ __launch_bounds__(FastShape<PIX>::THREADS) void k_raster_fast_px(FrameDev f, WsDev ws,
                                                                         const uint32_t* __restrict__ vals) {
    using S = FastShape<PIX>;
    constexpr int WAVES = S::WAVES;
    constexpr int CAP = S::CAP;
    constexpr float SKIP = EXPM == EXP_HW2 ? -LOG2_255F : -LN255F;
    // per-wave lists of folded Gaussians, in depth order
    __shared__ float4 s_a[WAVES][CAP];               // C1, C2, C3, C4
    __shared__ float4 s_b[WAVES][CAP];               // C5, C6, r, g
    __shared__ float2 s_c[WAVES][CAP];               // b, list position (as float bits)
    __shared__ uint32_t s_cnt[WAVES][WAVES];         // [wave of the staging thread][list]
    if (blockIdx.x >= (uint32_t)f.n_tiles) return;
    const uint32_t tile = f.ordered ? ws.order[blockIdx.x] : blockIdx.x;
    const uint32_t tx = tile % (uint32_t)f.tiles_x, ty = tile / (uint32_t)f.tiles_x;
    const uint32_t tid = threadIdx.x;
    const uint32_t wave = tid / 64, lane = tid % 64;
    const uint32_t lx = tid % TILE, ly = PIX * (tid / TILE);
    const uint32_t px = tx * TILE + lx, py = ty * TILE + ly;
    const uint32_t start = ws.ranges[2 * tile], end = ws.ranges[2 * tile + 1];
    // tile-centre coordinates
    const float ox = (float)(tx * TILE) + 7.5f, oy = (float)(ty * TILE) + 7.5f;
    const float x = (float)lx - 7.5f, y = (float)ly - 7.5f;
    const float x2 = x * x, xy = x * y, y2 = y * y;
    // the row factor 2 (y + k) + 1 of Eq. dual_pixel's step from row y + k to y + k + 1
    float yk[PIX > 1 ? PIX - 1 : 1];
#pragma unroll
    for (int k = 0; k + 1 < PIX; ++k) yk[k] = fmaf(2.0f, y + (float)k, 1.0f);

    float T[PIX], cr[PIX], cg[PIX], cb[PIX];
    uint32_t stop[PIX], nbl[PIX];
    // Whether pixel i is still blending.  Held in four scalars rather than an
    // array, so that each stays a lane mask in scalar registers (an array of
    // bools is kept as bytes in vector registers, two more VALU per pixel).
    bool live0 = px < (uint32_t)f.width && py < (uint32_t)f.height;
    bool live1 = PIX > 1 && px < (uint32_t)f.width && py + 1 < (uint32_t)f.height;
    bool live2 = PIX > 2 && px < (uint32_t)f.width && py + 2 < (uint32_t)f.height;
    bool live3 = PIX > 3 && px < (uint32_t)f.width && py + 3 < (uint32_t)f.height;
    auto live = [&](int i) -> bool& { return i == 0 ? live0 : i == 1 ? live1 : i == 2 ? live2 : live3; };
#pragma unroll
    for (int i = 0; i < PIX; ++i) {
        T[i] = 1.0f;
        cr[i] = cg[i] = cb[i] = 0.0f;
        stop[i] = 0xffffffffu;
        nbl[i] = 0;
    }
    uint32_t steps = 0;         // counting renders: list entries this wave evaluated
    const uint64_t lt = lanemask_lt();

    for (uint32_t base = start; base < end; base += S::BATCH) {
        const bool any = live0 || live1 || live2 || live3;
        if (__syncthreads_count(any) == 0) break;
        // ---- stage: fold, cull against every wave's band, compact per wave ----
        const uint32_t idx = base + tid;
        bool hit[WAVES];
#pragma unroll
        for (int w = 0; w < WAVES; ++w) hit[w] = false;
        float4 ca = make_float4(0.f, 0.f, 0.f, 0.f), cbv = make_float4(0.f, 0.f, 0.f, 0.f);
        float cbb = 0.f;
        if (idx < end) {
            const uint32_t g = vals[idx];
            const Record rec = ws.records[g < f.n_gaussians ? g : 0u];
            const float u = (rec.u_hi - ox) + rec.u_lo;
            const float v = (rec.v_hi - oy) + rec.v_lo;
            const float A = rec.A, B = rec.B, C = rec.C;
            const float C0 = fmaf(A * u, u, fmaf(2.0f * B * u, v, C * v * v));
            ca = make_float4(-0.5f * A, -B, -0.5f * C, fmaf(A, u, B * v));
            cbv = make_float4(fmaf(C, v, B * u), fmaf(-0.5f, C0, rec.opa), rec.r, rec.g);
            cbb = rec.b;
            if (EXPM == EXP_HW2) {       // P log2 e directly: alpha = exp2 of it
                ca = make_float4(ca.x * LOG2E_F, ca.y * LOG2E_F, ca.z * LOG2E_F, ca.w * LOG2E_F);
                cbv.x *= LOG2E_F;
                cbv.y *= LOG2E_F;
            }
            // the box |x - u| <= hx, |y - v| <= hy holds every pixel with
            // P >= -ln 255 (half-extents from the front end, rounded up, then
            // widened); a band outside it has no pair that passes the skip
            // test; then the ellipse itself: the band must hold a point with
            // q <= tau = 2 (ln 255 + ln o), up to the margin.  Comparisons are
            // phrased so that a NaN keeps the Gaussian.
            const float hx = fmaf(half_lo(rec.extra), 1.0f + BOX_MARGIN_REL, BOX_MARGIN_ABS);
            const float hy = fmaf(half_hi(rec.extra), 1.0f + BOX_MARGIN_REL, BOX_MARGIN_ABS);
            const bool x_out = u - hx > 7.5f || u + hx < -7.5f;
            const float qlim = fmaf(2.0f * (LN255F + rec.opa), 1.0f + Q_MARGIN_REL, Q_MARGIN_ABS);
            // the reciprocals only place the nearest point of an edge, where q is
            // then evaluated exactly; an error of an ulp moves q by ~C (1e-6 px)^2
            const float iA = __builtin_amdgcn_rcpf(A), iC = __builtin_amdgcn_rcpf(C);
#pragma unroll
            for (int w = 0; w < WAVES; ++w) {
                const float y0 = (float)(w * S::ROWS) - 7.5f, y1 = y0 + (float)(S::ROWS - 1);
                hit[w] = !(x_out || v - hy > y1 || v + hy < y0);
                if (hit[w]) hit[w] = !(conic_rect_min(u, v, A, B, C, iA, iC, y0, y1) > qlim);
            }
        }
        uint64_t mk[WAVES];
#pragma unroll
        for (int w = 0; w < WAVES; ++w) mk[w] = __ballot(hit[w]);
        if (lane == 0) {
#pragma unroll
            for (int w = 0; w < WAVES; ++w) s_cnt[wave][w] = (uint32_t)__popcll(mk[w]);
        }
        __syncthreads();
        const float posf = __uint_as_float(idx);
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            if (hit[w]) {
                uint32_t p = (uint32_t)__popcll(mk[w] & lt);
                for (uint32_t sw = 0; sw < wave; ++sw) p += s_cnt[sw][w];
                s_a[w][p] = ca;
                s_b[w][p] = cbv;
                s_c[w][p] = make_float2(cbb, posf);
            }
        }
        uint32_t nl[WAVES];
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            nl[w] = 0;
#pragma unroll
            for (int sw = 0; sw < WAVES; ++sw) nl[w] += s_cnt[sw][w];
        }
        // inert padding up to a multiple of the unroll: P = -1e30 is always skipped
        if (tid < WAVES * LIST_UNROLL) {
            const uint32_t w = tid / LIST_UNROLL, k = tid % LIST_UNROLL;
            const uint32_t p = nl[w] + k;
            s_a[w][p] = make_float4(0.f, 0.f, 0.f, 0.f);
            s_b[w][p] = make_float4(0.f, -1.0e30f, 0.f, 0.f);
            s_c[w][p] = make_float2(0.f, 0.f);
        }
        __syncthreads();

        // ---- blend this wave's list ----
        // (the list length is the same for the whole wave: keep it scalar)
        const uint32_t n = __builtin_amdgcn_readfirstlane(nl[wave]);
        const float4* la = s_a[wave];
        const float4* lb = s_b[wave];
        const float2* lc = s_c[wave];
        if (__ballot(any) != 0) {
            bool wave_done = false;     // every pixel of the wave has stopped
            for (uint32_t k0 = 0; k0 < n && !wave_done; k0 += LIST_UNROLL) {
                if (COUNT) steps += LIST_UNROLL;
#pragma unroll
                for (int u = 0; u < LIST_UNROLL; ++u) {
                    const float4 a = la[k0 + u];
                    const float4 m = lb[k0 + u];
                    const float2 c = lc[k0 + u];
                    float P[PIX];
                    P[0] = fmaf(a.x, x2, fmaf(a.y, xy, fmaf(a.z, y2, fmaf(a.w, x, fmaf(m.x, y, m.y)))));
#pragma unroll
                    for (int i = 1; i < PIX; ++i) P[i] = P[i - 1] + fmaf(a.y, x, fmaf(a.z, yk[i - 1], m.x));
                    float Tn[PIX], nr[PIX], ng[PIX], nb[PIX];
                    bool st[PIX];
                    bool any_stop = false;
#pragma unroll
                    for (int i = 0; i < PIX; ++i) {
                        // a skipped or finished pixel takes alpha = 0
                        const float al = (live(i) && P[i] >= SKIP) ? kept_alpha<EXPM>(P[i]) : 0.0f;
                        const float w = al * T[i];
                        Tn[i] = T[i] - w;
                        nr[i] = fmaf(w, m.z, cr[i]);
                        ng[i] = fmaf(w, m.w, cg[i]);
                        nb[i] = fmaf(w, c.x, cb[i]);
                        st[i] = Tn[i] < T_MIN;
                        any_stop |= st[i];
                        if (COUNT) nbl[i] += (al > 0.0f && !st[i]) ? 1u : 0u;
                    }
                    if (__ballot(any_stop) != 0) {
                        // a pixel reached the stop: that pair is not blended
                        const uint32_t at = __float_as_uint(c.y);
#pragma unroll
                        for (int i = 0; i < PIX; ++i) {
                            if (st[i]) {
                                live(i) = false;
                                stop[i] = at;
                                Tn[i] = T[i];
                                nr[i] = cr[i];
                                ng[i] = cg[i];
                                nb[i] = cb[i];
                            }
                        }
                        wave_done = __ballot(live0 || live1 || live2 || live3) == 0;
                    }
#pragma unroll
                    for (int i = 0; i < PIX; ++i) {
                        T[i] = Tn[i];
                        cr[i] = nr[i];
                        cg[i] = ng[i];
                        cb[i] = nb[i];
                    }
                }
            }
        }
        __syncthreads();
    }
    if (COUNT && lane == 0 && steps) atomicAdd(reinterpret_cast<unsigned long long*>(&ws.header->list_steps),
                                               (unsigned long long)steps);
    const uint64_t plane = (uint64_t)f.width * f.height;
    float* __restrict__ out = ws.params->out;
    const float bg0 = ws.params->cam.bg[0], bg1 = ws.params->cam.bg[1], bg2 = ws.params->cam.bg[2];
#pragma unroll
    for (int i = 0; i < PIX; ++i) {
        if (px < (uint32_t)f.width && py + i < (uint32_t)f.height) {
            const uint64_t o = (uint64_t)(py + i) * f.width + px;
            out[o] = fmaf(T[i], bg0, cr[i]);
            out[plane + o] = fmaf(T[i], bg1, cg[i]);
            out[2 * plane + o] = fmaf(T[i], bg2, cb[i]);
            if (COUNT) {                // the debug render's per-pixel outputs
                ws.t_final[o] = T[i];
                ws.n_proc[o] = stop[i] != 0xffffffffu ? (stop[i] - start + 1) | N_PROC_STOPPED : end - start;
                ws.n_blend[o] = nbl[i];
            }
        }
    }
}

// A frame of few tiles leaves most SIMDs with a wave or two, and its time is the
// chain of instructions of the wave with the longest lists: a pixel per lane in
// a quarter of a tile nearly halves that chain, for more instructions in all.
// Frame times with dual and with single pixels (us): 256 tiles, 10K Gaussians
// fast 97 and 83, plain 140 and 106; 1M Gaussians, fast and plain, 300 tiles
// 400, 602 and 340, 463; 1200 tiles 270, 431 and 226, 337; 2040 tiles 205, 333 and
// 182, 280; 3072 tiles 216, 351 and 206, 320; the kernel alone, fast, at 3600 tiles
// 79 and 89, at 4056 60 and 70, at 8160 88 and 124 us.  Counting renders keep the
// dual pixel (the counts are in its units); both give the same bits.
constexpr int32_t SINGLE_MAX_TILES = 3072;

template <int EXPM, bool TRAIN = false>
static void launch_raster(hipStream_t s, const FrameDev& f, const WsDev& ws, const uint32_t* vals, bool count) {
    const uint32_t groups = ((uint32_t)f.n_tiles + XCDS - 1) / XCDS * XCDS;
    const dim3 block(64);
    if (count) hipLaunchKernelGGL((k_raster<true, EXPM, TRAIN, 2>), dim3(2 * groups), block, 0, s, f, ws, vals);
    else if (f.n_tiles > SINGLE_MAX_TILES)
        hipLaunchKernelGGL((k_raster<false, EXPM, TRAIN, 2>), dim3(2 * groups), block, 0, s, f, ws, vals);
    else hipLaunchKernelGGL((k_raster<false, EXPM, TRAIN, 1>), dim3(4 * groups), block, 0, s, f, ws, vals);
}

template <int EXPM, int PIX>
static void launch_fast_px(hipStream_t s, const FrameDev& f, const WsDev& ws, const uint32_t* vals, bool count) {
    const dim3 grid((uint32_t)f.n_tiles), block(FastShape<PIX>::THREADS);
    if (count)
        hipLaunchKernelGGL((k_raster_fast_px<true, EXPM, PIX>), grid, block, 0, s, f, ws, vals);
    else
        hipLaunchKernelGGL((k_raster_fast_px<false, EXPM, PIX>), grid, block, 0, s, f, ws, vals);
}

void launch_raster_fast(hipStream_t s, const FrameDev& f, const WsDev& ws, const uint32_t* vals, bool count,
                        uint32_t opts) {
    const bool exact = (opts & OPT_FASTEXP) != 0, single = (opts & OPT_DUALPIXEL) != 0;
    if (opts & OPT_QUAD) launch_fast_px<EXP_BITS, 4>(s, f, ws, vals, count);        // not with the two below
    else if (opts & OPT_HW_EXP2) launch_raster<EXP_HW2>(s, f, ws, vals, count);  // not with the two below
    else if (!exact && !single) launch_raster<EXP_BITS>(s, f, ws, vals, count);
    else if (exact && !single) launch_raster<EXP_LIBM>(s, f, ws, vals, count);
    else if (!exact && single) launch_fast_px<EXP_BITS, 1>(s, f, ws, vals, count);
    else launch_fast_px<EXP_LIBM, 1>(s, f, ws, vals, count);
}

void launch_raster_plain(hipStream_t s, const FrameDev& f, const WsDev& ws, const uint32_t* vals, bool count) {
    launch_raster<EXP_PLAIN, true>(s, f, ws, vals, count);
}

void launch_raster_train(hipStream_t s, const FrameDev& f, const WsDev& ws, const uint32_t* vals, bool count) {
    launch_raster<EXP_HW2, true>(s, f, ws, vals, count);
}

}  // namespace rgs
