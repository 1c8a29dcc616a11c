// Depth sort of the duplicated entries and per-tile ranges (Sec. III-C, IV-A).
//
// LSD radix sort with 8-bit digits over the significant bits of the key
// (plain: 32 + b_t bits of the 64-bit key; fast: the 32-bit key, 4 passes),
// value = Gaussian index.  Eq. sort_memory counts one read and one write of
// every (key, value) entry per pass.
//
// The kernel that writes the keys (the front end) also counts every pass's
// digits into the workspace histogram and clears the first pass's look-back
// words; each pass is then one kernel over radix tiles of SIZE keys (4608 for
// 32-bit keys, 5632 for 64-bit ones), block b taking keys [SIZE b, SIZE (b + 1)):
//   * the tile loads its keys, ranks each key among equal digits of the tile
//     with wave64 ballots (stable: tile order is input order) and publishes
//     its 256 digit counts;
//   * it then sums the counts of the tiles before it: the earlier tiles of its
//     group of SORT_GROUP, and one published total per earlier group (the last
//     tile of a group publishes the group's total).  A frame's tiles mostly
//     run at once and publish at about the same time; this two-level sum keeps
//     every tile's wait at two round trips instead of a chain through all its
//     predecessors;
//   * it reorders the tile in LDS by digit and writes it out, so consecutive
//     threads store consecutive positions of a digit bucket.
// Nothing guarantees that the workgroups of a grid run at once or in order
// (another stream's kernels may hold the CUs), so no tile waits without
// bound: a word still unpublished after LOOKBACK_POLLS polls is replaced by
// counting that tile's keys directly (a decoupled look-back with fallback).
// Taking tiles from an atomic ticket instead, which would make waiting safe,
// costs more than the whole look-back: tickets on one address serialise at
// about 11 ns each.  The two sets of look-back words alternate between
// passes: a pass clears its tile's words of the set the next pass uses.
// Ties keep input order, and the front end emits entries in Gaussian-index
// order, so equal keys end ordered by Gaussian index.
//
// Grids are sized for the workspace capacity; the entry count is read from
// the workspace header on the device and tiles beyond it return at once, so
// no host round trip sits between the front end and the sort.
//
// Frames of at least 2^8 tiles take the tile index's top bits first, in one such
// pass, and the rest per bucket in LDS (the split sort below), which also writes
// the tile ranges.
#include "rgs_internal.h"

namespace rgs {


// A radix pass's shape: digit width, threads and keys per thread of a tile.
template <int BITS_, int THREADS_, int ITEMS_>
struct PassShape {
    static constexpr int BITS = BITS_, THREADS = THREADS_, ITEMS = ITEMS_;
    static constexpr uint32_t DIGITS = 1u << BITS;
    static constexpr int WAVES = THREADS / 64;
    static constexpr uint32_t SIZE = THREADS * ITEMS;
    static constexpr uint32_t SPLIT = THREADS / DIGITS;      // threads per digit in the look-back
    static_assert(THREADS % DIGITS == 0 && THREADS >= (int)DIGITS, "whole digit rows per block");
};
template <typename KeyT>
using LsdShape = PassShape<RADIX_BITS, SORT_THREADS, SortTile<KeyT>::ITEMS>;
template <int BITS>
using SplitShape = PassShape<BITS, SPLIT_THREADS, SPLIT_ITEMS>;

__device__ inline uint32_t entry_count(const WsHeader* h) {
    uint64_t n = h->n_entries;
    uint64_t cap = h->capacity;
    return (uint32_t)(n < cap ? n : cap);
}

constexpr uint32_t SORT_READY = 0x80000000u;   // look-back word: published

// A barrier that orders the workgroup's LDS accesses and leaves its global loads
// in flight (__syncthreads would wait for them).
__device__ inline void lds_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);      // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Exclusive scan of one value per digit (threads 0 .. DIGITS - 1; other threads
// pass anything and get an unspecified result).  s_wtot holds DIGITS / 64 words.
// Every thread of the block must call it: it holds two barriers.
// LDS_ONLY: the barriers leave global loads in flight.
template <uint32_t DIGITS, bool LDS_ONLY = false>
__device__ inline uint32_t digit_exclusive_scan(uint32_t x, uint32_t* s_wtot) {
    auto barrier = [] {
        if (LDS_ONLY) lds_barrier();
        else __syncthreads();
    };
    const uint32_t lane = lane_id(), wave = threadIdx.x / 64;
    const uint32_t incl = wave_inclusive_scan(x);
    if (lane == 63 && wave < DIGITS / 64) s_wtot[wave] = incl;
    barrier();
    uint32_t before = 0;
#pragma unroll
    for (uint32_t w = 0; w < DIGITS / 64; ++w)
        if (w < wave) before += s_wtot[w];
    barrier();
    return incl - x + before;
}

// Polls of a not yet published look-back word (each a short sleep and a
// reload, a microsecond or two) before the waiting tile counts the missing row
// itself: a bound of milliseconds, far above any real wait.  When several
// streams' frames share the GPU, a running predecessor can be slow for tens of
// microseconds; 64 polls then sent ~47K rows per pass into the fallback over a
// 600-request serving burst on four streams (2040 frames/s), 4096 polls none
// (3270 frames/s).
constexpr uint32_t LOOKBACK_POLLS = 4096;

// Shared memory of the look-back (inside the pass kernel's s_whist once the
// tile is reordered): per-thread partial sums, a block-wide flag, and two
// count rows for the fallback.
struct LookbackLds {
    uint32_t* part;     // [SPLIT][DIGITS]
    uint32_t* flag;     // one word
    uint32_t* fb;       // [DIGITS] digit counts of one tile
    uint32_t* acc;      // [DIGITS] digit counts of one group
};

// Block-wide: fb[d] = keys of tile t (of the pass input) whose digit is d.
template <typename S, typename KeyT>
__device__ inline void count_tile(const KeyT* __restrict__ kin, uint32_t t, uint32_t n, uint32_t shift,
                                  uint32_t* fb) {
    for (uint32_t i = threadIdx.x; i < S::DIGITS; i += S::THREADS) fb[i] = 0;
    __syncthreads();
    const uint32_t base = t * S::SIZE, cnt = min(S::SIZE, n - base);
    for (uint32_t i = threadIdx.x; i < cnt; i += S::THREADS)
        atomicAdd(&fb[(uint32_t)(kin[base + i] >> shift) & (S::DIGITS - 1)], 1u);
    __syncthreads();
}

// Block-wide: out[d] = the counts of tile row t, from its published words
// where all are ready, else counted from the tile's keys.
template <typename S, typename KeyT>
__device__ inline void tile_row(const uint32_t* tiles, const KeyT* __restrict__ kin, uint32_t t, uint32_t n,
                                uint32_t shift, const LookbackLds& L, uint32_t* out, bool force) {
    const uint32_t tid = threadIdx.x;
    if (tid == 0) *L.flag = force ? 1u : 0u;
    __syncthreads();
    uint32_t w = SORT_READY;
    if (tid < S::DIGITS && !force) {
        w = ld_state(&tiles[(uint64_t)t * S::DIGITS + tid]);
        if (!(w & SORT_READY)) *L.flag = 1;
    }
    __syncthreads();
    if (*L.flag) {
        count_tile<S>(kin, t, n, shift, L.fb);
        if (tid < S::DIGITS) out[tid] = L.fb[tid];
    } else if (tid < S::DIGITS) {
        out[tid] = w & ~SORT_READY;
    }
    __syncthreads();
}

// Keys of digit d = tid % DIGITS in rows [r0, r1) of a look-back table (tile
// rows, or group rows of SORT_GROUP tiles), this thread's share: rows
// r0 + s, r0 + s + SPLIT, ... with s = tid / DIGITS.  Each word is polled
// at most LOOKBACK_POLLS times; `ok` turns false when one is still unpublished.  No
// barrier: the block votes on `ok` later and, if any thread missed a word,
// takes the range again with fallback_range.
template <typename S>
__device__ inline uint32_t poll_range(const uint32_t* tab, uint32_t r0, uint32_t r1, bool& ok) {
    constexpr int BATCH = 16;
    const uint32_t d = threadIdx.x % S::DIGITS, s = threadIdx.x / S::DIGITS;
    uint32_t sum = 0;
    for (uint32_t r = r0 + s; r < r1; r += BATCH * S::SPLIT) {
        uint32_t v[BATCH];
#pragma unroll
        for (int m = 0; m < BATCH; ++m) {
            const uint32_t rr = r + m * S::SPLIT;
            v[m] = rr < r1 ? ld_state(&tab[(uint64_t)rr * S::DIGITS + d]) : SORT_READY;
        }
#pragma unroll
        for (int m = 0; m < BATCH; ++m) {
            const uint32_t rr = r + m * S::SPLIT;
            uint32_t spins = 0;
            while (!(v[m] & SORT_READY)) {
                if (++spins > LOOKBACK_POLLS) {
                    ok = false;
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
                v[m] = ld_state(&tab[(uint64_t)rr * S::DIGITS + d]);
            }
            sum += v[m] & ~SORT_READY;
        }
    }
    return sum;
}

// The same share as poll_range, taken row by row by the whole block (every
// thread calls it with the same range): each row is read from its published
// words where all are there, else counted from the keys.  No tile ever
// waits on another without bound: the workgroups of a grid are not
// guaranteed to run at once.
template <typename S, typename KeyT>
__device__ uint32_t fallback_range(const uint32_t* tiles, bool groups, uint32_t r0, uint32_t r1,
                                   const KeyT* __restrict__ kin, uint32_t n, uint32_t shift, const LookbackLds& L,
                                   bool force) {
    const uint32_t tid = threadIdx.x, d = tid % S::DIGITS, s = tid / S::DIGITS;
    uint32_t sum = 0;
    for (uint32_t r = r0; r < r1; ++r) {
        const bool mine = (r - r0) % S::SPLIT == s;
        if (!groups) {
            tile_row<S>(tiles, kin, r, n, shift, L, L.acc, force);
        } else {
            for (uint32_t i = tid; i < S::DIGITS; i += S::THREADS) L.acc[i] = 0;
            __syncthreads();
            for (uint32_t t = r * SORT_GROUP; t < (r + 1) * SORT_GROUP; ++t) {
                tile_row<S>(tiles, kin, t, n, shift, L, L.fb, force);
                if (tid < S::DIGITS) L.acc[tid] += L.fb[tid];
                __syncthreads();
            }
        }
        if (mine) sum += L.acc[d];
        __syncthreads();
    }
    return sum;
}

// Where a pass leaves its entries: the LSD passes a key and a value array, the
// split pass (local key, value) pairs (see the split sort below).
template <typename KeyT>
struct ArraysOut {
    using Held = KeyT;                   // what the tile holds of a key in LDS
    KeyT* keys;
    uint32_t* vals;
    __host__ __device__ Held hold(KeyT k) const { return k; }
    __host__ __device__ uint32_t digit(Held h, uint32_t shift, uint32_t mask) const { return (uint32_t)(h >> shift) & mask; }
    __device__ void put(uint32_t at, Held h, uint32_t v) const {
        keys[at] = h;
        vals[at] = v;
    }
};
template <typename KeyT>
struct PairsOut;
// 32-bit keys: the local key is the key below its top digit.
template <>
struct PairsOut<uint32_t> {
    using Held = uint32_t;
    uint2* pairs;
    LocalKey lk;
    const FrameParams* prm;
    __host__ __device__ Held hold(uint32_t k) const { return k; }
    __host__ __device__ uint32_t digit(Held h, uint32_t shift, uint32_t) const { return h >> shift; }
    __device__ void put(uint32_t at, Held h, uint32_t v) const { pairs[at] = make_uint2(h & ((1u << lk.bits) - 1u), v); }
};
// 64-bit keys: (tile bits below the top digit, float32 depth bits above the
// nearest depth's).  The digit is masked, as where the tile ranks its keys: after a
// front end that gave up, keys are whatever memory held, and their bits above the
// tile index must not index the digit tables.
template <>
struct PairsOut<uint64_t> {
    using Held = uint64_t;
    uint2* pairs;
    LocalKey lk;
    const FrameParams* prm;
    __host__ __device__ Held hold(uint64_t k) const { return k; }
    __host__ __device__ uint32_t digit(Held h, uint32_t shift, uint32_t mask) const { return (uint32_t)(h >> shift) & mask; }
    __device__ void put(uint32_t at, Held h, uint32_t v) const {
        const uint32_t tile = (uint32_t)(h >> 32) & ((1u << lk.tile_bits) - 1u);
        const uint32_t depth = (uint32_t)h - depth_key_base(prm->cam);
        pairs[at] = make_uint2((tile << (lk.bits - lk.tile_bits)) | depth, v);
    }
};

// One stable radix pass on the digit at `shift`.  hist[c][d]: HIST_COPIES copies,
// hist_stride words apart, of the digit counts of the whole input.  tiles,
// groups: this pass's look-back words; next_tiles, next_groups: those of the
// frame's next pass, cleared here (null: none).  bases: if not null, receives
// each digit's first output place and, after the last, the entry count.
// FORCE: take every look-back from the keys (fallback_range), for tests.
//
// The split pass at 1M / 1080p, 241 tiles of 9216 keys, one a CU, all running at
// once: 2.9 us loading, 4.3 ranking (vector ALUs: ten ballots a key), 4 counting and
// reordering in LDS, 4.2 looking back, 1.8 storing, bound by these in turn.
// The digits' first places are scanned while the keys are on their way, each
// wave's places of a digit start at its place in the tile, and the last tile of a
// group publishes the group before it reorders: 23.3 -> 21.3 us (plain, 313
// tiles in two rounds, 41.2 -> 40.5; 3M / 4K 63.3 -> 62.7).  Tiles of 4096, two a CU:
// 33 and 87 us.
template <typename KeyT, typename S, typename Out, bool FORCE>
__global__ __launch_bounds__(S::THREADS) void k_radix_pass(const KeyT* __restrict__ kin,
                                                           const uint32_t* __restrict__ vin, Out out,
                                                           const WsHeader* header, const uint32_t* hist,
                                                           uint32_t hist_stride, uint32_t* tiles, uint32_t* groups,
                                                           uint32_t* next_tiles, uint32_t* next_groups, uint32_t shift,
                                                           uint32_t* bases) {
    constexpr int ITEMS = S::ITEMS;
    constexpr uint32_t SIZE = S::SIZE, DIGITS = S::DIGITS;
    using Held = typename Out::Held;
    // per-wave digit counts (at most 64 ITEMS each), then where each wave's run of a
    // digit starts in the reordered tile; reused for the look-back once the tile is
    // reordered
    constexpr uint32_t WHIST_WORDS = S::WAVES * DIGITS / 2 > (S::SPLIT + 3) * DIGITS ? S::WAVES * DIGITS / 2
                                                                                     : (S::SPLIT + 3) * DIGITS;
    __shared__ uint32_t s_whist[WHIST_WORDS];
    __shared__ uint32_t s_bstart[DIGITS];   // first LDS position of digit d in the reordered tile
    __shared__ uint32_t s_gbase[DIGITS];    // bucket base of d, then output position minus s_bstart[d]
    __shared__ uint32_t s_tot[DIGITS];      // the tile's count of digit d
    __shared__ uint32_t s_wtot[DIGITS / 64];
    __shared__ uint32_t s_missed[2];        // look-back votes: some thread found an unpublished word
    __shared__ Held s_keys[SIZE];
    __shared__ uint32_t s_vals[SIZE];

    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid / 64;
    const uint32_t n = entry_count(header);
    const uint32_t vb = blockIdx.x;      // the radix tile: keys [vb * SIZE, (vb + 1) * SIZE)
    const uint32_t tile_base = vb * SIZE;
    if (tile_base >= n) {
        if (bases && n == 0 && vb == 0)
            for (uint32_t i = tid; i <= DIGITS; i += S::THREADS) bases[i] = 0;
        return;
    }
    const uint32_t n_valid = min(SIZE, n - tile_base);
    // the bucket sizes do not depend on this tile: start the loads first
    uint32_t copies[HIST_COPIES];
#pragma unroll
    for (int c = 0; c < HIST_COPIES; ++c) copies[c] = tid < DIGITS ? hist[(uint64_t)c * hist_stride + tid] : 0u;

    // wave w owns entries [tile_base + w*ITEMS*64, +ITEMS*64); round r, lane l
    // holds entry tile_base + w*ITEMS*64 + r*64 + l
    const uint32_t wbase = tile_base + wave * (ITEMS * 64);
    KeyT k[ITEMS];
    uint32_t v[ITEMS];
    uint32_t rank[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const uint32_t idx = wbase + r * 64 + lane;
        const bool valid = idx < n;
        k[r] = valid ? kin[idx] : (KeyT)0;
        v[r] = valid ? vin[idx] : 0u;
    }
    // the next pass's look-back words of this tile (its set was last read by
    // the previous pass, which has finished)
    if (next_tiles && tid < DIGITS) {
        st_state(&next_tiles[(uint64_t)vb * DIGITS + tid], 0u);
        if (vb % SORT_GROUP == 0) st_state(&next_groups[(uint64_t)(vb / SORT_GROUP) * DIGITS + tid], 0u);
    }
    for (uint32_t i = tid; i < WHIST_WORDS; i += S::THREADS) s_whist[i] = 0;
    if (tid < 2) s_missed[tid] = 0;
    // the digits' first output places, while this tile's entries are on their way
    // (the barriers wait for LDS only)
    uint32_t bucket = 0;
#pragma unroll
    for (int c = 0; c < HIST_COPIES; ++c) bucket += copies[c];
    const uint32_t bbase = digit_exclusive_scan<DIGITS, true>(bucket, s_wtot);
    // Lanes of a wave read counters that other lanes of the same wave wrote in
    // the previous round.  The LDS unit executes one wave's accesses in issue
    // order; the empty asm with a memory clobber keeps the compiler from
    // moving or reusing accesses across rounds.  (A volatile pointer would do
    // the same but loses the LDS address space: every access becomes a flat
    // access that waits on all outstanding global memory operations.)
    uint16_t* my_hist = reinterpret_cast<uint16_t*>(s_whist) + wave * DIGITS;
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        asm volatile("" ::: "memory");
        const uint32_t idx = wbase + r * 64 + lane;
        const bool valid = idx < n;
        const uint32_t d = (uint32_t)(k[r] >> shift) & (DIGITS - 1);
        // lanes whose digit differs from this lane's: for each bit b the
        // ballot M_b of lanes holding a 1, XOR-ed with this lane's bit spread
        // to a whole word (0 or all ones), marks the lanes that disagree on b.
        // One three-input bit operation per half-mask folds M_b ^ spread into
        // the running OR (truth table 0xBE: S2 | (S0 ^ S1)).
        uint32_t diff_lo = 0, diff_hi = 0;
#pragma unroll
        for (int b = 0; b < S::BITS; ++b) {
            const uint32_t spread = (uint32_t)((int32_t)(d << (31 - b)) >> 31);
            const uint64_t m = __ballot(spread != 0);
            diff_lo = __builtin_amdgcn_bitop3_b32((uint32_t)m, spread, diff_lo, 0xBE);
            diff_hi = __builtin_amdgcn_bitop3_b32((uint32_t)(m >> 32), spread, diff_hi, 0xBE);
        }
        const uint64_t vmask = __ballot(valid);
        const uint32_t peers_lo = ~diff_lo & (uint32_t)vmask, peers_hi = ~diff_hi & (uint32_t)(vmask >> 32);
        const uint32_t below = __builtin_amdgcn_mbcnt_hi(peers_hi, __builtin_amdgcn_mbcnt_lo(peers_lo, 0u));
        const uint32_t prev = valid ? my_hist[d] : 0u;
        rank[r] = prev + below;
        if (valid && below == 0) my_hist[d] = (uint16_t)(prev + (uint32_t)(__popc(peers_lo) + __popc(peers_hi)));
    }
    __syncthreads();

    // digit d = tid: the tile's count, published at once
    uint32_t tot = 0;
    uint32_t c[S::WAVES];
    uint16_t* h = reinterpret_cast<uint16_t*>(s_whist) + tid;
    if (tid < DIGITS) {
#pragma unroll
        for (int w = 0; w < S::WAVES; ++w) c[w] = h[w * DIGITS];
#pragma unroll
        for (int w = 0; w < S::WAVES; ++w) tot += c[w];
        st_state(&tiles[(uint64_t)vb * DIGITS + tid], SORT_READY | tot);
        s_tot[tid] = tot;
    }
    // The last tile of a look-back group publishes the group's counts before it
    // goes on, so that they are there when later groups look for them.
    const uint32_t d = tid % DIGITS, s = tid / DIGITS;
    const uint32_t g = vb / SORT_GROUP, g0 = g * SORT_GROUP;
    const bool closes = vb % SORT_GROUP == SORT_GROUP - 1;
    constexpr bool force = FORCE;
    bool ok = !force, published = false;
    uint32_t part = 0;
    if (closes && !force) {
        uint32_t* early = reinterpret_cast<uint32_t*>(s_keys);     // [SPLIT][DIGITS], before the reorder
        part = poll_range<S>(tiles, g0, vb, ok);
        early[s * DIGITS + d] = part;
        if (__ballot(!ok) != 0 && lane == 0) s_missed[0] = 1;
        __syncthreads();
        published = s_missed[0] == 0;
        if (published && tid < DIGITS) {
            uint32_t gsum = tot;
#pragma unroll
            for (uint32_t q = 0; q < S::SPLIT; ++q) gsum += early[q * DIGITS + tid];
            st_state(&groups[(uint64_t)g * DIGITS + tid], SORT_READY | gsum);
        }
        __syncthreads();
    }
    const uint32_t bstart = digit_exclusive_scan<DIGITS>(tot, s_wtot);
    if (tid < DIGITS) {
        s_bstart[tid] = bstart;
        s_gbase[tid] = bbase;
        uint32_t at = bstart;
#pragma unroll
        for (int w = 0; w < S::WAVES; ++w) {
            h[w * DIGITS] = (uint16_t)at;
            at += c[w];
        }
        if (bases && vb == 0) {
            bases[tid] = min(bbase, n);
            if (tid == 0) bases[DIGITS] = n;
        }
    }
    __syncthreads();

    // reorder the tile by digit in LDS
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const uint32_t idx = wbase + r * 64 + lane;
        if (idx < n) {
            const uint32_t d = (uint32_t)(k[r] >> shift) & (DIGITS - 1);
            const uint32_t pos = my_hist[d] + rank[r];
            s_keys[pos] = out.hold(k[r]);
            s_vals[pos] = v[r];
        }
    }
    __syncthreads();

    // keys of digit d in earlier tiles: SPLIT threads per digit share the rows
    uint32_t* s_part = s_whist;    // [SPLIT][DIGITS]
    const LookbackLds L{s_whist, s_whist + S::SPLIT * DIGITS, s_whist + (S::SPLIT + 1) * DIGITS,
                        s_whist + (S::SPLIT + 2) * DIGITS};
    if (closes && !published) {
        part = fallback_range<S>(tiles, false, g0, vb, kin, n, shift, L, force);
        s_part[s * DIGITS + d] = part;
        __syncthreads();
        ok = !force;
        if (tid < DIGITS) {
            uint32_t gsum = s_tot[tid];
#pragma unroll
            for (uint32_t q = 0; q < S::SPLIT; ++q) gsum += s_part[q * DIGITS + tid];
            st_state(&groups[(uint64_t)g * DIGITS + tid], SORT_READY | gsum);
        }
        __syncthreads();
    }
    if (!closes && !force) part = poll_range<S>(tiles, g0, vb, ok);
    if (!force) part += poll_range<S>(groups, 0, g, ok);
    s_part[s * DIGITS + d] = part;
    if (__ballot(!ok) != 0 && lane == 0) s_missed[1] = 1;
    __syncthreads();
    if (s_missed[1]) {
        // a predecessor's counts were not published in time: take both ranges again
        part = fallback_range<S>(tiles, false, g0, vb, kin, n, shift, L, force) +
               fallback_range<S>(tiles, true, 0, g, kin, n, shift, L, force);
        s_part[s * DIGITS + d] = part;
        __syncthreads();
    }
    if (tid < DIGITS) {
        uint32_t before = 0;
#pragma unroll
        for (uint32_t q = 0; q < S::SPLIT; ++q) before += s_part[q * DIGITS + tid];
        s_gbase[tid] = s_gbase[tid] + before - s_bstart[tid];
    }
    __syncthreads();

    for (uint32_t p = tid; p < n_valid; p += S::THREADS) {
        const Held h = s_keys[p];
        const uint32_t dst = s_gbase[out.digit(h, shift, DIGITS - 1)] + p;
        if (dst < n)          // always true for consistent counts; guards the bounds regardless
            out.put(dst, h, s_vals[p]);
    }
}

template <typename KeyT>
static void sort_typed(hipStream_t s, const WsDev& ws, uint32_t passes, bool force) {
    using S = LsdShape<KeyT>;
    KeyT* ka = reinterpret_cast<KeyT*>(ws.keys_a);
    KeyT* kb = reinterpret_cast<KeyT*>(ws.keys_b);
    const dim3 grid(ws.sort_rows), block(S::THREADS);
    for (uint32_t p = 0; p < passes; ++p) {
        const bool from_a = (p % 2) == 0;
        const ArraysOut<KeyT> out{from_a ? kb : ka, from_a ? ws.vals_b : ws.vals_a};
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, grid, block, 0, s, from_a ? ka : kb, from_a ? ws.vals_a : ws.vals_b, out,
                               ws.header, ws.hist + p * RADIX, (uint32_t)(MAX_PASSES * RADIX),
                               sort_state_tiles(ws, p & 1), sort_state_groups(ws, p & 1),
                               sort_state_tiles(ws, (p + 1) & 1), sort_state_groups(ws, (p + 1) & 1),
                               (uint32_t)(RADIX_BITS * p), (uint32_t*)nullptr);
        };
        if (force) launch(k_radix_pass<KeyT, S, ArraysOut<KeyT>, true>);
        else launch(k_radix_pass<KeyT, S, ArraysOut<KeyT>, false>);
    }
}

void launch_sort(hipStream_t s, const WsDev& ws, uint32_t key_bytes, uint32_t passes, bool force) {
    // force (a context's RGS_DEBUG_SORT_FALLBACK, for tests): every look-back
    // counts its rows from the keys instead of reading the published words
    if (key_bytes == 8) sort_typed<uint64_t>(s, ws, passes, force);
    else sort_typed<uint32_t>(s, ws, passes, force);
}

// ---------------------------------------------------------------------------
// The split sort, for frames of at least 2^SPLIT_MIN_BT tiles.  The same stable
// sort, reorganised:
//   * one radix pass as above on the tile index's top D bits moves every entry
//     to its digit's bucket, in input order: a bucket holds 2^(b_t - D) whole
//     tiles.  It leaves (local key, value) pairs, the local key being what is
//     left to sort: the remaining tile bits, then the depth (32-bit keys: the
//     quantised depth; 64-bit keys: the float32 depth's bits above those of
//     z_near, which no depth is below);
//   * one workgroup per bucket then takes the bucket's local key, least
//     significant digit first, each a stable counting pass in LDS
//     (bucket_rank).  A bucket of at most CAP entries stays in LDS for all of
//     them; one of at most 2 CAP is sorted as two runs in LDS, each written back
//     in place, and the two merged; a larger one streams through global memory
//     in chunks of CAP, one stable pass at a time;
//   * the same workgroup, holding its bucket sorted, writes its tiles' ranges.
// Every pass is stable and the top digit is taken first, then the rest least
// significant first; as a stable sort on the top digit followed by a stable
// sort on the rest leaves the keys ordered by (top digit, rest) with ties in
// input order, the result is the LSD sort's, bit for bit.  The frame then needs
// two sort kernels instead of four (32-bit keys) or six (64-bit keys, 1080p and
// 4K) passes and the ranges kernel.

constexpr uint32_t BK_LOAD_BATCH = 8;       // loads of a thread in flight where a loop stages or merges

// A bucket's workgroup: threads, and entries each holds.
template <int THREADS_, int ITEMS_>
struct BucketShape {
    static constexpr int THREADS = THREADS_, ITEMS = ITEMS_;
    static constexpr int WAVES = THREADS / 64;
    static constexpr uint32_t CAP = THREADS * ITEMS;
};

// Shared memory of the bucket sort.
template <typename B>
struct BucketLds {
    static constexpr int WORDS = B::WAVES > RADIX / 64 ? B::WAVES : RADIX / 64;
    uint2 pair[B::CAP];                        // (local key, value)
    uint16_t whist[B::WAVES * RADIX];          // per-wave digit counts, then places (below CAP)
    uint32_t tot[RADIX], bs[RADIX], base[RADIX];
    uint32_t wtot[WORDS];
};

// The digit of a local key at `shift` (0 past its end).
__device__ inline uint32_t digit_at(uint32_t k, uint32_t shift) {
    return shift < 32 ? (k >> shift) & (RADIX - 1) : 0u;
}

// Block-wide stable ranking of up to CAP keys.  Wave w holds entries
// [w R 64, (w + 1) R 64) of the chunk, round r and lane l holding entry
// (w R + r) 64 + l, with R = ceil(cnt / THREADS) <= ITEMS rounds, so that
// all waves share the work.  pos[r] is the key's place when the chunk is
// ordered by the RADIX_BITS-bit digit at `shift` (ties in entry order), tot[d]
// the chunk's count of digit d and bs[d] its first place.  lds.pair is scratch:
// every entry has been read from it before the call, and it may be overwritten
// on return.  Every thread calls it (barriers).
//
// The lanes of a round that share a digit are found through LDS: each lane ORs
// its bit into its digit's 64-bit mask in the wave's row, reads the mask back (a
// wave's LDS accesses execute in issue order), and the lowest lane of the digit
// clears it again.  Eight ballots and their bit operations, as in the radix
// pass, cost twice the VALU instructions of the whole kernel.
template <typename B>
__device__ inline void bucket_rank(const uint32_t (&k)[B::ITEMS], uint32_t cnt, uint32_t R, uint32_t shift,
                                   uint32_t (&pos)[B::ITEMS], BucketLds<B>& lds) {
    constexpr int WAVES = B::WAVES, THREADS = B::THREADS, BK_ITEMS = B::ITEMS;
    static_assert(sizeof(lds.pair) >= WAVES * RADIX * 8, "the masks fit the entries' LDS");
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid / 64;
    // entries of this wave that exist: round r, lane l holds one when r < R and r * 64 + l < lim
    const int lim = __builtin_amdgcn_readfirstlane((int)cnt - (int)(wave * R * 64));
    uint64_t* match = reinterpret_cast<uint64_t*>(lds.pair);
    __syncthreads();            // every entry has been read
    uint32_t* zero = reinterpret_cast<uint32_t*>(lds.whist);
    for (uint32_t i = tid; i < WAVES * RADIX / 2; i += THREADS) zero[i] = 0;
    for (uint32_t i = tid; i < WAVES * RADIX / 2; i += THREADS)
        reinterpret_cast<uint4*>(match)[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    uint16_t* my_hist = lds.whist + wave * RADIX;
    uint64_t* my_match = match + wave * RADIX;
    const uint64_t my_bit = 1ull << lane;
#pragma unroll
    for (int r = 0; r < BK_ITEMS; ++r) {
        if ((uint32_t)r >= R) break;
        // a wave's rounds read what its lanes wrote in the round before;
        // pos[r] holds the rank among the wave's keys of the same digit until
        // the scan below
        asm volatile("" ::: "memory");
        pos[r] = 0;
        if ((int)lane < lim - r * 64) {
            const uint32_t d = digit_at(k[r], shift);
            atomicOr(reinterpret_cast<unsigned long long*>(&my_match[d]), (unsigned long long)my_bit);
            const uint64_t peers = my_match[d];
            const uint32_t prev = my_hist[d];
            const uint32_t below =
                __builtin_amdgcn_mbcnt_hi((uint32_t)(peers >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)peers, 0u));
            pos[r] = prev + below;
            if (below == 0) {
                my_hist[d] = (uint16_t)(prev + (uint32_t)__popcll(peers));
                my_match[d] = 0ull;
            }
        }
    }
    __syncthreads();
    // digit d = tid: each wave's first place in the chunk
    uint32_t tot = 0, off = 0;
    uint32_t c[WAVES];
    if (tid < RADIX) {
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            c[w] = lds.whist[w * RADIX + tid];
            tot += c[w];
        }
        lds.tot[tid] = tot;
    }
    const uint32_t bs = digit_exclusive_scan<RADIX>(tot, lds.wtot);
    if (tid < RADIX) {
        lds.bs[tid] = bs;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            lds.whist[w * RADIX + tid] = (uint16_t)(bs + off);
            off += c[w];
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < BK_ITEMS; ++r) {
        if ((uint32_t)r >= R) break;
        pos[r] += my_hist[digit_at(k[r], shift)];
    }
}

// Digits of a local key of `bits` bits.
__device__ inline uint32_t digit_passes(uint32_t bits) { return bits ? (bits + RADIX_BITS - 1) / RADIX_BITS : 1u; }

// Where the sorted entries of a bucket go: the values, the tiles' ranges, and
// (debug renders) the full keys.
struct BucketOut {
    uint32_t* vals;
    uint32_t* ranges;
    uint32_t* keys32;       // 32-bit keys, or null
    uint64_t* keys64;       // 64-bit keys, or null
    uint32_t* order;        // the rasterizers' schedule, or null
    uint32_t* error;
    const FrameParams* prm;
    LocalKey lk;
    uint32_t n_tiles;

    __device__ uint32_t tile_of(uint32_t local) const {
        const uint32_t depth_bits = lk.bits - lk.tile_bits;
        return (blockIdx.x << lk.tile_bits) | (lk.tile_bits ? local >> depth_bits : 0u);
    }
    // The tile's run starts at entry `at` of the frame / ended before it.
    __device__ void start(uint32_t at, uint32_t local) const {
        const uint32_t t = tile_of(local);
        if (t < n_tiles) ranges[2 * t] = at;
        else atomicOr(error, 4u);       // only after a failed front end
    }
    __device__ void end(uint32_t at, uint32_t local) const {
        const uint32_t t = tile_of(local);
        if (t < n_tiles) ranges[2 * t + 1] = at;
        else atomicOr(error, 4u);
    }
    // Entry `at` and the one before it have these local keys.
    __device__ void boundary(uint32_t at, uint32_t before, uint32_t local) const {
        if (lk.tile_bits && (before ^ local) >> (lk.bits - lk.tile_bits)) {
            end(at, before);
            start(at, local);
        }
    }
    __device__ bool want_keys() const { return keys32 || keys64; }
    __device__ void put_key(uint32_t at, uint32_t local) const {
        const uint32_t depth_bits = lk.bits - lk.tile_bits;
        const uint32_t depth = lk.tile_bits ? local & ((1u << depth_bits) - 1u) : local, t = tile_of(local);
        if (keys32) keys32[at] = (t << depth_bits) | depth;
        if (keys64) keys64[at] = ((uint64_t)t << 32) | (depth_key_base(prm->cam) + depth);
    }
};

// Sorts m <= CAP pairs of src by their local key in LDS, all digits, leaving
// them in lds.pair.  Every thread calls it (barriers).
template <typename B>
__device__ inline void bucket_lds_sort(const uint2* src, uint32_t m, uint32_t bits, BucketLds<B>& lds) {
    constexpr int THREADS = B::THREADS, BK_ITEMS = B::ITEMS;
    const uint32_t lane = lane_id(), wave = threadIdx.x / 64;
    // Entry e is held in round r < R by (wave, lane) with e = (wave R + r) 64
    // + lane, the layout of bucket_rank.  The bounds are wave-uniform counts
    // against the lane index, so that no per-entry index stays live across the
    // passes.  The first pass takes its pairs straight from global memory in
    // that layout, every load of a thread in flight at once.
    uint32_t k[BK_ITEMS], v[BK_ITEMS], pos[BK_ITEMS];
    const uint32_t R = (m + THREADS - 1) / THREADS;
    const int lim = __builtin_amdgcn_readfirstlane((int)m - (int)(wave * R * 64));
    const uint2* mine = src + wave * R * 64 + lane;
    const uint2* held = lds.pair + wave * R * 64 + lane;
#pragma unroll
    for (int r = 0; r < BK_ITEMS; ++r) {
        const uint2 p = (uint32_t)r < R && (int)lane < lim - r * 64 ? mine[r * 64] : make_uint2(0u, 0u);
        k[r] = p.x;
        v[r] = p.y;
    }
    const uint32_t passes = digit_passes(bits);
    for (uint32_t q = 0; q < passes; ++q) {
        if (q > 0) {
#pragma unroll
            for (int r = 0; r < BK_ITEMS; ++r) {
                const uint2 p = (uint32_t)r < R && (int)lane < lim - r * 64 ? held[r * 64] : make_uint2(0u, 0u);
                k[r] = p.x;
                v[r] = p.y;
            }
        }
        bucket_rank<B>(k, m, R, RADIX_BITS * q, pos, lds);
        __syncthreads();        // the masks are done with
#pragma unroll
        for (int r = 0; r < BK_ITEMS; ++r)
            if ((uint32_t)r < R && (int)lane < lim - r * 64) lds.pair[pos[r]] = make_uint2(k[r], v[r]);
        __syncthreads();
    }
}

// The rasterizers' schedule from the buckets: the tiles of the busiest bucket
// first, in row-major order within a bucket (2^tile_bits neighbouring tiles, whose
// lists are alike), buckets of equal size in order.  Every workgroup counts the
// buckets before its own, so the schedule needs no kernel of its own (7 to 10 us
// between the sort and the rasterizer; counting takes 1.5 us of the bucket
// sort).  At 1M / 1080p the rasterizer takes 99 us with it, 91 with the order by
// tile, 102 with none; with each bucket's longer tiles in a first run over the
// buckets and its shorter ones in a second, 107.  Every thread calls it
// (barriers); scratch: a word per wave.
template <int THREADS>
__device__ inline void place_tiles(const uint32_t* __restrict__ bases, const BucketOut& out, uint32_t* scratch) {
    const uint32_t b = blockIdx.x, bits = out.lk.tile_bits;
    const uint32_t in_use = (out.n_tiles - 1) >> bits;      // the last bucket that has tiles, perhaps fewer
    if (b > in_use) return;
    const uint32_t size = bases[b + 1] - bases[b];
    uint32_t before = 0;
    for (uint32_t e = threadIdx.x; e <= in_use; e += THREADS) {
        const uint32_t other = bases[e + 1] - bases[e];
        before += (uint32_t)__popcll(__ballot(other > size || (other == size && e < b)));
    }
    if (lane_id() == 0) scratch[threadIdx.x / 64] = before;     // (lane 0 takes part in every round of its wave)
    __syncthreads();
    before = 0;
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) before += scratch[w];
    __syncthreads();
    const uint32_t last = out.n_tiles - (in_use << bits);       // tiles of the last bucket
    const uint32_t tiles = b == in_use ? last : 1u << bits;
    uint32_t at = before << bits;
    if (b != in_use && bases[in_use + 1] - bases[in_use] > size) at -= (1u << bits) - last;
    for (uint32_t t = threadIdx.x; t < tiles; t += THREADS)
        if (at + t < out.n_tiles) out.order[at + t] = (b << bits) + t;
}

__device__ inline uint2 ld_pair(const uint2* p) {
    const uint64_t w = ld_state(reinterpret_cast<const uint64_t*>(p));
    return make_uint2((uint32_t)w, (uint32_t)(w >> 32));
}

// FORCE: every bucket through the global-memory path (for tests).
// pairs: the split pass's output; tmp_keys, out.vals: a second buffer for that
// path (this bucket's own entries of both).
template <typename B, bool FORCE>
__global__ __launch_bounds__(B::THREADS) void k_bucket_sort(uint2* pairs, uint32_t* tmp_keys, const uint32_t* bases,
                                                         BucketOut out) {
    constexpr int THREADS = B::THREADS, BK_ITEMS = B::ITEMS;
    constexpr uint32_t CAP = B::CAP;
    __shared__ __align__(16) BucketLds<B> lds;
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid / 64;
    const uint32_t b0 = bases[blockIdx.x];
    const uint32_t b1 = bases[blockIdx.x + 1];
    if (out.order) place_tiles<THREADS>(bases, out, lds.wtot);
    if (b1 <= b0) return;
    const uint32_t cnt = b1 - b0, bits = out.lk.bits;
    uint2* src = pairs + b0;

    uint32_t* akeys = tmp_keys + b0;
    uint32_t* avals = out.vals + b0;
    // a debug render's keys, from the bucket's sorted local keys in akeys
    auto put_keys = [&]() {
        if (!out.want_keys()) return;
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        for (uint32_t e = tid; e < cnt; e += THREADS) out.put_key(b0 + e, ld_state(&akeys[e]));
    };
    if (!FORCE && cnt <= 2 * CAP) {
        // ---- the bucket in LDS, or in two runs: each half sorted in LDS and
        // written back in place, then the two merged ----
        const uint32_t runs = cnt <= CAP ? 1u : 2u;
        const uint32_t cA = runs == 1 ? cnt : (cnt + 1) / 2, cB = cnt - cA;
        for (uint32_t h = 0; h < runs; ++h) {
            const uint32_t o = h ? cA : 0u, m = h ? cB : cA;
            bucket_lds_sort<B>(src + o, m, bits, lds);
            if (runs == 1) {
                for (uint32_t e = tid; e < cnt; e += THREADS) {
                    const uint2 p = lds.pair[e];
                    out.vals[b0 + e] = p.y;
                    if (e == 0) out.start(b0, p.x);
                    else out.boundary(b0 + e, lds.pair[e - 1].x, p.x);
                    if (e + 1 == cnt) out.end(b0 + cnt, p.x);
                    if (out.want_keys()) out.put_key(b0 + e, p.x);
                }
                return;
            }
            for (uint32_t e = tid; e < m; e += THREADS) src[o + e] = lds.pair[e];
            __syncthreads();     // the first run's LDS before the second's loads
        }
        // both runs' keys into LDS, read past the CU's vector cache (it may
        // hold the first run's lines from before they were sorted)
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        uint32_t* keys = reinterpret_cast<uint32_t*>(lds.pair);
        for (uint32_t e0 = tid; e0 < cnt; e0 += BK_LOAD_BATCH * THREADS) {
            uint32_t t[BK_LOAD_BATCH];
#pragma unroll
            for (uint32_t j = 0; j < BK_LOAD_BATCH; ++j)
                t[j] = e0 + j * THREADS < cnt ? ld_state(&src[e0 + j * THREADS].x) : 0u;
#pragma unroll
            for (uint32_t j = 0; j < BK_LOAD_BATCH; ++j)
                if (e0 + j * THREADS < cnt) keys[e0 + j * THREADS] = t[j];
        }
        __syncthreads();
        // Merge path: thread t writes outputs [t S, (t + 1) S).  Its first
        // output takes i entries from A and o - i from B, i the least index
        // with A[i] > B[o - i - 1]; then the two are merged sequentially, A
        // first on equal keys (A holds the earlier entries: stable).
        const uint32_t* A = keys;
        const uint32_t* Bk = keys + cA;
        const uint32_t S = (cnt + THREADS - 1) / THREADS;
        const uint32_t o0 = tid * S, o1 = min(o0 + S, cnt);
        if (o0 < cnt) {
            uint32_t lo = o0 > cB ? o0 - cB : 0u, hi = min(o0, cA);
            while (lo < hi) {
                const uint32_t mid = (lo + hi) / 2;
                if (A[mid] <= Bk[o0 - mid - 1]) lo = mid + 1;
                else hi = mid;
            }
            uint32_t ia = lo, ib = o0 - lo;
            // the key before this thread's first output, for the tile runs
            uint32_t before = max(ia > 0 ? A[ia - 1] : 0u, ib > 0 ? Bk[ib - 1] : 0u);
            // BK_LOAD_BATCH outputs at a time: their value loads in flight together
            for (uint32_t ob = o0; ob < o1; ob += BK_LOAD_BATCH) {
                uint32_t key[BK_LOAD_BATCH], val[BK_LOAD_BATCH];
#pragma unroll
                for (uint32_t j = 0; j < BK_LOAD_BATCH; ++j) {
                    if (ob + j >= o1) break;
                    const bool take_a = ib >= cB || (ia < cA && A[ia] <= Bk[ib]);
                    const uint32_t at = take_a ? ia : cA + ib;
                    key[j] = take_a ? A[ia] : Bk[ib];
                    val[j] = ld_state(&src[at].y);
                    if (take_a) ++ia;
                    else ++ib;
                }
#pragma unroll
                for (uint32_t j = 0; j < BK_LOAD_BATCH; ++j) {
                    if (ob + j >= o1) break;
                    const uint32_t o = ob + j;
                    out.vals[b0 + o] = val[j];
                    if (o == 0) out.start(b0, key[j]);
                    else out.boundary(b0 + o, before, key[j]);
                    if (o + 1 == cnt) out.end(b0 + cnt, key[j]);
                    if (out.want_keys()) akeys[o] = key[j];
                    before = key[j];
                }
            }
        }
        put_keys();
        return;
    }

    // ---- a bucket larger than the LDS ----
    // Each pass streams it through global memory in chunks of CAP: a
    // histogram sweep, then the chunks in order, each ranked in LDS and
    // scattered after the chunks before it.  Passes alternate between the pairs
    // and the second buffer's arrays and their number is odd, so that the last
    // ends in the arrays.  Reads of what this workgroup wrote in the previous
    // pass bypass the CU's vector cache.
    uint32_t k[BK_ITEMS], v[BK_ITEMS], pos[BK_ITEMS];
    const uint32_t passes = digit_passes(bits) | 1u;
    for (uint32_t q = 0; q < passes; ++q) {
        const uint32_t shift = RADIX_BITS * q;
        const bool from_pairs = q % 2 == 0;
        if (tid < RADIX) lds.tot[tid] = 0;
        __syncthreads();
        for (uint32_t i0 = tid; i0 < cnt; i0 += BK_LOAD_BATCH * THREADS) {
            uint32_t t[BK_LOAD_BATCH];
#pragma unroll
            for (uint32_t j = 0; j < BK_LOAD_BATCH; ++j) {
                const uint32_t i = i0 + j * THREADS;
                t[j] = i < cnt ? ld_state(from_pairs ? &src[i].x : &akeys[i]) : 0u;
            }
#pragma unroll
            for (uint32_t j = 0; j < BK_LOAD_BATCH; ++j)
                if (i0 + j * THREADS < cnt) atomicAdd(&lds.tot[digit_at(t[j], shift)], 1u);
        }
        __syncthreads();
        const uint32_t base = digit_exclusive_scan<RADIX>(tid < RADIX ? lds.tot[tid] : 0u, lds.wtot);
        if (tid < RADIX) lds.base[tid] = base;
        __syncthreads();
        for (uint32_t c0 = 0; c0 < cnt; c0 += CAP) {
            const uint32_t ccnt = min(CAP, cnt - c0);
            const uint32_t R = (ccnt + THREADS - 1) / THREADS;
            const int lim = __builtin_amdgcn_readfirstlane((int)ccnt - (int)(wave * R * 64));
#pragma unroll
            for (int r = 0; r < BK_ITEMS; ++r) {
                k[r] = v[r] = 0u;
                if ((uint32_t)r < R && (int)lane < lim - r * 64) {
                    const uint32_t e = c0 + (wave * R + r) * 64 + lane;
                    if (from_pairs) {
                        const uint2 p = ld_pair(&src[e]);
                        k[r] = p.x;
                        v[r] = p.y;
                    } else {
                        k[r] = ld_state(&akeys[e]);
                        v[r] = ld_state(&avals[e]);
                    }
                }
            }
            bucket_rank<B>(k, ccnt, R, shift, pos, lds);
#pragma unroll
            for (int r = 0; r < BK_ITEMS; ++r) {
                if ((uint32_t)r < R && (int)lane < lim - r * 64) {
                    const uint32_t d = digit_at(k[r], shift);
                    const uint32_t dst = lds.base[d] + pos[r] - lds.bs[d];
                    if (dst < cnt) {      // always true for consistent counts
                        if (from_pairs) {
                            akeys[dst] = k[r];
                            avals[dst] = v[r];
                        } else {
                            src[dst] = make_uint2(k[r], v[r]);
                        }
                    }
                }
            }
            // the stores reach the L2 before any thread of the workgroup reads
            // them back (the next pass, the ranges)
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
            if (tid < RADIX) lds.base[tid] += lds.tot[tid];
            __syncthreads();
        }
    }
    // the arrays hold the bucket sorted
    for (uint32_t e = tid; e < cnt; e += THREADS) {
        const uint32_t key = ld_state(&akeys[e]);
        if (e == 0) out.start(b0, key);
        else out.boundary(b0 + e, ld_state(&akeys[e - 1]), key);
        if (e + 1 == cnt) out.end(b0 + cnt, key);
    }
    put_keys();
}

template <typename B>
static void launch_bucket(hipStream_t s, uint2* pairs, uint32_t* tmp_keys, const WsDev& ws, uint32_t buckets,
                          const BucketOut& out, bool force) {
    if (force)
        hipLaunchKernelGGL((k_bucket_sort<B, true>), dim3(buckets), dim3(B::THREADS), 0, s, pairs, tmp_keys,
                           ws.bases, out);
    else
        hipLaunchKernelGGL((k_bucket_sort<B, false>), dim3(buckets), dim3(B::THREADS), 0, s, pairs, tmp_keys,
                           ws.bases, out);
}

template <typename KeyT, int BITS>
static void launch_split_pass(hipStream_t s, const FrameDev& f, const WsDev& ws, uint2* pairs, bool force) {
    using S = SplitShape<BITS>;
    const PairsOut<KeyT> out{pairs, f.lk, ws.params};
    uint32_t* tiles = ws.sort_state;
    uint32_t* groups = ws.sort_state + (uint64_t)ws.sort_rows * S::DIGITS;
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(ws.sort_rows), dim3(S::THREADS), 0, s,
                           reinterpret_cast<const KeyT*>(ws.keys_a), ws.vals_a, out, ws.header, ws.hist,
                           (uint32_t)(MAX_PASSES * RADIX), tiles, groups, (uint32_t*)nullptr, (uint32_t*)nullptr,
                           f.split_shift, ws.bases);
    };
    if (force) launch(k_radix_pass<KeyT, S, PairsOut<KeyT>, true>);
    else launch(k_radix_pass<KeyT, S, PairsOut<KeyT>, false>);
}

void launch_sort_split(hipStream_t s, const FrameDev& f, const WsDev& ws, uint32_t key_bytes, bool force,
                       bool want_keys) {
    // pairs in the second key and value arrays (32-bit keys: the two are
    // adjacent); sorted values in the first value array
    uint2* pairs = reinterpret_cast<uint2*>(ws.keys_b);
    if (key_bytes == 8) {
        if (f.split_bits == 10) launch_split_pass<uint64_t, 10>(s, f, ws, pairs, force);
        else launch_split_pass<uint64_t, 8>(s, f, ws, pairs, force);
    } else {
        if (f.split_bits == 10) launch_split_pass<uint32_t, 10>(s, f, ws, pairs, force);
        else launch_split_pass<uint32_t, 8>(s, f, ws, pairs, force);
    }
    const uint32_t buckets = 1u << f.split_bits;
    BucketOut out{};
    out.vals = ws.vals_a;
    out.ranges = ws.ranges;
    // 32-bit keys replace the emitted ones; 64-bit keys take the place of their own pairs
    out.keys32 = want_keys && key_bytes == 4 ? reinterpret_cast<uint32_t*>(ws.keys_a) : nullptr;
    out.keys64 = want_keys && key_bytes == 8 ? reinterpret_cast<uint64_t*>(ws.keys_b) : nullptr;
    out.order = f.ordered == ORDER_BUCKETS ? ws.order : nullptr;
    out.error = &ws.header->error;
    out.prm = ws.params;
    out.lk = f.lk;
    out.n_tiles = (uint32_t)f.n_tiles;
    uint32_t* tmp_keys = reinterpret_cast<uint32_t*>(ws.keys_a);
    // The workgroup by the entries a bucket may hold on average (what the
    // workspace holds, usually 1.25 to 2 times the frame's): the busiest bucket
    // has about twice the frame's average, and should still be one run in LDS,
    // while smaller workgroups start together and share a CU better.  Kernel
    // times in us with 512 x 9, 512 x 16 and 1024 x 16 entries:
    // 1280x720 28, 35, 56; 1080p (1M) 33, 42, 68 (plain 65, 63, 94); 4K (3M) 94, 73, 104.
    const uint32_t room = f.capacity >> f.split_bits;
    if (room <= 4608) launch_bucket<BucketShape<512, 9>>(s, pairs, tmp_keys, ws, buckets, out, force);
    else if (room <= 12288) launch_bucket<BucketShape<512, 16>>(s, pairs, tmp_keys, ws, buckets, out, force);
    else launch_bucket<BucketShape<1024, 16>>(s, pairs, tmp_keys, ws, buckets, out, force);
}

// ---------------------------------------------------------------------------
// Tile ranges: the run of each tile in the sorted keys.  Entry i starts a run
// when its tile differs from entry i-1's, and ends the previous run there.
// Each thread takes RANGES_ITEMS consecutive keys with 16-byte loads.

constexpr int RANGES_ITEMS = 8;

template <typename KeyT>
__device__ inline void load_run(const KeyT* __restrict__ keys, uint64_t i0, uint32_t n, KeyT (&k)[RANGES_ITEMS]) {
    if (i0 + RANGES_ITEMS <= n) {
        // i0 is a multiple of RANGES_ITEMS and the buffers are 256-byte aligned
        const uint4* p = reinterpret_cast<const uint4*>(keys + i0);
        constexpr int VEC = RANGES_ITEMS * sizeof(KeyT) / 16;
        uint4 v[VEC];
#pragma unroll
        for (int q = 0; q < VEC; ++q) v[q] = p[q];
        __builtin_memcpy(k, v, sizeof(k));
    } else {
#pragma unroll
        for (int r = 0; r < RANGES_ITEMS; ++r) k[r] = i0 + r < n ? keys[i0 + r] : (KeyT)0;
    }
}

template <typename KeyT>
__global__ __launch_bounds__(256) void k_ranges(const KeyT* __restrict__ keys, WsDev ws,
                                                uint32_t shift, uint32_t n_tiles) {
    const uint32_t n = entry_count(ws.header);
    const uint64_t i0 = ((uint64_t)blockIdx.x * 256 + threadIdx.x) * RANGES_ITEMS;
    if (i0 >= n) return;
    KeyT k[RANGES_ITEMS];
    load_run(keys, i0, n, k);
    uint32_t tp = i0 ? (uint32_t)(keys[i0 - 1] >> shift) : 0xffffffffu;
#pragma unroll
    for (int r = 0; r < RANGES_ITEMS; ++r) {
        const uint64_t i = i0 + r;
        if (i >= n) break;
        const uint32_t t = (uint32_t)(k[r] >> shift);
        if (t >= n_tiles || (i && tp >= n_tiles)) {     // only after a failed sort
            atomicOr(&ws.header->error, 4u);
            return;
        }
        if (i == 0) {
            ws.ranges[2 * t] = 0;
        } else if (tp != t) {
            ws.ranges[2 * tp + 1] = (uint32_t)i;
            ws.ranges[2 * t] = (uint32_t)i;
        }
        if (i == n - 1) ws.ranges[2 * t + 1] = n;
        tp = t;
    }
}

void launch_ranges(hipStream_t s, const FrameDev& f, const WsDev& ws, uint32_t key_bytes,
                   bool result_in_b) {
    const uint64_t per_block = 256ull * RANGES_ITEMS;
    const uint32_t blocks = (uint32_t)((f.capacity + per_block - 1) / per_block);
    if (key_bytes == 8)
        hipLaunchKernelGGL(k_ranges<uint64_t>, dim3(blocks), dim3(256), 0, s,
                           reinterpret_cast<const uint64_t*>(result_in_b ? ws.keys_b : ws.keys_a), ws, 32u,
                           (uint32_t)f.n_tiles);
    else
        hipLaunchKernelGGL(k_ranges<uint32_t>, dim3(blocks), dim3(256), 0, s,
                           reinterpret_cast<const uint32_t*>(result_in_b ? ws.keys_b : ws.keys_a), ws,
                           (uint32_t)f.b_d, (uint32_t)f.n_tiles);
}

// ---------------------------------------------------------------------------
// The rasterizers' schedule.  A tile's time grows with its list, and list
// lengths differ several-fold between tiles; workgroups are dispatched in
// grid order, so a grid that ends on long tiles leaves most CUs idle while
// they finish.  In frames that take this schedule (ORDER_TILES; most frames take
// the bucket sort's), workgroup b renders tile order[b], where order lists the tiles of each
// chunk of ORDER_CHUNK longest first: each tile falls in one of ORDER_CLASSES
// classes of equal width in entry count (up to the chunk's longest list) and
// the classes follow one another in decreasing length (a
// longest-processing-time-first schedule; on the tile costs of the 1M / 1080p
// frame, 32 classes come within 0.2 % of an exact sort in a list-scheduling
// model).  Inside a class tiles stay in row-major order, so that tiles that
// run at about the same time still share some records in the caches.  No
// result depends on the order.
//
// One workgroup per chunk, no atomics: thread i takes tiles i, i + 1024, ...
// (round k), each wave ranks the tiles of one round within their class with
// five ballots (as the radix passes rank digits), and a scan over the
// (class, round, wave) counts places them.  The kernel takes about 10 us at
// 1M / 1080p: about 3 us to load the ranges, 2.4 us of ballots on the four
// SIMDs of a single CU, 1 us of scan and 2 us of stores; the fast rasterizer
// went from 0.123 to 0.106 ms, the plain one from 0.646 to 0.567 ms.

constexpr uint32_t ORDER_THREADS = 1024;
constexpr uint32_t ORDER_WAVES = ORDER_THREADS / 64;
constexpr uint32_t ORDER_CHUNK = 8192;
constexpr uint32_t ORDER_PER = ORDER_CHUNK / ORDER_THREADS;
constexpr uint32_t ORDER_CLASS_BITS = 5;
constexpr uint32_t ORDER_CLASSES = 1u << ORDER_CLASS_BITS;
static_assert(ORDER_CLASSES * ORDER_WAVES * ORDER_PER == 4 * ORDER_THREADS, "four (class, k, wave) groups per thread");

__global__ __launch_bounds__(ORDER_THREADS) void k_tile_order(WsDev ws, uint32_t n_tiles) {
    constexpr uint32_t GROUPS = ORDER_CLASSES * ORDER_WAVES * ORDER_PER;
    // tiles per (class, k, wave) group, class-major; the scan turns them into places
    __shared__ uint4 s_grp4[GROUPS / 4];
    __shared__ uint32_t s_red[ORDER_WAVES];
    uint32_t* s_grp = reinterpret_cast<uint32_t*>(s_grp4);
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid / 64;
    const uint32_t t0 = blockIdx.x * ORDER_CHUNK;
    const uint32_t t1 = min(t0 + ORDER_CHUNK, n_tiles);
    s_grp4[tid] = make_uint4(0u, 0u, 0u, 0u);
    // tile t0 + k * ORDER_THREADS + tid: its entry count, then the chunk's longest
    const uint2* __restrict__ rg = reinterpret_cast<const uint2*>(ws.ranges);
    uint32_t len[ORDER_PER];
    uint32_t longest = 0;
#pragma unroll
    for (uint32_t k = 0; k < ORDER_PER; ++k) {
        const uint32_t t = t0 + k * ORDER_THREADS + tid;
        len[k] = 0;
        if (t < t1) {
            const uint2 r = rg[t];
            len[k] = r.y > r.x ? r.y - r.x : 0u;
        }
        longest = max(longest, len[k]);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) longest = max(longest, (uint32_t)__shfl_xor((int)longest, off, 64));
    if (lane == 0) s_red[wave] = longest;
    __syncthreads();
    longest = 0;
#pragma unroll
    for (uint32_t w = 0; w < ORDER_WAVES; ++w) longest = max(longest, s_red[w]);
    const float scale = (float)ORDER_CLASSES / ((float)longest + 1.0f);
    // class (0 = longest lists) and rank among the tiles of the same (wave, k) group
    uint32_t cls[ORDER_PER], rank[ORDER_PER];
#pragma unroll
    for (uint32_t k = 0; k < ORDER_PER; ++k) {
        const bool valid = t0 + k * ORDER_THREADS + tid < t1;
        const uint32_t c = ORDER_CLASSES - 1 - min(ORDER_CLASSES - 1, (uint32_t)((float)len[k] * scale));
        uint32_t diff_lo = 0, diff_hi = 0;
#pragma unroll
        for (uint32_t b = 0; b < ORDER_CLASS_BITS; ++b) {
            const uint32_t spread = (uint32_t)((int32_t)(c << (31 - b)) >> 31);
            const uint64_t m = __ballot(spread != 0);
            diff_lo = __builtin_amdgcn_bitop3_b32((uint32_t)m, spread, diff_lo, 0xBE);
            diff_hi = __builtin_amdgcn_bitop3_b32((uint32_t)(m >> 32), spread, diff_hi, 0xBE);
        }
        const uint64_t vmask = __ballot(valid);
        const uint32_t peers_lo = ~diff_lo & (uint32_t)vmask, peers_hi = ~diff_hi & (uint32_t)(vmask >> 32);
        const uint32_t below = __builtin_amdgcn_mbcnt_hi(peers_hi, __builtin_amdgcn_mbcnt_lo(peers_lo, 0u));
        cls[k] = c;
        rank[k] = below;
        if (valid && below == 0)
            s_grp[(c * ORDER_PER + k) * ORDER_WAVES + wave] = (uint32_t)(__popc(peers_lo) + __popc(peers_hi));
    }
    __syncthreads();
    // places: exclusive scan of the group counts, four consecutive groups per thread
    const uint4 g = s_grp4[tid];
    const uint32_t sum4 = g.x + g.y + g.z + g.w;
    const uint32_t incl = wave_inclusive_scan(sum4);
    if (lane == 63) s_red[wave] = incl;
    __syncthreads();
    uint32_t before = incl - sum4;
    for (uint32_t w = 0; w < wave; ++w) before += s_red[w];
    s_grp4[tid] = make_uint4(before, before + g.x, before + g.x + g.y, before + g.x + g.y + g.z);
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < ORDER_PER; ++k) {
        const uint32_t t = t0 + k * ORDER_THREADS + tid;
        if (t < t1) ws.order[t0 + s_grp[(cls[k] * ORDER_PER + k) * ORDER_WAVES + wave] + rank[k]] = t;
    }
}

void launch_tile_order(hipStream_t s, const FrameDev& f, const WsDev& ws) {
    const uint32_t n_tiles = (uint32_t)f.n_tiles;
    hipLaunchKernelGGL(k_tile_order, dim3((n_tiles + ORDER_CHUNK - 1) / ORDER_CHUNK), dim3(ORDER_THREADS), 0, s,
                       ws, n_tiles);
}

}  // namespace rgs
