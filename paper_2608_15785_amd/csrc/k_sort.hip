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
// Frames of more than 2^7 tiles (8 tile bits) take the index's top bits first, in one such
// pass, and the rest per bucket in LDS (the split sort below), which also writes
// the tile ranges.
#include "rgs_internal.h"

namespace rgs {


// A radix pass's shape: digit width, threads and keys per thread of a tile, and the
// waves a SIMD that the registers must allow, two workgroups a CU of the LSD passes
// (64-bit keys, six passes at 1M / 1080p: 136 us, with one workgroup 177; 32-bit keys
// with three, as their LDS allows, spill: four passes of 1M at 176x176 78 us, 65 with two).
template <int BITS_, int THREADS_, int ITEMS_, int WAVES_SIMD_>
struct PassShape {
    static constexpr int BITS = BITS_, THREADS = THREADS_, ITEMS = ITEMS_, WAVES_SIMD = WAVES_SIMD_;
    static constexpr uint32_t DIGITS = 1u << BITS;
    static constexpr int WAVES = THREADS / 64;
    static constexpr uint32_t SIZE = THREADS * ITEMS;
    static constexpr uint32_t SPLIT = THREADS / DIGITS;      // threads per digit in the look-back
    static_assert(THREADS % DIGITS == 0 && THREADS >= (int)DIGITS, "whole digit rows per block");
};
template <typename KeyT>
using LsdShape = PassShape<RADIX_BITS, SORT_THREADS, SortTile<KeyT>::ITEMS, 4>;
template <int BITS>
using SplitShape = PassShape<BITS, SPLIT_THREADS, SPLIT_ITEMS, 4>;

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
// VOTE: bit 31 of the totals tells every thread (any) whether a thread below DIGITS has
// set its flag.
template <uint32_t DIGITS, bool LDS_ONLY, bool VOTE>
__device__ inline uint32_t digit_exclusive_scan(uint32_t x, uint32_t* s_wtot, bool flag, bool& any) {
    constexpr uint32_t FLAG = VOTE ? 0x80000000u : 0u;
    auto barrier = [] {
        if (LDS_ONLY) lds_barrier();
        else __syncthreads();
    };
    const uint32_t lane = lane_id(), wave = threadIdx.x / 64;
    const uint32_t incl = wave_inclusive_scan(x);
    const uint32_t mark = VOTE && __ballot(flag) != 0 ? FLAG : 0u;
    if (lane == 63 && wave < DIGITS / 64) s_wtot[wave] = incl | mark;
    barrier();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (uint32_t w = 0; w < DIGITS / 64; ++w) {
        if (w < wave) before += s_wtot[w] & ~FLAG;
        all |= s_wtot[w];
    }
    barrier();
    any = VOTE && __builtin_amdgcn_readfirstlane(all) >= FLAG;
    return incl - x + before;
}
template <uint32_t DIGITS>
__device__ inline uint32_t digit_exclusive_scan(uint32_t x, uint32_t* s_wtot) {
    bool any;
    return digit_exclusive_scan<DIGITS, false, false>(x, s_wtot, false, any);
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

// What the split pass leaves for the bucket sort beside the entries.  In a frame with a
// bucket of more than `limit` entries, every bucket of more than `alone` is sorted by
// several workgroups, about `part` entries each.
struct SplitPlan {
    uint32_t* bases;        // each bucket's first place and, after the last, the entry count
    uint32_t* n_parts;      // parts of all such buckets together
    uint32_t* parts;        // of the buckets up to this one (if there are any)
    uint32_t limit, alone, part;
};

// Where a pass leaves its entries: the LSD passes a key and a value array, the
// split pass (local key, value) pairs (see the split sort below).
template <typename KeyT>
struct ArraysOut {
    static constexpr bool PAIRS = false;
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
    static constexpr bool PAIRS = true;
    using Held = uint32_t;
    uint2* pairs;
    LocalKey lk;
    const FrameParams* prm;
    __host__ __device__ Held hold(uint32_t k) const { return k; }
    __host__ __device__ uint32_t digit(Held h, uint32_t shift, uint32_t) const { return h >> shift; }
    __device__ uint32_t local(Held h) const { return h & ((1u << lk.bits) - 1u); }
    __device__ void put(uint32_t at, Held h, uint32_t v) const { pairs[at] = make_uint2(local(h), v); }
};
// 64-bit keys: (tile bits below the top digit, float32 depth bits above the
// nearest depth's).  The digit is masked, as where the tile ranks its keys: after a
// front end that gave up, keys are whatever memory held, and their bits above the
// tile index must not index the digit tables.
template <>
struct PairsOut<uint64_t> {
    static constexpr bool PAIRS = true;
    using Held = uint64_t;
    uint2* pairs;
    LocalKey lk;
    const FrameParams* prm;
    __host__ __device__ Held hold(uint64_t k) const { return k; }
    __host__ __device__ uint32_t digit(Held h, uint32_t shift, uint32_t mask) const { return (uint32_t)(h >> shift) & mask; }
    __device__ uint32_t local(Held h) const {
        const uint32_t tile = (uint32_t)(h >> 32) & ((1u << lk.tile_bits) - 1u);
        const uint32_t depth = (uint32_t)h - depth_key_base(prm->cam);
        return lk.tile_bits ? (tile << (lk.bits - lk.tile_bits)) | depth : depth;
    }
    __device__ void put(uint32_t at, Held h, uint32_t v) const { pairs[at] = make_uint2(local(h), v); }
};

// The digit of a local key at `shift` (0 past its end).
__device__ inline uint32_t digit_at(uint32_t k, uint32_t shift) {
    return shift < 32 ? (k >> shift) & (RADIX - 1) : 0u;
}

// Digits of a local key of `bits` bits.
__device__ inline uint32_t digit_passes(uint32_t bits) { return bits ? (bits + RADIX_BITS - 1) / RADIX_BITS : 1u; }

// Ranks the keys of one wave among those with equal digits, in entry order: round r,
// lane l holds entry first + r * 64 + l, existing ones below n.  my_hist: the wave's
// digit counts, from zero on.
// Lanes of a wave read counters that other lanes of the same wave wrote in
// the previous round.  The LDS unit executes one wave's accesses in issue
// order; the empty asm with a memory clobber keeps the compiler from
// moving or reusing accesses across rounds.  (A volatile pointer would do
// the same but loses the LDS address space: every access becomes a flat
// access that waits on all outstanding global memory operations.)
template <int BITS, int ITEMS, typename KeyT, typename DigitFn>
__device__ inline void rank_wave(const KeyT (&k)[ITEMS], uint32_t first, uint32_t n, DigitFn digit, uint16_t* my_hist,
                                 uint32_t (&rank)[ITEMS]) {
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        asm volatile("" ::: "memory");
        const bool valid = first + r * 64 + lane_id() < n;
        const uint32_t d = digit(k[r]);
        // lanes whose digit differs from this lane's: for each bit b the
        // ballot M_b of lanes holding a 1, XOR-ed with this lane's bit spread
        // to a whole word (0 or all ones), marks the lanes that disagree on b.
        // One three-input bit operation per half-mask folds M_b ^ spread into
        // the running OR (truth table 0xBE: S2 | (S0 ^ S1)).
        uint32_t diff_lo = 0, diff_hi = 0;
#pragma unroll
        for (int b = 0; b < BITS; ++b) {
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
}

// Orders a radix tile by its entries' local keys, all digits, in LDS: the entries come
// and leave in registers, in rank_wave's layout with wave w's first entry at w ITEMS
// 64.  Every thread calls it (barriers); whist is scratch.
template <typename S, typename KeyT, typename Out>
__device__ inline void sort_tile_local(KeyT (&k)[S::ITEMS], uint32_t (&v)[S::ITEMS], uint32_t n_valid, const Out& out,
                                       uint32_t* whist, uint32_t* wtot, KeyT* keys, uint32_t* vals) {
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid / 64;
    const uint32_t first = wave * (S::ITEMS * 64);
    uint16_t* my_hist = reinterpret_cast<uint16_t*>(whist) + wave * RADIX;
    uint32_t rank[S::ITEMS];
    for (uint32_t q = 0; q < digit_passes(out.lk.bits); ++q) {
        auto digit = [&](KeyT key) { return digit_at(out.local(key), RADIX_BITS * q); };
        __syncthreads();
        for (uint32_t i = tid; i < S::WAVES * RADIX / 2; i += S::THREADS) whist[i] = 0;
        __syncthreads();
        rank_wave<RADIX_BITS>(k, first, n_valid, digit, my_hist, rank);
        __syncthreads();
        uint16_t* h = reinterpret_cast<uint16_t*>(whist) + tid;
        uint32_t tot = 0;
        if (tid < RADIX)
            for (int w = 0; w < S::WAVES; ++w) tot += h[w * RADIX];
        uint32_t at = digit_exclusive_scan<RADIX>(tot, wtot);
        if (tid < RADIX)
            for (int w = 0; w < S::WAVES; ++w) {
                const uint32_t c = h[w * RADIX];
                h[w * RADIX] = (uint16_t)at;
                at += c;
            }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < S::ITEMS; ++r) {
            if (first + r * 64 + lane < n_valid) {
                const uint32_t pos = my_hist[digit(k[r])] + rank[r];
                keys[pos] = k[r];
                vals[pos] = v[r];
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < S::ITEMS; ++r) {
            const uint32_t e = first + r * 64 + lane;
            k[r] = e < n_valid ? keys[e] : (KeyT)0;
            v[r] = e < n_valid ? vals[e] : 0u;
        }
    }
    __syncthreads();
}

// Shared memory of a radix pass.
template <typename S, typename Held>
struct alignas(8) TileLds {
    // per-wave digit counts (at most 64 ITEMS each), then where each wave's run of a
    // digit starts in the reordered tile; reused for the look-back once the tile is
    // reordered
    static constexpr uint32_t WHIST_WORDS = S::WAVES * S::DIGITS / 2 > (S::SPLIT + 3) * S::DIGITS
                                                ? S::WAVES * S::DIGITS / 2
                                                : (S::SPLIT + 3) * S::DIGITS;
    Held keys[S::SIZE];
    uint32_t vals[S::SIZE];
    uint32_t whist[WHIST_WORDS];
    uint32_t bstart[S::DIGITS];   // first LDS position of digit d in the reordered tile
    uint32_t gbase[S::DIGITS];    // bucket base of d, then output position minus bstart[d]
    uint32_t tot[S::DIGITS];      // the tile's count of digit d
    uint32_t wtot[S::DIGITS / 64];
    uint32_t missed[2];           // look-back votes: some thread found an unpublished word
};

// The split pass in a frame with a bucket for more than one workgroup, a function of its own
// (radix_tile).  Its arguments come in LDS, as what a call cannot pass in registers
// would make the kernel's stack larger.
template <typename KeyT, typename Out>
struct PassArgs {
    const KeyT* kin;
    const uint32_t* vin;
    Out out;
    const WsHeader* header;
    const uint32_t* hist;
    uint32_t *tiles, *groups;
    uint32_t hist_stride, shift;
    SplitPlan plan;
};
template <typename T>
using Lds = __attribute__((address_space(3))) T;
template <typename KeyT, typename S, typename Out, bool FORCE>
__device__ void crowded_tile(Lds<TileLds<S, typename Out::Held>>* lds);

// One stable radix pass on the digit at `shift`.  hist[c][d]: HIST_COPIES copies,
// hist_stride words apart, of the digit counts of the whole input.  tiles,
// groups: this pass's look-back words; next_tiles, next_groups: those of the
// frame's next pass, cleared here (null: none).  The split pass also leaves the
// bucket sort's plan (SplitPlan).
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
// SORTED: with the tile's entries ordered by their local keys first (sort_tile_local).
template <typename KeyT, typename S, typename Out, bool FORCE, bool SORTED>
__device__ inline void radix_tile(const KeyT* __restrict__ kin, const uint32_t* __restrict__ vin, const Out& out,
                                  const WsHeader* header, const uint32_t* hist, uint32_t hist_stride, uint32_t* tiles,
                                  uint32_t* groups, uint32_t* next_tiles, uint32_t* next_groups, uint32_t shift,
                                  const SplitPlan& plan, TileLds<S, typename Out::Held>& lds) {
    constexpr int ITEMS = S::ITEMS;
    constexpr uint32_t SIZE = S::SIZE, DIGITS = S::DIGITS;
    constexpr uint32_t WHIST_WORDS = TileLds<S, typename Out::Held>::WHIST_WORDS;
    using Held = typename Out::Held;
    uint32_t *s_whist = lds.whist, *s_bstart = lds.bstart, *s_gbase = lds.gbase, *s_tot = lds.tot;
    uint32_t *s_wtot = lds.wtot, *s_missed = lds.missed, *s_vals = lds.vals;
    Held* s_keys = lds.keys;

    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid / 64;
    const uint32_t n = entry_count(header);
    const uint32_t vb = blockIdx.x;      // the radix tile: keys [vb * SIZE, (vb + 1) * SIZE)
    const uint32_t tile_base = vb * SIZE;
    if (tile_base >= n) {
        if (Out::PAIRS && n == 0 && vb == 0) {
            for (uint32_t i = tid; i <= DIGITS; i += S::THREADS) plan.bases[i] = 0;
            if (tid == 0) *plan.n_parts = 0;
        }
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
    bool crowded;
    const uint32_t bbase =
        digit_exclusive_scan<DIGITS, true, Out::PAIRS>(bucket, s_wtot, bucket > plan.limit, crowded);
    uint16_t* my_hist = reinterpret_cast<uint16_t*>(s_whist) + wave * DIGITS;
    // A crowded frame starts over in code of its own, so that the pass of other frames stays
    // as it is: as a function it takes 0 to 0.5 us from them (one copy of the rest after a
    // branch 1 to 3 us).  Small frames of 32-bit keys and 8 bits, for which the
    // function's stack costs 1 us, take a second copy of the rest.
    if constexpr (Out::PAIRS && !SORTED) {
        if (__builtin_expect(crowded, false)) {
            __syncthreads();
            if constexpr (sizeof(KeyT) == 4 && S::BITS == 8) {
                radix_tile<KeyT, S, Out, FORCE, true>(kin, vin, out, header, hist, hist_stride, tiles, groups, nullptr,
                                                      nullptr, shift, plan, lds);
            } else {
                using Args = PassArgs<KeyT, Out>;
                static_assert(sizeof(Args) <= sizeof(lds.keys) && alignof(Args) <= 8, "the arguments fit");
                if (tid == 0) {         // (field by field: a temporary would live in LDS, a copy per thread)
                    Args* a = reinterpret_cast<Args*>(s_keys);
                    a->kin = kin;
                    a->vin = vin;
                    a->out.pairs = out.pairs;
                    a->out.lk.bits = out.lk.bits;
                    a->out.lk.tile_bits = out.lk.tile_bits;
                    a->out.prm = out.prm;
                    a->header = header;
                    a->hist = hist;
                    a->tiles = tiles;
                    a->groups = groups;
                    a->hist_stride = hist_stride;
                    a->shift = shift;
                    a->plan.bases = plan.bases;
                    a->plan.n_parts = plan.n_parts;
                    a->plan.parts = plan.parts;
                    a->plan.limit = plan.limit;
                    a->plan.alone = plan.alone;
                    a->plan.part = plan.part;
                }
                __syncthreads();
                crowded_tile<KeyT, S, Out, FORCE>((Lds<TileLds<S, Held>>*)&lds);
            }
            return;
        }
    }
    if constexpr (SORTED) {
        sort_tile_local<S>(k, v, n_valid, out, s_whist, s_wtot, s_keys, s_vals);
        for (uint32_t i = tid; i < WHIST_WORDS; i += S::THREADS) s_whist[i] = 0;
        __syncthreads();
    }
    uint32_t rank[ITEMS];
    rank_wave<S::BITS>(k, wbase, n, [&](KeyT key) { return (uint32_t)(key >> shift) & (DIGITS - 1); }, my_hist, rank);
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
    }
    __syncthreads();

    if (Out::PAIRS && vb == 0) {
        const uint32_t size = tid < DIGITS ? min(bbase + bucket, n) - min(bbase, n) : 0u;
        const uint32_t parts = size > plan.alone ? (size + plan.part - 1) / plan.part : 0u;
        const uint32_t before = SORTED ? digit_exclusive_scan<DIGITS>(parts, s_wtot) : 0u;
        if (tid < DIGITS) {
            plan.bases[tid] = min(bbase, n);
            if (tid == 0) plan.bases[DIGITS] = n;
            if (SORTED) plan.parts[tid] = before + parts;
            if (tid == DIGITS - 1) *plan.n_parts = SORTED ? before + parts : 0u;
        }
    }

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

template <typename KeyT, typename S, typename Out, bool FORCE>
__device__ __attribute__((noinline)) void crowded_tile(Lds<TileLds<S, typename Out::Held>>* lds) {
    auto& tile = *(TileLds<S, typename Out::Held>*)lds;
    union Words {
        PassArgs<KeyT, Out> args;
        int word[sizeof(PassArgs<KeyT, Out>) / 4];
        __device__ Words() {}
    } a;
#pragma unroll
    for (uint32_t i = 0; i < sizeof(a.word) / 4; ++i)
        a.word[i] = __builtin_amdgcn_readfirstlane(reinterpret_cast<const int*>(tile.keys)[i]);
    __syncthreads();
    const PassArgs<KeyT, Out>& p = a.args;
    radix_tile<KeyT, S, Out, FORCE, true>(p.kin, p.vin, p.out, p.header, p.hist, p.hist_stride, p.tiles, p.groups,
                                          nullptr, nullptr, p.shift, p.plan, tile);
}

template <typename KeyT, typename S, typename Out, bool FORCE>
__global__ __launch_bounds__(S::THREADS, S::WAVES_SIMD) void k_radix_pass(const KeyT* __restrict__ kin,
                                                           const uint32_t* __restrict__ vin, Out out,
                                                           const WsHeader* header, const uint32_t* hist,
                                                           uint32_t hist_stride, uint32_t* tiles, uint32_t* groups,
                                                           uint32_t* next_tiles, uint32_t* next_groups, uint32_t shift,
                                                           SplitPlan plan) {
    __shared__ TileLds<S, typename Out::Held> lds;
    radix_tile<KeyT, S, Out, FORCE, false>(kin, vin, out, header, hist, hist_stride, tiles, groups, next_tiles,
                                           next_groups, shift, plan, lds);
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
                               (uint32_t)(RADIX_BITS * p), SplitPlan{});
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
// The split sort, for frames of SPLIT_MIN_BT tile bits or more (129 tiles).  The same
// stable sort, reorganised:
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
//     in place, and the two merged;
//   * one of more, up to the shape's LIMIT, is streamed by its workgroup through global
//     memory, digit by digit (stream_bucket);
//   * the entries of a view from afar crowd into few tiles, and then into few
//     buckets.  In a crowded frame, one with a bucket beyond the LIMIT, every bucket of
//     more than CAP entries is divided among workgroups (sort_part).  The split pass, whose
//     tiles all know the bucket sizes, then leaves its tiles sorted by the whole
//     key, so that the bucket consists of one sorted run per radix tile; a part finds
//     its two cuts through the runs by their keys, gathers its entries and sorts
//     them in LDS.  No workgroup waits for another;
//   * a workgroup, holding its entries sorted, writes its tiles' ranges.
// Every pass is stable and the top digit is taken first, then the rest least
// significant first; as a stable sort on the top digit followed by a stable
// sort on the rest leaves the keys ordered by (top digit, rest) with ties in
// input order, the result is the LSD sort's, bit for bit.  The frame then needs
// two sort kernels instead of four (32-bit keys) or six (64-bit keys, 1080p and
// 4K) passes and the ranges kernel.

constexpr uint32_t BK_LOAD_BATCH = 8;       // loads of a thread in flight where a loop stages or merges

// A bucket's workgroup: threads, entries each holds, the waves a SIMD that its LDS
// allows (the registers must not allow fewer), and the limit of the buckets that one
// workgroup sorts.
//
// The limit: streaming costs a time with the one bucket's entries, dividing one with all the
// frame's, which the split pass sorts by the whole key.  Sort in us, streamed and
// divided: 512 x 9, busiest bucket of 2 to 3 CAP (1M Gaussians / 1080p from 40) 80, 80 (plain
// 194, 215), of 3 to 4 CAP (from 60) 156, 133 (312, 174), of more (from 200) 707, 141 (1378,
// 184); 512 x 16 of 3 to 4 CAP (3M / 4K from 100, plain) 522, 571, of more (from 300) 1600,
// 490; 1024 x 16 of 3 to 4 CAP (6M / 4K from 100, plain) 850, 1190.
template <int THREADS_, int ITEMS_, int WAVES_SIMD_, uint32_t LIMIT_CAPS>
struct BucketShape {
    static constexpr int THREADS = THREADS_, ITEMS = ITEMS_, WAVES_SIMD = WAVES_SIMD_;
    static constexpr int WAVES = THREADS / 64;
    static constexpr uint32_t CAP = THREADS * ITEMS;
    static constexpr uint32_t LIMIT = LIMIT_CAPS * CAP;
    // a part of a divided bucket: CAP entries at most with both cuts off by the tolerance
    static constexpr uint32_t TOLERANCE = CAP / 8, PART = CAP - 2 * TOLERANCE;
};

// Shared memory of the bucket sort.
template <typename B>
struct BucketLds {
    static constexpr int WORDS = B::WAVES > RADIX / 64 ? B::WAVES : RADIX / 64;
    uint2 pair[B::CAP];                        // (local key, value)
    uint16_t whist[B::WAVES * RADIX];          // per-wave digit counts, then places (below CAP)
    uint32_t tot[RADIX], bs[RADIX], base[RADIX];
    uint32_t wtot[WORDS];
    uint32_t red[2][6][B::WAVES];              // block-wide sums and extremes
};

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
    uint32_t bucket;        // set by the workgroup

    __device__ uint32_t tile_of(uint32_t local) const {
        const uint32_t depth_bits = lk.bits - lk.tile_bits;
        return (bucket << lk.tile_bits) | (lk.tile_bits ? local >> depth_bits : 0u);
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

// Sorts m <= CAP pairs by their local key in LDS, all digits, leaving them in
// lds.pair.  Entry e is held in round r < R = ceil(m / THREADS) by (wave, lane)
// with e = (wave R + r) 64 + lane, the layout of bucket_rank; it comes from
// load(a, b), e = a + b, every load of a thread in flight at once.  The bounds are wave-uniform counts
// against the lane index, so that no per-entry index stays live across the
// passes.  Every thread calls it (barriers).
template <typename B, typename LoadFn>
__device__ inline void bucket_lds_sort(LoadFn load, uint32_t m, uint32_t bits, BucketLds<B>& lds) {
    constexpr int THREADS = B::THREADS, BK_ITEMS = B::ITEMS;
    const uint32_t lane = lane_id(), wave = threadIdx.x / 64;
    uint32_t k[BK_ITEMS], v[BK_ITEMS], pos[BK_ITEMS];
    const uint32_t R = (m + THREADS - 1) / THREADS;
    const int lim = __builtin_amdgcn_readfirstlane((int)m - (int)(wave * R * 64));
    const uint32_t first = wave * R * 64 + lane;
    const uint2* held = lds.pair + first;
#pragma unroll
    for (int r = 0; r < BK_ITEMS; ++r) {
        const uint2 p = (uint32_t)r < R && (int)lane < lim - r * 64 ? load(first, r * 64) : make_uint2(0u, 0u);
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

// Writes the m sorted entries in lds.pair to the frame's places from `at` on.  head,
// tail: they begin, end the bucket; if not head, `before` is the key before them.
template <typename B>
__device__ inline void write_sorted(const BucketLds<B>& lds, uint32_t at, uint32_t m, bool head, bool tail,
                                    uint32_t before, const BucketOut& out) {
    for (uint32_t e = threadIdx.x; e < m; e += B::THREADS) {
        const uint2 p = lds.pair[e];
        out.vals[at + e] = p.y;
        if (e > 0) out.boundary(at + e, lds.pair[e - 1].x, p.x);
        else if (head) out.start(at, p.x);
        else out.boundary(at, before, p.x);
        if (e + 1 == m && tail) out.end(at + m, p.x);
        if (out.want_keys()) out.put_key(at + e, p.x);
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

// Merges the two sorted runs src[0, cA) and src[cA, cA + cB) of a bucket, which this
// workgroup has just written.
template <typename B>
__device__ inline void merge_runs(const uint2* src, uint32_t cA, uint32_t cB, uint32_t b0, const BucketOut& out,
                                  BucketLds<B>& lds) {
    constexpr int THREADS = B::THREADS;
    const uint32_t tid = threadIdx.x, cnt = cA + cB;
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
    if (o0 >= cnt) return;
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
            if (out.want_keys()) out.put_key(b0 + o, key[j]);
            before = key[j];
        }
    }
}

__device__ inline uint2 ld_pair(const uint2* p) {
    const uint64_t w = ld_state(reinterpret_cast<const uint64_t*>(p));
    return make_uint2((uint32_t)w, (uint32_t)(w >> 32));
}

// Sorts a bucket of any size by one workgroup, bound by the latency of one chunk after
// another: each pass streams it through global memory in chunks of CAP, a histogram sweep,
// then the chunks in order, each ranked in LDS and scattered after the chunks before it.
// Passes alternate between the pairs and the second buffer's arrays (akeys, and the
// bucket's output values) and their number is odd, so that the last ends in the arrays.
// Reads of what this workgroup wrote in the previous pass bypass the CU's vector cache.
// Every thread calls it (barriers).
template <typename B>
__device__ inline void stream_bucket(uint2* src, uint32_t* akeys, uint32_t cnt, uint32_t b0, const BucketOut& out,
                                     BucketLds<B>& lds) {
    constexpr int THREADS = B::THREADS, BK_ITEMS = B::ITEMS;
    constexpr uint32_t CAP = B::CAP;
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid / 64;
    uint32_t* avals = out.vals + b0;
    uint32_t k[BK_ITEMS], v[BK_ITEMS], pos[BK_ITEMS];
    const uint32_t passes = digit_passes(out.lk.bits) | 1u;
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
    if (!out.want_keys()) return;
    __syncthreads();             // 32-bit keys take the place of the local ones
    for (uint32_t e = tid; e < cnt; e += THREADS) out.put_key(b0 + e, ld_state(&akeys[e]));
}

// Block-wide exclusive scan of one value a thread, and the total.  Every thread calls
// it (barriers).
template <typename B>
__device__ inline uint32_t block_scan(uint32_t x, uint32_t* wtot, uint32_t& total) {
    const uint32_t wave = threadIdx.x / 64, incl = wave_inclusive_scan(x);
    if (lane_id() == 63) wtot[wave] = incl;
    __syncthreads();
    uint32_t before = 0;
    total = 0;
#pragma unroll
    for (uint32_t w = 0; w < B::WAVES; ++w) {
        if (w < wave) before += wtot[w];
        total += wtot[w];
    }
    __syncthreads();
    return before + incl - x;
}

// Block-wide combination of N values a thread (value j by op(j, ..)), in place.  red: one of two sets of words
// that successive calls alternate between, so that one barrier is enough.
template <typename B, int N, typename Op>
__device__ inline void block_reduce(uint32_t (&x)[N], uint32_t (*red)[B::WAVES], Op op) {
    const uint32_t wave = threadIdx.x / 64;
#pragma unroll
    for (int j = 0; j < N; ++j) {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) x[j] = op(j, x[j], (uint32_t)__shfl_xor((int)x[j], off, 64));
        if (lane_id() == 0) red[j][wave] = x[j];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < N; ++j) {
        x[j] = red[j][0];
#pragma unroll
        for (int w = 1; w < B::WAVES; ++w) x[j] = op(j, x[j], red[j][w]);
    }
}

// A part's samples are every 2^SAMPLE_SKIP-th key at least: the count they give is off by
// a third of that and the square root of the runs (a few hundred), within the tolerance.
constexpr uint32_t SAMPLE_SKIP = 4;

// One sorted run of a divided bucket: its first entry, for each of the part's two cuts the
// places between which it lies, and those of a step's two pivots.  Then the part's
// share of the run.
struct PartRun {
    uint32_t start;
    uint16_t lo[2], hi[2], cut[2][2];
};
struct PartShare {
    uint32_t at, from;               // first place among the part's entries, first entry of the bucket
};

// Sorts part q of P of a bucket that consists of n_runs sorted runs, run r of counts[r *
// stride] entries: those from about the place size q / P of the sorted bucket to about
// size (q + 1) / P.  A cut is a key that divides the bucket within the tolerance of
// its place, or where equal keys leave none the exact place, and the same whichever
// of the two parts beside it looks for it.  The key at a
// place K is the least one that more than K entries do not exceed; of the entries
// with just that key, the first ones in run order lie before the cut.  The key is
// first narrowed down on the runs' samples (every 2^skip-th key, in LDS), by estimates
// of the count; then by two pivots a step, the first of them the key so found, each step
// a search for both in every run, a run per thread.  The searches' loads, each a cache
// line of its own, are what costs, so there are to be few of them: one such step
// is usually enough.  Every thread calls it (barriers).
template <typename B>
__device__ void sort_part(const uint2* __restrict__ src, uint32_t size, uint32_t q, uint32_t P,
                          const uint32_t* __restrict__ counts, uint32_t stride, uint32_t n_runs, uint32_t b0,
                          const BucketOut& out, BucketLds<B>& lds) {
    constexpr uint32_t THREADS = B::THREADS;
    const uint32_t tid = threadIdx.x;
    PartRun* runs = reinterpret_cast<PartRun*>(lds.pair);
    uint32_t* samples = reinterpret_cast<uint32_t*>(runs + n_runs);     // run r's from start >> skip on
    uint32_t skip = SAMPLE_SKIP;
    while (size >> skip > 2 * B::CAP - n_runs * (uint32_t)(sizeof(PartRun) / 4)) ++skip;
    auto sum = [](int, uint32_t x, uint32_t y) { return x + y; };
    uint32_t K[2] = {(uint32_t)((uint64_t)size * q / P), (uint32_t)((uint64_t)size * (q + 1) / P)};
    uint32_t first = 0, total;
    uint32_t ends[2] = {0xffffffffu, 0xffffffffu};      // least key, and the complement of the greatest
    for (uint32_t r0 = 0; r0 < n_runs; r0 += THREADS) {
        const uint32_t r = r0 + tid;
        const uint32_t len = r < n_runs ? min(counts[(uint64_t)r * stride] & ~SORT_READY, SPLIT_SIZE) : 0u;
        const uint32_t start = first + block_scan<B>(len, lds.wtot, total);
        first += total;
        if (r >= n_runs) continue;
        const uint16_t l = (uint16_t)len;
        runs[r] = PartRun{start, {0, 0}, {l, l}, {{0, 0}, {0, 0}}};
        if (len && start + len <= size) {
            ends[0] = min(ends[0], src[start].x);
            ends[1] = min(ends[1], ~src[start + len - 1].x);
        }
    }
    if (first != size || size == 0) {            // (uniform) only after a failed front end
        if (tid == 0) atomicOr(out.error, 4u);
        return;
    }
    block_reduce<B>(ends, lds.red[0], [](int, uint32_t x, uint32_t y) { return min(x, y); });
    // the samples, by as many threads a run as there are; from here on run r is thread r % THREADS's alone
    uint32_t per_run = 1;
    while (per_run < 64 && 2 * per_run * n_runs <= THREADS) per_run *= 2;
    for (uint32_t r = tid / per_run; r < n_runs; r += THREADS / per_run) {
        const uint32_t start = runs[r].start, n = (uint32_t)runs[r].hi[0] >> skip;
        const uint2* from = src + start + (1u << skip) - 1;
#pragma unroll 4
        for (uint32_t q = tid % per_run; q < n; q += per_run) samples[(start >> skip) + q] = from[q << skip].x;
    }
    __syncthreads();
    // the keys at both cuts lie in [a, b]: lo = entries below a, hi = entries up to b, ca and cb in all
    uint32_t a[2], b[2], ca[2], cb[2], guess[2];
    bool found[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        found[j] = K[j] == 0 || K[j] == size;
        a[j] = ends[0];
        b[j] = found[j] ? a[j] : ~ends[1];
        ca[j] = 0;
        cb[j] = size;
    }
    // where the key would be if the keys in [x, y], counts cx and cy, were evenly spread, in [x, y - 1]
    auto even = [](uint32_t x, uint32_t y, uint32_t cx, uint32_t cy, uint32_t k, float shift) {
        const uint32_t w = y - x;
        const float wide = fminf((float)w, 4294967040.0f);        // (a float that fits 32 bits)
        const float share = ((float)(k - cx) + 0.5f) / (float)(cy - cx) + shift;
        return x + min((uint32_t)(fminf(fmaxf(share, 0.0f), 1.0f) * wide), w - 1);
    };
    {
        // on the samples: a run's entries up to a key are those up to its last sample up to it, and
        // half a gap
        uint32_t x[2] = {a[0], a[1]}, y[2] = {b[0], b[1]}, cx[2] = {0, 0}, cy[2] = {size, size};
        auto open = [&](int j) { return x[j] < y[j] && cy[j] > cx[j]; };
        const uint32_t half = (1u << skip) / 2;
#pragma unroll
        for (int j = 0; j < 2; ++j) guess[j] = x[j];
        for (uint32_t step = 0; open(0) || open(1); ++step) {
            // the counts, the samples next below the key, and (complemented) next above it
            uint32_t got[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll
            for (int j = 0; j < 2; ++j)
                if (open(j)) guess[j] = step % 2 ? x[j] + (y[j] - x[j]) / 2 : even(x[j], y[j], cx[j], cy[j], K[j], 0.0f);
            for (uint32_t r = tid; r < n_runs; r += THREADS) {
                const uint32_t base = runs[r].start >> skip, n = (uint32_t)runs[r].hi[0] >> skip;
                uint32_t s0[2] = {0, 0}, s1[2] = {n, n};
                while (s0[0] < s1[0] || s0[1] < s1[1]) {
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const uint32_t m = (s0[j] + s1[j]) / 2;
                        if (s0[j] >= s1[j]) continue;
                        if (samples[base + m] <= guess[j]) s0[j] = m + 1;
                        else s1[j] = m;
                    }
                }
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    got[j] += min((s0[j] << skip) + half, (uint32_t)runs[r].hi[0]);
                    if (s0[j] > 0) got[2 + j] = max(got[2 + j], samples[base + s0[j] - 1]);
                    if (s0[j] < n) got[4 + j] = max(got[4 + j], ~samples[base + s0[j]]);
                }
            }
            block_reduce<B>(got, lds.red[step & 1],
                            [](int i, uint32_t p, uint32_t q) { return i < 2 ? p + q : max(p, q); });
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                if (!open(j)) continue;
                const uint32_t upto = got[j];
                if (max(upto, K[j]) - min(upto, K[j]) <= B::TOLERANCE / 4) {        // near enough
                    y[j] = x[j];
                } else if (upto > K[j]) {        // no sample between the next below and the key: neither is the cut
                    y[j] = max(x[j], min(guess[j], got[2 + j]));
                    cy[j] = max(upto, cx[j]);
                    guess[j] = y[j];
                } else {
                    x[j] = min(y[j], max(guess[j] + 1, ~got[4 + j]));
                    cx[j] = min(upto, cy[j]);
                    guess[j] = x[j];
                }
            }
        }
        __syncthreads();
    }
    auto open = [&](int j) { return !found[j] && a[j] < b[j]; };
    for (uint32_t step = 0; open(0) || open(1); ++step) {
        uint32_t pivot[2][2], upto[4] = {0, 0, 0, 0};
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const uint32_t w = b[j] - a[j];
            if (step == 0) {
                pivot[j][0] = pivot[j][1] = open(j) ? min(guess[j], b[j] - 1) : a[j];
            } else if (step % 3 == 0) {                  // (sure to narrow it down, whatever the keys)
                pivot[j][0] = a[j] + w / 3;
                pivot[j][1] = open(j) ? min(a[j] + w / 3 * 2, b[j] - 1) : a[j];
            } else {
                pivot[j][0] = open(j) ? even(a[j], b[j], ca[j], cb[j], K[j], -1.0f / 16.0f) : a[j];
                pivot[j][1] = open(j) ? even(a[j], b[j], ca[j], cb[j], K[j], 1.0f / 16.0f) : a[j];
            }
        }
        for (uint32_t r = tid; r < n_runs; r += THREADS) {
            PartRun run = runs[r];
            const uint32_t base = run.start >> skip;
            const uint2* from = src + run.start;
            uint32_t lo[4], hi[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int j = i / 2;
                lo[i] = run.lo[j];
                hi[i] = open(j) && (step > 0 || i % 2 == 0) ? run.hi[j] : lo[i];     // (the first step has one pivot)
                // the sampled places between them
                uint32_t s0 = lo[i] >> skip, s1 = hi[i] >> skip;
                while (s0 < s1) {
                    const uint32_t m = (s0 + s1) / 2;
                    if (samples[base + m] <= pivot[j][i % 2]) s0 = m + 1;
                    else s1 = m;
                }
                lo[i] = max(lo[i], s0 << skip);
                hi[i] = min(hi[i], ((s0 + 1) << skip) - 1);
            }
            // then the others, the four searches' loads together
            while (lo[0] < hi[0] || lo[1] < hi[1] || lo[2] < hi[2] || lo[3] < hi[3]) {
                uint32_t key[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) key[i] = lo[i] < hi[i] ? from[(lo[i] + hi[i]) / 2].x : 0u;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t m = (lo[i] + hi[i]) / 2;
                    if (lo[i] >= hi[i]) continue;
                    if (key[i] <= pivot[i / 2][i % 2]) lo[i] = m + 1;
                    else hi[i] = m;
                }
            }
            if (step == 0) {
                lo[1] = lo[0];
                lo[3] = lo[2];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                run.cut[i / 2][i % 2] = (uint16_t)lo[i];
                upto[i] += lo[i];
            }
            runs[r] = run;
        }
        block_reduce<B>(upto, lds.red[step & 1], sum);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if (!open(j)) continue;
            const uint32_t up0 = upto[2 * j], up1 = upto[2 * j + 1];
            const bool raise0 = up0 <= K[j], raise1 = up1 <= K[j];        // the key is above the pivot
            const uint32_t off0 = max(up0, K[j]) - min(up0, K[j]), off1 = max(up1, K[j]) - min(up1, K[j]);
            found[j] = min(off0, off1) <= B::TOLERANCE;
            const int at = off0 <= off1 ? 0 : 1;
            for (uint32_t r = tid; r < n_runs; r += THREADS) {
                if (found[j]) {
                    runs[r].lo[j] = runs[r].hi[j] = runs[r].cut[j][at];
                } else {
                    if (raise0) runs[r].lo[j] = runs[r].cut[j][raise1 ? 1 : 0];
                    if (!raise1) runs[r].hi[j] = runs[r].cut[j][raise0 ? 1 : 0];
                }
            }
            if (found[j]) {
                K[j] = ca[j] = at ? up1 : up0;
            } else {
                if (raise0) {
                    a[j] = pivot[j][raise1 ? 1 : 0] + 1;
                    ca[j] = raise1 ? up1 : up0;
                }
                if (!raise1) {
                    b[j] = pivot[j][raise0 ? 1 : 0];
                    cb[j] = raise0 ? up1 : up0;
                }
            }
        }
    }
    // the cuts: entries below the key, and (equal keys) the first ones of those that equal it
    const uint32_t K0 = K[0], K1 = K[1];
    if (K1 <= K0 || K1 - K0 > B::CAP) {             // (uniform) never, by the tolerance
        if (tid == 0) atomicOr(out.error, 4u);
        return;
    }
    uint32_t rest[2] = {K0 - ca[0], K1 - ca[1]};
    uint32_t at = 0, before[1] = {0};
    PartShare* shares = reinterpret_cast<PartShare*>(lds.pair);
    for (uint32_t r0 = 0; r0 < n_runs; r0 += THREADS) {
        const uint32_t r = r0 + tid;
        uint32_t cut[2] = {0, 0}, start = 0;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            // (K at an end of the bucket: lo = 0, hi = all, and rest is 0 or everything)
            const uint32_t lo = r < n_runs ? runs[r].lo[j] : 0u, equal = r < n_runs ? runs[r].hi[j] - lo : 0u;
            const uint32_t earlier = block_scan<B>(equal, lds.wtot, total);
            cut[j] = lo + (rest[j] > earlier ? min(rest[j] - earlier, equal) : 0u);
            rest[j] -= min(rest[j], total);
        }
        if (r < n_runs) start = runs[r].start;
        const uint32_t place = at + block_scan<B>(cut[1] - cut[0], lds.wtot, total);      // (the runs have been read)
        at += total;
        if (r < n_runs) {
            if (cut[0] > 0) before[0] = max(before[0], src[start + cut[0] - 1].x);
            shares[r] = PartShare{place, start + cut[0]};
        }
    }
    block_reduce<B>(before, lds.red[0], [](int, uint32_t x, uint32_t y) { return max(x, y); });
    // entry e of the part is in the last run whose share begins at or before it
    auto entry = [&](uint32_t a, uint32_t b) {
        const uint32_t e = a + b;
        uint32_t lo = 0, hi = n_runs - 1;
        while (lo < hi) {
            const uint32_t m = (lo + hi + 1) / 2;
            if (shares[m].at <= e) lo = m;
            else hi = m - 1;
        }
        return src[min(shares[lo].from + (e - shares[lo].at), size - 1)];
    };
    bucket_lds_sort<B>(entry, K1 - K0, out.lk.bits, lds);
    write_sorted<B>(lds, b0 + K0, K1 - K0, K0 == 0, K1 == size, before[0], out);
}

// This workgroup's share of a crowded frame's parts.  A function of its own, its arguments in
// LDS: with its registers in the kernel, which then spills, frames without parts take 10 to
// 30 us more (1M / 1080p, 3M / 4K).  The call makes the parts 10 to 40 us slower.
struct PartsArgs {
    uint2* pairs;
    const uint32_t* counts;
    SplitPlan plan;
    BucketOut out;
};
template <typename B>
__device__ __attribute__((noinline)) void bucket_parts(Lds<BucketLds<B>>* lds_) {
    BucketLds<B>& lds = *(BucketLds<B>*)lds_;
    union Words {
        PartsArgs args;
        int word[sizeof(PartsArgs) / 4];
        __device__ Words() {}
    } a;
#pragma unroll
    for (uint32_t i = 0; i < sizeof(a.word) / 4; ++i)
        a.word[i] = __builtin_amdgcn_readfirstlane(reinterpret_cast<const int*>(lds.pair)[i]);
    __syncthreads();
    const SplitPlan& plan = a.args.plan;
    BucketOut out = a.args.out;
    const uint32_t* __restrict__ bases = plan.bases;
    const uint32_t n_parts = *plan.n_parts, buckets = gridDim.x;
    const uint32_t n_runs = (bases[buckets] + SPLIT_SIZE - 1) / SPLIT_SIZE;
    for (uint32_t p = blockIdx.x; p < n_parts; p += buckets) {
        uint32_t lo = 0, hi = buckets - 1;           // the bucket: the first that parts up to it exceed p
        while (lo < hi) {
            const uint32_t m = (lo + hi) / 2;
            if (plan.parts[m] > p) hi = m;
            else lo = m + 1;
        }
        const uint32_t first = bases[lo], before = lo ? plan.parts[lo - 1] : 0u;
        out.bucket = lo;
        __syncthreads();             // the LDS of what this workgroup did before
        sort_part<B>(a.args.pairs + first, bases[lo + 1] - first, p - before, plan.parts[lo] - before,
                     a.args.counts + lo, buckets, n_runs, first, out, lds);
    }
}

// pairs: the split pass's output; tmp_keys: a second buffer for streamed buckets (with the
// values' place).  plan.limit is LIMIT and plan.alone CAP, or both 0 to divide every bucket
// (for tests).  counts: the split pass's tiles' digit counts.
template <typename B>
__global__ __launch_bounds__(B::THREADS, B::WAVES_SIMD) void k_bucket_sort(uint2* pairs, uint32_t* tmp_keys,
                                                                        SplitPlan plan, const uint32_t* counts,
                                                                        BucketOut out) {
    constexpr int THREADS = B::THREADS;
    constexpr uint32_t CAP = B::CAP;
    __shared__ __align__(16) BucketLds<B> lds;
    const uint32_t tid = threadIdx.x;
    const uint32_t* __restrict__ bases = plan.bases;
    const uint32_t n_parts = *plan.n_parts;
    const uint32_t b0 = bases[blockIdx.x];
    const uint32_t b1 = bases[blockIdx.x + 1];
    if (out.order) place_tiles<THREADS>(bases, out, lds.wtot);
    const uint32_t cnt = b1 > b0 ? b1 - b0 : 0u, bits = out.lk.bits;
    uint2* src = pairs + b0;
    out.bucket = blockIdx.x;
    if (cnt > 0 && cnt <= (n_parts ? plan.alone : 2 * CAP)) {
        // ---- the bucket in LDS, or in two runs: each half sorted in LDS and
        // written back in place, then the two merged ----
        const uint32_t runs = cnt <= CAP ? 1u : 2u;
        const uint32_t cA = runs == 1 ? cnt : (cnt + 1) / 2, cB = cnt - cA;
        for (uint32_t h = 0; h < runs; ++h) {
            const uint32_t o = h ? cA : 0u, m = h ? cB : cA;
            const uint2* from = src + o;
            bucket_lds_sort<B>([&](uint32_t a, uint32_t b) { return (from + a)[b]; }, m, bits, lds);
            if (runs == 1) {
                write_sorted<B>(lds, b0, cnt, true, true, 0u, out);
            } else {
                for (uint32_t e = tid; e < m; e += THREADS) src[o + e] = lds.pair[e];
                __syncthreads();     // the first run's LDS before the second's loads
            }
        }
        if (__builtin_expect(runs == 2, false)) merge_runs<B>(src, cA, cB, b0, out, lds);
    } else if (__builtin_expect(cnt > 0 && n_parts == 0, false)) {
        stream_bucket<B>(src, tmp_keys + b0, cnt, b0, out, lds);
    }
    if (__builtin_expect(n_parts == 0, true)) return;
    static_assert(sizeof(PartsArgs) <= sizeof(lds.pair), "the arguments fit");
    __syncthreads();                 // the LDS of the bucket before the arguments
    if (tid == 0) {                  // (field by field: a temporary would live in LDS, a copy per thread)
        PartsArgs* a = reinterpret_cast<PartsArgs*>(lds.pair);
        a->pairs = pairs;
        a->counts = counts;
        a->plan.bases = plan.bases;
        a->plan.n_parts = plan.n_parts;
        a->plan.parts = plan.parts;
        a->plan.limit = plan.limit;
        a->plan.alone = plan.alone;
        a->plan.part = plan.part;
        a->out.vals = out.vals;
        a->out.ranges = out.ranges;
        a->out.keys32 = out.keys32;
        a->out.keys64 = out.keys64;
        a->out.order = out.order;
        a->out.error = out.error;
        a->out.prm = out.prm;
        a->out.lk.bits = out.lk.bits;
        a->out.lk.tile_bits = out.lk.tile_bits;
        a->out.n_tiles = out.n_tiles;
        a->out.bucket = out.bucket;
    }
    __syncthreads();
    bucket_parts<B>((Lds<BucketLds<B>>*)&lds);
}

template <typename KeyT, int BITS>
static void launch_split_pass(hipStream_t s, const FrameDev& f, const WsDev& ws, uint2* pairs, const SplitPlan& plan,
                              bool force) {
    using S = SplitShape<BITS>;
    const PairsOut<KeyT> out{pairs, f.lk, ws.params};
    uint32_t* tiles = ws.sort_state;
    uint32_t* groups = ws.sort_state + (uint64_t)ws.sort_rows * S::DIGITS;
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(ws.sort_rows), dim3(S::THREADS), 0, s,
                           reinterpret_cast<const KeyT*>(ws.keys_a), ws.vals_a, out, ws.header, ws.hist,
                           (uint32_t)(MAX_PASSES * RADIX), tiles, groups, (uint32_t*)nullptr, (uint32_t*)nullptr,
                           f.split_shift, plan);
    };
    if (force) launch(k_radix_pass<KeyT, S, PairsOut<KeyT>, true>);
    else launch(k_radix_pass<KeyT, S, PairsOut<KeyT>, false>);
}

// The two kernels with bucket workgroups B, for buckets of up to ROOM entries on average.
template <typename B, uint32_t ROOM>
static void launch_split(hipStream_t s, const FrameDev& f, const WsDev& ws, uint32_t key_bytes, uint2* pairs,
                         const BucketOut& out, bool force) {
    // the digit counts' copies are as wide as two split digits: the parts table takes
    // the unused half of the first
    static_assert(2 * SPLIT_DIGITS_MAX <= MAX_PASSES * RADIX, "the parts table fits");
    // the frame's radix tiles, the runs of a divided bucket, fit the entries' LDS
    static_assert(((uint64_t)(ROOM + 1) << SPLIT_WIDE_BT) / SPLIT_SIZE * sizeof(PartRun) < B::CAP * sizeof(uint2),
                  "the runs, and samples of them, fit");
    const SplitPlan plan{ws.bases, ws.bases + SPLIT_DIGITS_MAX + 1, ws.hist + SPLIT_DIGITS_MAX, force ? 0u : B::LIMIT,
                         force ? 0u : B::CAP, B::PART};
    if (key_bytes == 8) {
        if (f.split_bits == 10) launch_split_pass<uint64_t, 10>(s, f, ws, pairs, plan, force);
        else launch_split_pass<uint64_t, 8>(s, f, ws, pairs, plan, force);
    } else {
        if (f.split_bits == 10) launch_split_pass<uint32_t, 10>(s, f, ws, pairs, plan, force);
        else launch_split_pass<uint32_t, 8>(s, f, ws, pairs, plan, force);
    }
    hipLaunchKernelGGL(k_bucket_sort<B>, dim3(1u << f.split_bits), dim3(B::THREADS), 0, s, pairs,
                       key_bytes == 8 ? ws.vals_b : reinterpret_cast<uint32_t*>(ws.keys_a), plan, ws.sort_state, out);
}

void launch_sort_split(hipStream_t s, const FrameDev& f, const WsDev& ws, uint32_t key_bytes, bool force,
                       bool want_keys) {
    // pairs in the second key and value arrays (32-bit keys: the two are
    // adjacent); sorted values in the first value array, where wanted sorted keys
    // in the first key array
    uint2* pairs = reinterpret_cast<uint2*>(ws.keys_b);
    BucketOut out{};
    out.vals = ws.vals_a;
    out.ranges = ws.ranges;
    out.keys32 = want_keys && key_bytes == 4 ? reinterpret_cast<uint32_t*>(ws.keys_a) : nullptr;
    out.keys64 = want_keys && key_bytes == 8 ? reinterpret_cast<uint64_t*>(ws.keys_a) : nullptr;
    out.order = f.ordered == ORDER_BUCKETS ? ws.order : nullptr;
    out.error = &ws.header->error;
    out.prm = ws.params;
    out.lk = f.lk;
    out.n_tiles = (uint32_t)f.n_tiles;
    // The workgroup by the entries a bucket may hold on average (what the
    // workspace holds, usually 1.25 to 2 times the frame's): the busiest bucket
    // has about twice the frame's average, and should still be one run in LDS,
    // while smaller workgroups start together and share a CU better.  Kernel
    // times in us with 512 x 9, 512 x 16 and 1024 x 16 entries:
    // 1280x720 28, 35, 56; 1080p (1M) 33, 42, 68 (plain 65, 63, 94); 4K (3M) 94, 73, 104.
    // Sort with 512 x 16 and 1024 x 16: plain 4K (4M), room 14000, 299, 285 (LSD passes 569).
    const uint32_t room = f.capacity >> f.split_bits;
    if (room <= 4608) launch_split<BucketShape<512, 9, 6, 3>, 4608>(s, f, ws, key_bytes, pairs, out, force);
    else if (room <= 12288) launch_split<BucketShape<512, 16, 4, 4>, 12288>(s, f, ws, key_bytes, pairs, out, force);
    else launch_split<BucketShape<1024, 16, 4, 4>, SPLIT_MAX_ROOM>(s, f, ws, key_bytes, pairs, out, force);
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
