// esc_join.hip -- gfx950 hash join over the outputs of exact selectivity
// computation: build hash tables on (filtered) build relations, then count
// the rows of the star join of the probe relation with them in one pass.
//
// Section 2.2 joins a probe relation (the largest) with build relations,
// hash tables being built on the build side, and pushes selections down
// only there; the build inputs are then the temporary tables of Section 2.1.
//
// A table is a header and an area of 8 bytes for each of S slots (S a power
// of two, at least two per key), which the build lays out in one of three
// forms by the keys themselves (the device decides, nothing waits):
//   bitmap  keys within 32 S of each other: one bit per value, in the lower
//           half of the area (surrogate keys of a filtered dimension: a
//           lookup is one 4-byte read of a structure 32 times smaller than
//           the keys' range).  A key seen before goes to a hash of
//           (key, further rows) in the upper half;
//   counts  more keys than values in their range: one row count per value;
//   hash    all others: buckets of four keys (one 16-byte read) with linear
//           probing over buckets in the lower half.  A key of several rows
//           has a second copy further along, so that a lookup reads the number
//           of its further rows (upper half, one word per key slot) only when
//           it has any.
// Lookups are bound by the rate of random reads (one line of the L1's tag
// look-up per lane and read), so each is one read, eight rows per lane are
// looked up at a time, and the probe's waves fill the chip.  With one slot
// read at a time along a chain that went on to the first empty slot, as
// before, the wave waited for its longest chain: 200M rows against 100K and
// 3M surrogate keys took 2.01 ms, 20M rows against 50K and 2M keys spread
// over the 32-bit integers 0.81 ms.
#include <hip/hip_runtime.h>
#include <limits.h>
#include <stdint.h>

#include <algorithm>

#include "esc_device.h"
#include "esc_runtime.h"

namespace esc {

constexpr int kJoinMaxTables = 4;
// rows per lane of a probe tile: four for three or four sides, whose rows and
// products would not fit 128 registers
constexpr int probe_rpt(int ntables) { return ntables <= 2 ? 8 : 4; }
constexpr uint32_t kNoKey = 0x80000000u;   // an empty key slot of the hash form (that key is counted in the header)

enum TableMode : uint32_t { TAB_NONE = 0, TAB_BITMAP = 1, TAB_COUNTS = 2, TAB_HASH = 3 };

constexpr int kMinMaxParts = 24;           // partial minima and maxima the header holds
constexpr int kMinMaxBlock = 1024;
constexpr int64_t kMinMaxNone = 1 << 14;   // keys up to which every fill block finds the range itself
constexpr int64_t kMinMaxFew = 1 << 20;    // keys up to which kMinMaxParts blocks find it

// the first 256 bytes of a table
struct TableHeader {
    uint32_t mode;       // written by the fill kernel
    int32_t kmin;        // smallest key
    uint32_t span;       // largest key - smallest key
    uint32_t dup;        // some key has several rows
    uint32_t nokey;      // rows whose key is kNoKey (hash form)
    uint32_t rows;       // build rows
    uint32_t parts;      // ranges of 2^kPartBits values that build_parts_kernel takes, 0: build_kernel inserts the keys
    uint32_t pad[9];
    int32_t part[kMinMaxParts][2];
};
static_assert(sizeof(TableHeader) == 256, "the slots follow at byte 256");

struct HashRef {
    const TableHeader *head[kJoinMaxTables];
    uint32_t slots[kJoinMaxTables];
};

// Fibonacci hashing: the top bits of key * 2^32 / golden ratio
__device__ __forceinline__ uint32_t hash_of(uint32_t key) { return key * 0x9E3779B1u; }

// 16 bytes of a table, which may begin at any multiple of 8
typedef uint32_t slot4 __attribute__((ext_vector_type(4), aligned(8)));

__device__ __forceinline__ uint32_t *area(const TableHeader *h) { return (uint32_t *)((char *)h + sizeof(TableHeader)); }

// ------------------------------------------------------------------ build

__global__ void begin_build_kernel(TableHeader *h)
{
    const int t = threadIdx.x;
    if (t < 2 * kMinMaxParts) (&h->part[0][0])[t] = (t & 1) ? INT_MIN : INT_MAX;
}

// Smallest and largest of the keys that the calling threads (number t of
// nthreads) read, over the block, in thread 0 (s: one pair per wave).
template <int NT>
__device__ __forceinline__ void block_range(const int32_t *__restrict__ keys, int64_t n, int64_t t, int64_t nthreads,
                                            int32_t (*s)[2], int32_t &lo, int32_t &hi)
{
    lo = INT_MAX;
    hi = INT_MIN;
    const int64_t n4 = ((uintptr_t)keys & 15) ? 0 : n / 4;   // whole 16-byte groups, if the keys are aligned for them
    for (int64_t i = t; i < n4; i += nthreads) {
        const u32x4 q = ((const u32x4 *)keys)[i];
#pragma unroll
        for (int e = 0; e < 4; e++) {
            lo = min(lo, (int32_t)q[e]);
            hi = max(hi, (int32_t)q[e]);
        }
    }
    for (int64_t i = 4 * n4 + t; i < n; i += nthreads) {
        lo = min(lo, keys[i]);
        hi = max(hi, keys[i]);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        lo = min(lo, __shfl_xor(lo, o, 64));
        hi = max(hi, __shfl_xor(hi, o, 64));
    }
    if (lane_id() == 0) {
        s[wave_id()][0] = lo;
        s[wave_id()][1] = hi;
    }
    __syncthreads();
    for (int w = 0; w < NT / kWave; w++) {
        lo = min(lo, s[w][0]);
        hi = max(hi, s[w][1]);
    }
}

// `few`: block b stores the range of its keys in part[b] (at most kMinMaxParts
// blocks), else every block adds its own to part[b % kMinMaxParts], which
// begin_build_kernel set.
__global__ __launch_bounds__(kMinMaxBlock) void minmax_kernel(const int32_t *__restrict__ keys, int64_t n,
                                                              TableHeader *h, int few)
{
    __shared__ int32_t s_range[kMinMaxBlock / kWave][2];
    int32_t lo, hi;
    block_range<kMinMaxBlock>(keys, n, blockIdx.x * (int64_t)kMinMaxBlock + threadIdx.x,
                              gridDim.x * (int64_t)kMinMaxBlock, s_range, lo, hi);
    if (threadIdx.x == 0) {
        if (few) {
            h->part[blockIdx.x][0] = lo;
            h->part[blockIdx.x][1] = hi;
        } else {
            atomicMin(&h->part[blockIdx.x % kMinMaxParts][0], lo);
            atomicMax(&h->part[blockIdx.x % kMinMaxParts][1], hi);
        }
    }
}

__device__ __forceinline__ void fill_words(uint32_t *p, int64_t n4, uint32_t v)
{
    const slot4 q = {v, v, v, v};
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n4; i += (int64_t)gridDim.x * blockDim.x)
        ((slot4 *)p)[i] = q;
}

// Bitmaps of many keys are built in LDS, 2^20 bits by block: a random atomic
// on memory costs as much as one on a whole 64-byte line (26 * 10^9 lines a
// second measured), so the blocks of a part of the range scan slices of the
// keys and then OR their 128 KiB into memory line by line.  3M keys of a range
// of 24 parts: a build of 97 us, against 141 by one atomic per key.  The
// estimate: n / 25000 us for the atomics, against 30 us to write and 150 us for
// each million keys of a slice.  Both ways in us, by parts and slices a part:
// 10M keys 40 (6) 301 and 424, 64 (4) 383 and 423, 96 (2) 640 and 427; 50M 48
// (5) 1,780 and 1,994, 64 (4) 2,068 and 2,012, 96 (2) 3,702 and 2,013; 2M 32 (8)
// 86 and 102, 64 (4) 112 and 102.
constexpr int kPartBits = 20;
constexpr int kPartBytes = 1 << (kPartBits - 3);
constexpr int kPartBlock = 1024;
constexpr int64_t kPartKeys = 1 << 20;   // keys from which this kernel is launched at all

// Parts of a table built so by `blocks` blocks, 0 if it is not: asked once, by
// the kernel that writes the header, so that exactly one of the two build
// kernels inserts the keys.
__device__ __forceinline__ uint32_t build_parts(uint32_t mode, uint32_t span, int64_t n, int blocks)
{
    const uint32_t parts = (span >> kPartBits) + 1u, keys = (uint32_t)n;   // at most 2^30
    if (n < kPartKeys || mode != TAB_BITMAP || parts > (uint32_t)blocks) return 0u;
    const bool pays =
        (float)keys * (1.0f / 25000.0f) > 30.0f + (float)(keys / ((uint32_t)blocks / parts)) * 150e-6f;
    return pays ? parts : 0u;
}

// Chooses the form from the keys' range (every block alike), clears what that
// form uses, and writes the header.  nparts: minima and maxima in the header,
// 0 for a range that every block finds itself (kMinMaxNone keys at most);
// part_blocks: blocks of build_parts_kernel.
constexpr int kFillBlock = 256;

__global__ __launch_bounds__(kFillBlock) void fill_table_kernel(const int32_t *__restrict__ keys, TableHeader *h,
                                                                int64_t n, int64_t slots, int nparts, int part_blocks)
{
    int32_t lo = INT_MAX, hi = INT_MIN;
    if (nparts == 0) {
        __shared__ int32_t s_range[kFillBlock / kWave][2];
        block_range<kFillBlock>(keys, n, threadIdx.x, kFillBlock, s_range, lo, hi);
    }
    for (int i = 0; i < nparts; i++) {
        lo = min(lo, h->part[i][0]);
        hi = max(hi, h->part[i][1]);
    }
    const uint32_t span = (uint32_t)hi - (uint32_t)lo;
    uint32_t mode = TAB_HASH;
    if (n == 0) mode = TAB_NONE;
    else if ((int64_t)span + 1 < n) mode = TAB_COUNTS;         // span + 1 < n <= slots / 2: four bytes each fit
    else if ((int64_t)span + 1 <= 32 * slots) mode = TAB_BITMAP;
    uint32_t *a = area(h);
    if (mode == TAB_COUNTS) {
        fill_words(a, ((int64_t)span + 4) / 4, 0u);
    } else if (mode == TAB_BITMAP) {
        fill_words(a, ((int64_t)span + 128) / 128, 0u);
        fill_words(a + slots, slots / 4, 0u);
    } else if (mode == TAB_HASH) {
        fill_words(a, slots / 4, kNoKey);
        fill_words(a + slots, slots / 4, 0u);
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        h->mode = mode;
        h->kmin = lo;
        h->span = span;
        h->dup = mode == TAB_COUNTS;
        h->nokey = 0u;
        h->rows = (uint32_t)n;
        h->parts = build_parts(mode, span, n, part_blocks);
    }
}

// a further row of a key of the bitmap form: (key, rows) in the upper half,
// slots / 2 words of 8 bytes
__device__ __forceinline__ void add_further_row(uint32_t *a, uint32_t slots, int shift, uint32_t key)
{
    unsigned long long *more = (unsigned long long *)(a + slots);
    uint32_t s = hash_of(key) >> (shift + 1);
    for (uint32_t step = 0; step < slots / 2; step++) {
        const unsigned long long old = atomicCAS(&more[s], 0ull, (1ull << 32) | key);
        if (old == 0ull) return;
        if ((uint32_t)old == key) {
            atomicAdd(&more[s], 1ull << 32);
            return;
        }
        s = (s + 1u) & (slots / 2 - 1u);
    }
}

__global__ __launch_bounds__(kPartBlock) void build_parts_kernel(const int32_t *__restrict__ keys, int64_t n,
                                                                 TableHeader *h, uint32_t slots, int shift)
{
    extern __shared__ uint32_t s_part[];
    const int32_t kmin = h->kmin;
    const uint32_t span = h->span;
    const int parts = (int)h->parts;
    if (parts == 0) return;
    const int slices = (int)gridDim.x / parts;
    const uint32_t part = blockIdx.x % (unsigned)parts;
    const int slice = (int)(blockIdx.x / (unsigned)parts);
    if (slice >= slices) return;
    constexpr uint32_t WORDS = kPartBytes / 4;
    for (uint32_t i = threadIdx.x; i < WORDS; i += kPartBlock) s_part[i] = 0u;
    __syncthreads();
    uint32_t *a = area(h);
    bool dup = false;
    auto add = [&](uint32_t key) {
        const uint32_t d = key - (uint32_t)kmin;
        if (d >> kPartBits != part) return;
        const uint32_t f = d & ((1u << kPartBits) - 1u), bit = 1u << (f & 31u);
        if (atomicOr(&s_part[f >> 5], bit) & bit) {
            dup = true;
            add_further_row(a, slots, shift, key);
        }
    };
    // this slice's keys: whole 16-byte groups where the keys are aligned for them
    const int64_t per = ((n + slices - 1) / slices + 3) / 4 * 4;
    const int64_t k0 = min(n, slice * per), k1 = min(n, k0 + per);
    const int64_t k4 = ((uintptr_t)keys & 15) ? k0 : k0 + (k1 - k0) / 4 * 4;
    for (int64_t i = k0 + 4 * (int64_t)threadIdx.x; i < k4; i += 4 * kPartBlock) {
        const u32x4 q = *(const u32x4 *)(keys + i);
#pragma unroll
        for (int e = 0; e < 4; e++) add(q[e]);
    }
    for (int64_t i = k4 + threadIdx.x; i < k1; i += kPartBlock) add((uint32_t)keys[i]);
    __syncthreads();
    const uint32_t w0 = part * WORDS, nw = min(WORDS, span / 32 + 1 - w0);
    for (uint32_t i = threadIdx.x; i < nw; i += kPartBlock) {
        const uint32_t w = s_part[i];
        if (!__any(w != 0u)) continue;
        // bits that another slice has set too: further rows
        uint32_t both = atomicOr(&a[w0 + i], w) & w;
        if (both) dup = true;
        for (; both; both &= both - 1u)
            add_further_row(a, slots, shift, (uint32_t)kmin + (w0 + i) * 32u + (uint32_t)__builtin_ctz(both));
    }
    if (__any(dup) && lane_id() == 0) h->dup = 1u;   // every writer stores the same value
}

// One thread per build row (grid-stride).  Keys never leave a slot once they
// are in it, so every search ends: at least half of the key slots stay empty (a key
// takes one slot, or two for its two or more rows).
__global__ __launch_bounds__(256) void build_kernel(const int32_t *__restrict__ keys, int64_t n, TableHeader *h,
                                                    uint32_t slots, int shift)
{
    uint32_t *a = area(h);
    const uint32_t mode = h->mode;
    const int32_t kmin = h->kmin;
    if (h->parts != 0u) return;
    bool dup = false;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t key = (uint32_t)keys[i];
        const uint32_t d = key - (uint32_t)kmin;
        if (mode == TAB_COUNTS) {
            atomicAdd(&a[d], 1u);
        } else if (mode == TAB_BITMAP) {
            const uint32_t bit = 1u << (d & 31u);
            if (!(atomicOr(&a[d >> 5], bit) & bit)) continue;
            dup = true;
            add_further_row(a, slots, shift, key);
        } else if (key == kNoKey) {
            dup |= atomicAdd(&h->nokey, 1u) != 0u;
        } else {
            uint32_t b = hash_of(key) >> (shift + 2);   // slots / 4 buckets
            bool done = false, second = false;   // second: looking for the second copy's slot
            for (uint32_t step = 0; !done && step < slots / 4; step++) {
                // a slot read as empty may have been taken since: the
                // exchange below says by whom
                const slot4 q = *(const slot4 *)(a + 4 * (int64_t)b);
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    if (done) continue;
                    uint32_t old = q[e];
                    if (old == kNoKey) old = atomicCAS(&a[4 * (int64_t)b + e], kNoKey, key);
                    if (old == kNoKey) {
                        done = true;
                    } else if (old == key && !second) {
                        // the first copy (slots fill in order, so every row
                        // of a key meets it first); whoever adds the first
                        // further row inserts the second copy
                        dup = true;
                        if (atomicAdd(&a[(int64_t)slots + 4 * (int64_t)b + e], 1u) == 0u) second = true;
                        else done = true;
                    }
                }
                b = (b + 1u) & (slots / 4 - 1u);
            }
        }
    }
    if (__any(dup) && lane_id() == 0) h->dup = 1u;   // every writer stores the same value
}

// ------------------------------------------------------------------ probe

// a table as the probe reads it
struct Side {
    const uint32_t *a;
    uint32_t mode, span, slots, nokey, rows;
    int32_t kmin;
    int shift;
    bool dup;
};

__device__ __forceinline__ Side side_of(const TableHeader *h, uint32_t slots)
{
    Side t;
    t.a = area(h);
    t.mode = h->mode;
    t.span = h->span;
    t.kmin = h->kmin;
    t.nokey = h->nokey;
    t.rows = h->rows;
    t.dup = h->dup != 0u;
    t.slots = slots;
    t.shift = __builtin_clz(slots) + 1;   // 32 - log2(slots), slots >= 64
    // a table that no build wrote matches nothing, and no read leaves it
    if (t.mode > TAB_HASH || (t.mode == TAB_BITMAP && t.span >= 32ull * slots) ||
        (t.mode == TAB_COUNTS && t.span >= 2ull * slots))
        t.mode = TAB_NONE;
    return t;
}

// further rows of a key that the bitmap form holds
__device__ __forceinline__ uint32_t further_rows(const Side &t, uint32_t key)
{
    const unsigned long long *more = (const unsigned long long *)(t.a + t.slots);
    uint32_t s = hash_of(key) >> (t.shift + 1);
    for (uint32_t step = 0; step < t.slots / 2; step++) {
        const unsigned long long v = more[s];
        if (v == 0ull) return 0u;
        if ((uint32_t)v == key) return (uint32_t)(v >> 32);
        s = (s + 1u) & (t.slots / 2 - 1u);
    }
    return 0u;
}

// The build rows of N probe keys, for the rows of `live` (bit r): cnt[r] rows
// (DUP), else the mask of the rows with a match.  Rows that are not live read
// the table's first words and are masked.
template <int N, bool DUP>
__device__ __forceinline__ uint32_t lookup(const Side &t, const uint32_t *key, uint32_t live, uint32_t (&cnt)[N])
{
    uint32_t hit = 0u;
    if (t.mode == TAB_BITMAP || t.mode == TAB_COUNTS) {
        const int down = t.mode == TAB_BITMAP ? 5 : 0;
        uint32_t w[N];
#pragma unroll
        for (int r = 0; r < N; r++) {
            const uint32_t d = key[r] - (uint32_t)t.kmin;
            if (d > t.span) live &= ~(1u << r);
            w[r] = t.a[((live >> r) & 1u) ? d >> down : 0u];
        }
        if (t.mode == TAB_BITMAP) {
#pragma unroll
            for (int r = 0; r < N; r++) {
                const uint32_t d = key[r] - (uint32_t)t.kmin;
                hit |= ((w[r] >> (d & 31u)) & 1u) << r;
            }
            hit &= live;
            if constexpr (DUP) {
#pragma unroll
                for (int r = 0; r < N; r++) {
                    cnt[r] = (hit >> r) & 1u;
                    if (t.dup && cnt[r]) cnt[r] += further_rows(t, key[r]);
                }
            }
        } else {
#pragma unroll
            for (int r = 0; r < N; r++) {
                cnt[r] = ((live >> r) & 1u) ? w[r] : 0u;
                hit |= (cnt[r] != 0u ? 1u : 0u) << r;
            }
        }
        return hit;
    }
    if constexpr (DUP) {
#pragma unroll
        for (int r = 0; r < N; r++) cnt[r] = 0u;
    }
    if (t.mode != TAB_HASH) return 0u;
    // all rows' buckets are in flight at once; the rare rows whose bucket is
    // full go on to the next one together
    const uint32_t nb = t.slots / 4;
    u32x4 q[N];
    uint32_t b[N], open = live;   // rows still looking
#pragma unroll
    for (int r = 0; r < N; r++) {
        b[r] = ((live >> r) & 1u) ? hash_of(key[r]) >> (t.shift + 2) : 0u;
        q[r] = *(const slot4 *)(t.a + 4 * (int64_t)b[r]);
        if (key[r] == kNoKey && ((live >> r) & 1u)) {
            open &= ~(1u << r);
            hit |= (t.nokey != 0u ? 1u : 0u) << r;
            if constexpr (DUP) cnt[r] = t.nokey;
        }
    }
    for (uint32_t step = 0; step < nb; step++) {
#pragma unroll
        for (int r = 0; r < N; r++) {
            if (!((open >> r) & 1u)) continue;
            const uint32_t k = key[r];
            const uint32_t m = (q[r].x == k ? 1u : 0u) | (q[r].y == k ? 2u : 0u) | (q[r].z == k ? 4u : 0u) |
                               (q[r].w == k ? 8u : 0u);
            const bool gap = q[r].w == kNoKey;   // a bucket fills in order
            if constexpr (DUP) {
                if (m && !((hit >> r) & 1u)) {
                    hit |= 1u << r;
                    cnt[r] = 1u;
                    if (t.dup) {
                        // a second copy, here or (in a full bucket) further on?
                        const uint32_t at = 4u * b[r] + (uint32_t)__builtin_ctz(m);
                        if (m & (m - 1u)) {
                            cnt[r] += t.a[(int64_t)t.slots + at];
                        } else if (!gap) {
                            cnt[r] = 1u + t.a[(int64_t)t.slots + at];
                        }
                    }
                    open &= ~(1u << r);
                }
            } else if (m) {
                hit |= 1u << r;
                open &= ~(1u << r);
            }
            if (gap) open &= ~(1u << r);
        }
        if (open == 0u) break;
#pragma unroll
        for (int r = 0; r < N; r++) {
            if (!((open >> r) & 1u)) continue;
            b[r] = (b[r] + 1u) & (nb - 1u);
            q[r] = *(const slot4 *)(t.a + 4 * (int64_t)b[r]);
        }
    }
    return hit;
}

// A filter of the first side's keys in LDS, for probes of many rows: one bit
// per value of its range modulo 2^20 (bitmap form; exact when the range is no
// larger), or per 20-bit hash (hash form).  A global lookup moves a 128-byte
// line into the L1 for four bytes (2.8 cycles of a CU per lane measured), an
// LDS read takes a tenth of that, and the rows that it drops read nothing
// more, here or on the sides that follow.
constexpr int kFilterBits = 20;
constexpr int kFilterBytes = 1 << (kFilterBits - 3);
enum FilterKind { FILTER_NONE, FILTER_FOLDED, FILTER_EXACT, FILTER_HASH };

// Whether a filter pays: reading the bitmap (16 words a cycle) or the key
// slots (a bit set costs about half a cycle) into LDS has to be small beside
// the block's rows, and a folded or hashed filter has to leave most bits clear.
__device__ __forceinline__ FilterKind filter_kind(const Side &t, int64_t rows_per_block)
{
    if (t.mode == TAB_BITMAP) {
        if ((int64_t)(t.span >> 9) + 4096 > rows_per_block) return FILTER_NONE;
        if (t.span >> kFilterBits == 0u) return FILTER_EXACT;
        return t.rows < (1u << (kFilterBits - 1)) && t.rows < t.span / 2 ? FILTER_FOLDED : FILTER_NONE;
    }
    if (t.mode == TAB_HASH)
        return t.rows < (1u << (kFilterBits - 2)) && 4ll * t.slots + 4096 <= rows_per_block ? FILTER_HASH : FILTER_NONE;
    return FILTER_NONE;
}

template <int NT>
__device__ __forceinline__ void load_filter(const Side &t, FilterKind kind, uint32_t *s_bits)
{
    constexpr uint32_t WORDS = kFilterBytes / 4;
    if (kind == FILTER_HASH) {
        for (uint32_t i = threadIdx.x; i < WORDS; i += NT) s_bits[i] = 0u;
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < t.slots; i += NT) {
            const uint32_t k = t.a[i];
            const uint32_t f = hash_of(k) >> (32 - kFilterBits);
            if (k != kNoKey) atomicOr(&s_bits[f >> 5], 1u << (f & 31u));
        }
        if (threadIdx.x == 0 && t.nokey != 0u) {
            const uint32_t f = hash_of(kNoKey) >> (32 - kFilterBits);
            atomicOr(&s_bits[f >> 5], 1u << (f & 31u));
        }
    } else {
        const uint32_t nw = t.span / 32 + 1;
        for (uint32_t i = threadIdx.x; i < WORDS; i += NT) {
            uint32_t w = 0u;
            for (uint32_t j = i; j < nw; j += WORDS) w |= t.a[j];
            s_bits[i] = w;
        }
    }
    __syncthreads();
}

// the rows of `live` that the filter lets through
template <int N>
__device__ __forceinline__ uint32_t filtered(const Side &t, FilterKind kind, const uint32_t *s_bits,
                                             const uint32_t *key, uint32_t live)
{
    uint32_t pass = 0u;
#pragma unroll
    for (int r = 0; r < N; r++) {
        const uint32_t d = key[r] - (uint32_t)t.kmin;
        const uint32_t f = kind == FILTER_HASH ? hash_of(key[r]) >> (32 - kFilterBits) : d & ((1u << kFilterBits) - 1u);
        const uint32_t bit = (s_bits[f >> 5] >> (f & 31u)) & 1u;
        pass |= (kind != FILTER_HASH && d > t.span ? 0u : bit) << r;
    }
    return pass & live;
}

// One wave tile: the sum over its rows of the product of the sides' row counts.
template <int K, bool DUP>
__device__ __forceinline__ unsigned long long join_rows(const Side (&side)[K], const uint32_t (&v)[K][probe_rpt(K)],
                                                        uint32_t live, FilterKind kind, const uint32_t *s_bits)
{
    constexpr int RPT = probe_rpt(K);
    uint32_t cnt[RPT];
    unsigned long long prod[DUP ? RPT : 1];
#pragma unroll
    for (int j = 0; j < K; j++) {
        bool counted = false;
        if (j == 0 && kind != FILTER_NONE) {
            live = filtered<RPT>(side[0], kind, s_bits, v[0], live);
            if (kind == FILTER_EXACT && !side[0].dup) {
#pragma unroll
                for (int r = 0; r < RPT; r++) cnt[r] = (live >> r) & 1u;
                counted = true;
            } else if (!__any(live != 0u)) {
                return 0ull;
            }
        }
        if (!counted) live = lookup<RPT, DUP>(side[j], v[j], live, cnt);
        if constexpr (DUP) {
#pragma unroll
            for (int r = 0; r < RPT; r++) prod[r] = j == 0 ? cnt[r] : prod[r] * cnt[r];
        }
        if (!__any(live != 0u)) return 0ull;
    }
    if constexpr (!DUP) return (unsigned long long)__popc(live);
    unsigned long long s = 0;
    if constexpr (DUP) {
#pragma unroll
        for (int r = 0; r < RPT; r++) s += ((live >> r) & 1u) ? prod[r] : 0ull;
    }
    return s;
}

// Star-join count: sum over probe rows of the product over build sides of
// the matching build rows.  The probe's key columns are read as in the scans
// (wave tiles of 64 * 8 or 64 * 4 rows, 16-byte coalesced loads).  Every block
// stores its sum in out[blockIdx.x], a word of pinned host memory each, which
// the host adds up: no counter to clear before the launch and no copy after it.
// NT = kProbeBig threads: one block per CU, with the LDS filter where
// `filter` says that the launch has the LDS for one; NT = kScanBlock: for
// probes with no more than one such block of four waves for each CU.
constexpr int kProbeBig = 1024;

template <int K, int NT>
__global__ __launch_bounds__(NT) void probe_count_kernel(const ColPtrs cp, int64_t n, const HashRef h, int filter,
                                                         unsigned long long *out)
{
    constexpr int RPT = probe_rpt(K);
    constexpr int TILE = kWave * RPT;
    constexpr int NW = NT / kWave;
    extern __shared__ uint32_t s_bits[];
    const int64_t ntiles = (n + TILE - 1) / TILE;
    const int64_t step = (int64_t)gridDim.x * NW;
    Side side[K];
    bool dup = false;
#pragma unroll
    for (int j = 0; j < K; j++) {
        side[j] = side_of(h.head[j], h.slots[j]);
        dup |= side[j].dup;
    }
    FilterKind kind = FILTER_NONE;
    if constexpr (NT == kProbeBig) {
        if (filter) kind = filter_kind(side[0], n / gridDim.x);
        if (kind != FILTER_NONE) load_filter<NT>(side[0], kind, s_bits);
    }
    unsigned long long acc = 0;   // per lane
    // the blocks take the tiles in turn, so that few tiles use every CU
    for (int64_t t = (int64_t)wave_id() * gridDim.x + blockIdx.x; t < ntiles; t += step) {
        uint32_t v[K][RPT];
        load_vals<K, RPT>(cp, t * TILE, n, v);
        const uint32_t valid = valid_bits<RPT>(t * TILE, n);
        acc += dup ? join_rows<K, true>(side, v, valid, kind, s_bits) : join_rows<K, false>(side, v, valid, kind, s_bits);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
    __shared__ unsigned long long s_acc[NW];
    if (lane_id() == 0) s_acc[wave_id()] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long b = 0;
        for (int w = 0; w < NW; w++) b += s_acc[w];
        out[blockIdx.x] = b;
    }
}

// capacity (slots) of a table of `bytes`; 0 if the size is not 256 + 8 * 2^m, m in [6, 31]
int64_t table_slots(size_t bytes)
{
    if (bytes < 256 + 8 * 64) return 0;
    const size_t s = (bytes - 256) / 8;
    if ((s & (s - 1)) != 0 || s > (1ull << 31)) return 0;
    return (int64_t)s;
}

int log2_exact(int64_t s)
{
    int m = 0;
    while ((1ll << m) < s) m++;
    return m;
}

}  // namespace esc

using namespace esc;

extern "C" {

int esc_hash_table_bytes(int64_t nkeys, size_t *bytes)
{
    if (!bytes || nkeys < 0) return fail(ESC_ERR_INVALID, "null argument or nkeys < 0");
    if (nkeys > (1ll << 30)) return fail(ESC_ERR_UNSUPPORTED, "more than 2^30 keys");
    int64_t s = 64;
    while (s < 2 * nkeys) s *= 2;
    *bytes = 256 + 8 * (size_t)s;
    return ESC_OK;
}

int esc_hash_build(esc_ctx *ctx, const int32_t *dev_keys, int64_t nkeys, void *dev_table, size_t table_bytes,
                   void *stream)
{
    if (!ctx || !dev_table || (nkeys > 0 && !dev_keys) || nkeys < 0) return fail(ESC_ERR_INVALID, "null argument");
    const int64_t slots = table_slots(table_bytes);
    if (slots == 0) return fail(ESC_ERR_INVALID, "table_bytes %zu is not a size from esc_hash_table_bytes", table_bytes);
    if (2 * nkeys > slots) return fail(ESC_ERR_INVALID, "%lld keys need %lld slots or more, the table has %lld",
                                      (long long)nkeys, (long long)(2 * nkeys), (long long)slots);
    int rc = set_device(ctx->device);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)stream;
    TableHeader *h = (TableHeader *)dev_table;
    const int grid = ctx->num_cus * 8;
    int nparts = 0;
    if (nkeys > kMinMaxNone) {
        const bool few = nkeys <= kMinMaxFew;
        const int64_t blocks = std::min<int64_t>((nkeys + 8191) / 8192, few ? kMinMaxParts : ctx->num_cus);
        if (!few) hipLaunchKernelGGL(begin_build_kernel, dim3(1), dim3(64), 0, s, h);
        hipLaunchKernelGGL(minmax_kernel, dim3((unsigned)blocks), dim3(kMinMaxBlock), 0, s, dev_keys, nkeys, h, few ? 1 : 0);
        nparts = (int)std::min<int64_t>(blocks, kMinMaxParts);
    }
    const int64_t fill_blocks = std::min<int64_t>((slots / 2 + kFillBlock - 1) / kFillBlock, grid);   // 16 bytes per thread
    hipLaunchKernelGGL(fill_table_kernel, dim3((unsigned)fill_blocks), dim3(kFillBlock), 0, s, dev_keys, h, nkeys, slots,
                       nparts, ctx->num_cus);
    if (nkeys > 0) {
        const int shift = 32 - log2_exact(slots);
        // one of the two kernels does the work, as the header says
        if (nkeys >= kPartKeys) {
            hipError_t e = hipFuncSetAttribute((const void *)build_parts_kernel,
                                               hipFuncAttributeMaxDynamicSharedMemorySize, kPartBytes);
            if (e != hipSuccess) return hip_fail(e, "build kernel LDS");
            hipLaunchKernelGGL(build_parts_kernel, dim3(ctx->num_cus), dim3(kPartBlock), kPartBytes, s, dev_keys, nkeys,
                               h, (uint32_t)slots, shift);
        }
        hipLaunchKernelGGL(build_kernel, dim3((unsigned)std::min<int64_t>((nkeys + 255) / 256, grid)), dim3(256), 0, s,
                           dev_keys, nkeys, h, (uint32_t)slots, shift);
    }
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? ESC_OK : hip_fail(e, "hash build launch");
}

int esc_join_count(esc_ctx *ctx, const esc_table *probe, const int32_t *key_cols, void *const *dev_tables,
                   const size_t *table_bytes, int ntables, void *dev_ws, size_t ws_bytes, void *stream,
                   uint64_t *out_count)
{
    if (!ctx || !probe || !key_cols || !dev_tables || !table_bytes || !out_count)
        return fail(ESC_ERR_INVALID, "null argument");
    if (!dev_ws || ((uintptr_t)dev_ws & 255)) return fail(ESC_ERR_ALIGN, "workspace must be non-null and 256-byte aligned");
    if (ws_bytes < sizeof(WsHeader)) return fail(ESC_ERR_OOM, "workspace of %zu bytes, %zu needed", ws_bytes, sizeof(WsHeader));
    if (ntables < 1 || ntables > kJoinMaxTables)
        return fail(ESC_ERR_INVALID, "ntables %d outside [1, %d]", ntables, kJoinMaxTables);
    if (!probe->has_data()) return fail(ESC_ERR_INVALID, "probe table has no device columns");
    HashRef h{};
    ColPtrs cp{};
    cp.nt = ctx->nt;
    for (int j = 0; j < ntables; j++) {
        const int c = key_cols[j];
        if (c < 0 || c >= (int)probe->dtypes.size()) return fail(ESC_ERR_INVALID, "key column %d out of range", c);
        if (probe->dtypes[c] == ESC_FLOAT32) return fail(ESC_ERR_TYPE, "key column %d is float32", c);
        const int64_t slots = table_slots(table_bytes[j]);
        if (slots == 0 || !dev_tables[j]) return fail(ESC_ERR_INVALID, "hash table %d: bad pointer or size", j);
        h.head[j] = (const TableHeader *)dev_tables[j];
        h.slots[j] = (uint32_t)slots;
        cp.p[j] = (const uint32_t *)probe->cols[c];
    }
    int rc = set_device(ctx->device);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)stream;
    const int64_t n = probe->nrows;
    if (n == 0) {
        *out_count = 0;
        return ESC_OK;
    }
    typedef void (*ProbeFn)(const ColPtrs, int64_t, const HashRef, int, unsigned long long *);
    const ProbeFn few[] = {probe_count_kernel<1, kScanBlock>, probe_count_kernel<2, kScanBlock>,
                           probe_count_kernel<3, kScanBlock>, probe_count_kernel<4, kScanBlock>};
    const ProbeFn many[] = {probe_count_kernel<1, kProbeBig>, probe_count_kernel<2, kProbeBig>,
                            probe_count_kernel<3, kProbeBig>, probe_count_kernel<4, kProbeBig>};
    const int64_t tile = kWave * probe_rpt(ntables);
    const int64_t ntiles = (n + tile - 1) / tile;
    const int cus = std::min(ctx->num_cus, kSlotWord);   // one word of the pinned block for each block's sum
    const bool big = ntiles > (int64_t)cus * (kScanBlock / kWave);
    // from two tiles for each wave of the large blocks on, a filter of the first side may pay
    const bool filter = ntiles >= 2ll * cus * (kProbeBig / kWave);
    const ProbeFn fn = (big ? many : few)[ntables - 1];
    const int lds = filter ? kFilterBytes : 0;
    hipError_t e;
    if (filter && (e = hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds)) != hipSuccess)
        return hip_fail(e, "probe kernel LDS");
    const int grid = (int)std::min<int64_t>(ntiles, cus);
    hipLaunchKernelGGL(fn, dim3((unsigned)grid), dim3(big ? kProbeBig : kScanBlock), lds, s, cp, n, h, filter ? 1 : 0,
                       ctx->pinned_dev);
    if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "join probe launch");
    if ((e = hipStreamSynchronize(s)) != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
    unsigned long long total = 0;
    for (int b = 0; b < grid; b++) total += ((volatile unsigned long long *)ctx->pinned)[b];
    *out_count = total;
    return ESC_OK;
}

}  // extern "C"
