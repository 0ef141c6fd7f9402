// esc_materialize.hip -- gfx950 kernels that materialize a selection as a
// temporary table in row order (Section 2, Section 2.1): order-preserving
// stream compaction in passes with no inter-block waiting, after the count
// pass of esc_count.hip stored per-tile counts and lane masks:
//   1. for tables of many tiles one block scans the tile counts into
//      row-order output offsets (the write pass finds its own otherwise);
//   2. the write pass reads the masks instead of the predicate's columns,
//      ranks the qualifying rows of each 1,024-row unit with ballot masks and
//      writes row ids and projected values as contiguous runs at offset + rank.
// When the count pass was the caller's own preceding esc_count on the same
// workspace, table and predicate (count, decide, then materialize),
// materialization never reads the predicate's columns again.  A
// single-pass compaction with decoupled look-back serves a materialization
// with no count before it when asked for.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <type_traits>
#include <utility>

#include "esc_device.h"
#include "esc_grid.h"
#include "esc_host.h"
#include "esc_kernels.h"

namespace esc {

// ------------------------------------------------------------------ scan

// Exclusive scan of m per-tile counts into offsets[0..m]; offsets[m] is the
// total, also stored in ws->result.  One block of 1024 threads walks the
// counts in rounds of 16384: each thread takes 16 consecutive counts (four
// 16-byte loads, coalesced across the block), the thread totals are scanned
// with wave shuffles and a 16-entry LDS pass, and a carry links the rounds.
__global__ __launch_bounds__(1024) void scan_kernel(const uint32_t *counts, int64_t m, uint32_t *offsets,
                                                    WsHeader *ws, unsigned long long *total)
{
    constexpr int PER = 16, NT = 1024, NWV = NT / 64;
    __shared__ uint32_t s_wave[NWV];
    __shared__ uint32_t s_carry;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    if (t == 0) s_carry = 0;
    __syncthreads();
    for (int64_t r0 = 0; r0 < m; r0 += (int64_t)PER * NT) {
        const int64_t i0 = r0 + (int64_t)t * PER;
        uint32_t c[PER];
        if (i0 + PER <= m) {
#pragma unroll
            for (int q = 0; q < PER / 4; q++) {
                const u32x4 v = *(const u32x4 *)(counts + i0 + 4 * q);
                c[4 * q] = v.x; c[4 * q + 1] = v.y; c[4 * q + 2] = v.z; c[4 * q + 3] = v.w;
            }
        } else {
#pragma unroll
            for (int q = 0; q < PER; q++) c[q] = i0 + q < m ? counts[i0 + q] : 0u;
        }
        uint32_t sum = 0;
#pragma unroll
        for (int q = 0; q < PER; q++) sum += c[q];
        // inclusive scan of the thread sums inside the wave
        uint32_t inc = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t x = __shfl_up(inc, o, 64);
            if (lane >= o) inc += x;
        }
        if (lane == 63) s_wave[wave] = inc;
        __syncthreads();
        uint32_t before = s_carry;
        for (int w = 0; w < wave; w++) before += s_wave[w];
        uint32_t run = before + inc - sum;   // exclusive prefix of this thread's first count
        uint32_t o16[PER];
#pragma unroll
        for (int q = 0; q < PER; q++) { o16[q] = run; run += c[q]; }
        if (i0 + PER <= m) {
#pragma unroll
            for (int q = 0; q < PER / 4; q++) {
                u32x4 v;
                v.x = o16[4 * q]; v.y = o16[4 * q + 1]; v.z = o16[4 * q + 2]; v.w = o16[4 * q + 3];
                *(u32x4 *)(offsets + i0 + 4 * q) = v;
            }
        } else {
#pragma unroll
            for (int q = 0; q < PER; q++)
                if (i0 + q < m) offsets[i0 + q] = o16[q];
        }
        __syncthreads();   // every thread has read s_wave and s_carry
        if (t == NT - 1) s_carry = run;
        __syncthreads();
    }
    if (t == 0) {
        offsets[m] = s_carry;
        ws->result = s_carry;
        if (total) *total = s_carry;
    }
}

// ------------------------------------------------------------------ write

// Orders a wave's LDS accesses before and after it.
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The write pass works on units of 1,024 rows (16 per lane of the tile's
// masks), one wave each.  The unit's qualifying rows are ranked in row order
// and their places in the unit gathered in LDS; lane i then takes the i-th
// qualifying row of 64 and reads and writes every output column for it:
// row ids and values go out as contiguous runs, and a projected column is
// read in ascending addresses, one sector after the other, only where a row
// qualifies.  What bounds it is the latency of a unit's chain (offset, masks,
// ranks, one read per column): values need no staging, so a wave keeps 12
// reads per lane in flight in few registers.  Staging each 256-row chunk of
// a tile column by column took 131 us for the temporary tables of the star
// selections (60M rows, 0.9-8 % of them, three columns), against 82 us now.
//
// Where many rows of a unit qualify, reading and writing a row a lane is the
// bound: four times the instructions of whole 16-byte groups, each touching
// lines that the next one shares.  A unit of dense_rows() and more reads each
// column's groups, places the values in LDS by rank and writes aligned
// 16-byte groups (the last tile's units, whose rows may end inside a group,
// excepted).  Two materializations on 40M rows, one, three and four columns,
// staged by chunks / a row a lane throughout / now: 79 % of the rows 320, 544,
// 659 / 358, 616, 804 / 248, 461, 531 us; 35 %: 235, 423, 513 / 240, 424, 528 /
// 198, 353, 393.  The line at a quarter of the rows instead of an eighth cost
// 18 to 22 % of them 3 to 10 % (200, 347, 402 against 195, 340, 366, with runs
// of units a wave); below it both ways meet.
template <int RPT>
__device__ __forceinline__ void write_unit(uint32_t bits, int64_t base, unsigned long long p, const ProjArgs &pa,
                                           int32_t *rowids, unsigned long long cap, bool whole, uint32_t dense,
                                           uint32_t *buf)
{
    constexpr int NJ = kUnitRows / (4 * kWave);   // chunks of 256 rows
    const int lane = lane_id();
    uint16_t *place = (uint16_t *)buf;
    uint32_t n = 0;   // wave-uniform: rows so far
    uint32_t first[NJ];   // rank of the lane's first qualifying row of each chunk
#pragma unroll
    for (int j = 0; j < NJ; j++) {
        const uint32_t nib = (bits >> (4 * j)) & 0xfu;
        uint32_t k = n;
#pragma unroll
        for (int e = 0; e < 4; e++) {
            // set bits of the ballot in the lanes below this one (mbcnt: no
            // 64-bit shift by a per-lane amount)
            const uint64_t m = __ballot((nib >> e) & 1u);
            k = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, k));
            n += (uint32_t)__popcll(m);
        }
        first[j] = k;
    }
    const uint32_t avail = (uint32_t)(p + n <= cap ? n : cap - p);
    if (whole && n >= dense) {
        // one column at a time: its values (or the row ids) to their ranks in
        // LDS, then out in 16-byte groups; a run begins at word `head` of one
        auto column = [&](const uint32_t *src, uint32_t *dst, bool ids) {
            u32x4 v[NJ];
            if (!ids) {
#pragma unroll
                for (int j = 0; j < NJ; j++)
                    if ((bits >> (4 * j)) & 0xfu)
                        v[j] = __builtin_nontemporal_load((const u32x4 *)(src + base + lane * 4 + j * 4 * kWave));
            } else {
#pragma unroll
                for (int j = 0; j < NJ; j++)
#pragma unroll
                    for (int e = 0; e < 4; e++) v[j][e] = (uint32_t)base + lane * 4 + j * 4 * kWave + e;
            }
            const uint32_t head = (uint32_t)((uintptr_t)dst >> 2) & 3u, end = head + avail;
#pragma unroll
            for (int j = 0; j < NJ; j++) {
                uint32_t k = head + first[j];
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const uint32_t on = (bits >> (4 * j + e)) & 1u;
                    if (on) buf[k] = v[j][e];
                    k += on;
                }
            }
            wave_lds_fence();
            for (uint32_t i = lane * 4; i < end; i += 4 * kWave) {
                const u32x4 q = *(const u32x4 *)(buf + i);
                if (i >= head && i + 4 <= end) {
                    __builtin_nontemporal_store(q, (u32x4 *)(dst - head + i));
                } else {
#pragma unroll
                    for (uint32_t e = 0; e < 4; e++)
                        if (i + e >= head && i + e < end) dst[(int64_t)(i + e) - head] = q[e];
                }
            }
            wave_lds_fence();
        };
        if (rowids) column(nullptr, (uint32_t *)rowids + p, true);
#pragma unroll 1
        for (int q = 0; q < pa.nproj; q++) column(pa.src[q], pa.dst[q] + p, false);
        return;
    }
#pragma unroll
    for (int j = 0; j < NJ; j++) {
        uint32_t k = first[j];
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const uint32_t on = (bits >> (4 * j + e)) & 1u;
            if (on) place[k] = (uint16_t)(j * 256 + lane * 4 + e);
            k += on;
        }
    }
    wave_lds_fence();
    constexpr int U = 4;
    for (uint32_t i0 = lane; i0 < avail; i0 += U * kWave) {
        uint32_t r[U];
#pragma unroll
        for (int u = 0; u < U; u++) r[u] = i0 + u * kWave < avail ? place[i0 + u * kWave] : 0u;
        auto put = [&](uint32_t *dst, const uint32_t (&x)[U]) {
#pragma unroll
            for (int u = 0; u < U; u++)
                if (i0 + u * kWave < avail) dst[p + i0 + u * kWave] = x[u];
        };
        auto get = [&](const uint32_t *src, uint32_t (&x)[U]) {
#pragma unroll
            for (int u = 0; u < U; u++)
                if (i0 + u * kWave < avail) x[u] = __builtin_nontemporal_load(src + base + r[u]);
        };
        uint32_t x0[U], x1[U], x2[U];
        int q = 0;
        for (; q + 3 <= pa.nproj; q += 3) {
            get(pa.src[q], x0);
            get(pa.src[q + 1], x1);
            get(pa.src[q + 2], x2);
            put(pa.dst[q], x0);
            put(pa.dst[q + 1], x1);
            put(pa.dst[q + 2], x2);
        }
        if (q + 2 == pa.nproj) {
            get(pa.src[q], x0);
            get(pa.src[q + 1], x1);
            put(pa.dst[q], x0);
            put(pa.dst[q + 1], x1);
        } else if (q < pa.nproj) {
            get(pa.src[q], x0);
            put(pa.dst[q], x0);
        }
        if (rowids) {
#pragma unroll
            for (int u = 0; u < U; u++) x0[u] = (uint32_t)base + r[u];
            put((uint32_t *)rowids, x0);
        }
    }
    wave_lds_fence();
}

// Writes the qualifying rows of every wave tile at its offset, in row order,
// from the lane masks of the count pass: one unit a wave, in as many blocks as
// that takes, everything that a unit needs before its rows (masks, counts or
// offsets) read at once.  OWN: the block sums the counts of the tiles before
// its own and the last one stores the total (kOwnPrefixTiles); else the
// offsets are scan_kernel's.
// A wave that goes on to another unit waits for its stores before it sees its
// next loads (one counter in order), so runs of units a wave cost dense tables
// most: write passes with their counts on 100M rows, 80 % of them, three
// columns: 623 us with 16 tiles a block in turn, 1,280 blocks, 553 now, and
// 604 with every 256-row chunk staged and plain stores; 60M, 80 %, one column:
// 185, 161 and 202; 60M, 2 %, one column: 92, 83 and 110.  One unit a wave
// costs sparse ones the launch of the blocks: 100M, 0.01 %, no column: 104,
// against 101 and 99.
template <int RPT, bool OWN>
__global__ __launch_bounds__(kScanBlock) void write_kernel(const uint32_t *__restrict__ tile_bits,
                                                           const uint32_t *__restrict__ counts,
                                                           const uint32_t *__restrict__ offsets, int64_t ntiles,
                                                           const ProjArgs pa, int32_t *rowids, unsigned long long cap,
                                                           uint32_t dense, WsHeader *ws, unsigned long long *total)
{
    constexpr int TILE = kWave * RPT;
    constexpr int NW = kScanBlock / kWave;
    constexpr int UPT = TILE / kUnitRows;   // units of a tile: 1 or 2
    static_assert(UPT == 1 || UPT == 2, "units of 1,024 rows");
    __shared__ __attribute__((aligned(16))) uint32_t s_buf[NW][kUnitRows + 4];
    const int wave = wave_id(), lane = lane_id();
    const int64_t nunits = ntiles * UPT;
    // the unit u of the tile's masks `bits`, whose first row goes to o0
    auto put = [&](int64_t u, uint32_t bits, uint32_t o0) {
        const int64_t t = u / UPT;
        int64_t base = t * TILE;
        if constexpr (UPT == 2) {
            if (u & 1) {
                o0 += wave_sum((uint32_t)__popc(bits & 0xffffu));
                bits >>= 16;
                base += kUnitRows;
            }
            bits &= 0xffffu;
        }
        if (!__any(bits != 0u) || o0 >= cap) return;   // wave-uniform
        write_unit<RPT>(bits, base, o0, pa, rowids, cap, t + 1 < ntiles, dense, s_buf[wave]);
    };
    if constexpr (OWN) {
        constexpr int TPB = NW / UPT;   // tiles of a block
        __shared__ uint32_t s_sum[NW];
        const int64_t t0 = (int64_t)blockIdx.x * TPB, u = (int64_t)blockIdx.x * NW + wave;
        const uint32_t bits = u < nunits ? tile_bits[u / UPT * kWave + lane] : 0u;
        const uint32_t cnt = lane < TPB && t0 + lane < ntiles ? counts[t0 + lane] : 0u;
        uint32_t sum = 0;
        constexpr int NQ = 4;   // loads in flight
        for (int64_t i0 = threadIdx.x * 4; i0 < t0; i0 += NQ * 4 * kScanBlock) {
            u32x4 q[NQ];
#pragma unroll
            for (int k = 0; k < NQ; k++) {
                const int64_t i = i0 + k * 4 * kScanBlock;
                q[k] = u32x4{0u, 0u, 0u, 0u};
                if (i < t0) q[k] = *(const u32x4 *)(counts + i);   // t0 may end inside the four
            }
#pragma unroll
            for (int k = 0; k < NQ; k++)
#pragma unroll
                for (int e = 0; e < 4; e++) sum += i0 + k * 4 * kScanBlock + e < t0 ? q[k][e] : 0u;
        }
        sum = wave_sum(sum);
        if (lane == 0) s_sum[wave] = sum;
        __syncthreads();
        uint32_t off = 0, mine = 0, all = 0;
        for (int w = 0; w < NW; w++) off += s_sum[w];
#pragma unroll
        for (int i = 0; i < TPB; i++) {
            const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)cnt, i);
            if (i < wave / UPT) off += c;
            else all += c;
            if (i == wave / UPT) mine = c;
        }
        if (t0 + TPB >= ntiles && threadIdx.x == 0) {   // wave 0: all of the block's tiles lie behind `off`
            ws->result = off + all;
            if (total) *total = off + all;
        }
        if (mine != 0u && off < cap) put(u, bits, off);
    } else {
        // the loop is for grids of fewer blocks (esc_ctx::mat_bpc)
        uint32_t bits = 0, o0 = 0, o1 = 0;
        auto load = [&](int64_t u) {
            if (u >= nunits) return;
            const int64_t t = u / UPT;
            bits = tile_bits[t * kWave + lane];
            o0 = offsets[t];
            o1 = offsets[t + 1];
        };
        int64_t u = (int64_t)blockIdx.x * NW + wave;
        for (load(u); u < nunits;) {
            const int64_t next = u + (int64_t)gridDim.x * NW;
            const uint32_t b = bits, first = o0, last = o1;
            load(next);
            if (first != last && first < cap) put(u, b, first);
            u = next;
        }
    }
}

// ------------------------------------------------------------------ single-pass compaction

// Stages up to 256 values of the current chunk in the wave's LDS buffer at
// their compacted slots, then writes the first `avail` of them to dst with
// consecutive lanes on consecutive words (coalesced).
template <typename V>
__device__ __forceinline__ void stage_and_flush(uint32_t *buf, uint32_t nib, const uint32_t (&slot)[4], V &&val,
                                                uint32_t *dst, uint32_t avail)
{
#pragma unroll
    for (int e = 0; e < 4; e++)
        if ((nib >> e) & 1u) buf[slot[e]] = val(e);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (uint32_t i = lane_id(); i < avail; i += kWave) dst[i] = buf[i];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Writes the qualifying rows of one wave tile (lane masks `bits`, rows from
// `base`) at output positions p onwards, in row order, at most up to `cap`.
// Chunk j of the tile (256 rows) is compacted in LDS (rank of a row = lanes
// below, from ballot masks, then e) and each output column is written as one
// contiguous run.  proj(q, j, e, r0) gives projected column q's value at row
// r0 + e of chunk j.
template <int RPT, typename Proj>
__device__ __forceinline__ void write_tile(uint32_t bits, int64_t base, unsigned long long p, const ProjArgs &pa,
                                           int32_t *rowids, unsigned long long cap, uint32_t *buf, Proj &&proj)
{
    constexpr int NJ = RPT / 4;
    const int lane = lane_id();
#pragma unroll
    for (int j = 0; j < NJ; j++) {
        const uint32_t nib = (bits >> (4 * j)) & 0xfu;
        uint32_t pre = 0, tot = 0;
#pragma unroll
        for (int e = 0; e < 4; e++) {
            // set bits of the ballot in the lanes below this one (mbcnt: no
            // 64-bit shift by a per-lane amount)
            const uint64_t b = __ballot((nib >> e) & 1u);
            pre = __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, pre));
            tot += (uint32_t)__popcll(b);
        }
        if (tot == 0) continue;
        if (p >= cap) break;
        const uint32_t avail = (uint32_t)(p + tot <= cap ? tot : cap - p);
        uint32_t slot[4];
        uint32_t k = pre;
#pragma unroll
        for (int e = 0; e < 4; e++) {
            slot[e] = k;
            k += (nib >> e) & 1u;
        }
        const int64_t r0 = base + (int64_t)j * (4 * kWave) + lane * 4;   // row of e = 0
        if (rowids)
            stage_and_flush(buf, nib, slot, [&](int e) { return (uint32_t)(r0 + e); }, (uint32_t *)rowids + p, avail);
        for (int q = 0; q < pa.nproj; q++) proj(q, j, r0, nib, slot, pa.dst[q] + p, avail);
        p += tot;
    }
}

// Status word of a wave tile in the single-pass compaction: flag in the top
// two bits (0 not yet published, 1 the tile's own count, 2 the inclusive
// prefix of all tiles up to it), the value in the low 62 bits.
constexpr unsigned long long kStAggregate = 1ull << 62, kStInclusive = 2ull << 62;
constexpr unsigned long long kStValue = (1ull << 62) - 1ull;

// Count and materialization in one pass (a materialization with no count
// before it): waves take wave tiles in increasing order from a counter,
// evaluate the predicate, publish the tile's count, and find the rows
// before the tile by looking back over the predecessors' status words (a
// predecessor that has published its inclusive prefix ends the walk; one
// that has published only its count adds it and the walk continues).  Every
// predecessor was taken by a running wave before this tile, so every wait
// ends.  The qualifying rows are then written at that offset, 256 rows staged
// at a time, taking the projected values of predicate columns from
// registers.  status (ntiles words) and ctr must be zero at launch.
template <int K, int RPT, bool UDF>
__global__ __launch_bounds__(kScanBlock) void compact_kernel(const Program P, const ColPtrs cp, int64_t n,
                                                             unsigned long long *status, unsigned int *ctr,
                                                             const ProjArgs pa, const ProjSlots ps, int32_t *rowids,
                                                             unsigned long long cap, uint32_t dense_min,
                                                             unsigned long long *total)
{
    constexpr int TILE = kWave * RPT;
    constexpr int KK = K > 0 ? K : 1;
    constexpr int NW = kScanBlock / kWave;
    __shared__ uint32_t s_buf[NW][4 * kWave];
    uint32_t *buf = s_buf[wave_id()];
    const int64_t ntiles = (n + TILE - 1) / TILE;
    const SlotTabs<kMaxTables> tabs = load_tables<kMaxTables>(P);
    for (;;) {
        uint32_t got = 0;
        if (lane_id() == 0) got = atomicAdd(ctr, 1u);
        const int64_t t = (int64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)got);
        if (t >= ntiles) break;
        const int64_t base = t * TILE;
        uint32_t v[KK][RPT];
        load_vals<K, RPT>(cp, base, n, v);
        const uint32_t bits = run_program<K, RPT, UDF, kMaxTables>(P, v, valid_bits<RPT>(base, n), tabs);
        const unsigned long long c = wave_sum((uint32_t)__popc(bits));
        unsigned long long before = 0;
        if (t > 0) {
            __hip_atomic_store(&status[t], kStAggregate | c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            for (int64_t j = t - 1;;) {
                // every lane reads the same word; its first lane's copy
                // makes the walk wave-uniform
                const unsigned long long w =
                    __hip_atomic_load(&status[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const uint32_t wlo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)w);
                const uint32_t whi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(w >> 32));
                const unsigned long long wu = ((unsigned long long)whi << 32) | wlo;
                if ((wu >> 62) == 0ull) {
                    __builtin_amdgcn_s_sleep(1);
                    continue;
                }
                before += wu & kStValue;
                if ((wu >> 62) == 2ull) break;
                j--;
            }
        }
        __hip_atomic_store(&status[t], kStInclusive | (before + c), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (t == ntiles - 1 && lane_id() == 0) *total = before + c;
        if (c == 0 || before >= cap) continue;
        const bool dense = base + TILE <= n && c >= dense_min;
        write_tile<RPT>(bits, base, before, pa, rowids, cap, buf,
                        [&](int q, int j, int64_t r0, uint32_t nib, const uint32_t(&slot)[4], uint32_t *dst,
                            uint32_t avail) {
                            const int s = ps.slot[q];
                            bool done = false;
                            for_slot<K>(s, [&](auto C) {
                                stage_and_flush(buf, nib, slot, [&](int e) { return v[C][4 * j + e]; }, dst, avail);
                                done = true;
                            });
                            if (done) return;
                            const uint32_t *src = pa.src[q];
                            if (dense) {
                                const u32x4 x = __builtin_nontemporal_load((const u32x4 *)(src + r0));
                                stage_and_flush(buf, nib, slot, [&](int e) { return x[e]; }, dst, avail);
                            } else {
                                stage_and_flush(buf, nib, slot, [&](int e) { return src[r0 + e]; }, dst, avail);
                            }
                        });
    }
}

__global__ void zero_kernel(unsigned long long *p, int64_t nwords)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < nwords; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0ull;
}

// ------------------------------------------------------------------ dispatch tables

template <bool UDF, int... Ks>
constexpr CompactFn compact_table_impl(int k, std::integer_sequence<int, Ks...>)
{
    CompactFn t[] = {compact_kernel<Ks, kCompactRPT, UDF>...};
    return t[k];
}

CompactFn compact_fn(int nslots, bool udf)
{
    using S = std::make_integer_sequence<int, kMaxSlots + 1>;
    return udf ? compact_table_impl<true>(nslots, S{}) : compact_table_impl<false>(nslots, S{});
}

WriteFn write_fn(int rpt, bool own)
{
    // counts that store tiles run 16 or 32 rows per lane
    if (own) return rpt == 16 ? write_kernel<16, true> : write_kernel<32, true>;
    return rpt == 16 ? write_kernel<16, false> : write_kernel<32, false>;
}

void launch_zero(unsigned long long *p, int64_t nwords, hipStream_t s)
{
    if (nwords <= 0) return;
    int64_t blocks = (nwords + 255) / 256;
    if (blocks > 1024) blocks = 1024;
    hipLaunchKernelGGL(zero_kernel, dim3((unsigned)blocks), dim3(256), 0, s, p, nwords);
}

void launch_scan(const uint32_t *counts, int64_t m, uint32_t *offsets, WsHeader *ws, unsigned long long *total,
                 hipStream_t s)
{
    hipLaunchKernelGGL(scan_kernel, dim3(1), dim3(1024), 0, s, counts, m, offsets, ws, total);
}

}  // namespace esc
