// esc_index.hip -- counts a group of up to 128 selections on one table by a
// predicate index (esc_index.h): per row and column one search among the
// interval boundaries that the group's constants cut, and one record of bit
// masks, ANDed over the columns; bit p of the result says whether predicate p
// selects the row.
//
// What bounds it: LDS reads and vector issue.  A search level costs one
// 4-byte LDS read and three vector ops per row, a record word a quarter of a
// 16-byte read and one op; the trees are stored breadth first, so the top six
// levels' 64 lanes read different banks.  The interpreter of esc_batch.hip
// costs about 5 ops per instruction of every program instead.  Counters: 2,048
// predicates on six columns of 10M rows keep vector issue 72 % and LDS 70 %
// busy; 128 three-table queries on tables of 1M to 100M rows 64 and 56 %; 32
// short predicates a table 58 and 40 %.  In between the waves, four on a
// SIMD, wait for their own searches' chains of LDS reads (53 to 66 % of their
// time).
//
// Counting uses bit-sliced counters: plane b of result word w holds bit b of
// 32 counters per lane, so adding a row's word costs a few three-input bit
// operations for 32 predicates; the lanes are summed only when the planes
// are full or the work item ends.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "esc_batch.h"
#include "esc_device.h"

namespace esc {

namespace {

constexpr int kPlanes = 10;                               // counts up to 1023 rows per lane
constexpr int kFlushTiles = ((1 << kPlanes) - 1) / 4;     // wave tiles between two flushes (four rows per lane each)

typedef const uint32_t __attribute__((address_space(1))) gu32;
typedef const u32x4 __attribute__((address_space(1))) gu32x4;

__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

__device__ __forceinline__ uint32_t majority(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0xE8);
}

// Adds four one-bit numbers per bit position to the bit-sliced counters.
__device__ __forceinline__ void add_rows(uint32_t (&pl)[kPlanes], uint32_t a, uint32_t b, uint32_t c, uint32_t d)
{
    const uint32_t s = xor3(pl[0], a, b), c1 = majority(pl[0], a, b);
    const uint32_t c2 = majority(s, c, d);
    pl[0] = xor3(s, c, d);
    uint32_t carry = majority(pl[1], c1, c2);
    pl[1] = xor3(pl[1], c1, c2);
#pragma unroll
    for (int k = 2; k < kPlanes; k++) {
        const uint32_t t = pl[k] & carry;
        pl[k] ^= carry;
        carry = t;
    }
}

// Sums the lanes' counters (bit-sliced addition over the six lane
// distances), adds the 32 totals to cnt and clears the counters.
__device__ __forceinline__ void flush_planes(uint32_t (&pl)[kPlanes], uint32_t *cnt)
{
    uint32_t t[kPlanes + 6];
#pragma unroll
    for (int k = 0; k < kPlanes; k++) {
        t[k] = pl[k];
        pl[k] = 0u;
    }
#pragma unroll
    for (int step = 0; step < 6; step++) {
        uint32_t carry = 0u;
#pragma unroll
        for (int k = 0; k < kPlanes + step; k++) {
            const uint32_t y = (uint32_t)__shfl_xor((int)t[k], 1 << step, 64);
            const uint32_t s = xor3(t[k], y, carry);
            carry = majority(t[k], y, carry);
            t[k] = s;
        }
        t[kPlanes + step] = carry;
    }
    const int p = lane_id() & 31;
    uint32_t n = 0u;
#pragma unroll
    for (int k = 0; k < kPlanes + 6; k++) n |= ((t[k] >> p) & 1u) << k;
    if (lane_id() < 32 && n) atomicAdd(&cnt[p], n);
}

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned char __attribute__((address_space(3))) lds_u8;

// the T at an LDS byte address
template <typename T>
__device__ __forceinline__ T lds_at(uint32_t addr)
{
    return *(const T __attribute__((address_space(3))) *)(uintptr_t)addr;
}

// The four rows' records of one column: x holds the rows' values, at[r]
// receives the LDS address of row r's record.
template <int R>
__device__ __forceinline__ void search(const IndexColumnRef &C, uint32_t lds, u32x4 x, uint32_t (&at)[4])
{
    int32_t v[4];
    const uint32_t keys = lds + C.key_byte;
#pragma unroll
    for (int r = 0; r < 4; r++) {
        v[r] = (int32_t)x[r];
        at[r] = keys + 4u;   // the root, node 1
    }
    if (C.is_float) {
#pragma unroll
        for (int r = 0; r < 4; r++) v[r] ^= (v[r] >> 31) & 0x7fffffff;
    }
    // node i -> 2i + (value >= boundary): a compare, a select and a
    // shift-and-add per level.  The two addends pass through mbcnt of an
    // empty mask (which adds nothing) so that they stay two registers: as
    // "4 or 0, minus keys" the step would be two operations longer.
    const uint32_t up = __builtin_amdgcn_mbcnt_lo(0u, 4u - keys), down = __builtin_amdgcn_mbcnt_hi(0u, 0u - keys);
    for (int l = 0; l < C.levels; l++) {
        int32_t b[4];
#pragma unroll
        for (int r = 0; r < 4; r++) b[r] = lds_at<int32_t>(at[r]);
#pragma unroll
        for (int r = 0; r < 4; r++) at[r] = 2u * at[r] + (v[r] >= b[r] ? up : down);
    }
    // leaf 2^levels + e holds record e
    const uint32_t recs = lds + C.rec_byte - (keys + (4u << C.levels)) * R;
#pragma unroll
    for (int r = 0; r < 4; r++) at[r] = recs + R * at[r];
}

template <int R>
__device__ __forceinline__ void load_record(uint32_t at, uint32_t (&m)[R])
{
    if constexpr (R == 2) {
        const u32x2 q = lds_at<u32x2>(at);
        m[0] = q.x;
        m[1] = q.y;
    } else {
#pragma unroll
        for (int k = 0; k < R / 4; k++) {
            const u32x4 q = lds_at<u32x4>(at + 16u * k);
#pragma unroll
            for (int e = 0; e < 4; e++) m[4 * k + e] = q[e];
        }
    }
}

// The result words of four rows per lane: x(c) gives the rows' values of
// column c, read one pair of columns ahead.  Two columns are searched at a
// time: eight independent chains of LDS reads, and one three-input AND takes
// both columns' record words.
template <int W, int R, typename X>
__device__ __forceinline__ void index_tile(const IndexGroupRef &g, uint32_t lds, X &&x, uint32_t (&acc)[4][R])
{
#pragma unroll
    for (int r = 0; r < 4; r++)
#pragma unroll
        for (int w = 0; w < R; w++) acc[r][w] = ~0u;
    const int ncols = g.ncols;
    u32x4 n0 = x(0), n1 = n0;
    if (ncols > 1) n1 = x(1);
    int c = 0;
    for (; c + 1 < ncols; c += 2) {
        const u32x4 x0 = n0, x1 = n1;
        if (c + 2 < ncols) n0 = x(c + 2);
        if (c + 3 < ncols) n1 = x(c + 3);
        uint32_t a0[4], a1[4];
        search<R>(g.cols[c], lds, x0, a0);
        search<R>(g.cols[c + 1], lds, x1, a1);
#pragma unroll
        for (int r = 0; r < 4; r++) {
            uint32_t m0[R], m1[R];
            load_record<R>(a0[r], m0);
            load_record<R>(a1[r], m1);
#pragma unroll
            for (int w = 0; w < R; w++) acc[r][w] = __builtin_amdgcn_bitop3_b32(acc[r][w], m0[w], m1[w], 0x80);
        }
    }
    if (c < ncols) {
        uint32_t a0[4];
        search<R>(g.cols[c], lds, n0, a0);
#pragma unroll
        for (int r = 0; r < 4; r++) {
            uint32_t m0[R];
            load_record<R>(a0[r], m0);
#pragma unroll
            for (int w = 0; w < R; w++) acc[r][w] &= m0[w];
        }
    }
    // OR layers hold the complement of their clause
    const int nor = g.nor;
#pragma unroll
    for (int j = 0; j < R - W; j++) {
        if (j >= nor) break;
        const int w = g.or_word[j];
#pragma unroll
        for (int q = 0; q < W; q++)
            if (w == q) {
#pragma unroll
                for (int r = 0; r < 4; r++) acc[r][q] &= ~acc[r][W + j];
            }
    }
}

template <int W, int R>
__device__ __forceinline__ void index_rows(const IndexGroupRef &g, const BatchItem &it, uint32_t lds,
                                           uint32_t *cnt)
{
    constexpr int NW = kIndexBlock / kWave;
    const int lane = lane_id();
    uint32_t pl[W][kPlanes];
#pragma unroll
    for (int w = 0; w < W; w++)
#pragma unroll
        for (int k = 0; k < kPlanes; k++) pl[w][k] = 0u;
    const int full = (it.r1 - it.r0) / kIndexTile;   // whole wave tiles of the item
    int room = kFlushTiles;
    for (int t = wave_id(); t <= full; t += NW) {
        const int64_t base = (int64_t)it.r0 + (int64_t)t * kIndexTile;
        uint32_t acc[4][R];
        if (t < full) {
            index_tile<W, R>(
                g, lds,
                [&](int c) { return *(gu32x4 *)((gu32 *)g.cols[c].ptr + base + lane * 4); }, acc);
        } else {
            const int rem = (int)(it.r1 - base);   // rows after the last whole tile
            if (rem <= 0) break;
            index_tile<W, R>(
                g, lds,
                [&](int c) {
                    gu32 *src = (gu32 *)g.cols[c].ptr + base;
                    u32x4 q;
#pragma unroll
                    for (int e = 0; e < 4; e++) q[e] = src[min(lane * 4 + e, rem - 1)];
                    return q;
                },
                acc);
#pragma unroll
            for (int r = 0; r < 4; r++)
                if (lane * 4 + r >= rem) {
#pragma unroll
                    for (int w = 0; w < W; w++) acc[r][w] = 0u;
                }
        }
#pragma unroll
        for (int w = 0; w < W; w++) add_rows(pl[w], acc[0][w], acc[1][w], acc[2][w], acc[3][w]);
        if (--room == 0) {
#pragma unroll
            for (int w = 0; w < W; w++) flush_planes(pl[w], cnt + 32 * w);
            room = kFlushTiles;
        }
    }
#pragma unroll
    for (int w = 0; w < W; w++) flush_planes(pl[w], cnt + 32 * w);
}

}  // namespace

// Persistent blocks pop (group, rows) items; a block loads a group's index
// into LDS when its group changes and publishes the counts of the old one.
__global__ __launch_bounds__(kIndexBlock) __attribute__((amdgpu_waves_per_eu(4)))
void index_kernel(BatchHeader *h, const char *__restrict__ lists, unsigned long long *counts)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char s_index[];
    __shared__ uint32_t s_cnt[kIndexMaxPreds];
    __shared__ int s_item;
    const int nitems = (int)h->nitems[1];
    const IndexGroupRef *__restrict__ groups = (const IndexGroupRef *)(lists + h->igroups);
    const BatchItem *__restrict__ items = (const BatchItem *)(lists + h->iitems);
    const uint32_t *__restrict__ blob = (const uint32_t *)(lists + h->blob);
    const int32_t *__restrict__ ids = (const int32_t *)(lists + h->ids);
    const uint32_t lds = (uint32_t)(uintptr_t)(lds_u8 *)s_index;
    int cur = -1;
    for (int i = threadIdx.x; i < kIndexMaxPreds; i += kIndexBlock) s_cnt[i] = 0u;
    for (;;) {
        __syncthreads();   // s_item and the index of the last item are no longer read
        if (threadIdx.x == 0) s_item = (int)atomicAdd(&h->next[1], 1u);
        __syncthreads();
        const int item = __builtin_amdgcn_readfirstlane(s_item);
        const bool done = item >= nitems;
        BatchItem it{};
        if (!done) it = items[item];
        if (done || it.group != cur) {
            if (cur >= 0) {
                const IndexGroupRef &o = groups[cur];
                if ((int)threadIdx.x < o.npred) {
                    const uint32_t n = s_cnt[threadIdx.x];
                    s_cnt[threadIdx.x] = 0u;
                    if (n) atomicAdd(&counts[ids[o.pbegin + threadIdx.x]], (unsigned long long)n);
                } else if ((int)threadIdx.x < kIndexMaxPreds) {
                    s_cnt[threadIdx.x] = 0u;   // bits beyond the group's predicates count nothing
                }
            }
            if (done) break;
            cur = it.group;
            const u32x4 *src = (const u32x4 *)(blob + groups[cur].blob);
            const int n4 = groups[cur].nwords / 4;
            for (int i = threadIdx.x; i < n4; i += kIndexBlock) ((u32x4 *)s_index)[i] = src[i];
            __syncthreads();
        }
        const IndexGroupRef &g = groups[cur];
        switch (g.words * 16 + g.rec) {
        case 16 + 2: index_rows<1, 2>(g, it, lds, s_cnt); break;
        case 16 + 4: index_rows<1, 4>(g, it, lds, s_cnt); break;
        case 16 + 8: index_rows<1, 8>(g, it, lds, s_cnt); break;
        case 32 + 2: index_rows<2, 2>(g, it, lds, s_cnt); break;
        case 32 + 4: index_rows<2, 4>(g, it, lds, s_cnt); break;
        case 32 + 8: index_rows<2, 8>(g, it, lds, s_cnt); break;
        case 64 + 4: index_rows<4, 4>(g, it, lds, s_cnt); break;
        default: index_rows<4, 8>(g, it, lds, s_cnt); break;
        }
    }
}

hipError_t prepare_index()
{
    return hipFuncSetAttribute((const void *)index_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                               kIndexMaxWords * 4);
}

void launch_index(BatchHeader *h, unsigned long long *counts, int grid, hipStream_t s)
{
    hipLaunchKernelGGL(index_kernel, dim3(grid), dim3(kIndexBlock), kIndexMaxWords * 4, s, h, (const char *)h, counts);
}

}  // namespace esc
