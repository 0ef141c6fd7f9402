// esc_count_kernel.h -- the count kernel, for the two files that instantiate
// it: esc_count.hip (counts that store tiles, and those with one result word)
// and esc_count_parts.hip (one host word per block), which compile side by side.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <utility>

#include "esc_device.h"
#include "esc_host.h"
#include "esc_kernels.h"

namespace esc {

// A wave's tile records wait in LDS (masks) and in a register (counts, one
// tile per lane) and go out kTileBuf tiles at a time: a global store inside
// the tile loop would make the next tile's loads wait for its
// acknowledgement (stores and loads share one counter of outstanding
// memory operations), and with one wave per SIMD nothing hides that wait.
__device__ __forceinline__ void flush_tiles(const TileOut &to, const uint32_t *buf, uint32_t tcnt, int64_t t0,
                                            int64_t step, int nbuf)
{
    for (int j = 0; j < nbuf; j++) to.bits[(t0 + j * step) * kWave + lane_id()] = buf[j * kWave + lane_id()];
    if (lane_id() < nbuf) to.counts[t0 + lane_id() * step] = tcnt;
}

// Grid-stride over wave tiles.  With TILES, every wave tile's count and lane
// masks are stored in to.counts and to.bits (the launch then gives the block
// kTileBufBytes of dynamic LDS); a plain count carries none of that code.
// UDF = false for programs without udf instructions.  PARTS (plain counts):
// every block has a host word of its own, out[blockIdx.x], which the host adds
// up: no chain of atomics on one word (about 10 ns a block).  A kernel of its
// own: as a branch at the end of the others, its few instructions moved the
// tile loop of programs with a udf against the instruction cache's lines and
// cost them 1 % (40M rows, the Section 1 selection 127.4 -> 128.6 us).
template <int K, int RPT, bool UDF, bool TILES, bool PARTS>
__global__ __launch_bounds__(kScanBlock) void count_kernel(const Program P, const ColPtrs cp, int64_t n,
                                                           WsHeader *ws, unsigned long long *out, const TileOut to)
{
    constexpr int TILE = kWave * RPT;
    constexpr int KK = K > 0 ? K : 1;
    constexpr int NW = kScanBlock / kWave;
    const int64_t ntiles = (n + TILE - 1) / TILE;
    const int64_t step = (int64_t)gridDim.x * NW;
    const int64_t first = (int64_t)blockIdx.x * NW + wave_id();
    // the workspace already holds this count's tiles: nothing to do (the
    // stamp is read from a previous launch's write, the same for every block)
    if (TILES && to.expect != 0ull && ws->stamp == to.expect) return;
    const SlotTabs<kMaxTables> tabs = load_tables<kMaxTables>(P);
    extern __shared__ uint32_t s_tbuf[];   // [NW][kTileBuf][kWave] lane masks
    const int wave = wave_id();
    uint32_t *buf = s_tbuf + wave * (kTileBuf * kWave);
    uint32_t tcnt = 0;   // lane j: count of the j-th buffered tile
    int nbuf = 0;
    int64_t t0 = first;  // the first buffered tile; the others follow at step
    uint32_t cnt = 0;    // per lane
    for (int64_t t = first; t < ntiles; t += step) {
        uint32_t v[KK][RPT];
        load_vals<K, RPT>(cp, t * TILE, n, v);
        const uint32_t bits = run_program<K, RPT, UDF, kMaxTables>(P, v, valid_bits<RPT>(t * TILE, n), tabs);
        const uint32_t c = (uint32_t)__popc(bits);
        if constexpr (TILES) {
            const uint32_t w = wave_sum(c);
            tcnt = lane_id() == nbuf ? w : tcnt;
            buf[nbuf * kWave + lane_id()] = bits;   // each lane reads back only its own words
            if (++nbuf == kTileBuf) {
                flush_tiles(to, buf, tcnt, t0, step, nbuf);
                nbuf = 0;
                t0 = t + step;
            }
        }
        cnt += c;
    }
    if (TILES && nbuf) flush_tiles(to, buf, tcnt, t0, step, nbuf);
    cnt = wave_sum(cnt);
    __shared__ uint32_t s_cnt[NW];
    if (lane_id() == 0) s_cnt[wave] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long b = 0;
        for (int w = 0; w < NW; w++) b += s_cnt[w];
        if constexpr (PARTS) {
            out[blockIdx.x] = b;
            return;
        }
        // One 64-bit word carries both the running row count (low
        // kTotalBits bits) and the number of blocks done (high bits), so
        // each block's contribution is one atomic read-modify-write of one
        // location.  All such RMWs are totally ordered and each reads the
        // value left by the previous ones, so the block whose RMW returns
        // gridDim.x - 1 blocks done has read the sum of every other block:
        // exact without fences and without any order between two
        // addresses.  That block publishes the total and resets the word,
        // so the next launch on the workspace starts from zero.
        const unsigned long long old = atomicAdd(&ws->total, (1ull << kTotalBits) | b);
        if ((old >> kTotalBits) == gridDim.x - 1u) {
            *out = (old & ((1ull << kTotalBits) - 1ull)) + b;
            atomicExch(&ws->total, 0ull);
            if (TILES) ws->stamp = to.stamp;
        }
    }
}

template <int RPT, bool UDF, bool TILES, bool PARTS, int... Ks>
constexpr CountFn count_table_impl(int k, std::integer_sequence<int, Ks...>)
{
    CountFn t[] = {count_kernel<Ks, RPT, UDF, TILES, PARTS>...};
    return t[k];
}

template <int RPT, bool TILES, bool PARTS>
static CountFn count_table(int k, bool udf)
{
    using S = std::make_integer_sequence<int, kMaxSlots + 1>;
    return udf ? count_table_impl<RPT, true, TILES, PARTS>(k, S{}) : count_table_impl<RPT, false, TILES, PARTS>(k, S{});
}

}  // namespace esc
