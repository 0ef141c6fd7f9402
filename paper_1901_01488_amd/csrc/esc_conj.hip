// esc_conj.hip -- gfx950 kernel of the per-conjunct counts of split
// selectivity: one scan gives the rows of every top-level conjunct alone and
// of every prefix of them.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <utility>

#include "esc_device.h"
#include "esc_host.h"
#include "esc_kernels.h"

namespace esc {

// Every conjunct's program runs on each loaded wave tile; a running AND of
// their masks gives the prefixes.  A lane keeps its counts of a conjunct in a
// 64-bit LDS word of its own (rows of the conjunct in the low half, of the
// prefix above): one add a tile and conjunct and no reduction across lanes
// before the last tile.  Each block stores its words of that form in pinned
// host memory, out[block * nconj + conjunct], and the host adds them up: no
// counters to clear before the scan and no copy after it.
// What bounds it: the columns' bytes for programs of little work (four star
// predicates, ten column reads in all, 40M rows 313 us = 5.1 TB/s; 354 before),
// the interpreter's vector instructions for others (conj_load), and below
// about 3M rows the call (10,000 rows 22 us; 10M star rows 198 -> 144 us for
// four, 36 us a call for 16 us of their bytes).
// PACKED: the programs come as one list in the kernel's arguments with their
// tables in registers; else from memory.
template <int K, int RPT, bool UDF, bool PACKED>
__global__ __launch_bounds__(kScanBlock) void conj_kernel(const ConjPack pack, const Program *__restrict__ progs,
                                                          int nconj, const ColPtrs cp, int64_t n,
                                                          unsigned long long *out)
{
    constexpr int TILE = kWave * RPT;
    constexpr int NW = kScanBlock / kWave;
    constexpr int NT = PACKED ? kMaxTables : 0;
    extern __shared__ unsigned long long s_acc[];   // [nconj][kScanBlock]
    __shared__ unsigned long long s_sum[NW][kMaxConj];
    const int wave = wave_id();
    unsigned long long *acc = s_acc + threadIdx.x;
    for (int i = 0; i < nconj; i++) acc[i * kScanBlock] = 0ull;
    SlotTabs<NT> tabs;
    if constexpr (PACKED) tabs = load_tables<NT>(pack);
    const int64_t ntiles = (n + TILE - 1) / TILE;
    const int64_t step = (int64_t)gridDim.x * NW;
    for (int64_t t = (int64_t)blockIdx.x * NW + wave; t < ntiles; t += step) {
        uint32_t v[K][RPT];
        load_vals<K, RPT>(cp, t * TILE, n, v);
        const uint32_t valid = valid_bits<RPT>(t * TILE, n);
        uint32_t prefix = valid;
        for (int i = 0; i < nconj; i++) {
            uint32_t m;
            if constexpr (PACKED) {
                const int a = pack.first[i];
                m = run_program<K, RPT, UDF, NT>(ProgView{pack.first[i + 1] - a, pack.insn + a, pack.kpool}, v, valid, tabs);
            } else {
                m = run_program<K, RPT, UDF>(progs[i], v, valid);
            }
            prefix &= m;
            const unsigned long long c = (unsigned long long)(uint32_t)__popc(prefix) << 32 | (uint32_t)__popc(m);
            __hip_atomic_fetch_add(&acc[i * kScanBlock], c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
        }
    }
    for (int i = 0; i < nconj; i++) {
        const unsigned long long c = acc[i * kScanBlock];
        const uint32_t c1 = wave_sum((uint32_t)c), c2 = wave_sum((uint32_t)(c >> 32));
        if (lane_id() == 0) s_sum[wave][i] = (unsigned long long)c2 << 32 | c1;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < nconj; i += kScanBlock) {
        unsigned long long b = 0;
#pragma unroll
        for (int w = 0; w < NW; w++) b += s_sum[w][i];
        out[(int64_t)blockIdx.x * nconj + i] = b;
    }
}

template <bool UDF, bool PACKED, int... Ks>
constexpr ConjFn conj_table_impl(int k, std::integer_sequence<int, Ks...>)
{
    ConjFn t[] = {conj_kernel<Ks + 1, 16, UDF, PACKED>...};
    return t[k - 1];
}

// nslots in [1, kMaxSlots]
ConjFn conj_fn(int nslots, bool udf, bool packed)
{
    using S = std::make_integer_sequence<int, kMaxSlots>;
    if (packed) return udf ? conj_table_impl<true, true>(nslots, S{}) : conj_table_impl<false, true>(nslots, S{});
    return udf ? conj_table_impl<true, false>(nslots, S{}) : conj_table_impl<false, false>(nslots, S{});
}

}  // namespace esc
