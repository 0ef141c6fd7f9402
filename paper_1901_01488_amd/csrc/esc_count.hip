// esc_count.hip -- gfx950 kernels of the COUNT(*) selectivity sub-query
// (Section 2).
//
// Data layout: every column is a contiguous array of nrows 4-byte values
// (int32, date32 or float32), 16-byte aligned.  The unit of work is a wave
// tile of 64*RPT consecutive rows (esc_device.h): its columns are read with
// coalesced 16-byte loads, the predicate program runs on registers with
// wave-uniform control, and the qualifying rows come out as per-lane bit
// masks.  Waves are independent; nothing per row is stored by a plain
// count.  A count that precedes a materialization also stores, per wave
// tile, its qualifying-row count and every lane's truth mask (1/32 of the
// bytes of one 4-byte column), which the write pass (esc_materialize.hip)
// reads instead of the predicate's columns.
#include "esc_count_kernel.h"

namespace esc {

// Rows per lane of a count (ESC_COUNT_VARIANT selects a variant, for
// comparisons).  variant 0: 16; variant 1: 32 for programs of up to four
// column slots, 16 above; variant 2: 8 for plain counts (variant 1 for
// counts that store tiles); variant 3: variant 1 when the count stores its
// tiles for a materialization, else 32 for one or two columns and 16 for
// more, with twice the blocks for one column; variant 4 (the default):
// plain counts as variant 3 except that programs longer than one test per
// column keep 32, and counts that store tiles run 32 up to six columns.
// Measured on the 60M-row star table: plain counts 6.05 TB/s back to back
// with variant 3 against 5.9 for variant 1 (one-column counts 5.2 against
// 4.8); counts that store tiles with 16 rows per lane store twice the mask
// bytes and give the offset scan twice the tiles (154 against 145 us per
// count).
static int rows_per_lane(int variant, int k, int ninsn, bool tiles)
{
    if (variant == 2 && !tiles) return 8;
    if (variant == 3 && !tiles) return k <= 2 ? 32 : 16;
    // plain counts of three or more columns: 16 rows per lane when the
    // program is one test per column; longer programs are interpreted once
    // per wave tile and keep 32 rows per lane to spread that over more rows
    if (variant == 4 && !tiles) return k <= 2 || ninsn > k ? 32 : 16;
    // counts that store tiles (variant 4): 32 rows per lane up to six
    // columns (at one wave per SIMD their values fit in registers: 280 and
    // 316 VGPRs for five and six), so the offset scan and the write pass
    // handle half the tiles
    return variant == 0 || k > (tiles && variant == 4 ? 6 : 4) ? 16 : 32;
}

// Plain counts of tables of few tiles take fewer rows per lane (variant 4),
// down to 8, while there are fewer than two tiles a CU: a wave's time is then
// the call's, and it interprets its program on all of its rows.  The Section 1
// selection with its udf on 100,000 rows 21.9 -> 17.9 us, 700,000 22.1 ->
// 19.0, 1M 21.5 -> 19.0, most of it of this rule.  With the line at 1.5 tiles
// a CU 1M rows stay at 21.1; at 3, 700,000 rows of the star table run in two
// rounds (eight selections 150 us, 136 here).  Counts that store tiles keep
// theirs: eight selections of 100,000 rows 184 us, 193 with half the rows per
// lane.
int count_rpt(int variant, int k, int ninsn, bool tiles, int64_t nrows, int cus)
{
    int rpt = rows_per_lane(variant, k, ninsn, tiles);
    if (variant != 4 || tiles) return rpt;
    while (rpt > 8 && (nrows + 64 * rpt - 1) / (64 * rpt) < 2 * (int64_t)cus) rpt /= 2;
    return rpt;
}

// blocks of four waves per CU; one-column counts run two to keep enough
// loads in flight (variant 3: plain counts only; variant 4: also counts
// that store tiles)
int count_bpc(int variant, int k, int bpc, bool tiles)
{
    if (k > 1 || variant < 3 || (tiles && variant == 3)) return bpc;
    return 2 * bpc;
}

CountFn count_fn(int k, int rpt, bool udf, bool tiles)
{
    // counts that store tiles run 16 or 32 rows per lane (count_rpt)
    if (tiles) return rpt == 16 ? count_table<16, true, false>(k, udf) : count_table<32, true, false>(k, udf);
    switch (rpt) {
    case 8: return count_table<8, false, false>(k, udf);
    case 16: return count_table<16, false, false>(k, udf);
    default: return count_table<32, false, false>(k, udf);
    }
}

}  // namespace esc
