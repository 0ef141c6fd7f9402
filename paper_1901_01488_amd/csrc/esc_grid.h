// esc_grid.h -- how many blocks the scans launch (host only, no HIP): rules on
// sizes, and the settings that override them.
#pragma once
#include <stdint.h>

namespace esc {

// Blocks of a count: per_cu for each of cus CUs, at most the `needed` ones.
// Long plain programs (more instructions than columns) on tables of up to two
// blocks per CU run them all at once (2.2M rows of the Section 1 selection: 28.6
// us in two rounds, 23.5), unless ESC_BLOCKS_PER_CU says how many (set).
inline int64_t count_grid(int cus, int per_cu, bool set, bool long_plain, int64_t needed)
{
    int64_t grid = (int64_t)cus * per_cu;
    if (!set && long_plain && needed <= 2 * (int64_t)cus) grid = needed;
    return grid < needed ? grid : needed;
}

// Tiles up to which every block of the write pass finds its own offset (the
// sum of the counts before it, read from the L2s) and no scan is launched.
// The sums grow with tiles times blocks: counts and write passes of 0.05 % of
// the rows, one column, with the scan and without, 6M rows 21 and 18 us, 12M
// 28 and 26, 20M (9,766 tiles) 34 and 34, 28M 42 and 44, 40M 53 and 58.
constexpr int64_t kOwnPrefixTiles = 12288;

// Whether the blocks of the write pass find their own offsets: they then have to
// be as many as its units fill, so not where ESC_MAT_BLOCKS_PER_CU (mat_bpc)
// sets their number.
inline bool own_offsets(int64_t ntiles, int mat_bpc) { return mat_bpc <= 0 && ntiles <= kOwnPrefixTiles; }

// Blocks of the write pass for `needed` blocks' units, occ resident per CU.
// sparse: few_written().
inline int64_t write_grid(int cus, int mat_bpc, int occ, bool sparse, int64_t needed)
{
    int64_t grid = needed;
    if (mat_bpc > 0) grid = (int64_t)cus * (mat_bpc < occ ? mat_bpc : occ);
    else if (sparse) grid = 16 * (int64_t)cus;
    return grid < needed ? grid : needed;
}

// Whether the outputs have room for so few of the rows that most units hold
// little: then waves that go on to further units, their masks read ahead, cost
// less than a launch for each (with its count, 0.001 % of the rows, one column,
// 100M rows 96 us, 100 with a wave for each unit; 200M 188 and 197).
inline bool few_written(uint64_t capacity, int64_t nrows) { return capacity < (uint64_t)nrows / 64; }

// Qualifying rows from which the write pass takes a unit's columns whole:
// an eighth of its 1,024 rows (measured beside write_unit), or the fraction
// 2^-shift that ESC_DENSE_SHIFT sets.
constexpr int kUnitRows = 1024;

inline uint32_t dense_rows(bool set, int shift)
{
    if (!set) return kUnitRows / 8;
    const uint32_t rows = (uint32_t)kUnitRows >> shift;
    return rows ? rows : 1u;
}

}  // namespace esc
