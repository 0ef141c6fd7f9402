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

}  // namespace esc
