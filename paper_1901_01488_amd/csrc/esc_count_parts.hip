// esc_count_parts.hip -- the plain counts of small tables whose blocks store
// their counts in host words of their own (esc_count_kernel.h).
#include "esc_count_kernel.h"

namespace esc {

CountFn count_parts_fn(int k, int rpt, bool udf)
{
    switch (rpt) {
    case 8: return count_table<8, false, true>(k, udf);
    case 16: return count_table<16, false, true>(k, udf);
    default: return count_table<32, false, true>(k, udf);
    }
}

}  // namespace esc
