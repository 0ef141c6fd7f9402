// Checks the numbers of blocks that the scans launch: the rules on sizes, and
// that a setting is followed wherever it is made.  Exit code 1 on a difference.
#include <stdio.h>

#include <algorithm>

#include "esc_grid.h"

using namespace esc;

static int bad = 0;

static void expect(const char *what, int64_t got, int64_t want)
{
    if (got != want) {
        printf("%s: %lld, expected %lld\n", what, (long long)got, (long long)want);
        bad = 1;
    }
}

int main()
{
    const int cus = 256;
    for (int64_t needed : {1, 255, 256, 257, 511, 512, 513, 5000})
        for (int per_cu : {1, 2, 3, 8}) {
            const int64_t plain = std::min<int64_t>(needed, (int64_t)cus * per_cu);
            expect("short count", count_grid(cus, per_cu, false, false, needed), plain);
            expect("long count", count_grid(cus, per_cu, false, true, needed), needed <= 512 ? needed : plain);
            // ESC_BLOCKS_PER_CU
            expect("set, short count", count_grid(cus, per_cu, true, false, needed), plain);
            expect("set, long count", count_grid(cus, per_cu, true, true, needed), plain);
        }
    for (int64_t tiles : {(int64_t)1, kOwnPrefixTiles - 1, kOwnPrefixTiles, kOwnPrefixTiles + 1, (int64_t)1000000}) {
        expect("own offsets", own_offsets(tiles, 0), tiles <= kOwnPrefixTiles);
        // ESC_MAT_BLOCKS_PER_CU: the scan's offsets, and its number of blocks
        for (int set : {1, 2, 5}) expect("set, own offsets", own_offsets(tiles, set), 0);
    }
    for (int64_t needed : {1, 255, 1024, 6144, 100000})
        for (bool sparse : {false, true}) {
            expect("write pass", write_grid(cus, 0, 6, sparse, needed), sparse ? std::min<int64_t>(needed, 4096) : needed);
            for (int set : {1, 2, 5, 9})
                expect("set, write pass", write_grid(cus, set, 6, sparse, needed), std::min<int64_t>(needed, 256 * std::min(set, 6)));
        }
    expect("few written", few_written(0, 64), 1);
    expect("few written", few_written(1, 64), 0);
    expect("few written", few_written(1562499, 100000000), 1);
    expect("few written", few_written(1562500, 100000000), 0);
    expect("dense rows", dense_rows(false, 7), 128);
    // ESC_DENSE_SHIFT
    for (int shift = 0; shift <= 12; shift++) expect("set, dense rows", dense_rows(true, shift), std::max(1, 1024 >> shift));
    if (!bad) printf("ok\n");
    return bad;
}
