// Checks the room that a batch's workspace keeps for indexes: whatever the
// sizes of the groups, those that are given room fit together with the
// programs of all others; groups of 16 predicates and more are never refused,
// nor the few with the largest indexes that a batch of few predicates may
// turn into, whose programs would take less than their index.  Exit code 1 on
// a difference.
#include <stdio.h>

#include <algorithm>
#include <random>

#include "esc_index.h"

using namespace esc;

int main()
{
    std::mt19937 rng(7);
    auto pick = [&](int lo, int hi) { return (int)(lo + rng() % (unsigned)(hi - lo + 1)); };
    long taken = 0, refused = 0;
    for (int trial = 0; trial < 20000; trial++) {
        const int tables = pick(1, 9), npreds = pick(1, 3000), cap = npreds + (pick(0, 1) ? pick(0, 2000) : 0);
        const int least = pick(0, 3) ? 1 : 16, most = pick(least, kIndexMaxPreds);
        IndexRoom room((size_t)cap, (size_t)npreds, (size_t)tables);
        size_t bytes = 0;
        for (int left = npreds; left >= least;) {
            const int n = pick(least, std::min(left, most));
            IndexGroup g{};
            g.nwords = pick(0, 1) ? kIndexMaxWords : 4 * pick(2, kIndexMaxWords / 4);
            if (room.take(g, n)) {
                bytes += 4 * (size_t)g.nwords + sizeof(IndexGroupRef);
                taken++;
            } else {
                if (n >= 16) { printf("a group of %d refused\n", n); return 1; }
                bytes += (size_t)n * sizeof(Program);
                refused++;
            }
            left -= n;
            if (bytes + (size_t)left * sizeof(Program) > index_room((size_t)cap, (size_t)tables)) {
                printf("%zu bytes and %d programs in %zu\n", bytes, left, index_room((size_t)cap, (size_t)tables));
                return 1;
            }
        }
    }
    // eight predicates of two tables, four in an index of the largest size each:
    // 17 KB of programs
    IndexRoom room(8, 8, 2);
    IndexGroup g{};
    g.nwords = kIndexMaxWords;
    if (!room.take(g, 4) || !room.take(g, 4)) { printf("few predicates refused\n"); return 1; }
    printf("ok %ld taken, %ld refused\n", taken, refused);
    return taken && refused ? 0 : 1;
}
