// Checks the order in which predicates are cut into groups: a permutation, in
// ascending order of OR clauses, with equal sets of columns together among
// equals, and fewer columns to search in groups of 128 than in the given
// order.  Exit code 1 on a difference.
#include <stdio.h>

#include <algorithm>
#include <random>
#include <set>
#include <vector>

#include "esc.h"
#include "esc_index.h"

using namespace esc;

static uint64_t columns(const IndexSource &s, int i)
{
    uint64_t m = 0;
    for (int l = s.preds[i].l0; l < s.preds[i].l1; l++) m |= 1ull << s.leaves[l].col;
    return m;
}

static int searched(const IndexSource &s, const std::vector<int> &order)
{
    int n = 0;
    for (size_t i = 0; i < order.size(); i += kIndexMaxPreds) {
        uint64_t m = 0;
        for (size_t j = i; j < std::min(order.size(), i + kIndexMaxPreds); j++) m |= columns(s, order[j]);
        n += __builtin_popcountll(m);
    }
    return n;
}

int main()
{
    std::mt19937 rng(99);
    for (int n : {1, 2, 127, 128, 129, 500, 2048}) {
        for (int ncols : {1, 6, 16, 64}) {
            IndexSource s;
            std::vector<int> plain;
            for (int i = 0; i < n; i++) {
                const int l0 = (int)s.leaves.size(), k = 1 + (int)(rng() % 4);
                for (int j = 0; j < k; j++) {
                    const int i0 = (int)s.intervals.size();
                    s.intervals.resize(i0 + 1 + rng() % 3);
                    s.leaves.push_back({(int)(rng() % ncols), -1, i0, (int)s.intervals.size()});
                }
                s.preds.push_back({rng() % 2 ? 0 : (int)(rng() % 3), l0, (int)s.leaves.size()});
                plain.push_back(i);
            }
            std::stable_sort(plain.begin(), plain.end(), [&](int x, int y) { return s.preds[x].nor < s.preds[y].nor; });
            for (bool by_columns : {false, true}) {
                std::vector<int> order;
                for (int i = 0; i < n; i++) order.push_back(i);
                index_order(s, order, by_columns);
                if (!by_columns && order != plain) { printf("not the plain order\n"); return 1; }
                std::vector<int> sorted = order;
                std::sort(sorted.begin(), sorted.end());
                std::set<std::pair<int, uint64_t>> done;
                for (int i = 0; i < n; i++) {
                    if (sorted[i] != i) { printf("not a permutation\n"); return 1; }
                    if (i && s.preds[order[i]].nor < s.preds[order[i - 1]].nor) { printf("OR clauses not ascending\n"); return 1; }
                    if (!by_columns) continue;
                    const std::pair<int, uint64_t> key(s.preds[order[i]].nor, columns(s, order[i]));
                    const bool same = i && s.preds[order[i - 1]].nor == key.first && columns(s, order[i - 1]) == key.second;
                    if (!same && !done.insert(key).second) { printf("a set of columns is apart\n"); return 1; }
                }
                if (by_columns && n >= 500 && ncols == 6 && searched(s, order) >= searched(s, plain)) {
                    printf("%d columns searched, %d in the plain order\n", searched(s, order), searched(s, plain));
                    return 1;
                }
            }
        }
    }
    printf("ok\n");
    return 0;
}
