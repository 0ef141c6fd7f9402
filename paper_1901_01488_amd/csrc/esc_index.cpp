// esc_index.cpp -- builds the predicate index of a group of selections from
// their compiled programs (host only; esc_index.h says what it holds).
#include "esc_index.h"

#include <limits.h>
#include <string.h>

#include <algorithm>

#include "esc.h"

namespace esc {

namespace {

typedef std::vector<IndexInterval> Set;

void add_values(Set &s, int64_t lo, int64_t hi)
{
    s.push_back({(int32_t)lo, (int32_t)hi});
}

// sorted, disjoint, touching intervals joined
void normalize(Set &s)
{
    bool apart = true;
    for (size_t i = 1; apart && i < s.size(); i++) apart = (int64_t)s[i - 1].hi + 1 < s[i].lo;
    if (apart) return;
    std::sort(s.begin(), s.end(), [](const IndexInterval &a, const IndexInterval &b) { return a.lo < b.lo; });
    size_t n = 0;
    for (const IndexInterval &v : s) {
        if (n && (int64_t)v.lo <= (int64_t)s[n - 1].hi + 1) s[n - 1].hi = std::max(s[n - 1].hi, v.hi);
        else s[n++] = v;
    }
    s.resize(n);
}

Set intersect(const Set &a, const Set &b)
{
    Set out;
    for (size_t i = 0, j = 0; i < a.size() && j < b.size();) {
        const int32_t lo = std::max(a[i].lo, b[j].lo), hi = std::min(a[i].hi, b[j].hi);
        if (lo <= hi) out.push_back({lo, hi});
        if (a[i].hi < b[j].hi) i++;
        else j++;
    }
    return out;
}

// events by their upper 32 bits: a radix sort that skips the bytes all share
void sort_by_value(std::vector<uint64_t> &v, std::vector<uint64_t> &other)
{
    if (v.size() < 64) {
        std::sort(v.begin(), v.end());
        return;
    }
    uint32_t count[4][256] = {};
    for (uint64_t x : v)
        for (int b = 0; b < 4; b++) count[b][(x >> (32 + 8 * b)) & 255u]++;
    other.resize(v.size());
    for (int b = 0; b < 4; b++) {
        const int shift = 32 + 8 * b;
        if (count[b][(v[0] >> shift) & 255u] == v.size()) continue;
        uint32_t at = 0;
        for (uint32_t &c : count[b]) {
            const uint32_t n = c;
            c = at;
            at += n;
        }
        for (uint64_t x : v) other[count[b][(x >> shift) & 255u]++] = x;
        v.swap(other);
    }
}

float as_float(uint32_t u)
{
    float f;
    memcpy(&f, &u, 4);
    return f;
}

// the float values in [lo, hi] (IEEE comparisons: both zeros are one value)
void add_floats(Set &s, uint32_t lo_bits, uint32_t hi_bits)
{
    const float lo = as_float(lo_bits), hi = as_float(hi_bits);
    if (!(lo <= hi)) return;
    const int32_t a = lo == 0.0f ? float_key(0x80000000u) : float_key(lo_bits);
    const int32_t b = hi == 0.0f ? float_key(0u) : float_key(hi_bits);
    add_values(s, a, b);
}

// the values a test on a column accepts
bool accepted(const Insn &t, const Program &P, bool is_float, Set &s)
{
    const uint32_t *k = P.kpool + t.a;
    switch (t.op) {
    case T_RANGE_I32: {
        const int32_t hi = (int32_t)((uint32_t)t.a + (uint32_t)t.b);
        if (hi >= t.a) {
            add_values(s, t.a, hi);
        } else {   // the range wraps around
            add_values(s, t.a, INT32_MAX);
            add_values(s, INT32_MIN, hi);
        }
        return true;
    }
    case T_RANGE_F32: add_floats(s, (uint32_t)t.a, (uint32_t)t.b); return true;
    case T_IN_I32:
        for (int i = 0; i < t.b; i++) add_values(s, (int32_t)k[i], (int32_t)k[i]);
        return true;
    case T_IN_F32:
        for (int i = 0; i < t.b; i++) add_floats(s, k[i], k[i]);
        return true;
    case T_BITSET: {
        const uint32_t w[2] = {(uint32_t)t.b, (uint32_t)t.c};
        for (uint32_t h = 0; h < 2; h++)
            for (uint32_t m = w[h]; m; m &= m - 1u) {
                const int32_t v = (int32_t)((uint32_t)t.a + 32u * h + (uint32_t)__builtin_ctz(m));
                add_values(s, v, v);
            }
        return true;
    }
    case T_IN_HASH:   // bit equality with one of the entries; empty slots hold the list's first key
        for (int i = 0, empty = -1; i < kSlotTable; i++) {
            if (empty >= 0 && k[i] == k[empty]) continue;
            if (empty < 0 && i + 1 < kSlotTable && k[i] == k[i + 1]) empty = i;
            const int32_t v = is_float ? float_key(k[i]) : (int32_t)k[i];
            add_values(s, v, v);
        }
        return true;
    case T_IN_BITMAP:
        for (uint32_t w = 0; w < kSlotTable; w++)
            for (uint32_t m = k[w]; m; m &= m - 1u) {
                const int32_t v = (int32_t)((uint32_t)t.b + 32u * w + (uint32_t)__builtin_ctz(m));
                add_values(s, v, v);
            }
        return true;
    }
    return false;
}

}  // namespace

void IndexSource::add(const Program &P, const int32_t *dtypes)
{
    const size_t nl = leaves.size(), ni = intervals.size();
    int nor = 0;
    bool ok = !(P.flags & (P_HAS_UDF | P_ALWAYS_TRUE | P_ALWAYS_FALSE));
    Set *and_set = scratch, *clause = scratch + kMaxSlots;   // per slot: the values its single-column clauses
    bool has_and[kMaxSlots] = {};                            // leave, and those of the open clause
    auto put = [&](int slot, int layer, const Set &s) {
        const int i0 = (int)intervals.size();
        intervals.insert(intervals.end(), s.begin(), s.end());
        leaves.push_back({P.slot_col[slot], layer, i0, (int)intervals.size()});
    };
    for (int i = 0; ok && i < P.ninsn;) {
        bool used[kMaxSlots] = {};
        for (; ok && i < P.ninsn; i++) {
            const Insn &t = P.insn[i];
            if (t.op >= U_LOAD || (t.flags & F_SRC_UDF) || t.src >= P.nslots) {
                ok = false;
                break;
            }
            if (!used[t.src]) clause[t.src].clear();
            used[t.src] = true;
            ok = accepted(t, P, dtypes[P.slot_col[t.src]] == ESC_FLOAT32, clause[t.src]);
            if (t.flags & (F_END_CLAUSE | F_SINGLE)) {
                i++;
                break;
            }
        }
        if (!ok) break;
        int nused = 0, last = 0;
        for (int s = 0; s < P.nslots; s++)
            if (used[s]) {
                normalize(clause[s]);
                nused++;
                last = s;
            }
        if (nused == 1) {
            if (has_and[last]) and_set[last] = intersect(and_set[last], clause[last]);
            else and_set[last].swap(clause[last]);
            has_and[last] = true;
        } else {
            for (int s = 0; s < P.nslots; s++)
                if (used[s]) put(s, nor, clause[s]);
            nor++;
        }
    }
    if (ok) {
        for (int s = 0; s < P.nslots; s++)
            if (has_and[s]) put(s, -1, and_set[s]);
        preds.push_back({nor, (int)nl, (int)leaves.size()});
    } else {
        leaves.resize(nl);
        intervals.resize(ni);
        preds.push_back({-1, (int)nl, (int)nl});
    }
}

void index_order(const IndexSource &src, std::vector<int> &order, bool by_columns)
{
    if (!by_columns) {
        std::stable_sort(order.begin(), order.end(),
                         [&](int x, int y) { return src.preds[x].nor < src.preds[y].nor; });
        return;
    }
    int64_t width[64] = {};   // intervals by column
    int bit[64], by_width[64];
    for (int i : order)
        for (int l = src.preds[i].l0; l < src.preds[i].l1; l++)
            width[src.leaves[l].col] += 1 + src.leaves[l].i1 - src.leaves[l].i0;
    for (int c = 0; c < 64; c++) by_width[c] = c;
    std::stable_sort(by_width, by_width + 64, [&](int a, int b) { return width[a] > width[b]; });
    for (int k = 0; k < 64; k++) bit[by_width[k]] = 63 - k;
    struct Key { uint64_t rank; int nor, pred; };
    std::vector<Key> keys;
    keys.reserve(order.size());
    for (int i : order) {
        uint64_t r = 0;
        for (int l = src.preds[i].l0; l < src.preds[i].l1; l++) r |= 1ull << bit[src.leaves[l].col];
        for (int s = 1; s < 64; s *= 2) r ^= r >> s;   // position in Gray code
        keys.push_back({r, src.preds[i].nor, i});
    }
    std::stable_sort(keys.begin(), keys.end(),
                     [](const Key &a, const Key &b) { return a.nor != b.nor ? a.nor < b.nor : a.rank < b.rank; });
    for (size_t k = 0; k < keys.size(); k++) order[k] = keys[k].pred;
}

bool build_index(const IndexSource &src, const int *member, int n, const int32_t *dtypes, IndexGroup &g,
                 std::vector<uint32_t> &blob)
{
    memset(&g, 0, sizeof g);
    if (n < 1 || n > kIndexMaxPreds) return false;
    g.words = n <= 32 ? 1 : n <= 64 ? 2 : 4;
    // OR layers: as many for each result word as its predicates' most
    int layer0[kIndexMaxPreds / 32] = {};   // record word of a result word's first layer
    for (int w = 0; w < g.words; w++) {
        int most = 0;
        for (int i = 32 * w; i < std::min(n, 32 * w + 32); i++) most = std::max(most, src.preds[member[i]].nor);
        if (g.words + g.nor + most > kIndexMaxRec) return false;
        layer0[w] = g.words + g.nor;
        for (int j = 0; j < most; j++) g.or_word[g.nor++] = (uint8_t)w;
    }
    g.rec = g.words + g.nor <= 2 ? 2 : g.words + g.nor <= 4 ? 4 : 8;

    // the leaves by column
    struct Item { int32_t next, leaf, pos; };   // pos: member position
    std::vector<Item> items;
    int col_of[kIndexMaxCols], head[kIndexMaxCols], slot_of_col[64];
    for (int c = 0; c < 64; c++) slot_of_col[c] = -1;
    for (int i = 0; i < n; i++) {
        const IndexPred &p = src.preds[member[i]];
        if (p.nor < 0) return false;
        for (int l = p.l0; l < p.l1; l++) {
            const int c = src.leaves[l].col;
            if (slot_of_col[c] < 0) {
                if (g.ncols == kIndexMaxCols) return false;
                slot_of_col[c] = g.ncols;
                col_of[g.ncols] = c;
                head[g.ncols++] = -1;
            }
            int &h = head[slot_of_col[c]];
            items.push_back({h, l, i});
            h = (int)items.size() - 1;
        }
    }
    if (g.ncols == 0) return false;

    const size_t blob0 = blob.size();
    // a column's events: at value v the bit `pos` of record word w flips
    // (v above the word and position, so that they sort by v)
    std::vector<uint64_t> event, other;
    const int R = g.rec;
    for (int k = 0; k < g.ncols; k++) {
        IndexColumn &C = g.cols[k];
        C.col = col_of[k];
        C.is_float = dtypes[C.col] == ESC_FLOAT32;
        event.clear();
        uint32_t first[kIndexMaxRec];   // record of the values below every cut
        for (int w = 0; w < R; w++) first[w] = ~0u;   // no condition on this column; layers: not through this column
        if (k == 0)
            for (int i = 0; i < n; i++) {
                // a predicate without some layer of its word passes it
                const int w = i >> 5;
                for (int j = src.preds[member[i]].nor; layer0[w] + j < g.words + g.nor; j++) {
                    const int at = layer0[w] + j;
                    if (g.or_word[at - g.words] != w) break;
                    first[at] &= ~(1u << (i & 31));
                }
            }
        for (int i = head[k]; i >= 0; i = items[i].next) {
            const IndexLeaf &L = src.leaves[items[i].leaf];
            const int pos = items[i].pos;
            const int w = L.layer < 0 ? pos >> 5 : layer0[pos >> 5] + L.layer;
            const uint32_t bit = 1u << (pos & 31);
            if (L.layer < 0) first[w] ^= bit;   // holds only inside its intervals
            const uint64_t flip = (uint64_t)(w * 32 + (pos & 31));
            for (int j = L.i0; j < L.i1; j++) {
                const IndexInterval &v = src.intervals[j];
                if (v.lo == INT32_MIN) first[w] ^= bit;
                else event.push_back((uint64_t)((uint32_t)v.lo ^ 0x80000000u) << 32 | flip);
                if (v.hi != INT32_MAX) event.push_back((uint64_t)((uint32_t)(v.hi + 1) ^ 0x80000000u) << 32 | flip);
            }
        }
        sort_by_value(event, other);
        int m = 0;   // cuts: distinct event values
        for (size_t i = 0; i < event.size(); i++) m += i == 0 || event[i] >> 32 != event[i - 1] >> 32;
        int s = 2;
        while ((1 << s) - 1 < m) s++;
        const int size = 1 << s;
        if (s > kIndexMaxLevels || g.nwords + size * (1 + R) > kIndexMaxWords) {
            blob.resize(blob0);
            return false;
        }
        C.levels = s;
        C.key_off = g.nwords;
        C.rec_off = g.nwords + size;
        g.nwords += size * (1 + R);
        blob.resize(blob0 + g.nwords);
        // record e: values with exactly e cuts at or below them
        int32_t *key = (int32_t *)&blob[blob0 + C.key_off];
        uint32_t *out = &blob[blob0 + C.rec_off];
        memcpy(out, first, R * sizeof(uint32_t));
        int32_t cut[1 << kIndexMaxLevels];
        size_t i = 0;
        for (int e = 1; e < size; e++) {
            memcpy(out + (size_t)e * R, out + (size_t)(e - 1) * R, R * sizeof(uint32_t));
            if (e > m) {   // beyond the last cut: INT32_MAX, which both sides of it may reach
                cut[e - 1] = INT32_MAX;
                continue;
            }
            const uint64_t v = event[i] >> 32;
            cut[e - 1] = (int32_t)((uint32_t)v ^ 0x80000000u);
            for (; i < event.size() && event[i] >> 32 == v; i++) {
                const uint32_t flip = (uint32_t)event[i];
                out[(size_t)e * R + (flip >> 5)] ^= 1u << (flip & 31u);
            }
        }
        // tree nodes in breadth-first order
        key[0] = INT32_MAX;
        for (int lev = 0, node = 1; lev < s; lev++)
            for (int p = 0; p < (1 << lev); p++, node++) key[node] = cut[((2 * p + 1) << (s - lev - 1)) - 1];
    }
    return true;
}

int cut_group(const IndexSource &src, const int *member, int n, const int32_t *dtypes, IndexGroup &g,
              std::vector<uint32_t> &blob)
{
    while (n > 0 && !build_index(src, member, n, dtypes, g, blob)) n = n > 32 ? std::max(32, n / 64 * 32) : n / 2;
    return n;
}

}  // namespace esc
