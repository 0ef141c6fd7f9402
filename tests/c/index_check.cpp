// Checks the predicate index of a batch against direct evaluation of the
// compiled programs, on the CPU: random trees over int, date and float columns
// (ranges, IN-lists of every compiled form, ORs over one and several columns),
// groups of the sizes given on the command line, rows around every constant
// and at the extremes.  Prints what it covered; exit code 1 on a difference.
#include <limits.h>
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <random>
#include <vector>

#include "esc.h"
#include "esc_host.h"
#include "esc_index.h"

using namespace esc;

static std::mt19937 rng(12345);
static int pick(int lo, int hi) { return (int)(lo + rng() % (unsigned)(hi - lo + 1)); }

static float bits_f(uint32_t u) { float f; memcpy(&f, &u, 4); return f; }
static uint32_t f_bits(float f) { uint32_t u; memcpy(&u, &f, 4); return u; }

// one test of a compiled program on a stored value
static bool test(const Insn &t, const uint32_t *pool, uint32_t x)
{
    const uint32_t *k = pool + t.a;
    const float f = bits_f(x);
    switch (t.op) {
    case T_RANGE_I32: return x - (uint32_t)t.a <= (uint32_t)t.b;
    case T_RANGE_F32: return bits_f((uint32_t)t.a) <= f && f <= bits_f((uint32_t)t.b);
    case T_IN_I32: for (int i = 0; i < t.b; i++) if (x == k[i]) return true; return false;
    case T_IN_F32: for (int i = 0; i < t.b; i++) if (f == bits_f(k[i])) return true; return false;
    case T_BITSET: {
        const uint32_t d = x - (uint32_t)t.a;
        return d < 64 && (((uint64_t)(uint32_t)t.c << 32 | (uint32_t)t.b) >> d & 1);
    }
    case T_IN_HASH: {
        const uint32_t h = (uint32_t)t.b;
        const uint32_t rot = h && h < 32 ? x >> h | x << (32 - h) : x;
        return k[h < 32 ? (rot >> 2) & 63 : (x * h) >> 26] == x;
    }
    case T_IN_BITMAP: {
        const uint32_t d = x - (uint32_t)t.b;
        return d < 2048 && (k[d >> 5] >> (d & 31) & 1);
    }
    }
    abort();
}

static bool evaluate(const Program &P, const uint32_t *row)
{
    bool acc = true, clause = false;
    for (int i = 0; i < P.ninsn; i++) {
        const Insn &t = P.insn[i];
        const bool m = test(t, P.kpool, row[P.slot_col[t.src]]);
        if (t.flags & F_SINGLE) acc = acc && m;
        else {
            clause = clause || m;
            if (t.flags & F_END_CLAUSE) { acc = acc && clause; clause = false; }
        }
    }
    return acc;
}

static bool by_index(const IndexGroup &g, const uint32_t *blob, const uint32_t *row, int bit)
{
    uint32_t acc[kIndexMaxRec];
    for (uint32_t &a : acc) a = ~0u;
    for (int c = 0; c < g.ncols; c++) {
        const IndexColumn &C = g.cols[c];
        const int32_t v = C.is_float ? float_key(row[C.col]) : (int32_t)row[C.col];
        uint32_t i = 1;
        for (int l = 0; l < C.levels; l++) i = 2 * i + (v >= (int32_t)blob[C.key_off + i]);
        const uint32_t e = i - (1u << C.levels);
        for (int w = 0; w < g.rec; w++) acc[w] &= blob[C.rec_off + e * g.rec + w];
    }
    for (int j = 0; j < g.nor; j++) acc[g.or_word[j]] &= ~acc[g.words + j];
    return acc[bit >> 5] >> (bit & 31) & 1;
}

static const int kCols = 6;
static const int32_t kTypes[kCols] = {ESC_INT32, ESC_DATE32, ESC_FLOAT32, ESC_INT32, ESC_FLOAT32, ESC_INT32};
static const float kFloats[] = {0.0f, -0.0f, 1e-45f, -1e-45f, INFINITY, -INFINITY, NAN, 1.0f, -1.0f, 3.4e38f, -3.4e38f};

static uint32_t constant(int col, std::vector<uint32_t> *seen)
{
    uint32_t b;
    if (kTypes[col] == ESC_FLOAT32) {
        b = pick(0, 3) == 0 ? f_bits(kFloats[pick(0, 10)]) : f_bits((float)pick(-2000, 2000) / 16.0f);
    } else {
        switch (pick(0, 9)) {
        case 0: b = (uint32_t)INT32_MIN + (uint32_t)pick(0, 2); break;
        case 1: b = (uint32_t)INT32_MAX - (uint32_t)pick(0, 2); break;
        case 2: b = (uint32_t)rng(); break;
        case 3: case 4: b = (uint32_t)pick(-3000, 3000); break;
        default: b = (uint32_t)pick(0, col == 3 ? 12 : 200); break;
        }
    }
    seen[col].push_back(b);
    return b;
}

struct Tree {
    std::vector<esc_node> nodes;
    std::vector<esc_const> consts;
};

static void leaf(Tree &t, int col, std::vector<uint32_t> *seen)
{
    esc_node n{};
    const int ops[] = {ESC_EQ, ESC_LT, ESC_GT, ESC_BETWEEN, ESC_BETWEEN, ESC_IN};
    n.op = ops[pick(0, 5)];
    n.col = col;
    auto add = [&](uint32_t b) {
        esc_const c{};
        c.dtype = kTypes[col];
        c.v.bits = b;
        t.consts.push_back(c);
        return (int)t.consts.size() - 1;
    };
    n.k0 = add(constant(col, seen));
    if (n.op == ESC_BETWEEN) n.k1 = add(constant(col, seen));
    if (n.op == ESC_IN) {
        n.k1 = pick(1, pick(0, 3) ? 6 : 40);
        const bool near = kTypes[col] != ESC_FLOAT32 && pick(0, 1);
        for (int i = 1; i < n.k1; i++) {
            uint32_t b = constant(col, seen);
            if (near) seen[col].push_back(b = t.consts[n.k0].v.bits + (uint32_t)pick(0, pick(0, 1) ? 60 : 1900));
            add(b);
        }
    }
    t.nodes.push_back(n);
}

int main(int argc, char **argv)
{
    esc_table *schema = nullptr;
    if (esc_table_create(0, kCols, kTypes, nullptr, &schema)) return 2;
    long checks = 0, groups = 0, refused = 0, layers = 0, ops[8] = {};
    for (int a = 1; a < argc; a++) {
        const int n = atoi(argv[a]);
        for (int trial = 0; trial < 12; trial++) {
            const int p_or = trial % 4;   // OR clauses: none, few, many
            std::vector<uint32_t> seen[kCols];
            std::vector<esc_pred *> preds;
            IndexSource src;
            while ((int)preds.size() < n) {
                Tree t;
                const int k = pick(1, 4);
                esc_node root{};
                root.op = ESC_AND;
                root.nchild = k;
                t.nodes.push_back(root);
                for (int i = 0; i < k; i++) {
                    if (pick(0, 5) < p_or) {
                        esc_node o{};
                        o.op = ESC_OR;
                        o.nchild = pick(2, 3);
                        t.nodes.push_back(o);
                        const int col = pick(0, kCols - 1), one = pick(0, 2) == 0;
                        for (int j = 0; j < o.nchild; j++) leaf(t, one ? col : pick(0, kCols - 1), seen);
                    } else {
                        leaf(t, pick(0, kCols - 1), seen);
                    }
                }
                esc_pred *p = nullptr;
                if (esc_compile_predicate(schema, t.nodes.data(), (int)t.nodes.size(), t.consts.data(),
                                          (int)t.consts.size(), nullptr, 0, &p)) continue;
                if (p->prog.flags & (P_ALWAYS_TRUE | P_ALWAYS_FALSE)) { esc_pred_destroy(p); continue; }
                for (int i = 0; i < p->prog.ninsn; i++) ops[p->prog.insn[i].op]++;
                preds.push_back(p);
                src.add(p->prog, kTypes);
            }
            std::vector<int> member;
            for (int i = 0; i < n; i++) {
                if (src.preds[i].nor < 0) { printf("predicate without udf not indexed\n"); return 1; }
                member.push_back(i);
            }
            std::stable_sort(member.begin(), member.end(), [&](int x, int y) { return src.preds[x].nor < src.preds[y].nor; });
            for (int at = 0; at < n;) {
                IndexGroup g;
                std::vector<uint32_t> blob(3, 7u);   // an index may follow others
                int m = std::min(n - at, kIndexMaxPreds);
                while (m && !build_index(src, &member[at], m, kTypes, g, blob)) {
                    if (blob.size() != 3) { printf("a refused group left words\n"); return 1; }
                    refused++;
                    m = m > 32 ? m / 64 * 32 : m / 2;
                }
                if (!m) { at++; continue; }
                if (blob.size() != 3 + (size_t)g.nwords) { printf("wrong size\n"); return 1; }
                groups++;
                layers += g.nor;
                std::vector<uint32_t> rows;
                for (int r = 0; r < 600; r++) {
                    uint32_t row[kCols];
                    for (int c = 0; c < kCols; c++) {
                        row[c] = seen[c].empty() || pick(0, 9) == 0 ? (uint32_t)rng() : seen[c][rng() % seen[c].size()];
                        if (kTypes[c] != ESC_FLOAT32 && pick(0, 2)) row[c] += (uint32_t)pick(-1, 1);
                        if (kTypes[c] == ESC_FLOAT32 && pick(0, 5) == 0) row[c] ^= 0x80000000u;
                        if (kTypes[c] == ESC_FLOAT32 && pick(0, 5) == 0) row[c] += (uint32_t)pick(-1, 1);
                    }
                    for (int i = 0; i < m; i++) {
                        checks++;
                        if (by_index(g, blob.data() + 3, row, i) != evaluate(preds[member[at + i]]->prog, row)) {
                            printf("differs: group of %d, predicate %d, nor %d\n", m, i, src.preds[member[at + i]].nor);
                            return 1;
                        }
                    }
                }
                at += m;
            }
            for (esc_pred *p : preds) esc_pred_destroy(p);
        }
    }
    esc_table_destroy(schema);
    printf("ok %ld checks, %ld groups, %ld refused, %ld layers, ops", checks, groups, refused, layers);
    for (int i = 0; i < 7; i++) {
        printf(" %ld", ops[i]);
        if (!ops[i]) { printf(" (an operation was not covered)\n"); return 1; }
    }
    printf("\n");
    return groups && layers && checks > 100000 ? 0 : 1;
}
