// Checks how a list of predicates is cut into groups with an index each:
// every predicate that fits an index by itself lands in a group, whatever the
// length of the list, and groups are as large as the way of cutting promises.
// Predicates whose groups hold at most 32 by their OR layers, and predicates
// of many constants on one column, whose groups hold few by their cuts.
#include <stdio.h>

#include <algorithm>
#include <random>
#include <vector>

#include "esc.h"
#include "esc_host.h"
#include "esc_index.h"

using namespace esc;

static std::mt19937 rng(99);

static const int kCols = 4;
static const int32_t kTypes[kCols] = {ESC_INT32, ESC_INT32, ESC_INT32, ESC_INT32};

static bool add(const esc_table *schema, const std::vector<esc_node> &nodes, const std::vector<int32_t> &values,
                IndexSource &src)
{
    std::vector<esc_const> consts;
    for (int32_t v : values) {
        esc_const c{};
        c.dtype = ESC_INT32;
        c.v.i = v;
        consts.push_back(c);
    }
    esc_pred *p = nullptr;
    if (esc_compile_predicate(schema, nodes.data(), (int)nodes.size(), consts.data(), (int)consts.size(), nullptr, 0, &p))
        return false;
    src.add(p->prog, kTypes);
    esc_pred_destroy(p);
    return true;
}

// four ORs, each over two columns
static bool add_ors(const esc_table *schema, IndexSource &src)
{
    std::vector<esc_node> nodes;
    std::vector<int32_t> values;
    esc_node root{};
    root.op = ESC_AND;
    root.nchild = 4;
    nodes.push_back(root);
    for (int i = 0; i < 4; i++) {
        esc_node o{};
        o.op = ESC_OR;
        o.nchild = 2;
        nodes.push_back(o);
        for (int c = 0; c < 2; c++) {
            esc_node leaf{};
            leaf.op = ESC_LT;
            leaf.col = (i + c) % kCols;
            leaf.k0 = (int)values.size();
            values.push_back((int32_t)(rng() % 20) * 10);
            nodes.push_back(leaf);
        }
    }
    return add(schema, nodes, values, src);
}

// an IN-list of 20 constants far apart: 40 cuts
static bool add_list(const esc_table *schema, IndexSource &src)
{
    std::vector<esc_node> nodes;
    std::vector<int32_t> values;
    esc_node leaf{};
    leaf.op = ESC_IN;
    leaf.k1 = 20;
    for (int i = 0; i < 20; i++) values.push_back((int32_t)rng());
    nodes.push_back(leaf);
    return add(schema, nodes, values, src);
}

int main()
{
    esc_table *schema = nullptr;
    if (esc_table_create(0, kCols, kTypes, nullptr, &schema)) return 2;
    long groups = 0;
    for (int kind = 0; kind < 2; kind++) {
        IndexSource src;
        for (int i = 0; i < 300; i++) {
            if (!(kind == 0 ? add_ors(schema, src) : add_list(schema, src))) return 2;
            if (src.preds.back().nor != (kind == 0 ? 4 : 0)) { printf("not the predicate meant\n"); return 1; }
        }
        std::vector<int> member;
        for (int i = 0; i < 300; i++) member.push_back(i);
        for (int n = 1; n <= 300; n++) {
            std::vector<uint32_t> blob(4, 7u);
            for (int at = 0; at < n;) {
                IndexGroup g;
                const size_t blob0 = blob.size();
                const int left = std::min(n - at, kIndexMaxPreds);
                const int m = cut_group(src, &member[at], left, kTypes, g, blob);
                if (m < 1 || m > left || blob.size() != blob0 + (size_t)g.nwords) {
                    printf("kind %d, %d predicates: %d of %d at %d\n", kind, n, m, left, at);
                    return 1;
                }
                // 32 with four layers fit; 25 lists of 40 cuts do, and a list is halved at most to 8 of them
                if (m < std::min(left, kind == 0 ? 32 : 8)) {
                    printf("kind %d, %d predicates: a group of %d of %d\n", kind, n, m, left);
                    return 1;
                }
                groups++;
                at += m;
            }
        }
    }
    esc_table_destroy(schema);
    printf("ok %ld groups\n", groups);
    return 0;
}
