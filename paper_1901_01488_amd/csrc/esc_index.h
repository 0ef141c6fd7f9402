// esc_index.h -- predicate index of a group of selections on one table,
// shared by the host planner of the batch and the gfx950 kernel.
//
// A group's predicates together cut every column into elementary intervals
// inside which no leaf changes its value.  The index of a column holds the
// sorted interval boundaries and, per interval, a record of bit masks: bit p
// says whether predicate p's condition on that column holds there.  Counting
// a row then costs one search and one record per column, whatever the number
// of predicates, instead of running every program on it:
//   result words  = AND over the columns of the records' AND words (bit p is
//                   set when p has no single-column clause on that column);
//   OR clauses over several columns live in extra words ("layers"): layer
//                   bit p is the complement of "p's clause holds through this
//                   column", so the same AND over columns leaves the
//                   complement of the clause.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <vector>

#include "esc_program.h"

namespace esc {

constexpr int kIndexMaxPreds = 128;   // predicates of a group: four 32-bit result words
constexpr int kIndexMaxCols = 16;     // columns of a group
constexpr int kIndexMaxRec = 8;       // words of a record
constexpr int kIndexMaxLevels = 10;   // levels of a column's search tree
// words of a group's index: two blocks of 512 threads share a CU's 160 KiB of LDS
constexpr int kIndexMaxWords = 19 * 1024;

struct IndexColumn {
    int32_t col;        // table column
    int32_t is_float;   // values are float32: compared through their order-preserving int32 image
    int32_t levels;     // the tree has 2^levels - 1 boundaries, the column 2^levels records
    int32_t key_off;    // word offset of the tree (in breadth-first order from word 1)
    int32_t rec_off;    // word offset of the records
};

struct IndexGroup {
    int32_t words;      // result words: 1, 2 or 4
    int32_t rec;        // words of a record: the result words, then the OR layers (2, 4 or 8)
    int32_t nor;        // OR layers in use
    int32_t ncols;
    int32_t nwords;     // words of the whole index
    uint8_t or_word[kIndexMaxRec];   // result word of each OR layer
    IndexColumn cols[kIndexMaxCols];
};

// Accepted values of a leaf: disjoint, ascending, inclusive intervals.
struct IndexInterval {
    int32_t lo, hi;
};

struct IndexLeaf {
    int32_t col;
    int32_t layer;      // -1: a clause on this column alone; else which OR clause of the predicate
    int32_t i0, i1;     // intervals
};

struct IndexPred {
    int32_t nor;        // OR clauses over several columns; -1: cannot be indexed (a udf)
    int32_t l0, l1;     // leaves
};

// The predicates of a batch as intervals.
struct IndexSource {
    std::vector<IndexPred> preds;
    std::vector<IndexLeaf> leaves;
    std::vector<IndexInterval> intervals;
    // appends P (nor = -1 when its conditions are not intervals of single columns)
    void add(const Program &P, const int32_t *dtypes);

private:
    std::vector<IndexInterval> scratch[2 * kMaxSlots];
};

// order-preserving int32 image of a float's bits (-0 directly below +0, NaNs
// beyond the infinities)
inline int32_t float_key(uint32_t bits)
{
    return (int32_t)(bits ^ (uint32_t)(((int32_t)bits >> 31) & 0x7fffffff));
}

// The same group as the kernel reads it (device memory).
struct IndexColumnRef {
    const uint32_t *ptr;
    uint32_t key_byte, rec_byte;   // byte offsets in the group's index
    int32_t levels, is_float;
};

struct IndexGroupRef {
    int32_t words, rec, nor, ncols;
    int32_t nwords;
    uint32_t blob;      // word offset of the index among all groups' indexes
    int32_t npred;
    int32_t pbegin;     // first entry of the group's predicate ids
    uint8_t or_word[kIndexMaxRec];
    IndexColumnRef cols[kIndexMaxCols];
};

// Orders source predicates (positions in src.preds, none with nor = -1) for
// being cut into groups: by their OR clauses, so that predicates with as many
// of them share the extra record words, and, when there are several groups,
// so that neighbours condition on much the same columns, since a group
// searches every column that one of its predicates names.  The sets of columns
// follow each other in Gray code, the columns with the most intervals as its
// upper bits: groups agree on those.  2,048 predicates of one to four
// conjuncts on a table of six columns: 102 columns in 17 groups before, 79
// after, and the kernel takes 1,305 us on 10M rows, 1,505 before.
void index_order(const IndexSource &src, std::vector<int> &order, bool by_columns);

// The index of source predicates member[0 .. n) (in ascending order of nor),
// bit i of the result words standing for member[i].  Appends g.nwords words
// to blob; false (and blob as before) when the group does not fit the limits
// above.
bool build_index(const IndexSource &src, const int *member, int n, const int32_t *dtypes, IndexGroup &g,
                 std::vector<uint32_t> &blob);

// The bytes of a workspace that hold programs and indexes: for each of the
// predicates it was sized for the sixteenth of a largest index and its group
// (more than a program takes), and a largest index for every table and one more.  A group
// that is given room leaves every other predicate its own, so the indexes a
// plan chooses always fit, whichever predicates an update brings; groups of 16
// and more always find room.
constexpr size_t kIndexPredBytes = (kIndexMaxWords * 4 + 512) / 16;
static_assert(kIndexPredBytes >= sizeof(Program), "a predicate's share holds its program");
static_assert(sizeof(IndexGroupRef) <= 512, "16 predicates' shares hold a largest index and its group");

inline size_t index_room(size_t npreds, size_t ntables)
{
    return npreds * kIndexPredBytes + (ntables + 1) * kIndexMaxWords * 4;
}

struct IndexRoom {
    int64_t left;   // beside the shares of the predicates without an index
    // of a workspace for cap predicates, when npreds are counted
    IndexRoom(size_t cap, size_t npreds, size_t ntables)
        : left((int64_t)index_room(cap, ntables) - (int64_t)(npreds * kIndexPredBytes)) {}
    // room for an index of g over n predicates, if there is; their shares go to it
    bool take(const IndexGroup &g, int n)
    {
        const int64_t after = left + n * (int64_t)kIndexPredBytes - 4 * (int64_t)g.nwords - (int64_t)sizeof(IndexGroupRef);
        if (after < 0) return false;
        left = after;
        return true;
    }
};

// The index of as many of member[0 .. n) as fit one, from the first on: all
// of them, else whole 32s, else halves; their number, 0 if none fits (and blob
// as before).  Fewer predicates need fewer boundaries, columns and layers.
int cut_group(const IndexSource &src, const int *member, int n, const int32_t *dtypes, IndexGroup &g,
              std::vector<uint32_t> &blob);

}  // namespace esc
