// esc_host.h -- host-side objects behind the opaque handles of esc.h.
#pragma once
#include <stdint.h>

#include <string>
#include <vector>

#include "esc.h"
#include "esc_program.h"

struct esc_table {
    uint64_t id = 0;   // unique per table handle (never reused)
    int64_t nrows = 0;
    std::vector<int32_t> dtypes;
    std::vector<const void *> cols;   // empty for a schema-only table
    bool has_data() const { return !cols.empty(); }
};

struct esc_pred {
    uint64_t id = 0;   // unique per predicate handle (never reused)
    esc::Program prog{};
    int ncols_schema = 0;
    std::vector<int32_t> schema_dtypes;
    // the source tree, kept for featurization
    std::vector<esc_node> nodes;
    std::vector<esc_const> consts;
    std::vector<esc_udf_insn> udf;
    uint64_t col_mask = 0;
    int nhashed = 0;   // IN-lists compiled to slot tables
};

namespace esc {

// thread-local error message; returns `status` so callers can `return fail(...)`
int fail(int status, const char *fmt, ...);
uint64_t next_handle_id();
void clear_error();

// host compiler (no HIP): fills p->prog from the tree
int compile(const esc_table *schema, const esc_node *nodes, int nnodes,
            const esc_const *consts, int nconsts, const esc_udf_insn *udf, int nudf,
            esc_pred *p);

// The top-level conjuncts of p (the children of a root AND; p itself
// otherwise), each compiled on its own, with their column slots mapped onto
// one common slot order (nslots, slot_col).
int split_conjuncts(const esc_pred *p, std::vector<Program> &out, int &nslots, int *slot_col);
// The programs as one list with one pool; false if they need more
// instructions, pool words or slot tables than it holds.
bool pack_conjuncts(const std::vector<Program> &progs, ConjPack &pack);
// How split conjuncts on nslots columns run.  Programs of little work for each
// column they load are bound by the loads and run two blocks a CU: four star
// predicates on 40M rows take 313 us so, 321 to 332 with four to eight.
// heavy: others are bound by their own instructions and run all the blocks
// that registers and LDS hold (an instruction counts one, each constant of a
// compare list one, a slot table eight).  40M rows, two blocks and all: two
// IN-lists of 40 on two columns 236 and 189 us, 12 ORs of three on three 288
// and 218, three udfs on two 161 and 124; two ORs of three 101 and 106.
// upload: on seven and eight columns heavy programs are read from memory: as an
// argument, with their tables in registers, they lose a wave (eight columns,
// six IN-lists, 60M rows 844 against 702 us).
struct ConjLoad {
    bool heavy, upload;
};
ConjLoad conj_load(const std::vector<Program> &progs, int nslots);

}  // namespace esc
