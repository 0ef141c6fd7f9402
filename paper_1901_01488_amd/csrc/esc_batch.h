// esc_batch.h -- the work list of a batched count as its two kernels read it
// from the batch's workspace: a header with byte offsets, then (packed, so
// that a new plan is one host-to-device copy) the predicate groups, work
// items and programs of the interpreter and the groups, work items and
// indexes of the predicate-index kernel.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "esc_index.h"
#include "esc_kernels.h"

namespace esc {

struct BatchItem {
    int32_t group;
    int32_t r0, r1;
    int32_t pad;
};

struct BatchHeader {
    unsigned int next[2];       // next work item of each kernel (reset before every launch)
    unsigned int nitems[2];     // [0] interpreter, [1] predicate index
    unsigned int ids;           // byte offsets from the header: predicate ids,
    unsigned int groups, items, progs;       // the interpreter's lists,
    unsigned int igroups, iitems, blob;      // the predicate index's lists
    unsigned int pad[53];
};
static_assert(sizeof(BatchHeader) == 256, "the header keeps the lists 256-byte aligned");

constexpr int kIndexBlock = 512;        // threads of an index block (8 waves)
constexpr int kIndexTile = 256;         // rows of a wave tile: four per lane
constexpr int kIndexBlocksPerCu = 2;    // by LDS (kIndexMaxWords) and registers

// counts every predicate of the header's index groups into counts[id]
void launch_index(BatchHeader *h, unsigned long long *counts, int grid, hipStream_t s);
// once per process and device before the first launch: the kernel's LDS
hipError_t prepare_index();

}  // namespace esc
