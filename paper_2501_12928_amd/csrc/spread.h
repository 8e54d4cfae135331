// Likelihood with the tiles of each theta spread over many workgroups
// (spread.hip).
#pragma once

#include "common.h"
#include "route.h"

namespace eor {

// Words of one theta's progress row beside the N counts of finished tiles:
// stop (the theta has failed), tails (diagonal tiles whose ln d is stored),
// done (finished units), handed (the last row whose X is in its diagonal
// tile's slot), inverses (diagonal tiles whose inverse is stored).
constexpr int SPREAD_EXTRA = 5;

struct SpreadParams {
    const InstDesc *inst;    // device [n_inst]
    const int2 *task;        // device [ntask] (instance, theta index), largest instance first, or NULL: (0, t)
    const int32_t *count;    // device [n_max + 1]: tasks of instances with at least that many tile rows, or NULL: ntask
    int32_t ntask;           // theta, each with a slot of its own
    int32_t n_max;           // tile rows of the largest instance
    int64_t units;           // tiles in all (< 2^31)
    unsigned int *counter;   // next unit; zero before and after a launch
    int32_t *prog;           // [ntask][n_max + SPREAD_EXTRA]; zero before and after a launch
    double2 *Lw;             // packed tiles of L, slot after slot
    const longlong2 *off;    // device [ntask]: first element of each slot in Lw and in yw, or NULL: slot * slot_elems, * slot_y
    int64_t slot_elems;
    double2 *yw;             // per-slot w, then y
    int64_t slot_y;
    int32_t per_cu;          // workgroups per CU, 1 or 2 (spread_per_cu)
    CallDesc call[MAX_INST];
};

hipError_t launch_spread(const SpreadParams &p, int num_cu, hipStream_t s);

}  // namespace eor
