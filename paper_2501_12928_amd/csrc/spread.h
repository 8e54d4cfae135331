// Likelihood with the tiles of each theta spread over many workgroups
// (spread.hip).
#pragma once

#include "common.h"

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

// Estimated times (us) of one launch, from which the callers choose (the
// results are the same bits either way). Measured at n = 64 .. 4096 with 1 ..
// 256 theta, and within 15% of that:
//  - one workgroup takes a theta of N tile rows in 30 N + 1.5 N^2 + 0.93 N^3
//    (200 us at n = 200, 4.7 ms at 1003, 253 ms at 4096), up to 15% more when
//    all workgroups run;
//  - spread, a theta's diagonal tiles follow one another every 27 us, and its
//    N (N + 1) / 2 tiles take the whole GPU 0.08 us each plus their products at
//    78 TFLOP/s. The chain and the work of all theta overlap almost wholly where
//    the chain is the longer, in part otherwise; with two to four tile rows there
//    is too little of either, and they add up (spread against one workgroup each:
//    n = 128, 60 theta 78 / 81 us, 128 109 / 89; n = 200, 64 160 / 205, 128 214 /
//    205, where the sum without this said spread in all four).
inline double lone_us(int64_t N) { return 30.0 * N + 1.5 * N * N + 0.93 * N * N * N; }
inline double spread_chain_us(int64_t N) { return 27.0 * N; }
inline double spread_work_us(int64_t N) { return 0.04 * N * (N + 1) + 4.0 / 3.0 * 262144.0 * N * N * N / 78e6; }
inline double spread_us(double chain, double work, int64_t N) {
    if (N >= 2 && N <= 4) return chain + work;
    return chain > work ? chain + 0.1 * work : work + 0.3 * chain;
}

// Where the chain bounds, one workgroup per CU: a second one's matrix
// instructions hold up the single wave that factors a diagonal tile (19 us
// beside them, 14 alone). With much more work than chain, two, so that one
// computes while the other waits. The line, as work over chain, rises with the
// tile rows N, since longer sums leave less waiting to cover. Measured, one
// against two per CU: N = 4, 64 theta (work 0.6 times the chain) 164 / 162 us; N = 9,
// 32 (0.9) 364 / 378, 40 (1.1) 415 / 388; N = 16, 14 (1.0) 550 / 638, 24 (1.6) 859 /
// 744; N = 24, 10 (1.3) 932 / 1022, 12 (1.6) 1129 / 1092; N = 32, 8 (1.8) 1531 /
// 1563, 10 (2.2) 1955 / 1830; N = 47, 4 (1.8) 2.21 / 2.37 ms, 6 (2.6) 3.19 / 3.18; N =
// 64, two (1.6) 2.64 / 3.06, four (3.1) 4.94 / 5.12.
inline int spread_per_cu(double chain, double work, int64_t N) { return work < (0.5 + N / 22.0) * chain ? 1 : 2; }

}  // namespace eor
