// State of a clip-ratio search (Algorithm 1, section 4.1) and what it keeps in device memory.
#pragma once
#include "rotq_internal.h"
#include "search_rule.h"

namespace rq {

// Search state: the best point so far and the nearest evaluated point on either side of it; probes go to the midpoint
// towards the left and the right neighbour in turn.
struct GbsState {
    double left, right;   // nearest evaluated points left and right of the best
    double best;
    int side;             // neighbour the next probe goes towards: 0 left, 1 right
    __host__ __device__ double width() const { return right - left; }
    __host__ __device__ double probe() const { return 0.5 * ((side ? right : left) + best); }
    // after probing x = probe(): `better` = the probe beat the best point, which then bounds the far side
    __host__ __device__ void next(double x, bool better) {
        const bool to_left = better ? side == 1 : side == 0;
        const double bound = better ? best : x;
        left = to_left ? bound : left;
        right = to_left ? right : bound;
        best = better ? x : best;
        side = 1 - side;
    }
};
__host__ __device__ inline GbsState gbs_start() { return GbsState{0.0, 1.0, 0.5, 0}; }

// What one launch of the stepped form hands to the next.
struct GbsCarry {
    GbsState st;
    float fm;             // objective at the best point
    int evals;
    int done;
};

struct GbsDev {
    GbsCarry carry[2];    // stepped form; the rest: batched form
    ClipList clips;       // the next batch
    GbsState st;
    float fm;             // objective at the best point
    int evals;
    int done;
    float trace_clips[256], trace_mse[256];
    // grid form: the workgroups' sums at every clip ratio of the grid (number m at m), their totals, the workgroups that
    // have contributed to them
    double grid_sums[kGridGroups][kGridRatios];
    double grid_totals[kGridRatios];
    uint32_t grid_ticket;
};

}  // namespace rq
