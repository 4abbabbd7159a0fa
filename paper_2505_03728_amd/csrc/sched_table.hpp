// Device-side description of a mixed batch for the persistent LM launches
// (lm_mixed.hip), built on the host by the scheduler (sched.hip).
//
// A batch is up to PK_MAX_GROUPS groups; each group is one robot with its
// problems, weights, outputs and resumable state (SolveParams) and the device
// path that solves it.  One round of the launch chain runs every unfinished
// problem of every group for at most k more LM iterations: a plan kernel
// turns the groups' active-list sizes into a table of work items, the
// persistent kernels' wavefronts pop items from their queue, and a compaction
// kernel packs the problems that are still unfinished into the next round's
// active lists.
#pragma once

#include "pk_internal.hpp"

namespace pk {

// Device paths of the persistent kernel (one per (lanes per problem, robot
// class) instantiation).
enum MixedPath : int32_t {
    MIX_LANE_ARM = 0,     // one problem per lane, serial 7-joint arm, one pose EE
    MIX_STAR_HAND = 1,    // four lanes per problem, 4 chains of 4 joints, 4 position EEs
    MIX_WAVE_16_4 = 2,    // one problem per wavefront, lane per joint, depth <= 16 levels, <= 4 EEs
    MIX_PATH_16_4 = 3,    // one problem per wavefront, lane per (joint, EE path) pair,
                          // depth <= 16 levels, <= 4 EEs
    MIX_WAVE_64_8 = 4,    // one problem per wavefront, any tree (<= 64 joints, 8 EEs)
    MIX_PATH_13_4 = 5,    // MIX_PATH_16_4 for trees of at most 13 levels,
    MIX_PATH_8_4 = 6,     // of at most 8 (the path-pair kernel's row lengths)
    MIX_PATHS = 7
};

// Launches of a round that is split, in order, and the one that serves a path: a
// kernel per path-pair instantiation, one for all other paths (lm_mixed.hip says
// why).  A kernel that holds every path serves the rounds that are not split.
constexpr int PK_MIX_LAUNCHES = 4;
constexpr int PK_MIX_ALL = PK_MIX_LAUNCHES;

inline int mixed_launch_of(int path)
{
    return path == MIX_PATH_16_4 ? 0 : path == MIX_PATH_13_4 ? 1 : path == MIX_PATH_8_4 ? 2 : 3;
}

// Groups one persistent launch serves (its description travels by value as
// kernel arguments, which keeps every buffer pointer a global-memory pointer).
constexpr int PK_MIX_GROUPS = 8;

struct MixedGroup {
    const RobotC *rb;
    const float *qr;          // rest pose: the caller's, else the robot's mid-range table
    SolveParams P;            // buffers, weights, options, resumable state and this
                              // round's active list, budget and resume flag
    int32_t *list[2];         // active lists of alternate rounds
    int32_t *count;           // [2] active-list sizes
    int32_t path;             // MixedPath
    int32_t per_item;         // problems per work item: 64 (lane), 16 (star) or 1 (wavefront paths)
};

struct MixedArgs {
    int32_t n_groups;
    int32_t round;
    MixedGroup g[PK_MIX_GROUPS];            // in launch, then queue order
};

// LDS floats one wavefront needs on a path.
int mixed_lds_floats(int path);

// Enqueues one round on stream s: plan (work items per group into item_end,
// queue heads reset), persistent solves (each problem at most P.iter_budget
// more iterations), and, unless it is the last round, compaction.  a holds
// this round's fields; item_end [PK_MIX_GROUPS] and heads [PK_MIX_LAUNCHES]
// are device buffers; wpc = persistent wavefronts per CU, cus = CUs; wg = threads
// per workgroup (64, 128 or 256); max_n = the largest group.
hipError_t launch_mixed_round(const MixedArgs &a, int32_t *item_end, int32_t *heads, int max_n,
                              bool last, int wpc, int cus, int wg, hipStream_t s);

}  // namespace pk
