// Launches of the star of four chains of four joints (lm_star.hpp).
#include "lm_star.hpp"

namespace pk {
namespace star {
namespace {

constexpr int PROBLEMS = lane::QUAD_PROBLEMS;
constexpr int THREADS = 4 * PROBLEMS;

// Up to 64 problems per workgroup of four wavefronts, best-of-K as in the quad
// kernel.
__global__ __launch_bounds__(THREADS) void lm_star_kernel(const RobotC *__restrict__ rb,
                                                          const float *__restrict__ qr, SolveParams P, BestOut B,
                                                          int per_block, int64_t block0)
{
    __shared__ float bc[PROBLEMS], bp[PROBLEMS];
    __shared__ int bv[PROBLEMS];
    const int slot = threadIdx.x >> 2, c = threadIdx.x & 3;
    const int64_t p = (block0 + blockIdx.x) * per_block + slot;   // (place in the active list, if there is one)
    const bool live = slot < per_block && p < (P.n_active ? (int64_t)*P.n_active : P.N);
    Final fin;
    if (live) star_problem<false>(rb, qr, P, p, &fin);
    if (!(B.index || B.joints || B.success)) return;   // uniform
    if (live && c == 0) {
        bc[slot] = fin.cost;
        bp[slot] = fin.pcost;
        bv[slot] = fin.conv ? PK_CONVERGED : PK_MAX_ITERS;
    }
    __syncthreads();
    if (!live) return;
    const int K = P.K, first = slot / K * K;
    bool any;
    const int b = best_of_k_pick(bv, bc, bp, first, K, any);
    if (slot != first + b) return;
    const int64_t t = p / K;
    if (B.joints)
#pragma unroll
        for (int i = 0; i < L; ++i) B.joints[(int64_t)(c * L + i) * P.T + t] = fin.q[i];
    if (c == 0) {
        if (B.index) B.index[t] = b;
        if (B.success) B.success[t] = any ? 1 : 0;
    }
}

// Persistent, resumable variant: wavefront w takes every gridDim-th 16 problems
// of the active list, from the w-th on.  No queue: 16 problems are little work
// for an atomic on one address (about 12 ns each, one after the other), and with
// few iterations per launch the atomics were the launch.  100000 hands, 50
// iterations in launches of 1, 2, 5 and 50, 16 wavefronts per CU, us: 7495, 3797,
// 1610 and 403 from a queue; 3143, 1504, 760 and 368 now (4162, 2239, 1285 and
// 859 with one lane per problem and 64 problems to a pop).
__global__ __launch_bounds__(64) void lm_star_persist_kernel(const RobotC *__restrict__ rb,
                                                             const float *__restrict__ qr, SolveParams P)
{
    const int64_t nact = P.n_active ? (int64_t)*P.n_active : P.N, nitems = (nact + 15) / 16;
    for (int64_t item = blockIdx.x; item < nitems; item += gridDim.x) {
        const int64_t i = item * 16 + (threadIdx.x >> 2);
        Final fin;
        if (i < nact) star_problem<true>(rb, qr, P, i, &fin);
    }
}

}  // namespace

hipError_t launch(const RobotC *rb, const SolveParams &P, int persist_blocks, hipStream_t s, const BestOut *best)
{
    const float *qr = P.q_rest ? P.q_rest : rb->mid;
    if (best && (P.K > PROBLEMS || P.queue_head || P.active || P.n_active)) return hipErrorInvalidValue;
    if (P.queue_head) {   // (the mark of a persistent launch)
        int64_t grid = (P.N + 15) / 16;
        if (persist_blocks > 0 && persist_blocks < grid) grid = persist_blocks;
        hipLaunchKernelGGL(lm_star_persist_kernel, dim3((unsigned)grid), dim3(64), 0, s, rb, qr, P);
        return hipGetLastError();
    }
    const BestOut B = best ? *best : BestOut{nullptr, nullptr, nullptr};
    const int per_block = lane::quad_per_block(P.K, best != nullptr);
    // (four threads a problem: above 2^30 problems one launch cannot hold them)
    return launch_parts((P.N + per_block - 1) / per_block, THREADS, [&](int64_t block0, unsigned blocks) {
        hipLaunchKernelGGL(lm_star_kernel, dim3(blocks), dim3(THREADS), 0, s, rb, qr, P, B, per_block, block0);
        return hipGetLastError();
    });
}

}  // namespace star
}  // namespace pk
