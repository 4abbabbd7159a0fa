// Which lane kernel serves a plain launch (no queue, no active list): one lane
// per problem, or four (lm_quad.hpp, lm_star.hpp).  Host code only, also
// compiled by the CPU test of the rule.
#pragma once

#include "pk_internal.hpp"

namespace pk {
namespace lane {

constexpr int QUAD_PROBLEMS = 64;   // per workgroup of the four-lane kernels

// Problems per workgroup: with best-of-K in the launch (K at most 64), whole
// targets.
inline int quad_per_block(int K, bool best) { return best ? QUAD_PROBLEMS / K * K : QUAD_PROBLEMS; }

// Workgroups (of four wavefronts) up to which single chains run with four lanes
// per problem.  256 give every SIMD one wavefront, 512 two; two take less than
// twice as long as one, three do not, and the per-lane kernel's time hardly
// depends on the batch up to 65536.  30 iterations, four lanes against one, us:
//   256: 3 joints 55 / 89, 7 joints 77 / 131, 8 joints 83 / 146, 10 joints
//        112 / 192; without the rest term (the redundant chains' steps then end
//        in the FP64 re-solve) 7 joints 104 / 236
//   512: 3 joints 80 / 83, 5 joints 103 / 108, 6 joints 110 / 122, 7 joints
//        118 / 136 (without the rest term 160 / 246), 8 joints with a position
//        EE 98 / 110; 10 joints 189 / 192, more than 256 registers and so one
//        wavefront per SIMD after the other
//   512, 8 joints with a pose EE: 163 / 152 while the FP32 factor holds (rest
//        weight 0.01 and above), 231 / 281 without the rest term and 243 / 281 at
//        1e-4, where its square is below the pivot test
//   848: 7 joints, 33 seeds per target and so a target per workgroup: 218 / 164;
//        146 with best-of-K in a launch of its own on 438 workgroups
inline int64_t quad_max_blocks(int chain_len, int ee_kind, const SolveParams &P)
{
    if (chain_len > 8) return 256;
    if (chain_len < 8 || ee_kind == PK_EE_POSITION) return 512;
    return P.w_rest * P.w_rest <= P.pivot_rel ? 512 : 256;
}

// best: with best-of-K in the launch.  (target_exit is defined on the per-lane
// kernel's runs of lanes.)
inline bool takes_quad(int chains, int chain_len, int ee_kind, const SolveParams &P, bool best)
{
    if (chains != 1 || P.target_exit || (best && P.K > QUAD_PROBLEMS)) return false;
    const int per_block = quad_per_block(P.K, best);
    return (P.N + per_block - 1) / per_block <= quad_max_blocks(chain_len, ee_kind, P);
}

// The star of four chains of four joints with position EEs runs with four lanes
// per problem, a chain each (lm_star.hpp: faster at every size measured, 64 to a
// million problems); the per-lane kernel keeps target_exit, which is defined on
// its runs of lanes.
inline bool takes_star(int chains, int chain_len, const SolveParams &P)
{
    return chains == 4 && chain_len == 4 && !P.target_exit;
}

// Whether the launch can take best-of-K itself: K divides 64, so that a
// target's problems share a wavefront, or they share a workgroup of a four-lane
// kernel.
inline bool takes_best(int chains, int chain_len, int ee_kind, const SolveParams &P)
{
    return 64 % P.K == 0 ||
           (P.K <= QUAD_PROBLEMS && (takes_quad(chains, chain_len, ee_kind, P, true) || takes_star(chains, chain_len, P)));
}

}  // namespace lane
}  // namespace pk
