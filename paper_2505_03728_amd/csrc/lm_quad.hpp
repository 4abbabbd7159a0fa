// Four-lanes-per-problem Levenberg-Marquardt IK kernel for single chains: the
// per-lane kernel's method and arithmetic (lm_lane.hpp), with a problem's
// rows spread over a quad of lanes.
//
// A batch of a few thousand problems leaves the per-lane kernel with a
// wavefront or less per SIMD, and the launch then takes one wavefront's
// instruction stream times the iterations (about 2.1 k VALU instructions per
// iteration for 7 joints).  Here lane r of a quad holds
//   * row r of every frame of the forward kinematics (lane 3 repeats row 2),
//     of the EE pose error and of the right-Jacobian-inverse blocks;
//   * joints r, r + 4, r + 8 (clamped to the last joint): their sine and
//     cosine, limit and rest terms, Jacobian columns and rows of J^T J, and
//     the rows of the Cholesky factor, all in registers;
// and the scalar chains in between (pose log, costs, back substitution, the
// LM controller) run on all four lanes alike.  Values pass between the lanes
// by quad_perm, a modifier of the reading instruction; the joints' axes and
// origins go from rows to columns through LDS.
//
// Every value is computed by the per-lane kernel's expressions in its order
// of operations (the right-looking factorisation subtracts the same products
// from an entry in the same order), so the results are the per-lane kernel's
// bit for bit.  Control flow is uniform over a quad: a lane that reads
// another by quad_perm finds it active.
//
// Bound: one wavefront's instruction stream (about 1.1 k VALU instructions
// per iteration for 7 joints, and the latencies that one wavefront per SIMD
// does not hide).  8 problems x 30 iterations, 7 joints: 148.0 -> 95.5 us;
// 16384 problems of the mobile base (10 joints): 223.5 -> 126.3 us.
#pragma once

#include "lm_lane_kernels.hpp"

namespace pk {
namespace quad {

using lane::ee_of;
using lane::LaneFinal;
using lane::LaneLds;
using lane::pris_of;

constexpr int PROBLEMS = 64;             // per workgroup
constexpr int THREADS = 4 * PROBLEMS;

// v of lane S of the quad.
template <int S>
PK_DEV float from(float v)
{
    const int i = __builtin_bit_cast(int, v);
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(i, S * 0x55, 0xf, 0xf, true));
}

// The same with the lane as a value known after unrolling.
PK_DEV float from(float v, int s)
{
    return s == 0 ? from<0>(v) : s == 1 ? from<1>(v) : s == 2 ? from<2>(v) : from<3>(v);
}

// v of the lane holding row (r + 1) mod 3, (r + 2) mod 3; lane 3 as lane 2.
PK_DEV float rot1(float v)
{
    const int i = __builtin_bit_cast(int, v);
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(i, 0x09, 0xf, 0xf, true));   // 1, 2, 0, 0
}
PK_DEV float rot2(float v)
{
    const int i = __builtin_bit_cast(int, v);
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(i, 0x52, 0xf, 0xf, true));   // 2, 0, 1, 1
}

PK_DEV float quad_max(float v)
{
    const int a = __builtin_bit_cast(int, v);
    v = fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(a, 0xb1, 0xf, 0xf, true)));   // 1, 0, 3, 2
    const int b = __builtin_bit_cast(int, v);
    return fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(b, 0x4e, 0xf, 0xf, true)));   // 2, 3, 0, 1
}

// LDS exchange between the lanes of a quad (one wavefront: in order).
PK_DEV void exchange()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int L, int KIND>
struct Geo {
    static constexpr int NS = (L + 3) / 4;                            // joints per lane
    static constexpr int ROWS = ee_of(KIND) == PK_EE_POSE ? 6 : 3;
    static constexpr int TGW = ee_of(KIND) == PK_EE_POSE ? 12 : 3;    // target slots, as lane::Slots<1, L, KIND>
    static constexpr int JW = 8;                                      // floats per joint: axis, origin, 2 unused
    static constexpr int EX = L * JW + 4;                             // floats per problem, banks staggered
    static constexpr int FLOATS = PROBLEMS * (TGW + EX);
};

// What a lane keeps over the whole solve.
template <int L, int KIND>
struct Lane {
    int r, row;                             // lane of the quad, its row (lane 3: row 2)
    float lo[Geo<L, KIND>::NS], hi[Geo<L, KIND>::NS], qr[Geo<L, KIND>::NS];
    bool pris[Geo<L, KIND>::NS];
    float tp, Rt[3];                        // target position's component, column `row` of its rotation
    float *ex;                              // the problem's exchange area
};

// a[min(r, n - 1)] of the N values a (n at most 4), by selects.  The values
// are opaque to the optimiser, which otherwise turns the selects into one
// load at a lane-dependent address and keeps the array in scratch memory.
template <int N>
PK_DEV float pick(int r, const float *a)
{
    float v = a[0];
    asm("" : "+v"(v));
#pragma unroll
    for (int i = 1; i < N; ++i) {
        float w = a[i];
        asm("" : "+v"(w));
        v = r >= i ? w : v;
    }
    return v;
}

// Normal equations of the taken point on this lane: rows 4 s + r of J^T J
// (entries up to the diagonal), the diagonal entry with its limit and rest
// terms, and J^T r.
template <int L, int KIND>
struct Normal {
    float A[Geo<L, KIND>::NS][L];
    float dg[Geo<L, KIND>::NS], g[Geo<L, KIND>::NS];
};

// One point: cost and errors at q and, when it is taken (lane::eval_point1's
// rule), its normal equations.
template <int L, int KIND>
PK_DEV void eval_point(const RobotC *__restrict__ rb, const SolveParams &P, const Lane<L, KIND> &Q,
                       const float *q, bool first, float cur, float &cost, float &pcost, float &perr,
                       float &rerr, Normal<L, KIND> &E)
{
    using G = Geo<L, KIND>;
    constexpr int NS = G::NS, ROWS = G::ROWS;
    constexpr bool POSE = ee_of(KIND) == PK_EE_POSE;
    float qo[NS], so[NS], co[NS];           // own joints: value, sine, cosine
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        qo[s] = L - 4 * s >= 4 ? pick<4>(Q.r, q + 4 * s) : pick<(L % 4 ? L % 4 : 4)>(Q.r, q + 4 * s);
        joint_sincos(qo[s], so[s], co[s]);
        if (pris_of(KIND)) {
            so[s] = Q.pris[s] ? 0.f : so[s];
            co[s] = Q.pris[s] ? 1.f : co[s];
        }
    }
    // forward kinematics, row by row
    float o[3], p = 0.f;
#pragma unroll
    for (int u = 0; u < 3; ++u) o[u] = Q.row == u ? 1.f : 0.f;
#pragma unroll
    for (int j = 0; j < L; ++j) {
        float on[3], pn;
        joint_step_row(o, p, rb->j[j].G, rb->j[j].t, from(so[j / 4], j % 4), from(co[j / 4], j % 4), on, pn);
        if (pris_of(KIND) && rb->j[j].type == PK_JOINT_PRISMATIC) pn += q[j] * on[2];   // joint_slide
#pragma unroll
        for (int u = 0; u < 3; ++u) o[u] = on[u];
        p = pn;
        Q.ex[j * G::JW + Q.row] = o[2];
        Q.ex[j * G::JW + 3 + Q.row] = p;
    }
    float Re[3], pe;
    ee_frame_row(o, p, rb->e[0].G, rb->e[0].t, Re, pe);
    // residual rows
    const float dr = pe - Q.tp;
    const float d[3] = {from<0>(dr), from<1>(dr), from<2>(dr)};
    perr = sqrtf(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
    float r[ROWS];
    PoseLog lg;
    if constexpr (POSE) {
        float e[3], RE[9], tE[3];
#pragma unroll
        for (int j = 0; j < 3; ++j)
            e[j] = Q.Rt[0] * from<0>(Re[j]) + Q.Rt[1] * from<1>(Re[j]) + Q.Rt[2] * from<2>(Re[j]);
        const float t = Q.Rt[0] * d[0] + Q.Rt[1] * d[1] + Q.Rt[2] * d[2];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
#pragma unroll
            for (int j = 0; j < 3; ++j) RE[3 * i + j] = from(e[j], i);
            tE[i] = from(t, i);
        }
        lg = pose_log_of(RE, tE);
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            r[u] = P.w_pos * lg.rho[u];
            r[3 + u] = P.w_rot * lg.phi[u];
        }
        rerr = lg.theta;
    } else {
#pragma unroll
        for (int u = 0; u < 3; ++u) r[u] = P.w_pos * d[u];
        rerr = 0.f;
    }
    float cp = 0.f, cj = 0.f, jc[NS];
#pragma unroll
    for (int u = 0; u < ROWS; ++u) cp += r[u] * r[u];
#pragma unroll
    for (int s = 0; s < NS; ++s) jc[s] = lane::joint_cost_at(P, qo[s], Q.lo[s], Q.hi[s], Q.qr[s]);
#pragma unroll
    for (int j = 0; j < L; ++j) cj += from(jc[j / 4], j % 4);
    pcost = cp;
    cost = cp + cj;
    if (!(first || cost < cur)) return;

    // own Jacobian columns: lane::jac_column on the own joints' axes and
    // origins, M and N of jr_inv_blocks by rows, then whole on every lane
    float pev[3], M[9], N[9];
#pragma unroll
    for (int u = 0; u < 3; ++u) pev[u] = from(pe, u);
    if constexpr (POSE) {
        const JrCoef J = jr_coef(lg);
        const float *f = lg.phi;
        const bool r0 = Q.row == 0, r1 = Q.row == 1;
        const float fi = r0 ? f[0] : r1 ? f[1] : f[2], ri = r0 ? lg.rho[0] : r1 ? lg.rho[1] : lg.rho[2],
                    ci = r0 ? J.c[0] : r1 ? J.c[1] : J.c[2];
        // rows of hat(f), hat(sk)
        const float hf[3] = {r0 ? 0.f : r1 ? f[2] : -f[1], r0 ? -f[2] : r1 ? 0.f : f[0], r0 ? f[1] : r1 ? -f[0] : 0.f};
        const float hs[3] = {r0 ? 0.f : r1 ? J.sk[2] : -J.sk[1], r0 ? -J.sk[2] : r1 ? 0.f : J.sk[0],
                             r0 ? J.sk[1] : r1 ? -J.sk[0] : 0.f};
        float Pr[3], Qr[3], m[3], qm[3], nr[3];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            jr_entry(J, f, lg.rho, fi, ri, ci, j, Q.row == j, Pr[j], Qr[j]);
            Pr[j] += 0.5f * hf[j];
            Qr[j] += hs[j];
        }
#pragma unroll
        for (int j = 0; j < 3; ++j)
            m[j] = Pr[0] * from(Re[0], j) + Pr[1] * from(Re[1], j) + Pr[2] * from(Re[2], j);
#pragma unroll
        for (int j = 0; j < 3; ++j) qm[j] = Qr[0] * from<0>(m[j]) + Qr[1] * from<1>(m[j]) + Qr[2] * from<2>(m[j]);
#pragma unroll
        for (int j = 0; j < 3; ++j)
            nr[j] = -(Pr[0] * from<0>(qm[j]) + Pr[1] * from<1>(qm[j]) + Pr[2] * from<2>(qm[j]));
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                M[3 * i + j] = from(m[j], i);
                N[3 * i + j] = from(nr[j], i);
            }
    }
    exchange();
    float col[NS][ROWS], gx[NS], dq[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int j = min(4 * s + Q.r, L - 1);
        float om[3], pj[3];
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            om[u] = Q.ex[j * G::JW + u];
            pj[u] = Q.ex[j * G::JW + 3 + u];
        }
        lane::jac_column<KIND>(P, M, N, om, pj, pev, pris_of(KIND) && Q.pris[s], col[s]);
        lane::joint_terms_at(P, qo[s], Q.lo[s], Q.hi[s], Q.qr[s], dq[s], gx[s]);
    }
    exchange();   // the next point's frames overwrite the area
    // own rows of J^T J and J^T r
#pragma unroll
    for (int s = 0; s < NS; ++s) {
#pragma unroll
        for (int k = 0; k < L; ++k) {
            if (k > 4 * s + 3) continue;
            float a = 0.f;
#pragma unroll
            for (int u = 0; u < ROWS; ++u) a += col[s][u] * from(col[k / 4][u], k % 4);
            E.A[s][k] = a;
        }
        E.dg[s] = (L - 4 * s >= 4 ? pick<4>(Q.r, E.A[s] + 4 * s) : pick<(L % 4 ? L % 4 : 4)>(Q.r, E.A[s] + 4 * s)) +
                  dq[s];
        float b = gx[s];
#pragma unroll
        for (int u = 0; u < ROWS; ++u) b += col[s][u] * r[u];
        E.g[s] = b;
    }
}

// Damped step: lane::lane_step's test and values, the factor right-looking
// with rows over the quad.  x whole on every lane; false on a small pivot.
template <int L, int KIND>
PK_DEV bool step(const SolveParams &P, int r, const Normal<L, KIND> &E, float lam, float *x)
{
    constexpr int NS = Geo<L, KIND>::NS;
    float dmax = 0.f, F[NS][L], ys[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) dmax = fmaxf(dmax, E.dg[s] + lam * fmaxf(E.dg[s], P.damping_floor));
    dmax = quad_max(dmax);
    const float thresh = P.pivot_rel * dmax;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        float dd = E.dg[s];
        dd += lam * (E.dg[s] > P.damping_floor ? E.dg[s] : P.damping_floor);
#pragma unroll
        for (int k = 0; k < L; ++k) {
            if (k > 4 * s + 3) continue;
            F[s][k] = k >= 4 * s && r == k - 4 * s ? dd : E.A[s][k];
        }
        ys[s] = -E.g[s];
    }
    bool ok = true;
    float inv[L], y[L];
#pragma unroll
    for (int l = 0; l < L; ++l) {
        float d = from(F[l / 4][l], l % 4);
        if (!(d > thresh) || !(d < INFINITY)) {
            ok = false;
            d = 1.f;
        }
        inv[l] = rsqrt_t(d);
        y[l] = from(ys[l / 4], l % 4) * inv[l];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            if (4 * s + 3 <= l) continue;       // rows up to l only
            F[s][l] *= inv[l];
            ys[s] -= F[s][l] * y[l];
        }
#pragma unroll
        for (int k = l + 1; k < L; ++k) {
            const float lk = from(F[k / 4][l], k % 4);
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                if (k > 4 * s + 3) continue;
                F[s][k] -= F[s][l] * lk;
            }
        }
    }
#pragma unroll
    for (int i = L - 1; i >= 0; --i) {
        float t = y[i];
#pragma unroll
        for (int l = i + 1; l < L; ++l) t -= from(F[l / 4][i], l % 4) * x[l];
        x[i] = t * inv[i];
    }
    return ok;
}

// Problem i on this quad: lane::lane_problem's loop.
template <int L, int KIND>
PK_DEV void quad_problem(const RobotC *__restrict__ rb, const float *__restrict__ qr, const SolveParams &P,
                         float *smem, int64_t p, LaneFinal<L> *fin)
{
    using G = Geo<L, KIND>;
    constexpr int NS = G::NS;
    const int slot = threadIdx.x >> 2;
    const LaneLds S{smem + slot};           // target slots, 64 problems side by side
    Lane<L, KIND> Q;
    Q.r = threadIdx.x & 3;
    Q.row = min(Q.r, 2);
    Q.ex = smem + PROBLEMS * G::TGW + slot * G::EX;
    float q[L], qt[L];
    if (!lane::load_problem<1, L, KIND>(P, S, P.seeds, p, q)) {
        if (Q.r == 0) lane::write_nonfinite<1, L, KIND>(P, p, q, false);
#pragma unroll
        for (int j = 0; j < L; ++j) fin->q[j] = q[j];
        fin->cost = fin->pcost = NAN;
        fin->conv = false;
        return;
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int j = min(4 * s + Q.r, L - 1);
        Q.lo[s] = rb->j[j].lo;
        Q.hi[s] = rb->j[j].hi;
        Q.qr[s] = qr[j];
        Q.pris[s] = pris_of(KIND) && rb->j[j].type == PK_JOINT_PRISMATIC;
    }
    exchange();
    Q.tp = S[Q.row];
    if constexpr (ee_of(KIND) == PK_EE_POSE) {
#pragma unroll
        for (int k = 0; k < 3; ++k) Q.Rt[k] = S[3 + 3 * k + Q.row];
    }
    int iters = 0, accepts = 0, itt = -1, flags = 0;
    bool done = false, stalled = false, first = true;
    float lam = P.lambda0, cost = 0.f, pcost = 0.f, perr[1] = {0.f}, rerr[1] = {0.f};
    Normal<L, KIND> E;
#pragma unroll
    for (int j = 0; j < L; ++j) qt[j] = q[j];
    for (;;) {
        bool ok = true;
        if (!first) {
            float delta[L];
            ok = step<L, KIND>(P, Q.r, E, lam, delta);
            if (!ok) {
                flags |= PK_FLAG_FP64;
                ok = lane::step_fp64_1<L, KIND>(rb, P, qr, S, q, lam, delta);
            }
#pragma unroll
            for (int j = 0; j < L; ++j) qt[j] = q[j] + delta[j];
        }
        float ct = INFINITY, pct = 0.f, pe_t[1] = {0.f}, re_t[1] = {0.f};
        if (ok) eval_point<L, KIND>(rb, P, Q, qt, first, cost, ct, pct, pe_t[0], re_t[0], E);
        if (first) {
            cost = ct;
            pcost = pct;
            perr[0] = pe_t[0];
            rerr[0] = re_t[0];
            itt = lane::meets_tol<1, L, KIND>(P, perr, rerr) ? 0 : -1;
            done = P.early_exit && itt == 0;
            first = false;
        } else {
            ++iters;
            const bool acc = ct < cost;
            if (acc) {
#pragma unroll
                for (int j = 0; j < L; ++j) q[j] = qt[j];
                cost = ct;
                pcost = pct;
                perr[0] = pe_t[0];
                rerr[0] = re_t[0];
                lam = fmaxf(lam / P.nu_down, P.lambda_min);
                ++accepts;
                if (lane::meets_tol<1, L, KIND>(P, perr, rerr)) {
                    if (itt < 0) itt = iters;
                    if (P.early_exit) done = true;
                }
            } else {
                if (lam >= P.lambda_max) {
                    stalled = true;
                    done = true;
                }
                lam = fminf(lam * P.nu_up, P.lambda_max);
            }
            if (P.trace_iters && Q.r == 0) lane::write_trace<1, L, KIND>(P, iters - 1, p, q, acc);
        }
        if (done || iters >= P.max_iters) break;
    }
    if (Q.r == 0)
        lane::write_result<1, L, KIND>(P, p, q, cost, pcost, perr, rerr, iters, accepts, itt, flags, stalled, true);
#pragma unroll
    for (int j = 0; j < L; ++j) fin->q[j] = q[j];
    fin->cost = cost;
    fin->pcost = pcost;
    fin->conv = lane::meets_tol<1, L, KIND>(P, perr, rerr);
}

// 64 problems per workgroup of four wavefronts; with B's pointers set, their
// targets' best-of-K as well (K divides 64).
template <int L, int KIND>
__global__ __launch_bounds__(THREADS) void lm_quad_kernel(const RobotC *__restrict__ rb,
                                                          const float *__restrict__ qr, SolveParams P,
                                                          BestOut B)
{
    using G = Geo<L, KIND>;
    __shared__ __attribute__((aligned(16))) float smem[G::FLOATS];
    __shared__ float bc[PROBLEMS], bp[PROBLEMS];
    __shared__ int bv[PROBLEMS];
    const int64_t base = (int64_t)blockIdx.x * PROBLEMS, p = base + (threadIdx.x >> 2);
    const bool live = p < P.N;
    LaneFinal<L> fin;
    if (live) quad_problem<L, KIND>(rb, qr, P, smem, p, &fin);
    if (!(B.index || B.joints || B.success)) return;   // uniform
    if (live && (threadIdx.x & 3) == 0) {
        bc[threadIdx.x >> 2] = fin.cost;
        bp[threadIdx.x >> 2] = fin.pcost;
        bv[threadIdx.x >> 2] = fin.conv ? PK_CONVERGED : PK_MAX_ITERS;
    }
    __syncthreads();
    if (!live) return;
    const int K = P.K, slot = threadIdx.x >> 2, first = slot / K * K;
    bool any;
    const int b = best_of_k_pick(bv, bc, bp, first, K, any);
    if (slot != first + b || (threadIdx.x & 3)) return;
    const int64_t t = p / K;
    if (B.joints)
#pragma unroll
        for (int j = 0; j < L; ++j) B.joints[(int64_t)j * P.T + t] = fin.q[j];
    if (B.index) B.index[t] = b;
    if (B.success) B.success[t] = any ? 1 : 0;
}

template <int L, int KIND>
hipError_t launch(const RobotC *rb, const SolveParams &P, hipStream_t s, const BestOut *best)
{
    const float *qr = P.q_rest ? P.q_rest : rb->mid;
    const BestOut B = best ? *best : BestOut{nullptr, nullptr, nullptr};
    hipLaunchKernelGGL((lm_quad_kernel<L, KIND>), dim3((unsigned)((P.N + PROBLEMS - 1) / PROBLEMS)), dim3(THREADS),
                       0, s, rb, qr, P, B);
    return hipGetLastError();
}

}  // namespace quad
}  // namespace pk
