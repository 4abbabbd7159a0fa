// Four-lanes-per-problem Levenberg-Marquardt IK for the star of four chains of
// four joints with position EEs: the per-lane kernel's method and arithmetic
// (lm_lane.hpp) with a chain per lane.
//
// The chains share nothing but the problem's decisions: J^T J is one 4 x 4
// block per chain, so frames, columns, factor and step of a chain are its own
// lane's, in registers.  Between the lanes go the residuals and joint costs
// (summed by every lane in the per-lane kernel's order), the largest damped
// diagonal and whether every chain's factorisation held, by quad_perm.  Values
// are the per-lane kernel's bit for bit; control flow is uniform over a quad.
//
// Bound: a wavefront's instruction stream.  The per-lane kernel runs the four
// chains one after the other on 250 registers and 26 KiB of LDS per wavefront,
// and 20000 problems are 313 wavefronts of it on 1024 SIMDs.  30 iterations of
// 64, 20000, 131072 and 1048576 problems: 230, 263, 569 and 2977 us there; 44,
// 79, 262 and 1818 here, so here for every size.
#pragma once

#include "lm_lane_kernels.hpp"

namespace pk {
namespace star {

using quad::from;
using quad::quad_max;

constexpr int C = 4, L = 4, N = C * L, ROWS = 3, NA = L * (L + 1) / 2;
constexpr int KIND = PK_EE_POSITION;

PK_DEV bool quad_all(bool v)
{
    int i = v ? 1 : 0;
    i &= __builtin_amdgcn_mov_dpp(i, 0xb1, 0xf, 0xf, true);   // 1, 0, 3, 2
    i &= __builtin_amdgcn_mov_dpp(i, 0x4e, 0xf, 0xf, true);   // 2, 3, 0, 1
    return i != 0;
}

// What a lane keeps of its chain over the whole solve.
struct Chain {
    float G[L][9], t[L][3], et[3];          // joint transforms, EE offset
    float lo[L], hi[L], qr[L], tp[3];       // limits, rest pose, target
};

// The chain's part of the point whose normal equations the next step solves.
struct Point {
    float col[L][ROWS], r[ROWS], dg[L], gx[L];
    float A[NA], g[L];                      // packed FP32 normal equations
};

template <typename T>
PK_DEV void form_normal(const Point &X, T *A, T *g)
{
#pragma unroll
    for (int i = 0; i < L; ++i) {
#pragma unroll
        for (int k = 0; k <= i; ++k) {
            T s = 0;
#pragma unroll
            for (int u = 0; u < ROWS; ++u) s += (T)X.col[i][u] * (T)X.col[k][u];
            if (k == i) s += (T)X.dg[i];
            A[lane::tri(i, k)] = s;
        }
        T s = (T)X.gx[i];
#pragma unroll
        for (int u = 0; u < ROWS; ++u) s += (T)X.col[i][u] * (T)X.r[u];
        g[i] = s;
    }
}

// One point: cost and this chain's EE error at q and, when it is taken
// (lane::eval_point1's rule), its normal equations.  Whether it was taken.
PK_DEV void eval_point(const SolveParams &P, const Chain &H, const float *q, bool first, float cur, float &cost,
                       float &pcost, float &perr, Point &X)
{
    float O[9], p[3], om[L][3], pj[L][3], pe[3], r[ROWS], jc[L];
#pragma unroll
    for (int i = 0; i < L; ++i) {
        float s, c, On[9], pn[3];
        joint_sincos(q[i], s, c);
        if (i == 0) {
#pragma unroll
            for (int u = 0; u < 3; ++u) {
                joint_turn_row(H.G[0][3 * u], H.G[0][3 * u + 1], H.G[0][3 * u + 2], s, c, On + 3 * u);
                pn[u] = H.t[0][u];
            }
        } else {
            joint_step(O, p, H.G[i], H.t[i], s, c, On, pn);
        }
#pragma unroll
        for (int u = 0; u < 9; ++u) O[u] = On[u];
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            p[u] = pn[u];
            om[i][u] = O[3 * u + 2];
            pj[i][u] = p[u];
        }
    }
    float d[3];
#pragma unroll
    for (int u = 0; u < 3; ++u) {
        // (ee_frame's origin)
        pe[u] = p[u] + O[3 * u] * H.et[0] + O[3 * u + 1] * H.et[1] + O[3 * u + 2] * H.et[2];
        d[u] = pe[u] - H.tp[u];
    }
    perr = sqrtf(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
#pragma unroll
    for (int u = 0; u < ROWS; ++u) r[u] = P.w_pos * d[u];
#pragma unroll
    for (int i = 0; i < L; ++i) jc[i] = lane::joint_cost_at(P, q[i], H.lo[i], H.hi[i], H.qr[i]);
    float cp = 0.f, cj = 0.f;
#pragma unroll
    for (int c = 0; c < C; ++c) {
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
            const float v = from(r[u], c);
            cp += v * v;
        }
#pragma unroll
        for (int i = 0; i < L; ++i) cj += from(jc[i], c);
    }
    pcost = cp;
    cost = cp + cj;
    if (!(first || cost < cur)) return;
#pragma unroll
    for (int i = 0; i < L; ++i) {
        lane::jac_column<KIND>(P, nullptr, nullptr, om[i], pj[i], pe, false, X.col[i]);
        lane::joint_terms_at(P, q[i], H.lo[i], H.hi[i], H.qr[i], X.dg[i], X.gx[i]);
    }
#pragma unroll
    for (int u = 0; u < ROWS; ++u) X.r[u] = r[u];
    form_normal<float>(X, X.A, X.g);
}

// lane::lane_step (and its FP64 re-solve) on the four chains.
PK_DEV bool step(const SolveParams &P, const Point &X, float lam, int &flags, float *delta)
{
    float dmax = 0.f, Lf[NA];
#pragma unroll
    for (int i = 0; i < L; ++i) {
        const float a = X.A[lane::tri(i, i)];
        dmax = fmaxf(dmax, a + lam * fmaxf(a, P.damping_floor));
    }
    const bool held = lane::chol_damped<L, float>(X.A, lam, P.damping_floor, P.pivot_rel * quad_max(dmax), Lf);
    lane::chol_solve_neg<L, float>(Lf, X.g, delta);
    if (quad_all(held)) return true;
    flags |= PK_FLAG_FP64;
    double A[NA], g[L], x[L];
    form_normal<double>(X, A, g);
    const bool ok = lane::chol_damped<L, double>(A, (double)lam, (double)P.damping_floor, 0.0, A);
    lane::chol_solve_neg<L, double>(A, g, x);
#pragma unroll
    for (int i = 0; i < L; ++i) delta[i] = (float)x[i];
    return quad_all(ok);
}

// How a problem ended, for a best-of-K in the launch that solved it.
struct Final {
    float q[L];                             // this chain's joints
    float cost, pcost;
    bool conv;
};

// The lane's share of a trace row (lane::write_trace).
PK_DEV void write_trace(const SolveParams &P, int it, int64_t p, int c, const float *q, bool acc)
{
    if (it >= P.trace_iters) return;
#pragma unroll
    for (int i = 0; i < L; ++i) P.trace_q[((int64_t)it * N + c * L + i) * P.N + p] = q[i];
    if (c == 0) P.trace_acc[(int64_t)it * P.N + p] = acc ? 1 : 0;
}

// Problem i of the active list on this quad: lane::lane_problem.
template <bool RESUMABLE>
PK_DEV void star_problem(const RobotC *__restrict__ rb, const float *__restrict__ qr, const SolveParams &P,
                         int64_t i0, Final *fin)
{
    const int c = threadIdx.x & 3;
    const int64_t p = P.active ? (int64_t)P.active[i0] : i0;
    const int64_t np = P.N, t = p / P.K;
    const bool resume = RESUMABLE && P.resume;
    Chain H;
    float q[L], qt[L];
    bool finite = true;
    const float *src = resume ? P.joints : P.seeds;
#pragma unroll
    for (int i = 0; i < L; ++i) {
        const int j = c * L + i;
        q[i] = src[j * np + p];
        finite &= isfinite(q[i]);
#pragma unroll
        for (int u = 0; u < 9; ++u) H.G[i][u] = rb->j[j].G[u];
#pragma unroll
        for (int u = 0; u < 3; ++u) H.t[i][u] = rb->j[j].t[u];
        H.lo[i] = rb->j[j].lo;
        H.hi[i] = rb->j[j].hi;
        H.qr[i] = qr[j];
    }
#pragma unroll
    for (int u = 0; u < 3; ++u) {
        H.et[u] = rb->e[c].t[u];
        H.tp[u] = P.targets[(int64_t)(c * 3 + u) * P.T + t];
        finite &= isfinite(H.tp[u]);
    }
    if (!quad_all(finite)) {
        // lane::write_nonfinite
#pragma unroll
        for (int i = 0; i < L; ++i) P.joints[(int64_t)(c * L + i) * np + p] = q[i];
        if (P.pos_err) P.pos_err[c * np + p] = NAN;
        if (P.rot_err) P.rot_err[c * np + p] = NAN;
        if (c == 0) {
            if (P.cost) P.cost[p] = NAN;
            if (P.pose_cost) P.pose_cost[p] = NAN;
            if (P.iters) P.iters[p] = 0;
            if (P.accepts) P.accepts[p] = 0;
            if (P.status) P.status[p] = PK_NONFINITE;
            if (P.iters_to_tol) P.iters_to_tol[p] = -1;
            if (RESUMABLE) P.st_state[p] = PK_ST_DONE;
        }
        for (int it = 0; it < P.trace_iters; ++it) write_trace(P, it, p, c, q, false);
#pragma unroll
        for (int i = 0; i < L; ++i) fin->q[i] = q[i];
        fin->cost = fin->pcost = NAN;
        fin->conv = false;
        return;
    }
    int iters = 0, accepts = 0, itt = -1, flags = 0;
    bool done = false, stalled = false, first = true;
    float lam = P.lambda0, cost = 0.f, pcost = 0.f, perr = 0.f;
    if (resume) {
        const int st = P.st_state[p];
        iters = P.iters[p];
        accepts = P.accepts[p];
        itt = P.iters_to_tol[p];
        flags = st & 0xffff;
        stalled = (st & PK_ST_STALLED) != 0;
        done = (st & PK_ST_DONE) != 0;
        lam = P.st_lambda[p];
    }
    const int iter_end = RESUMABLE ? min(P.max_iters, iters + P.iter_budget) : P.max_iters;
    Point X;
#pragma unroll
    for (int i = 0; i < L; ++i) qt[i] = q[i];
    for (;;) {
        bool ok = true;
        if (!first) {
            float delta[L];
            ok = step(P, X, lam, flags, delta);
#pragma unroll
            for (int i = 0; i < L; ++i) qt[i] = q[i] + delta[i];
        }
        float ct = INFINITY, pct = 0.f, pe_t = 0.f;
        if (ok) eval_point(P, H, qt, first, cost, ct, pct, pe_t, X);
        const bool meets = quad_all(pe_t <= P.tol_pos);
        if (first) {
            cost = ct;
            pcost = pct;
            perr = pe_t;
            if (!resume) {
                itt = meets ? 0 : -1;
                done = P.early_exit && itt == 0;
            }
            first = false;
        } else {
            ++iters;
            const bool acc = ct < cost;
            if (acc) {
#pragma unroll
                for (int i = 0; i < L; ++i) q[i] = qt[i];
                cost = ct;
                pcost = pct;
                perr = pe_t;
                lam = fmaxf(lam / P.nu_down, P.lambda_min);
                ++accepts;
                if (meets) {
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
            write_trace(P, iters - 1, p, c, q, acc);
        }
        if (done || iters >= iter_end) break;
    }
    // lane::write_result
    const bool finished = done || iters >= P.max_iters;
    if (finished)
        for (int it = iters; it < P.trace_iters; ++it) write_trace(P, it, p, c, q, false);
    const bool conv = quad_all(perr <= P.tol_pos);
#pragma unroll
    for (int i = 0; i < L; ++i) P.joints[(int64_t)(c * L + i) * np + p] = q[i];
    if (P.pos_err) P.pos_err[c * np + p] = perr;
    if (P.rot_err) P.rot_err[c * np + p] = 0.f;
    if (c == 0) {
        if (P.cost) P.cost[p] = cost;
        if (P.pose_cost) P.pose_cost[p] = pcost;
        if (P.iters) P.iters[p] = iters;
        if (P.accepts) P.accepts[p] = accepts;
        if (P.status) P.status[p] = (conv ? PK_CONVERGED : (stalled ? PK_STALLED : PK_MAX_ITERS)) | flags;
        if (P.iters_to_tol) P.iters_to_tol[p] = itt;
        if (RESUMABLE) {
            P.st_lambda[p] = lam;
            P.st_state[p] = flags | (stalled ? PK_ST_STALLED : 0) | (finished ? PK_ST_DONE : 0);
        }
    }
#pragma unroll
    for (int i = 0; i < L; ++i) fin->q[i] = q[i];
    fin->cost = cost;
    fin->pcost = pcost;
    fin->conv = conv;
}

}  // namespace star
}  // namespace pk
