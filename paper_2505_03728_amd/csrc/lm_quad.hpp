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
// Bound: one wavefront's instruction stream: about 1.2 k instructions per pass
// for 7 joints, 1.07 k of them VALU, so 55 of a launch's 85 us; the rest is
// latencies that one wavefront per SIMD does not hide.  Against one lane per
// problem, 30 iterations: 8 problems of 7 joints 144 -> 85 us; 16384 of the
// mobile base (10 joints) 192 -> 112; 16384 of 7 joints without the rest term,
// where most steps end in the FP64 re-solve, 236 -> 104.
#pragma once

#include "lm_lane_kernels.hpp"

namespace pk {
namespace quad {

using lane::ee_of;
using lane::LaneFinal;
using lane::LaneLds;
using lane::pris_of;

constexpr int PROBLEMS = lane::QUAD_PROBLEMS;
constexpr int THREADS = 4 * PROBLEMS;

// v of lane S of the quad.
template <int S>
PK_DEV float from(float v)
{
    const int i = __builtin_bit_cast(int, v);
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(i, S * 0x55, 0xf, 0xf, true));
}

template <int S>
PK_DEV double from(double v)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)b, S * 0x55, 0xf, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(b >> 32), S * 0x55, 0xf, 0xf, true);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// The same with the lane as a value known after unrolling.
template <typename T>
PK_DEV T from(T v, int s)
{
    return s == 0 ? from<0>(v) : s == 1 ? from<1>(v) : s == 2 ? from<2>(v) : from<3>(v);
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
    // The own row of the first joint's transform, the others and the EE's whole
    // (G, then t).  Read with scalar loads where they
    // are used, each joint's wait for them stood in the one wavefront's way.
    float g0[3], t0, fr[L][12];
    float *ex;                              // the problem's exchange area
};

// a[min(r, n - 1)] of the N values a (n at most 4), by selects.  The values
// are opaque to the optimiser, which otherwise turns the selects into one
// load at a lane-dependent address and keeps the array in scratch memory.
template <int N, typename T>
PK_DEV T pick(int r, const T *a)
{
    T v = a[0];
    asm("" : "+v"(v));
#pragma unroll
    for (int i = 1; i < N; ++i) {
        T w = a[i];
        asm("" : "+v"(w));
        v = r >= i ? w : v;
    }
    return v;
}

// The taken point on this lane: Jacobian columns of the own joints, their
// limit and rest terms (of the diagonal, of J^T r) and the residual rows.
template <int L, int KIND>
struct Point {
    float col[Geo<L, KIND>::NS][Geo<L, KIND>::ROWS], dq[Geo<L, KIND>::NS], gx[Geo<L, KIND>::NS];
    float r[Geo<L, KIND>::ROWS];
};

// Its normal equations in precision T: rows 4 s + r of J^T J (entries up to
// the diagonal), the diagonal entry with its limit and rest terms, and J^T r.
template <int L, typename T>
struct Normal {
    static constexpr int NS = (L + 3) / 4;
    T A[NS][L], dg[NS], g[NS];
};

template <int L, int KIND, typename T>
PK_DEV void form_normal(int lr, const Point<L, KIND> &X, Normal<L, T> &E)
{
    constexpr int NS = Geo<L, KIND>::NS, ROWS = Geo<L, KIND>::ROWS;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
#pragma unroll
        for (int k = 0; k < L; ++k) E.A[s][k] = 0;
    }
#pragma unroll
    for (int k = 0; k < L; ++k)
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
            const T ck = (T)from(X.col[k / 4][u], k % 4);
#pragma unroll
            for (int s = k / 4; s < NS; ++s) E.A[s][k] += (T)X.col[s][u] * ck;
        }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        E.dg[s] = (L - 4 * s >= 4 ? pick<4>(lr, E.A[s] + 4 * s) : pick<(L % 4 ? L % 4 : 4)>(lr, E.A[s] + 4 * s)) +
                  (T)X.dq[s];
        T b = (T)X.gx[s];
#pragma unroll
        for (int u = 0; u < ROWS; ++u) b += (T)X.col[s][u] * (T)X.r[u];
        E.g[s] = b;
    }
}

// One point: cost and errors at q and, when it is taken (lane::eval_point1's
// rule), what its normal equations are formed from.  Whether it was taken.
template <int L, int KIND>
PK_DEV bool eval_point(const RobotC *__restrict__ rb, const SolveParams &P, const Lane<L, KIND> &Q,
                       const float *q, bool first, float cur, float &cost, float &pcost, float &perr,
                       float &rerr, Point<L, KIND> &X)
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
    float o[3], p;
#pragma unroll
    for (int j = 0; j < L; ++j) {
        float on[3], pn = Q.t0;
        const float s = from(so[j / 4], j % 4), c = from(co[j / 4], j % 4);
        if (j == 0)
            joint_turn_row(Q.g0[0], Q.g0[1], Q.g0[2], s, c, on);   // (the identity times it)
        else
            joint_step_row(o, p, Q.fr[j - 1], Q.fr[j - 1] + 9, s, c, on, pn);
        if (pris_of(KIND) && rb->j[j].type == PK_JOINT_PRISMATIC) pn += q[j] * on[2];   // joint_slide
#pragma unroll
        for (int u = 0; u < 3; ++u) o[u] = on[u];
        p = pn;
        Q.ex[j * G::JW + Q.row] = o[2];
        Q.ex[j * G::JW + 3 + Q.row] = p;
    }
    float Re[3], pe;
    ee_frame_row(o, p, Q.fr[L - 1], Q.fr[L - 1] + 9, Re, pe);
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
    if (!(first || cost < cur)) return false;

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
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int j = min(4 * s + Q.r, L - 1);
        float om[3], pj[3];
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            om[u] = Q.ex[j * G::JW + u];
            pj[u] = Q.ex[j * G::JW + 3 + u];
        }
        lane::jac_column<KIND>(P, M, N, om, pj, pev, pris_of(KIND) && Q.pris[s], X.col[s]);
        lane::joint_terms_at(P, qo[s], Q.lo[s], Q.hi[s], Q.qr[s], X.dq[s], X.gx[s]);
    }
    exchange();   // the next point's frames overwrite the area
#pragma unroll
    for (int u = 0; u < ROWS; ++u) X.r[u] = r[u];
    return true;
}

// x = -(A + lam diag(max(A_ii, floor)))^-1 g, whole on every lane: the values
// of lane::chol_damped and chol_solve_neg, the factor right-looking with its
// rows over the quad.  False if a pivot is not above thresh (or not finite).
template <int L, typename T>
PK_DEV bool solve(int r, const Normal<L, T> &E, T lam, T floor_, T thresh, T *x)
{
    constexpr int NS = Normal<L, T>::NS;
    T F[NS][L], ys[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        T dd = E.dg[s];
        dd += lam * (E.dg[s] > floor_ ? E.dg[s] : floor_);
#pragma unroll
        for (int k = 0; k < L; ++k) {
            if (k > 4 * s + 3) continue;
            F[s][k] = k >= 4 * s && r == k - 4 * s ? dd : E.A[s][k];
        }
        ys[s] = -E.g[s];
    }
    bool ok = true;
    T inv[L], y[L];
#pragma unroll
    for (int l = 0; l < L; ++l) {
        T d = from(F[l / 4][l], l % 4);
        if (!(d > thresh) || !(d < (T)INFINITY)) {
            ok = false;
            d = 1;
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
            const T lk = from(F[k / 4][l], k % 4);
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                if (k > 4 * s + 3) continue;
                F[s][k] -= F[s][l] * lk;
            }
        }
    }
#pragma unroll
    for (int i = L - 1; i >= 0; --i) {
        T t = y[i];
#pragma unroll
        for (int l = i + 1; l < L; ++l) t -= from(F[l / 4][i], l % 4) * x[l];
        x[i] = t * inv[i];
    }
    return ok;
}

// Damped step from the taken point: lane::lane_step's pivot test on the
// FP32 factor and the FP64 re-solve, here from the columns the point kept
// (the per-lane kernel, short of registers, forms them again).  False if
// that fails too.
template <int L, int KIND>
PK_DEV bool step(const SolveParams &P, int r, const Point<L, KIND> &X, const Normal<L, float> &E, float lam,
                 int &flags, float *delta)
{
    constexpr int NS = Geo<L, KIND>::NS;
    float dmax = 0.f;
#pragma unroll
    for (int s = 0; s < NS; ++s) dmax = fmaxf(dmax, E.dg[s] + lam * fmaxf(E.dg[s], P.damping_floor));
    dmax = quad_max(dmax);
    if (solve<L, float>(r, E, lam, P.damping_floor, P.pivot_rel * dmax, delta)) return true;
    flags |= PK_FLAG_FP64;
    Normal<L, double> D;
    double x[L];
    form_normal<L, KIND, double>(r, X, D);
    const bool ok = solve<L, double>(r, D, (double)lam, (double)P.damping_floor, 0.0, x);
#pragma unroll
    for (int j = 0; j < L; ++j) delta[j] = (float)x[j];
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
#pragma unroll
    for (int u = 0; u < 3; ++u) Q.g0[u] = rb->j[0].G[3 * Q.row + u];
    Q.t0 = rb->j[0].t[Q.row];
#pragma unroll
    for (int j = 1; j <= L; ++j)
#pragma unroll
        for (int u = 0; u < 12; ++u) {
            Q.fr[j - 1][u] = j < L ? (u < 9 ? rb->j[j].G[u] : rb->j[j].t[u - 9])
                                   : (u < 9 ? rb->e[0].G[u] : rb->e[0].t[u - 9]);
            asm("" : "+v"(Q.fr[j - 1][u]));     // in vector registers over the whole solve
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
    Point<L, KIND> X;
    Normal<L, float> E;
#pragma unroll
    for (int j = 0; j < L; ++j) qt[j] = q[j];
    for (;;) {
        bool ok = true;
        if (!first) {
            float delta[L];
            ok = step<L, KIND>(P, Q.r, X, E, lam, flags, delta);
#pragma unroll
            for (int j = 0; j < L; ++j) qt[j] = q[j] + delta[j];
        }
        float ct = INFINITY, pct = 0.f, pe_t[1] = {0.f}, re_t[1] = {0.f};
        if (ok && eval_point<L, KIND>(rb, P, Q, qt, first, cost, ct, pct, pe_t[0], re_t[0], X))
            form_normal<L, KIND, float>(Q.r, X, E);
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

// Up to 64 problems per workgroup of four wavefronts; with B's pointers set,
// whole targets per workgroup (K at most 64) and their best-of-K as well.
template <int L, int KIND>
__global__ __launch_bounds__(THREADS) void lm_quad_kernel(const RobotC *__restrict__ rb,
                                                          const float *__restrict__ qr, SolveParams P,
                                                          BestOut B, int per_block)
{
    using G = Geo<L, KIND>;
    __shared__ __attribute__((aligned(16))) float smem[G::FLOATS];
    __shared__ float bc[PROBLEMS], bp[PROBLEMS];
    __shared__ int bv[PROBLEMS];
    const int slot = threadIdx.x >> 2;
    const int64_t p = (int64_t)blockIdx.x * per_block + slot;
    const bool live = slot < per_block && p < P.N;
    LaneFinal<L> fin;
    if (live) quad_problem<L, KIND>(rb, qr, P, smem, p, &fin);
    if (!(B.index || B.joints || B.success)) return;   // uniform
    if (live && (threadIdx.x & 3) == 0) {
        bc[slot] = fin.cost;
        bp[slot] = fin.pcost;
        bv[slot] = fin.conv ? PK_CONVERGED : PK_MAX_ITERS;
    }
    __syncthreads();
    if (!live) return;
    const int K = P.K, first = slot / K * K;
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
    if (best && P.K > PROBLEMS) return hipErrorInvalidValue;
    const BestOut B = best ? *best : BestOut{nullptr, nullptr, nullptr};
    const int per_block = lane::quad_per_block(P.K, best != nullptr);
    const dim3 grid((unsigned)((P.N + per_block - 1) / per_block));
    hipLaunchKernelGGL((lm_quad_kernel<L, KIND>), grid, dim3(THREADS), 0, s, rb, qr, P, B, per_block);
    return hipGetLastError();
}

}  // namespace quad
}  // namespace pk
