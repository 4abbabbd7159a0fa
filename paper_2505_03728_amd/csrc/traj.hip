// Trajectory optimisation: LM over a trajectory of T configurations of a
// single-chain robot (Sec. II: a configuration interacts only with its
// temporal neighbours, so the normal equations are banded).  One trajectory
// per workgroup of four wavefronts:
//   * lanes 0 and 1 run FK, the pose log and the pose Jacobian at the first
//     and the last configuration (start and goal pose costs);
//   * every thread takes its share of the T*n variables for the limit,
//     smoothness, velocity-limit and five-point acceleration/jerk terms;
//   * J^T J is banded (half-bandwidth 4n in time-major order): it is formed
//     straight into a band in LDS, damped, factored by a band L D L^T
//     blocked by timestep and solved, all in FP64: the jerk rows outweigh
//     the smoothness rows by ~1e5 in J^T J, and at that conditioning an FP32
//     factorisation steers LM off the FP64 path (FP64 FMAs issue at the
//     unpacked FP32 rate).
#include <stddef.h>
#include <string.h>

#include <cmath>

#include "pk_ctx.hpp"
#include "pk_device.hpp"

namespace pk {
namespace {

constexpr int TRAJ_VMAX = 256;   // T * n variables per trajectory
constexpr int TRAJ_THREADS = 256; // four wavefronts per trajectory

struct TrajParams {
    int64_t B;
    int T;
    float dt, w_pos, w_rot, w_limit, w_smooth, w_vel, w_acc, w_jerk;
    const float *vmax;                 // [n] or null (no velocity-limit term)
    const float *start, *goal;         // [7][B]: p, quaternion wxyz
    const float *init;                 // [B][T][n]
    float *out;                        // [B][T][n]
    float *cost, *pos_err, *rot_err;   // [B], [2][B], [2][B]
    int32_t *iters, *accepts, *status;
    float lambda0, nu_up, nu_down, lambda_min, lambda_max, tol_pos, tol_rot, damping_floor,
        pivot_rel;
    int max_iters, early_exit;
};

// Five-point stencils on offsets -2..2: second derivative times dt^2 and
// third derivative times dt^3 (copied to LDS per workgroup).
constexpr float ACC5[5] = {-1.f / 12.f, 16.f / 12.f, -30.f / 12.f, 16.f / 12.f, -1.f / 12.f};
constexpr float JERK5[5] = {-0.5f, 1.f, 0.f, -1.f, 0.5f};

template <int NJ>
struct TrajLds {
    static constexpr int HB = 4 * NJ, W = HB + 1;
    static constexpr int NPAIR = HB * (HB + 1) / 2;
    double b[TRAJ_VMAX];
    double invd[TRAJ_VMAX];                            // 1 / D_j of the L D L^T factorisation
    double dump[64];                                   // where masked stores go
    static constexpr int NX = (NJ + 1) / 2 * 2;
    double next[(NJ + 1) * NX];                        // the next block's rows of the block just eliminated (+ dump row)
    float Q[TRAJ_VMAX], Qt[TRAJ_VMAX];
    float J0[6 * NJ], J1[6 * NJ], r0[6], r1[6];        // pose rows at the current point
    float Jt0[6 * NJ], Jt1[6 * NJ], rt0[6], rt1[6];    // ... at the trial point
    float err[4], errt[4];                             // pos/rot errors (start, goal)
    // per-joint limits and allowed step, the stencils: read per band entry,
    // so they sit in LDS rather than behind lane-indexed global loads
    float lo[NJ], hi[NJ], vdt[NJ], acc5[5], jerk5[5];
    float red[4];                                      // per-wavefront partials of a reduction
    // the part of the normal matrix that does not depend on the trajectory:
    // smoothness and the two stencils, A(t, t - dtk) per joint at t * 5 + dtk
    double ctab[5 * (TRAJ_VMAX / NJ)];
    float racc[TRAJ_VMAX], rjerk[TRAJ_VMAX];          // stencil rows at the current point
    int fail;                                          // a pivot failed in the factorisation
    // A(v, v - k) at v * W + k.  The factorisation reads some entries beside
    // the band before it discards them: up to 64 past its end, and up to 16
    // rows before its start (the arrays above).
    double band[TRAJ_VMAX * W + 64];
    // What those indices rely on: masked stores reach the dump from invd and from
    // b, and the backward solve's last chunk reads 15 rows of diagonals above row 0.
    static constexpr bool laid_out()
    {
        return offsetof(TrajLds, invd) == offsetof(TrajLds, b) + sizeof(b) &&
               offsetof(TrajLds, dump) == offsetof(TrajLds, invd) + sizeof(invd) &&
               offsetof(TrajLds, band) >= 15 * (W + 1) * sizeof(double) && offsetof(TrajLds, band) % sizeof(double) == 0;
    }
};

PK_DEV float wsum(float v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

PK_DEV float wmax(float v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}

// Sum and maximum over the workgroup (four wavefronts): butterflies within
// each wavefront, then the four partials through LDS, added in one order so
// that every thread gets the same value.
PK_DEV float block_sum(float v, float *red)
{
    v = wsum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return (red[0] + red[1]) + (red[2] + red[3]);
}

PK_DEV float block_max(float v, float *red)
{
    v = wmax(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}

// FK of the chain at q (NJ values), the pose residual rows against target
// tp (p, quaternion) and, with jac, the weighted pose Jacobian [6][NJ].
template <int NJ>
PK_DEV void endpoint(const RobotC *__restrict__ rb, const TrajParams &P, const float *q,
                     const float *tp, float *r6, float *J, float &perr, float &rerr)
{
    float O[9] = {1.f, 0.f, 0.f, 0.f, 1.f, 0.f, 0.f, 0.f, 1.f}, p[3] = {0.f, 0.f, 0.f};
    float om[NJ][3], pj[NJ][3];
#pragma unroll
    for (int i = 0; i < NJ; ++i) {
        const bool pri = rb->j[i].type == PK_JOINT_PRISMATIC;
        float s = 0.f, c = 1.f, On[9], pn[3];
        if (!pri) joint_sincos(q[i], s, c);
        joint_step(O, p, rb->j[i].G, rb->j[i].t, s, c, On, pn);
        if (pri) joint_slide(On, q[i], pn);
#pragma unroll
        for (int u = 0; u < 9; ++u) O[u] = On[u];
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            p[u] = pn[u];
            om[i][u] = O[3 * u + 2];
            pj[i][u] = p[u];
        }
    }
    float Re[9], pe[3], Rt[9], d[3];
    ee_frame(O, p, rb->e[0].G, rb->e[0].t, Re, pe);
#pragma unroll
    for (int u = 0; u < 3; ++u) d[u] = pe[u] - tp[u];
    perr = sqrtf(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
    quat_to_rot(tp[3], tp[4], tp[5], tp[6], Rt);
    const PoseLog lg = pose_log(Rt, Re, d);
    rerr = lg.theta;
#pragma unroll
    for (int u = 0; u < 3; ++u) {
        r6[u] = P.w_pos * lg.rho[u];
        r6[3 + u] = P.w_rot * lg.phi[u];
    }
    float M[9], Nb[9];
    jr_inv_blocks(lg, Re, M, Nb);
#pragma unroll
    for (int i = 0; i < NJ; ++i) {
        float v[3], w[3];
        joint_twist(rb->j[i].type == PK_JOINT_PRISMATIC, om[i], pj[i], pe, v, w);
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            const float mv = M[3 * u] * v[0] + M[3 * u + 1] * v[1] + M[3 * u + 2] * v[2];
            const float nw = Nb[3 * u] * w[0] + Nb[3 * u + 1] * w[1] + Nb[3 * u + 2] * w[2];
            const float mw = M[3 * u] * w[0] + M[3 * u + 1] * w[1] + M[3 * u + 2] * w[2];
            J[u * NJ + i] = P.w_pos * (mv + nw);
            J[(3 + u) * NJ + i] = P.w_rot * mw;
        }
    }
}

// Per-variable pieces at Q: limit residual and derivative, and the
// velocity-limit residual and sign of the step into timestep t.
template <int NJ>
PK_DEV void limit_row(const TrajLds<NJ> &S, const TrajParams &P, float q, int i, float &rl, float &dl)
{
    const float over = q - S.hi[i], under = S.lo[i] - q;
    rl = P.w_limit * (fmaxf(over, 0.f) + fmaxf(under, 0.f));
    const float wl = P.w_limit;
    dl = over > 0.f ? wl : (under > 0.f ? -wl : 0.f);
}

template <int NJ>
PK_DEV void vel_row(const TrajLds<NJ> &S, const TrajParams &P, const float *Q, int v, int i, float &rv,
                    float &sv)
{
    const float d = Q[v] - Q[v - NJ];
    const float ex = fabsf(d) - S.vdt[i];
    rv = ex > 0.f ? P.w_vel * ex : 0.f;
    sv = ex > 0.f ? (d > 0.f ? P.w_vel : -P.w_vel) : 0.f;
}

PK_DEV float acc_row(const TrajParams &P, const float *Q, int v, int n)
{
    float a = 0.f;
#pragma unroll
    for (int k = 0; k < 5; ++k) a += ACC5[k] * Q[v + (k - 2) * n];
    return a * (P.w_acc / (P.dt * P.dt));
}

PK_DEV float jerk_row(const TrajParams &P, const float *Q, int v, int n)
{
    float a = 0.f;
#pragma unroll
    for (int k = 0; k < 5; ++k) a += JERK5[k] * Q[v + (k - 2) * n];
    return a * (P.w_jerk / (P.dt * P.dt * P.dt));
}

// Sum of squares of the non-pose rows at Q (every lane; wave total).
template <int NJ>
PK_DEV float path_cost(TrajLds<NJ> &S, const TrajParams &P, const float *Q, int lane)
{
    const int T = P.T, V = T * NJ;
    float s = 0.f;
    for (int v = lane; v < V; v += TRAJ_THREADS) {
        const int t = v / NJ, i = v - t * NJ;
        float rl, dl;
        limit_row<NJ>(S, P, Q[v], i, rl, dl);
        s += rl * rl;
        if (t >= 1) {
            const float rs = P.w_smooth * (Q[v] - Q[v - NJ]);
            s += rs * rs;
            if (P.vmax) {
                float rv, sv;
                vel_row<NJ>(S, P, Q, v, i, rv, sv);
                s += rv * rv;
            }
        }
        if (t >= 2 && t <= T - 3) {
            const float ra = acc_row(P, Q, v, NJ), rj = jerk_row(P, Q, v, NJ);
            s += ra * ra + rj * rj;
        }
    }
    return block_sum(s, S.red);
}

// Band of A + lambda diag(max(A_vv, floor)) and the right-hand side -J^T r at
// the current point, in precision T: A(v, v - k) at band[v * W + k].
template <int NJ, typename T>
PK_DEV void form_system(const RobotC *__restrict__ rb, const TrajParams &P, TrajLds<NJ> &S,
                        float lam, int lane, T *band, T *rhs)
{
    constexpr int W = TrajLds<NJ>::W;
    const int TT = P.T, V = TT * NJ;
    const T sa = (T)P.w_acc / ((T)P.dt * (T)P.dt), sj = (T)P.w_jerk / ((T)P.dt * (T)P.dt * (T)P.dt);
    for (int v = lane; v < V; v += TRAJ_THREADS) {
        const int t = v / NJ;
        if (t >= 2 && t <= TT - 3) {
            S.racc[v] = acc_row(P, S.Q, v, NJ);
            S.rjerk[v] = jerk_row(P, S.Q, v, NJ);
        }
    }
    // one band row per thread: A(v, v - k) for k = 0 .. W-1.  Nonzero are the
    // same joint's entries (k a multiple of NJ: smoothness, stencils, the
    // velocity rows and, on the diagonal, the limit row) and, at the first
    // and the last timestep, the pose block (k <= i); the rest is zero.
    for (int v = lane; v < V; v += TRAJ_THREADS) {
        const int t = v / NJ, i = v - t * NJ;
        float rl, dl, rv = 0.f, sv = 0.f, rv1 = 0.f, sv1 = 0.f;
        limit_row<NJ>(S, P, S.Q[v], i, rl, dl);
        if (P.vmax) {   // velocity rows tau = t and tau = t + 1, where active
            if (t >= 1) vel_row<NJ>(S, P, S.Q, v, i, rv, sv);
            if (t + 1 <= TT - 1) vel_row<NJ>(S, P, S.Q, v + NJ, i, rv1, sv1);
        }
        const bool endp = t == 0 || t == TT - 1;
        const float *J = t == 0 ? S.J0 : S.J1;
        T *row = band + v * W;
#pragma unroll
        for (int k = 0; k < W; ++k) {
            T a = 0;
            if (v - k >= 0) {
                if (k % NJ == 0) {
                    a = (T)S.ctab[t * 5 + k / NJ];
                    if (k == 0) {
                        a += (T)dl * (T)dl;
                        a += (T)sv * (T)sv + (T)sv1 * (T)sv1;
                    }
                    if (k == NJ) a -= (T)sv * (T)sv;
                }
                if (k < NJ && endp && k <= i) {
#pragma unroll
                    for (int r = 0; r < 6; ++r) a += (T)J[r * NJ + i] * (T)J[r * NJ + i - k];
                }
                if (k == 0) a += (T)lam * (a > (T)P.damping_floor ? a : (T)P.damping_floor);
            }
            row[k] = a;
        }
    }
    __syncthreads();   // stencil rows
    for (int v = lane; v < V; v += TRAJ_THREADS) {
        const int t = v / NJ, i = v - t * NJ;
        T g = 0;
        float rl, dl;
        limit_row<NJ>(S, P, S.Q[v], i, rl, dl);
        g += (T)dl * (T)rl;
        if (t >= 1) g += (T)P.w_smooth * (T)P.w_smooth * ((T)S.Q[v] - (T)S.Q[v - NJ]);
        if (t <= TT - 2) g -= (T)P.w_smooth * (T)P.w_smooth * ((T)S.Q[v + NJ] - (T)S.Q[v]);
        if (P.vmax) {
            float rv, sv;
            if (t >= 1) {
                vel_row<NJ>(S, P, S.Q, v, i, rv, sv);
                g += (T)sv * (T)rv;
            }
            if (t <= TT - 2) {
                vel_row<NJ>(S, P, S.Q, v + NJ, i, rv, sv);
                g -= (T)sv * (T)rv;
            }
        }
        for (int tc = t - 2; tc <= t + 2; ++tc) {
            if (tc < 2 || tc > TT - 3) continue;
            const int o = t - tc + 2, vc = tc * NJ + i;
            g += sa * (T)S.acc5[o] * (T)S.racc[vc] + sj * (T)S.jerk5[o] * (T)S.rjerk[vc];
        }
        if (t == 0 || t == TT - 1) {
            const float *J = t == 0 ? S.J0 : S.J1;
            const float *r = t == 0 ? S.r0 : S.r1;
#pragma unroll
            for (int q = 0; q < 6; ++q) g += (T)J[q * NJ + i] * (T)r[q];
        }
        rhs[v] = -g;
    }
}

// The part of a block step's trailing triangle beyond the next block's
// columns: entries (R, R2) = (c0 + NJ - 1 + di, c0 + NJ - 1 + dk) with
// NJ < dk <= di <= HB, spread over wavefronts 1..3.
template <int NJ>
struct Pairs {
    static constexpr int HB = TrajLds<NJ>::HB;
    static constexpr int NB = (HB - NJ) * (HB - NJ + 1) / 2;
    static constexpr int PB = (NB + TRAJ_THREADS - 64 - 1) / (TRAJ_THREADS - 64);
};

// Entries p = t + stride m of the part with dk in [dlo, HB], listed dk-major
// (di = dk .. HB within a dk), packed di | dk << 8; 0 for t < 0 and past total.
template <int NJ, int M>
PK_DEV void part_pairs(int t, int stride, int dlo, int total, int (&mp)[M])
{
    constexpr int HB = TrajLds<NJ>::HB;
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const int p = t + stride * m;
        int dk = dlo, rem = p;
        while (dk <= HB && rem >= HB - dk + 1) {
            rem -= HB - dk + 1;
            ++dk;
        }
        mp[m] = t >= 0 && p < total ? ((dk + rem) | (dk << 8)) : 0;
    }
}

// Rank-NJ update of the listed entries of the trailing triangle of the block
// step at c0: A(R, R2) -= sum_cc A(R, cc) A(R2, cc) / D_cc over the block's
// columns (unscaled entries).  Addresses are clamped into the band so that
// every load is issued unconditionally; padding entries store nothing.
template <int NJ, typename T, int M>
PK_DEV void trail(T *band, const T *invd, int V, int c0_, const int (&mp)[M])
{
    constexpr int HB = TrajLds<NJ>::HB, W = TrajLds<NJ>::W;
    // the block offset as an opaque uniform value: addresses are recomputed
    // per block step rather than carried as induction variables across the
    // factorisation (which spilled them)
    const int c0 = __builtin_amdgcn_readfirstlane(c0_);
    T dinv[NJ];
#pragma unroll
    for (int cc = 0; cc < NJ; ++cc) dinv[cc] = invd[c0 + cc];
#pragma unroll
    for (int m = 0; m < M; ++m) {
        // likewise for the pair: its offsets are derived here, not hoisted
        int pm = mp[m];
        asm volatile("" : "+v"(pm));
        const int di = pm & 0xff, dk = pm >> 8;
        const int R = c0 + NJ - 1 + di, R2 = c0 + NJ - 1 + dk;
        const bool ok = di && R < V;
        const int Rc = min(R, V - 1), R2c = min(R2, V - 1);
        // every load first (the target included), so that they are in flight
        // together; the band-edge selects come after
        T a1[NJ], a2[NJ];
#pragma unroll
        for (int cc = 0; cc < NJ; ++cc) {
            a1[cc] = band[Rc * W + min(NJ - 1 + di - cc, HB)];
            a2[cc] = band[R2c * W + min(NJ - 1 + dk - cc, HB)];
        }
        const T tv = band[Rc * W + (di - dk)];
        T term[NJ];
#pragma unroll
        for (int cc = 0; cc < NJ; ++cc) {
            const int k1 = NJ - 1 + di - cc, k2 = NJ - 1 + dk - cc;
            term[cc] = (k1 <= HB ? a1[cc] : (T)0) * dinv[cc] * (k2 <= HB ? a2[cc] : (T)0);
        }
        // pairwise sum: a short dependent chain
#pragma unroll
        for (int w = 1; w < NJ; w *= 2)
#pragma unroll
            for (int cc = 0; cc + w < NJ; cc += 2 * w) term[cc] += term[cc + w];
        if (ok) band[R * W + (di - dk)] = tv - term[0];
    }
}

// Value of v in lane l (l uniform) broadcast to the wavefront.
PK_DEV double readlane_d(double v, int l)
{
    const long long u = __double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, l);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), l);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// 1 / d for a positive normal d: the hardware reciprocal estimate refined by
// one Newton-Raphson step r <- r + r (1 - d r), which squares its relative
// error (measured on gfx950 over 2^20 values across 60 binades: below
// 2^-24.4 for the estimate, below 2^-48.7 after the step).  It sits on the
// factorisation's dependent chain; the solution is rounded to FP32 anyway.
PK_DEV double recip(double d)
{
    const double r = __builtin_amdgcn_rcp(d);
    return fma(r, fma(-d, r, 1.0), r);
}

// Columns c0 .. c0 + NJ - 1 of the factor scaled by 1 / D (wavefronts 1..3,
// thread t of them).
template <int NJ>
PK_DEV void scale_columns(double *band, const double *invd, int V, int c0, int t)
{
    constexpr int HB = TrajLds<NJ>::HB, W = TrajLds<NJ>::W;
#pragma unroll
    for (int e0 = 0; e0 < NJ * HB; e0 += TRAJ_THREADS - 64) {
        const int e = e0 + t, cc = e / HB, k = e % HB + 1, R = c0 + cc + k;
        if (e < NJ * HB && R < V) band[R * W + k] *= invd[c0 + cc];
    }
}

// In-place band L D L^T factorisation of S.band (half-bandwidth HB, unit L)
// and the solve of L D L^T x = rhs (x over S.b).  A pivot D_j not above
// thresh_rel times the largest damped diagonal fails the factorisation
// (returns false).  No square roots.
//
// Bound: the dependent chain of pivots, so the first wavefront runs it with
// as little in between as possible: no branches (a masked store goes to the
// lane's own slot of a dump) and one workgroup barrier per block of NJ
// columns.  Row R lives in lane R mod 64 while it is
// in the window of a block (the block's rows and the HB rows below),
// restricted to the block's columns, with the right-hand side as one more
// column (the forward substitution).  Per block the first wavefront
//   * eliminates the NJ columns in registers, broadcasting each pivot row's
//     entries with readlane, and stores them (unscaled entries D_j L_ij);
//   * after the barrier applies the rank-NJ update to the next block's
//     columns in registers, the multiplying rows read back from LDS by every
//     lane alike (the loads issued before the barrier; by readlane this phase
//     took twice as long),
// while wavefronts 1..3 apply the rest of the block's update to the columns
// beyond (disjoint entries) and scale finished columns by 1 / D_j.
// The backward solve L^T x = D^-1 y runs on the first wavefront with row i in
// lane i mod 64 (a finished entry reaches the HB rows above it only): per
// step one readlane pair and one FMA depend on the step before.
// With two barriers per block, the next block's columns updated through LDS
// by the whole workgroup and two register slots per lane in the backward
// solve, 1024 trajectories of 32 x 7 variables took 3.10 ms and 37 of 25 x 6
// (one workgroup's time) 0.979 ms; now 2.74 and 0.805.  (7 joints: 20 of the 256
// registers' values are spilled, reloaded once per iteration.)
template <int NJ>
PK_DEV bool band_solve(TrajLds<NJ> &S, int V, float thresh_rel, const int (&mpb)[Pairs<NJ>::PB], int tid)
{
    constexpr int HB = TrajLds<NJ>::HB, W = TrajLds<NJ>::W, NR = NJ + HB, NX = TrajLds<NJ>::NX, CH = 16;
    static_assert(TrajLds<NJ>::laid_out(), "indices beside b, invd and band stay in S");
    static_assert(NR + NJ <= 64, "the windows of a block and the next fit one wavefront");
    static_assert(HB + CH < 64, "a finished row's lane takes its next row before that is updated");
    double *band = S.band, *rhs = S.b, *invd = S.invd;
    float mx = 0.f;
    for (int v = tid; v < V; v += TRAJ_THREADS) mx = fmaxf(mx, (float)band[v * W]);
    const double thresh = (double)thresh_rel * (double)block_max(mx, S.red);
    if (tid == 0) S.fail = 0;
    // (a scalar branch: every wavefront passes one barrier per block)
    if (__builtin_amdgcn_readfirstlane(tid >> 6) != 0) {
        for (int c0 = 0; c0 < V; c0 += NJ) {
            __syncthreads();
            trail<NJ, double>(band, invd, V, c0, mpb);
            if (c0 > 0) scale_columns<NJ>(band, invd, V, c0 - NJ, tid - 64);
        }
        scale_columns<NJ>(band, invd, V, V - NJ, tid - 64);
    } else {
        const int lane = tid, dump = (int)(&S.dump[lane] - band);   // as an index of the band
        bool bad = false;
        double x[NJ], bv;
#pragma unroll
        for (int cc = 0; cc < NJ; ++cc) {
            const bool ok = (unsigned)(lane - cc) <= (unsigned)HB && lane < V;
            const double v = band[ok ? lane * W + lane - cc : 0];
            x[cc] = ok ? v : 0.0;
        }
        bv = rhs[min(lane, V - 1)];
        for (int c0_ = 0; c0_ < V; c0_ += NJ) {
            // (opaque and uniform: addresses are formed per block, not carried)
            const int c0 = __builtin_amdgcn_readfirstlane(c0_);
            const int r = (lane - c0) & 63, R = c0 + r;
            double inv[NJ];
#pragma unroll
            for (int jj = 0; jj < NJ; ++jj) {
                // a failed pivot discards the whole factorisation, so the
                // test stays off the dependent chain
                const int pl = (c0 + jj) & 63;
                const double d = readlane_d(x[jj], pl);
                bad |= !(d > thresh) || !(d < (double)INFINITY);
                inv[jj] = recip(d);
                const double ell = r > jj ? x[jj] : 0.0;   // unscaled D_jj L_(R, jj)
#pragma unroll
                for (int cc = jj + 1; cc < NJ; ++cc)
                    x[cc] -= ell * (readlane_d(x[jj], (c0 + cc) & 63) * inv[jj]);
                bv -= ell * (readlane_d(bv, pl) * inv[jj]);
            }
            {   // the next block's rows, for every lane to read back
                const int n = r >= NJ && r < 2 * NJ ? r - NJ : NJ;
#pragma unroll
                for (int cc = 0; cc < NJ; ++cc) S.next[n * NX + cc] = x[cc];
            }
            const int rw = R < V ? r : 127;            // rows past the end store nothing
#pragma unroll
            for (int cc = 0; cc < NJ; ++cc)
                band[(unsigned)(rw - cc) <= (unsigned)HB ? R * W + r - cc : dump] = x[cc];
            double iv = inv[0];
#pragma unroll
            for (int jj = 1; jj < NJ; ++jj) iv = r == jj ? inv[jj] : iv;
            invd[r < NJ ? R : TRAJ_VMAX + lane] = iv;              // (else the dump, which follows)
            rhs[r < NJ ? R : 2 * TRAJ_VMAX + lane] = bv;
            double a2[NJ][NX];
#pragma unroll
            for (int i = 0; i < NJ; ++i)
#pragma unroll
                for (int cc = 0; cc < NX; ++cc) a2[i][cc] = S.next[i * NX + cc];
            __builtin_amdgcn_sched_barrier(0);         // (all in flight, not one by one where they are used)
            __syncthreads();
            if (c0 + NJ >= V) break;
            // the next block's columns: rows R1 (this lane) x c0 + NJ + i
            const int r1 = (lane - c0 - NJ) & 63, R1 = min(c0 + NJ + r1, V - 1);
            double tv[NJ], m[NJ];
#pragma unroll
            for (int i = 0; i < NJ; ++i) tv[i] = band[R1 * W + r1 - i];   // (in S where not in the band)
            const double bn = rhs[R1];
            bv = r1 >= NR - NJ ? bn : bv;              // rows entering the window
#pragma unroll
            for (int cc = 0; cc < NJ; ++cc) m[cc] = x[cc] * inv[cc];
#pragma unroll
            for (int i = 0; i < NJ; ++i) {
                double term[NJ];
#pragma unroll
                for (int cc = 0; cc < NJ; ++cc) term[cc] = m[cc] * a2[i][cc];
                // pairwise sum: a short dependent chain
#pragma unroll
                for (int w = 1; w < NJ; w *= 2)
#pragma unroll
                    for (int cc = 0; cc + w < NJ; cc += 2 * w) term[cc] += term[cc + w];
                tv[i] -= term[0];
            }
#pragma unroll
            for (int i = 0; i < NJ; ++i) x[i] = (unsigned)(r1 - i) <= (unsigned)HB ? tv[i] : 0.0;
        }
        if (bad && lane == 0) S.fail = 1;
    }
    __syncthreads();
    if (S.fail) return false;
    // S.b now holds y of L y = rhs (forward substitution rode along with the
    // elimination), S.band L
    if (__builtin_amdgcn_readfirstlane(tid >> 6) == 0) {
        const int lane = tid;
        // row i of the 64 up to j: i = j - ((j - lane) mod 64); D z = y
        auto row = [&](int i) { return i >= 0 ? rhs[max(i, 0)] * invd[max(i, 0)] : 0.0; };
        double x = row(V - 1 - ((V - 1 - lane) & 63));
        double c[CH], cn[CH];
        // entries L(j0 - u, row of this lane), 0 outside the band: every load
        // at its place on the row's diagonal, then the selects
        auto load = [&](double(&o)[CH], int j0) {
            const int k0 = (j0 - lane) & 63, kk = k0 <= j0 ? k0 : -1;
            const double *p = band + max(j0, 0) * W + k0;
#pragma unroll
            for (int u = 0; u < CH; ++u) o[u] = p[-u * (W + 1)];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < CH; ++u) o[u] = (unsigned)(kk - u - 1) < (unsigned)HB ? o[u] : 0.0;
        };
        load(c, V - 1);
        for (int j0_ = V - 1; j0_ >= 0; j0_ -= CH) {
            const int j0 = __builtin_amdgcn_readfirstlane(j0_);
            const int q = (j0 - lane) & 63, i = j0 - q;
            const double z = row(i - 64);
            load(cn, j0 - CH);
#pragma unroll
            for (int u = 0; u < CH; ++u) {
                const double y = readlane_d(x, (j0 - u) & 63);
                x -= c[u] * y;
            }
            // the chunk's rows are finished; their lanes take the rows 64 above
            rhs[q < CH && i >= 0 ? i : 2 * TRAJ_VMAX + lane] = x;
            x = q < CH ? z : x;
#pragma unroll
            for (int u = 0; u < CH; ++u) c[u] = cn[u];
        }
    }
    __syncthreads();
    return true;
}

// Two workgroups per CU where their LDS fits (up to 7 joints), which also
// holds the register budget to 256 per lane.
template <int NJ>
__global__ __launch_bounds__(TRAJ_THREADS, NJ <= 7 ? 2 : 1) void traj_kernel(const RobotC *__restrict__ rb,
                                                                             TrajParams P)
{
    using L = TrajLds<NJ>;
    __shared__ L S;
    const int lane = threadIdx.x;
    const int64_t b = blockIdx.x;
    if (b >= P.B) return;   // uniform per workgroup
    const int TT = P.T, V = TT * NJ;
    int mpb[Pairs<NJ>::PB];
    part_pairs<NJ>(lane - 64, TRAJ_THREADS - 64, NJ + 1, Pairs<NJ>::NB, mpb);
    const float *src = P.init + b * (int64_t)V;
    for (int v = lane; v < V; v += TRAJ_THREADS) S.Q[v] = src[v];
    if (lane < NJ) {
        S.lo[lane] = rb->j[lane].lo;
        S.hi[lane] = rb->j[lane].hi;
        S.vdt[lane] = P.vmax ? P.vmax[lane] * P.dt : 0.f;
    }
    if (lane < 5) {
        S.acc5[lane] = ACC5[lane];
        S.jerk5[lane] = JERK5[lane];
    }
    {
        // smoothness rows q_tau - q_{tau-1} (tau = 1..T-1), then the
        // acceleration and jerk rows centred at tc = 2..T-3
        const double ws2 = (double)P.w_smooth * (double)P.w_smooth;
        const double sa = (double)P.w_acc / ((double)P.dt * (double)P.dt);
        const double sj = (double)P.w_jerk / ((double)P.dt * (double)P.dt * (double)P.dt);
        for (int x = lane; x < 5 * P.T; x += TRAJ_THREADS) {
            const int t = x / 5, dtk = x - 5 * t, t2 = t - dtk;
            double a = 0;
            if (dtk == 0) a += (t >= 1 ? ws2 : 0.0) + (t <= P.T - 2 ? ws2 : 0.0);
            if (dtk == 1) a -= ws2;
            for (int tc = t - 2; tc <= t2 + 2; ++tc) {
                if (tc < 2 || tc > P.T - 3) continue;
                const int o1 = t - tc + 2, o2 = t2 - tc + 2;
                a += sa * sa * (double)ACC5[o1] * (double)ACC5[o2] +
                     sj * sj * (double)JERK5[o1] * (double)JERK5[o2];
            }
            S.ctab[x] = a;
        }
    }
    __syncthreads();

    float tgt[7];
    const float *tplane = lane == 0 ? P.start : P.goal;
#pragma unroll
    for (int u = 0; u < 7; ++u) tgt[u] = tplane[(int64_t)u * P.B + b];

    int iters = 0, accepts = 0;
    bool stalled = false, done = false, first = true, evaluate = true;
    float lam = P.lambda0, cost = 0.f;
    // Each pass evaluates one point (first the initial trajectory, then each
    // trial), takes or rejects it, then forms and solves the next step; a
    // failed solve is a rejected trial.  All decisions are workgroup-uniform.
    for (;;) {
        bool acc = false;
        if (evaluate) {
            const float *Qe = first ? S.Q : S.Qt;
            if (lane < 2) {
                float q[NJ], perr, rerr;
                const int t = lane == 0 ? 0 : TT - 1;
#pragma unroll
                for (int i = 0; i < NJ; ++i) q[i] = Qe[t * NJ + i];
                endpoint<NJ>(rb, P, q, tgt, lane == 0 ? S.rt0 : S.rt1, lane == 0 ? S.Jt0 : S.Jt1,
                             perr, rerr);
                S.errt[lane] = perr;
                S.errt[2 + lane] = rerr;
            }
            const float pc = path_cost<NJ>(S, P, Qe, lane);
            __syncthreads();
            float pose = 0.f;
#pragma unroll
            for (int u = 0; u < 6; ++u) pose += S.rt0[u] * S.rt0[u] + S.rt1[u] * S.rt1[u];
            const float ct = pc + pose;
            acc = first || ct < cost;
            if (acc) {
                if (!first)
                    for (int v = lane; v < V; v += TRAJ_THREADS) S.Q[v] = S.Qt[v];
                for (int e = lane; e < 6 * NJ; e += TRAJ_THREADS) {
                    S.J0[e] = S.Jt0[e];
                    S.J1[e] = S.Jt1[e];
                }
                if (lane < 6) {
                    S.r0[lane] = S.rt0[lane];
                    S.r1[lane] = S.rt1[lane];
                }
                if (lane < 4) S.err[lane] = S.errt[lane];
                cost = ct;
            }
        }
        if (!first) {
            ++iters;
            if (acc) {
                lam = fmaxf(lam / P.nu_down, P.lambda_min);
                ++accepts;
            } else {
                if (lam >= P.lambda_max) {
                    stalled = true;
                    done = true;
                }
                lam = fminf(lam * P.nu_up, P.lambda_max);
            }
        }
        if (acc && P.early_exit && S.errt[0] <= P.tol_pos && S.errt[1] <= P.tol_pos &&
            S.errt[2] <= P.tol_rot && S.errt[3] <= P.tol_rot)
            done = true;
        first = false;
        __syncthreads();
        if (done || iters >= P.max_iters) break;
        // damped step from the current point (a pivot test failure is a
        // rejected trial, as when the IK re-solve fails)
        form_system<NJ, double>(rb, P, S, lam, lane, S.band, S.b);
        __syncthreads();
        const bool ok = band_solve<NJ>(S, V, P.pivot_rel, mpb, lane);
        for (int v = lane; v < V; v += TRAJ_THREADS) S.Qt[v] = S.Q[v] + (ok ? (float)S.b[v] : 0.f);
        evaluate = ok;
        __syncthreads();
    }
    float *dst = P.out + b * (int64_t)V;
    for (int v = lane; v < V; v += TRAJ_THREADS) dst[v] = S.Q[v];
    if (lane == 0) {
        const bool meets = S.err[0] <= P.tol_pos && S.err[1] <= P.tol_pos && S.err[2] <= P.tol_rot &&
                           S.err[3] <= P.tol_rot;
        if (P.cost) P.cost[b] = cost;
        if (P.iters) P.iters[b] = iters;
        if (P.accepts) P.accepts[b] = accepts;
        if (P.status) P.status[b] = meets ? PK_CONVERGED : (stalled ? PK_STALLED : PK_MAX_ITERS);
        if (P.pos_err) {
            P.pos_err[b] = S.err[0];
            P.pos_err[P.B + b] = S.err[1];
        }
        if (P.rot_err) {
            P.rot_err[b] = S.err[2];
            P.rot_err[P.B + b] = S.err[3];
        }
    }
}

inline bool traj_variant(int n) { return n == 4 || n == 6 || n == 7 || n == 10; }

hipError_t launch_traj(const RobotC *rb, int n, const TrajParams &P, hipStream_t s)
{
    return launch_parts(P.B, TRAJ_THREADS, [&](int64_t b, unsigned blocks) {
        // trajectory b is the part's first (planes keep their stride P.B)
        TrajParams Q = P;
        Q.start += b; Q.goal += b;
        Q.init += b * P.T * n; Q.out += b * P.T * n;
        for (float **p : {&Q.cost, &Q.pos_err, &Q.rot_err})
            if (*p) *p += b;
        for (int32_t **p : {&Q.iters, &Q.accepts, &Q.status})
            if (*p) *p += b;
        const dim3 grid(blocks), block(TRAJ_THREADS);
        switch (n) {
        case 4: hipLaunchKernelGGL(traj_kernel<4>, grid, block, 0, s, rb, Q); break;
        case 6: hipLaunchKernelGGL(traj_kernel<6>, grid, block, 0, s, rb, Q); break;
        case 7: hipLaunchKernelGGL(traj_kernel<7>, grid, block, 0, s, rb, Q); break;
        case 10: hipLaunchKernelGGL(traj_kernel<10>, grid, block, 0, s, rb, Q); break;
        default: return hipErrorInvalidValue;
        }
        return hipGetLastError();
    });
}

}  // namespace
}  // namespace pk

using namespace pk;

extern "C" int pk_traj_solve(pk_ctx *ctx, int32_t robot_id, const pk_traj_problem *pr,
                             const pk_traj_costs *c, const pk_lm_options *o,
                             const pk_traj_outputs *out, void *stream)
{
    if (!ctx) return fail(nullptr, PK_EINVAL, "pk_traj_solve: ctx is NULL");
    RobotEntry *rb = robot_of(ctx, robot_id);
    if (!rb) return fail(ctx, PK_ENOTFOUND, "pk_traj_solve: unknown robot %d", robot_id);
    if (!pr || !c || !o || !out) return fail(ctx, PK_EINVAL, "pk_traj_solve: NULL argument");
    const RobotC &H = rb->host;
    const int n = H.n;
    if (H.chains != 1 || H.m != 1 || H.e[0].kind != PK_EE_POSE || H.n_mimic != 0 || !traj_variant(n))
        return fail(ctx, PK_EUNSUPPORTED, "pk_traj_solve: needs a single chain of 4, 6, 7 or 10 "
                    "non-mimic joints with one pose EE");
    if (pr->B < 0 || pr->T < 5 || (int64_t)pr->T * n > TRAJ_VMAX)
        return fail(ctx, PK_EINVAL, "pk_traj_solve: B=%lld T=%d (need T >= 5, T * n <= %d)",
                    (long long)pr->B, pr->T, TRAJ_VMAX);
    if (pr->B == 0) return PK_OK;
    if (pr->B >= (int64_t)1 << 31) return fail(ctx, PK_EUNSUPPORTED, "pk_traj_solve: B too large");
    if (!pr->start || !pr->goal || !pr->init || !out->traj)
        return fail(ctx, PK_EINVAL, "pk_traj_solve: NULL start/goal/init/traj");
    if (!(c->dt > 0) || !std::isfinite(c->w_pos) || !std::isfinite(c->w_rot) ||
        !std::isfinite(c->w_limit) || !std::isfinite(c->w_smooth) || !std::isfinite(c->w_vel) ||
        !std::isfinite(c->w_acc) || !std::isfinite(c->w_jerk))
        return fail(ctx, PK_EINVAL, "pk_traj_solve: bad costs");
    if (c->w_vel != 0.f && !c->vmax)
        return fail(ctx, PK_EINVAL, "pk_traj_solve: w_vel != 0 needs vmax (velocity limits)");
    if (o->max_iters < 0 || !(o->lambda0 > 0) || !(o->nu_up > 1) || !(o->nu_down > 1) ||
        !(o->lambda_min > 0) || !(o->lambda_max >= o->lambda_min) || !(o->damping_floor > 0) ||
        !(o->pivot_rel >= 0))
        return fail(ctx, PK_EINVAL, "pk_traj_solve: invalid LM options");
    PK_HIP(ctx, hipSetDevice(ctx->device));
    TrajParams P;
    memset(&P, 0, sizeof P);
    P.B = pr->B;
    P.T = pr->T;
    P.dt = c->dt;
    P.w_pos = c->w_pos; P.w_rot = c->w_rot; P.w_limit = c->w_limit; P.w_smooth = c->w_smooth;
    P.w_vel = c->w_vel; P.w_acc = c->w_acc; P.w_jerk = c->w_jerk; P.vmax = c->vmax;
    P.start = pr->start; P.goal = pr->goal; P.init = pr->init;
    P.out = out->traj; P.cost = out->cost; P.pos_err = out->pos_err; P.rot_err = out->rot_err;
    P.iters = out->iters; P.accepts = out->accepts; P.status = out->status;
    P.lambda0 = o->lambda0; P.nu_up = o->nu_up; P.nu_down = o->nu_down;
    P.lambda_min = o->lambda_min; P.lambda_max = o->lambda_max;
    P.tol_pos = o->tol_pos; P.tol_rot = o->tol_rot;
    P.damping_floor = o->damping_floor; P.pivot_rel = o->pivot_rel;
    P.max_iters = o->max_iters; P.early_exit = o->early_exit ? 1 : 0;
    PK_HIP(ctx, launch_traj(rb->dev, n, P, (hipStream_t)stream));
    return PK_OK;
}
