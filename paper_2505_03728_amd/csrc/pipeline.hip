// Learned seeds + LM refinement, a restart of the unsolved targets' problems
// from their refined joints, and a random-seed LM fallback on the targets
// still unsolved.  Everything stays on the device: each later pass's
// problems are compacted into an active list that a persistent LM launch
// (wavefronts popping items from a device queue) reads, so the host never
// synchronises and a pass costs what its listed problems cost.
#include <limits.h>
#include <string.h>

#include <algorithm>

#include "pk_ctx.hpp"
#include "pk_device.hpp"

namespace pk {
namespace {

__global__ void fill_i32_kernel(int64_t count, int32_t v, int32_t *p)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = v;
}

// Threads of a block whose targets are to be listed take consecutive places:
// one atomic per counter and block (with one per target the counter's line
// served 30000 of them one after the other: 131072 targets, lists of 29634 and
// 12080, 49 and 78 us; 6.6 and 7.9 now).  per: problems a target lists.
// Returns the place of this thread's target in units of targets.
constexpr int LIST_BLOCK = 1024;

PK_DEV int list_places(bool need, int per, int32_t *count_t, int32_t *count_p, int32_t *count_stage)
{
    __shared__ int wave_n[LIST_BLOCK / 64], base;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const uint64_t mask = __ballot(need);
    if (lane == 0) wave_n[w] = __popcll(mask);
    __syncthreads();
    if (threadIdx.x == 0) {
        int sum = 0;
        for (int u = 0; u < LIST_BLOCK / 64; ++u) {
            const int c = wave_n[u];
            wave_n[u] = sum;
            sum += c;
        }
        base = 0;
        if (sum) {
            // the list's own counter gives the place; the others only count
            const int at = atomicAdd(count_stage ? count_stage : count_p, sum * per);
            base = at / per;
            if (count_stage) atomicAdd(count_p, sum * per);
            if (count_t) atomicAdd(count_t, sum);
        }
    }
    __syncthreads();
    return base + wave_n[w] + __popcll(mask & ((1ull << lane) - 1));
}

// The listed targets' problems t * Kf + c0 + k, k < per, at place * per of the
// list; the wavefront writes them for one of its targets after the other.
PK_DEV void list_write(bool need, int64_t t, int place, int Kf, int c0, int per, int32_t *active)
{
    const int lane = threadIdx.x & 63;
    for (uint64_t mask = __ballot(need); mask; mask &= mask - 1) {
        const int src = __builtin_ctzll(mask);
        const int64_t tt = __shfl(t, src, 64), at = (int64_t)__shfl(place, src, 64) * per;
        for (int k = lane; k < per; k += 64) active[at + k] = (int32_t)(tt * Kf + c0 + k);
    }
}

// Targets not solved (success[t] == 0) -> active problem list of a later
// pass (Kf problems per target, problem t * Kf + k).
__global__ __launch_bounds__(LIST_BLOCK) void fallback_list_kernel(int64_t T, int Kf,
                                                                   const int32_t *__restrict__ success,
                                                                   int32_t *count_t, int32_t *count_p,
                                                                   int32_t *active)
{
    const int64_t t = (int64_t)blockIdx.x * LIST_BLOCK + threadIdx.x;
    const bool need = t < T && !success[t];
    list_write(need, t, list_places(need, Kf, count_t, count_p, nullptr), Kf, 0, Kf, active);
}

// Fallback stage [c0, c1) of every target's Kf random seeds.  Stage 0 lists
// the targets the earlier passes left unsolved; a later stage lists those
// that ran the previous stage [cp, c0) and got no converged problem from it.
// done[t] counts the target's fallback seeds run so far.
__global__ __launch_bounds__(LIST_BLOCK) void fallback_stage_kernel(
    int64_t T, int Kf, int cp, int c0, int c1, const int32_t *__restrict__ success,
    const int32_t *__restrict__ status, int32_t *done, int32_t *count_t, int32_t *count_p,
    int32_t *count_stage, int32_t *active)
{
    const int64_t t = (int64_t)blockIdx.x * LIST_BLOCK + threadIdx.x;
    const int lane = threadIdx.x & 63;
    bool need = t < T;
    if (c0 == 0) {
        if (need && success[t]) {
            done[t] = 0;
            need = false;
        }
    } else {
        need = need && done[t] == c0;
        for (uint64_t mask = __ballot(need); mask; mask &= mask - 1) {
            const int src = __builtin_ctzll(mask);
            const int64_t tt = __shfl(t, src, 64);
            bool conv = false;
            for (int k = cp + lane; k < c0; k += 64) conv |= (status[tt * Kf + k] & 0xff) == PK_CONVERGED;
            if (__ballot(conv) && lane == src) need = false;
        }
    }
    if (need) done[t] = c1;
    const int w = c1 - c0;
    list_write(need, t, list_places(need, w, count_t, count_p, count_stage), Kf, c0, w, active);
}

struct MergeArgs {
    int64_t T;
    int K, Kf, n, refine_its;
    const int32_t *best_a, *succ_a, *succ_r, *itt_a;
    const float *joints_a;
    const int32_t *status_b, *itt_b, *done_b;
    const float *cost_b, *pcost_b, *joints_b;
    float *best_joints;
    int32_t *success, *source, *itt;
};

// A number whose order is the float's by `<` (-0 made +0, equal to it), a NaN
// after every number; with the index below it the least is the first smallest.
PK_DEV uint64_t pick_key(float v, int k)
{
    const uint32_t u = __float_as_uint(v + 0.f);
    const uint32_t o = v != v ? 0xffffffffu : u ^ ((u >> 31) ? 0xffffffffu : 0x80000000u);
    return (uint64_t)o << 32 | (uint32_t)k;
}

PK_DEV uint64_t wave_min(uint64_t v)
{
#pragma unroll
    for (int d = 1; d < 64; d *= 2) {
        const uint64_t o = __shfl_xor((unsigned long long)v, d, 64);
        v = o < v ? o : v;
    }
    return v;
}

// best_of_k_pick by a whole wavefront, K >= 1.  (Its comparisons are `<` from
// the first candidate on, so a NaN wins exactly where it is that first one.)
PK_DEV int wave_best_of_k(const int32_t *status, const float *cost, const float *pcost, int64_t base, int K,
                          bool &any)
{
    uint64_t bc = ~0ull, bp = ~0ull, first = ~0ull;
    for (int k = threadIdx.x & 63; k < K; k += 64) {
        const int32_t st = status[base + k];
        const float c = cost[base + k], pc = pcost[base + k];
        if ((st & 0xff) == PK_CONVERGED) {
            const uint64_t key = pick_key(c, k);
            bc = key < bc ? key : bc;
            // the first candidate's index, then whether it is a NaN
            const uint64_t f = (uint64_t)k << 1 | (c != c ? 1 : 0);
            first = f < first ? f : first;
        }
        const uint64_t key = pick_key(pc, k);
        bp = key < bp ? key : bp;
        if (k == 0 && pc != pc) bp = 0;   // (lane 0, its first candidate: stays the least)
    }
    first = wave_min(first);
    any = first != ~0ull;
    if (any) return first & 1 ? (int)(first >> 1) : (int)(uint32_t)wave_min(bc);
    return (int)(uint32_t)wave_min(bp);
}

// Eight lanes per target: its iterations to tolerance and its joints are a
// read each of consecutive values.  The fallback's targets take the whole
// wavefront, one after the other.  131072 targets of 8 seeds, 12080 of them in a
// fallback of 128: 103 us with a thread per target (chains of dependent reads
// 32 bytes and more apart), 33 now.
constexpr int MERGE_LANES = 8, MERGE_BLOCK = 256;

__global__ __launch_bounds__(MERGE_BLOCK) void merge_kernel(MergeArgs a)
{
    const int64_t t = ((int64_t)blockIdx.x * MERGE_BLOCK + threadIdx.x) / MERGE_LANES;
    const int lane = threadIdx.x & 63, sub = lane % MERGE_LANES;
    const int64_t NA = a.T * a.K, NB = a.T * a.Kf;
    const bool live = t < a.T;
    // pass A (learned seeds), or its restart: best_a / itt_a then hold the
    // restart's values for the targets that were restarted
    const bool sa = live && a.succ_a[t] != 0;
    const bool restarted = live && a.succ_r && !sa;
    const bool solved = sa || (restarted && a.succ_r[t] != 0);
    const bool fallback = live && !solved && a.Kf > 0;
    int src = solved ? (restarted ? 2 : 0) : -1, it = INT_MAX;
    if (live && !fallback) {
        const int b = a.best_a[t];
        for (int j = sub; j < a.n; j += MERGE_LANES)
            a.best_joints[(int64_t)j * a.T + t] = a.joints_a[(int64_t)j * NA + t * a.K + b];
        if (solved)
            for (int k = sub; k < a.K; k += MERGE_LANES) {
                const int v = a.itt_a[t * a.K + k];
                it = v >= 0 && v < it ? v : it;
            }
    }
#pragma unroll
    for (int d = 1; d < MERGE_LANES; d *= 2) it = min(it, __shfl_xor(it, d, 64));
    it = it == INT_MAX ? -1 : it;
    if (solved && restarted) it += a.refine_its;
    for (uint64_t mask = __ballot(fallback && sub == 0); mask; mask &= mask - 1) {
        // the fallback seeds this target ran (every stage up to its first
        // converged problem)
        const int from = __builtin_ctzll(mask);
        const int64_t tt = __shfl(t, from, 64);
        const int kr = a.done_b[tt];
        bool any;
        const int b = wave_best_of_k(a.status_b, a.cost_b, a.pcost_b, tt * a.Kf, kr, any);
        for (int j = lane; j < a.n; j += 64)
            a.best_joints[(int64_t)j * a.T + tt] = a.joints_b[(int64_t)j * NB + tt * a.Kf + b];
        if (any) {
            int v = INT_MAX;
            for (int k = lane; k < kr; k += 64) {
                const int u = a.itt_b[tt * a.Kf + k];
                v = u >= 0 && u < v ? u : v;
            }
#pragma unroll
            for (int d = 1; d < 64; d *= 2) v = min(v, __shfl_xor(v, d, 64));
            if (lane == from) {
                src = 1;
                it = v == INT_MAX ? -1 : v;
            }
        }
    }
    if (!live || sub != 0) return;
    if (a.success) a.success[t] = src >= 0 ? 1 : 0;
    if (a.source) a.source[t] = src;
    if (a.itt) a.itt[t] = it;
}

inline unsigned nblk(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

}  // namespace
}  // namespace pk

using namespace pk;

extern "C" int pk_ik_solve_seeded(pk_ctx *ctx, int32_t robot_id, int64_t T, const float *targets,
                                  const pk_cost_weights *w, const pk_seeded_options *o,
                                  const pk_seeded_outputs *out, void *stream)
{
    if (!ctx) return fail(nullptr, PK_EINVAL, "pk_ik_solve_seeded: ctx is NULL");
    RobotEntry *rb = robot_of(ctx, robot_id);
    if (!rb) return fail(ctx, PK_ENOTFOUND, "pk_ik_solve_seeded: unknown robot %d", robot_id);
    if (!w || !o || !out) return fail(ctx, PK_EINVAL, "pk_ik_solve_seeded: NULL argument");
    if (T < 0) return fail(ctx, PK_EINVAL, "pk_ik_solve_seeded: T < 0");
    if (T == 0) return PK_OK;
    if (!targets || !out->best_joints) return fail(ctx, PK_EINVAL, "pk_ik_solve_seeded: NULL targets/best_joints");
    if (o->fallback_K < 0 || (o->fallback_K > 0 && !o->fallback_seeds))
        return fail(ctx, PK_EINVAL, "pk_ik_solve_seeded: fallback seeds missing");
    if (o->fallback_chunk < 0) return fail(ctx, PK_EINVAL, "pk_ik_solve_seeded: fallback_chunk < 0");
    hipStream_t s = (hipStream_t)stream;
    PK_HIP(ctx, hipSetDevice(ctx->device));
    SolveParams PA, PB;
    int va = 0, vb = 0;
    int rc = prepare_solve(ctx, *rb, w, &o->refine, PA, va);
    if (rc) return rc;
    rc = prepare_solve(ctx, *rb, w, &o->fallback, PB, vb);
    if (rc) return rc;
    // Seeds from the network (also validates the seeder / robot pairing).
    int32_t K = 0, srobot = -1;
    {
        // probe K and robot without launching
        rc = seeder_infer_into(ctx, o->seeder_id, targets, 0, nullptr, s, &K, &srobot);
        if (rc) return rc;
    }
    if (srobot != robot_id) return fail(ctx, PK_EINVAL, "pk_ik_solve_seeded: seeder belongs to robot %d", srobot);
    const int n = rb->host.nv, Kf = o->fallback_K;
    const int Kc = o->fallback_chunk > 0 && o->fallback_chunk < Kf ? o->fallback_chunk : Kf;
    const int64_t NA = T * K, NB = T * Kf;
    if (NA >= (int64_t)1 << 31 || NB >= (int64_t)1 << 31)
        return fail(ctx, PK_EUNSUPPORTED, "pk_ik_solve_seeded: too many problems");
    const int R = o->restart_iters;
    if (R < 0) return fail(ctx, PK_EINVAL, "pk_ik_solve_seeded: restart_iters < 0");
    const int wpc = o->persist_waves_per_cu > 0 ? o->persist_waves_per_cu : 8;
    hipDeviceProp_t prop;
    PK_HIP(ctx, hipGetDeviceProperties(&prop, ctx->device));
    const int persist = wpc * prop.multiProcessorCount;
    const int64_t NS = std::max(NA, NB);   // resumable-state words of the persistent passes
    // Workspace layout (4-byte words).
    const size_t words = (size_t)NA * (2 * n + 6) + 4 * T + 16 + (size_t)NB * (n + 6) + 2 * (size_t)NS;
    if (words * 4 > ctx->ws2_bytes) {
        if (ctx->ws2) (void)hipFree(ctx->ws2);
        ctx->ws2 = nullptr;
        ctx->ws2_bytes = 0;
        if (hipMalloc(&ctx->ws2, words * 4) != hipSuccess)
            return fail(ctx, PK_ENOMEM, "pk_ik_solve_seeded: workspace of %zu bytes", words * 4);
        ctx->ws2_bytes = words * 4;
    }
    float *f = (float *)ctx->ws2;
    float *seeds_a = f;                 f += (size_t)NA * n;
    float *joints_a = f;                f += (size_t)NA * n;
    float *cost_a = f;                  f += NA;
    float *pcost_a = f;                 f += NA;
    int32_t *status_a = (int32_t *)f;   f += NA;
    int32_t *itt_a = (int32_t *)f;      f += NA;
    int32_t *spare_a = (int32_t *)f;    f += NA;
    int32_t *best_a = (int32_t *)f;     f += T;
    int32_t *succ_a = (int32_t *)f;     f += T;
    int32_t *succ_r = (int32_t *)f;     f += T;
    int32_t *list_r = (int32_t *)f;     f += NA;
    int32_t *done_b = (int32_t *)f;     f += T;
    // [0..1] fallback targets and problems, [2..3] restart list, [4] queue
    // head, [5] problems of the current fallback stage
    int32_t *counters = (int32_t *)f;   f += 16;
    float *st_lambda = f;               f += NS;
    int32_t *st_state = (int32_t *)f;   f += NS;
    float *joints_b = f;                f += (size_t)NB * n;
    float *cost_b = f;                  f += NB;
    float *pcost_b = f;                 f += NB;
    int32_t *status_b = (int32_t *)f;   f += NB;
    int32_t *itt_b = (int32_t *)f;      f += NB;
    int32_t *active = (int32_t *)f;     f += NB;
    (void)spare_a;

    rc = seeder_infer_into(ctx, o->seeder_id, targets, T, seeds_a, s, nullptr, nullptr);
    if (rc) return rc;
    // Pass A: LM from the learned seeds.
    PA.K = K; PA.N = NA; PA.T = T;
    PA.targets = targets; PA.seeds = seeds_a;
    PA.joints = joints_a; PA.cost = cost_a; PA.pose_cost = pcost_a; PA.status = status_a;
    PA.iters = out->refine_iters; PA.accepts = out->refine_accepts; PA.iters_to_tol = itt_a;
    if (o->refine_iters_per_launch > 0) {
        // Persistent, compacted schedule (same per-problem results).
        pk_ik_group g;
        memset(&g, 0, sizeof g);
        g.robot_id = robot_id;
        g.problem.n_targets = T;
        g.problem.K = K;
        g.problem.targets = targets;
        g.problem.seeds = seeds_a;
        g.weights = *w;
        g.out.joints = joints_a;
        g.out.cost = cost_a;
        g.out.iters = out->refine_iters;
        g.out.accepts = out->refine_accepts;
        g.out.status = status_a;
        g.out.iters_to_tol = itt_a;
        g.out.best_index = best_a;
        g.out.target_success = succ_a;
        pk_sched_options so;
        memset(&so, 0, sizeof so);
        so.iters_per_launch = o->refine_iters_per_launch;
        so.waves_per_cu = o->refine_blocks_per_cu > 0 ? o->refine_blocks_per_cu : 4;
        so.workgroup_size = 64;
        so.use_graph = 1;
        rc = sched_run(ctx, 1, &g, &o->refine, so, s);
        if (rc) return rc;
    } else if (va == PK_VARIANT_LANE && 64 % K == 0) {
        const BestOut B{best_a, nullptr, succ_a};   // best-of-K in the same launch
        PK_HIP(ctx, launch_lm(*rb, PA, va, s, 0, &B));
    } else {
        PK_HIP(ctx, launch_lm(*rb, PA, va, s));
        PK_HIP(ctx, launch_best_of_k(PA, n, best_a, nullptr, succ_a, s));
    }
    hipLaunchKernelGGL(fill_i32_kernel, dim3(1), dim3(64), 0, s, (int64_t)16, 0, counters);
    // Pass A': the K problems of each unsolved target again from their
    // refined joints (lambda back at lambda0), in place, then best-of-K again.
    const int32_t *succ_now = succ_a;
    if (R > 0) {
        if (out->restart_iters)
            hipLaunchKernelGGL(fill_i32_kernel, dim3(nblk(NA, 256)), dim3(256), 0, s, NA, 0, out->restart_iters);
        if (out->restart_accepts)
            hipLaunchKernelGGL(fill_i32_kernel, dim3(nblk(NA, 256)), dim3(256), 0, s, NA, 0, out->restart_accepts);
        hipLaunchKernelGGL(fallback_list_kernel, dim3(nblk(T, LIST_BLOCK)), dim3(LIST_BLOCK), 0, s, T, K, succ_a,
                           counters + 2, counters + 3, list_r);
        SolveParams PR = PA;
        PR.max_iters = R;
        PR.seeds = joints_a;            // each problem reads its joints before writing them
        PR.iters = out->restart_iters; PR.accepts = out->restart_accepts;
        PR.active = list_r; PR.n_active = counters + 3;
        PR.st_lambda = st_lambda; PR.st_state = st_state;
        PR.resume = 0; PR.iter_budget = R;
        PR.queue_head = counters + 4;
        PK_HIP(ctx, launch_lm(*rb, PR, va, s, persist));
        PK_HIP(ctx, launch_best_of_k(PA, n, best_a, nullptr, succ_r, s));
        succ_now = succ_r;
    }
    // Pass B: random seeds on the targets still unsolved.
    if (Kf > 0) {
        if (out->fallback_iters)
            hipLaunchKernelGGL(fill_i32_kernel, dim3(nblk(NB, 256)), dim3(256), 0, s, NB, 0, out->fallback_iters);
        if (out->fallback_accepts)
            hipLaunchKernelGGL(fill_i32_kernel, dim3(nblk(NB, 256)), dim3(256), 0, s, NB, 0, out->fallback_accepts);
        PB.K = Kf; PB.N = NB; PB.T = T;
        PB.targets = targets; PB.seeds = o->fallback_seeds;
        PB.joints = joints_b; PB.cost = cost_b; PB.pose_cost = pcost_b; PB.status = status_b;
        PB.iters = out->fallback_iters; PB.accepts = out->fallback_accepts; PB.iters_to_tol = itt_b;
        PB.active = active; PB.n_active = counters + 5;
        PB.st_lambda = st_lambda; PB.st_state = st_state;
        PB.resume = 0; PB.iter_budget = PB.max_iters;
        PB.queue_head = counters + 4;
        for (int cp = 0, c0 = 0; c0 < Kf; cp = c0, c0 += Kc) {
            const int c1 = std::min(Kf, c0 + Kc);
            hipLaunchKernelGGL(fill_i32_kernel, dim3(1), dim3(64), 0, s, (int64_t)2, 0, counters + 4);
            hipLaunchKernelGGL(fallback_stage_kernel, dim3(nblk(T, LIST_BLOCK)), dim3(LIST_BLOCK), 0, s, T, Kf, cp, c0,
                               c1, succ_now, status_b, done_b, c0 == 0 ? counters : nullptr, counters + 1,
                               counters + 5, active);
            PK_HIP(ctx, hipGetLastError());
            PK_HIP(ctx, launch_lm(*rb, PB, vb, s, persist));
        }
    }
    MergeArgs m;
    m.T = T; m.K = K; m.Kf = Kf; m.n = n; m.refine_its = o->refine.max_iters;
    m.best_a = best_a; m.succ_a = succ_a; m.succ_r = R > 0 ? succ_r : nullptr; m.itt_a = itt_a;
    m.joints_a = joints_a;
    m.status_b = status_b; m.itt_b = itt_b; m.done_b = done_b; m.cost_b = cost_b; m.pcost_b = pcost_b; m.joints_b = joints_b;
    m.best_joints = out->best_joints; m.success = out->target_success; m.source = out->source;
    m.itt = out->iters_to_tol;
    hipLaunchKernelGGL(merge_kernel, dim3(nblk(T * MERGE_LANES, MERGE_BLOCK)), dim3(MERGE_BLOCK), 0, s, m);
    PK_HIP(ctx, hipGetLastError());
    if (out->n_fallback)
        PK_HIP(ctx, hipMemcpyAsync(out->n_fallback, counters, 4, hipMemcpyDeviceToDevice, s));
    if (out->n_restart)
        PK_HIP(ctx, hipMemcpyAsync(out->n_restart, counters + 2, 4, hipMemcpyDeviceToDevice, s));
    if (out->n_fallback_problems)
        PK_HIP(ctx, hipMemcpyAsync(out->n_fallback_problems, counters + 1, 4, hipMemcpyDeviceToDevice, s));
    return PK_OK;
}
