// Persistent LM launches over a mixed batch: the wavefronts of a grid pop work
// items from a device queue; an item is (group, range of that group's active
// problems): 64 problems for a per-lane path, 16 for the star's four lanes per
// problem, one for a per-wavefront path.
// The wavefront branches (uniformly) to the device path of the item's group,
// which runs the problems for at most k more LM iterations with their state in
// HBM (resumable), so a problem's result does not depend on k, on the grid or
// on which wavefront takes it.
//
// A round of a large batch is up to four launches, one after the other: one per
// row length of the path-pair kernel (one tree problem per wavefront), then one
// for all other paths.  A kernel that holds every path takes the registers of
// the per-lane arm (253: two wavefronts per SIMD), and the trees, which need four
// to cover their LDS and dependency waits, run at 16 levels' row length.  4096
// trees of 34 joints, 50 iterations, in us: 1454 in such a kernel; 1326 in one of
// their own (128 VGPRs, 9.4 KiB, two row lengths, the LDS slice of unknown
// alignment: 32-bit accesses); 935 with the slice's alignment and the robot in
// constant memory known; 833 at their own row length.  With 60000 arms and
// 20000 hands the batch took 2246, 1390 with these launches, 1129 with the hands
// on four lanes per problem (lm_star.hpp), 1121 with grids no larger than the
// items.
//
// Method: Sec. III-A (LM over the sum of squared weighted residuals) for each
// problem, as in the per-lane and per-wavefront kernels it instantiates.
#include <algorithm>

#include "lm_path.hpp"
#include "lm_star.hpp"
#include "lm_wave.hpp"
#include "sched_table.hpp"

namespace pk {
namespace {

constexpr int align4(int f) { return (f + 3) & ~3; }

// Work items per group for this round, the queue heads reset, and the next
// round's list size cleared (the compaction after this round fills it).
__global__ void mixed_plan_kernel(MixedArgs a, int32_t *item_end, int32_t *heads)
{
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    const int cur = a.round & 1;
    int acc = 0;
    for (int g = 0; g < a.n_groups; ++g) {
        const MixedGroup &G = a.g[g];
        const int64_t cnt = a.round > 0 ? (int64_t)G.count[cur] : G.P.N;
        acc += (int)((cnt + G.per_item - 1) / G.per_item);
        item_end[g] = acc;
        G.count[cur ^ 1] = 0;
    }
    for (int i = 0; i < PK_MIX_LAUNCHES; ++i) heads[i] = 0;
}

// Unfinished problems of this round's list -> next round's list (one grid
// row per group).
__global__ void mixed_compact_kernel(MixedArgs a)
{
    const int g = blockIdx.y;
    if (g >= a.n_groups) return;
    const MixedGroup &G = a.g[g];
    const int cur = a.round & 1;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t nc = a.round > 0 ? (int64_t)G.count[cur] : G.P.N;
    if (i >= nc) return;
    const int32_t p = a.round > 0 ? G.list[cur][i] : (int32_t)i;
    if (!(G.P.st_state[p] & PK_ST_DONE)) G.list[cur ^ 1][atomicAdd(&G.count[cur ^ 1], 1)] = p;
}

// A pointer of the group's as one to constant memory, which no kernel writes:
// loads through it are scalar loads that a store does not stand in the way of.
// (As a kernel's own restricted argument it is known to be that; read from the
// group it was not, and every pass fetched its robot with vector loads.)
template <typename T>
PK_DEV const T *constant(const T *p)
{
    return (const T *)(const __attribute__((address_space(4))) T *)(uint64_t)p;
}

// Per-lane path: problems first*64 + lane of the group's active list.
template <int C, int L, int KIND>
PK_DEV void run_lane(const MixedGroup &G, float *ws, int64_t first, int lane)
{
    const SolveParams &P = G.P;
    const int64_t nact = P.n_active ? (int64_t)*P.n_active : P.N;
    const int64_t i = first * 64 + lane;
    if (i < nact) lane::lane_problem<C, L, KIND, true>(constant(G.rb), constant(G.qr), P, lane::LaneLds{ws + lane}, i);
}

// Star path: problems first*16 + quad of the group's active list.
PK_DEV void run_star(const MixedGroup &G, int64_t first, int lane)
{
    const SolveParams &P = G.P;
    const int64_t nact = P.n_active ? (int64_t)*P.n_active : P.N;
    const int64_t i = first * 16 + (lane >> 2);
    star::Final fin;
    if (i < nact) star::star_problem<true>(constant(G.rb), constant(G.qr), P, i, &fin);
}

// One tree problem on this wavefront.
template <int DMAX, int RW>
PK_DEV void run_path(const MixedGroup &G, int g, float *ws, int64_t first)
{
    path::path_problem<DMAX, 4, RW>(
        constant(G.rb), path::kernel_params_at(offsetof(MixedArgs, g) + g * sizeof(MixedGroup) + offsetof(MixedGroup, P)),
        ws, first);
}

// Groups [g0, g1) of the batch.  MixedArgs is the first kernel argument
// (offset 0 of the argument segment).
template <int WG, int LAUNCH>
__global__ __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(LAUNCH < 3 ? 4 : 2))) void lm_mixed_kernel(
    const MixedArgs a, int g0, int g1, const int32_t *__restrict__ item_end, int32_t *head, int lds_quads)
{
    extern __shared__ __attribute__((aligned(16))) float smem[];
    const int lane = threadIdx.x & 63;
    // 16-byte aligned to the compiler too: its LDS accesses are 128 bits wide
    float *ws = WG == 64 ? smem : smem + 4 * ((threadIdx.x >> 6) * lds_quads);
    const int start = g0 > 0 ? item_end[g0 - 1] : 0;
    const int total = item_end[g1 - 1];
    for (;;) {
        int v = 0;
        if (lane == 0) v = atomicAdd(head, 1);
        const int item = start + __builtin_amdgcn_readfirstlane(__shfl(v, 0, 64));
        if (item >= total) break;
        int g = g0;
        while (g < g1 - 1 && item >= item_end[g]) ++g;
        g = __builtin_amdgcn_readfirstlane(g);   // uniform: item is
        const MixedGroup &G = a.g[g];
        const int64_t first = item - (g > 0 ? item_end[g - 1] : 0);
        if constexpr (LAUNCH == 0) {
            run_path<16, 16>(G, g, ws, first);
        } else if constexpr (LAUNCH == 1) {
            run_path<16, 12>(G, g, ws, first);
        } else if constexpr (LAUNCH == 2) {
            run_path<8, 8>(G, g, ws, first);
        } else {
            switch (G.path) {
            case MIX_LANE_ARM:
                run_lane<1, 7, PK_EE_POSE>(G, ws, first, lane);
                break;
            case MIX_STAR_HAND:
                run_star(G, first, lane);
                break;
            case MIX_WAVE_16_4:
                wave::wave_problem<16, 4>(constant(G.rb), G.P, ws, first);
                break;
            default:   // rows for any tree; only in the kernel with every path
                static_assert(path::Lds<8, 4>::FLOATS == path::Lds<16, 4>::FLOATS, "mixed_lds_floats gives the tree's own");
                if constexpr (LAUNCH == PK_MIX_ALL) run_path<16, 16>(G, g, ws, first);
                break;
            }
        }
        // the next item reuses this wavefront's LDS slice
        wave::wave_sync();
    }
}

inline unsigned nblk(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

}  // namespace

int mixed_lds_floats(int path)
{
    switch (path) {
    case MIX_LANE_ARM: return align4(lane::Slots<1, 7, PK_EE_POSE>::TOTAL * lane::BLOCK);
    case MIX_STAR_HAND: return 0;
    case MIX_WAVE_16_4: return align4(wave::Lds<16, 4>::FLOATS);
    case MIX_PATH_16_4:
    case MIX_PATH_13_4: return align4(path::Lds<16, 4>::FLOATS);
    case MIX_PATH_8_4: return align4(path::Lds<8, 4>::FLOATS);
    default: return 0;
    }
}

namespace {

int64_t items_of(const MixedGroup &G) { return (G.P.N + G.per_item - 1) / G.per_item; }

// The launch of the batch's LAUNCH groups (from g0, which moves past them),
// with the LDS of the largest of their paths.
template <int LAUNCH>
hipError_t launch_groups(const MixedArgs &a, int &g0, int32_t *item_end, int32_t *heads, int waves, int wg,
                         hipStream_t s)
{
    int ldsf = 0, g1 = g0;
    int64_t items = 0;
    for (; g1 < a.n_groups && (LAUNCH == PK_MIX_ALL || mixed_launch_of(a.g[g1].path) == LAUNCH); ++g1) {
        ldsf = std::max(ldsf, mixed_lds_floats(a.g[g1].path));
        items += items_of(a.g[g1]);
    }
    if (g1 == g0) return hipSuccess;
    const int first = g0;
    int32_t *head = heads + LAUNCH % PK_MIX_LAUNCHES;
    g0 = g1;
    // No more wavefronts than items: the dispatcher spreads a grid over the SIMDs,
    // but which of too many wavefronts reach the queue first is chance, and two
    // items on one SIMD leave another idle (60000 arms, 938 items: 302 us from a
    // grid of 2048, 227 from one of 938).
    const int wpb = wg / 64;
    const dim3 grid(nblk(std::min<int64_t>(waves, items), wpb)), block(wg);
    const size_t lds = (size_t)wpb * ldsf * sizeof(float);
    switch (wg) {
    case 64:
        hipLaunchKernelGGL((lm_mixed_kernel<64, LAUNCH>), grid, block, lds, s, a, first, g1, item_end, head, ldsf / 4);
        break;
    case 128:
        hipLaunchKernelGGL((lm_mixed_kernel<128, LAUNCH>), grid, block, lds, s, a, first, g1, item_end, head, ldsf / 4);
        break;
    case 256:
        hipLaunchKernelGGL((lm_mixed_kernel<256, LAUNCH>), grid, block, lds, s, a, first, g1, item_end, head, ldsf / 4);
        break;
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Whether one launch serves the whole round: the batch has more than one kernel
// and the kernel with every path holds all its trees at once (they are first in
// the queue).  Then they run beside the other items; split, the launches' times
// add up.  Past that they queue behind each other there.  50 iterations, 8
// wavefronts per CU (so up to 2048 trees), one launch against split, us: 60000
// arms and 20000 hands with 200 trees 498 / 728, 1000 585 / 774, 2048 812 / 854,
// 2300 1026 / 924, 4096 1347 / 1123; 1000 arms and 1000 hands with 2048 652 / 761,
// 2300 1015 / 832; 100000 arms and 2000 hands with 2048 877 / 849.  With 4 per CU (up
// to 1024): 60000 and 20000 with 500 559 / 775, 1000 822 / 799, 1500 1048 / 854.
bool one_launch(const MixedArgs &a, int wpc, int cus, int wg)
{
    int64_t trees = 0;
    int ldsf = 0;
    bool same = true;
    for (int g = 0; g < a.n_groups; ++g) {
        if (mixed_launch_of(a.g[g].path) < PK_MIX_LAUNCHES - 1) trees += a.g[g].P.N;
        ldsf = std::max(ldsf, mixed_lds_floats(a.g[g].path));
        same = same && mixed_launch_of(a.g[g].path) == mixed_launch_of(a.g[0].path);
    }
    const int wpb = wg / 64, block_lds = std::max(1, wpb * ldsf * (int)sizeof(float));
    const int held = std::min(8, wpb * (160 * 1024 / block_lds));   // per CU (237 VGPRs: 2 per SIMD)
    return !same && trees <= (int64_t)std::min(wpc, held) * cus;
}

}  // namespace

hipError_t launch_mixed_round(const MixedArgs &a, int32_t *item_end, int32_t *heads, int max_n,
                              bool last, int wpc, int cus, int wg, hipStream_t s)
{
    hipLaunchKernelGGL(mixed_plan_kernel, dim3(1), dim3(64), 0, s, a, item_end, heads);
    const int waves = wpc * cus;
    int g = 0;
    hipError_t e = hipSuccess;
    if (one_launch(a, wpc, cus, wg)) {
        e = launch_groups<PK_MIX_ALL>(a, g, item_end, heads, waves, wg, s);
    } else {
        // (the path-pair kernels take half the registers: twice the wavefronts)
        e = launch_groups<0>(a, g, item_end, heads, 2 * waves, wg, s);
        if (e == hipSuccess) e = launch_groups<1>(a, g, item_end, heads, 2 * waves, wg, s);
        if (e == hipSuccess) e = launch_groups<2>(a, g, item_end, heads, 2 * waves, wg, s);
        if (e == hipSuccess) e = launch_groups<3>(a, g, item_end, heads, waves, wg, s);
    }
    if (e != hipSuccess) return e;
    if (!last)
        hipLaunchKernelGGL(mixed_compact_kernel, dim3(nblk(max_n, 256), a.n_groups), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace pk
