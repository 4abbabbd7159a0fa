// CPU check of the rule that sends a batch to the kernel with four lanes per
// problem (lane_rule.hpp): over batch sizes, seeds per target and chain lengths
// the workgroups of the launch it chooses stay at two per CU of 256 (one from 9
// joints), counted as the kernel counts them; and the parts that a batch too large
// for one launch is split into.  Prints one line per failure.
#include <cstdio>
#include <cstring>

#include "lane_rule.hpp"

using namespace pk;

static int failures = 0;

static SolveParams batch(int64_t T, int K, float w_rest)
{
    SolveParams P;
    memset(&P, 0, sizeof P);
    P.T = T;
    P.K = K;
    P.N = T * K;
    P.w_rest = w_rest;
    P.pivot_rel = 1e-6f;
    return P;
}

static void line(const char *what, int L, int kind, float w_rest, int K, bool best, int64_t most)
{
    const bool in = lane::takes_quad(1, L, kind, batch(most / K, K, w_rest), best),
               out = lane::takes_quad(1, L, kind, batch(most / K + 1, K, w_rest), best);
    if (!in || out) {
        ++failures;
        printf("FAIL %s: L=%d K=%d best=%d: %d at %lld, %d above\n", what, L, K, best, in, (long long)most, out);
    }
}

int main()
{
    for (int L = 2; L <= 10; ++L)
        for (int K = 1; K <= 130; ++K)
            for (int64_t T = 1; T * K <= 70000; T += T / 40 + 1)
                for (int kind : {PK_EE_POSE, PK_EE_POSITION})
                    for (float w_rest : {0.f, 0.01f}) {
                        const SolveParams P = batch(T, K, w_rest);
                        const bool quad = lane::takes_quad(1, L, kind, P, true), takes = lane::takes_best(1, L, kind, P);
                        const int targets = K <= 64 ? 64 / K : 0;   // per workgroup, best-of-K in the launch
                        const int64_t blocks = targets ? (T + targets - 1) / targets : 0;
                        if (quad && (K > 64 || blocks > (L > 8 ? 256 : 512))) {
                            ++failures;
                            printf("FAIL L=%d K=%d T=%lld: %lld workgroups\n", L, K, (long long)T, (long long)blocks);
                        }
                        // best-of-K without a launch of its own needs a kernel that can
                        if (takes && 64 % K != 0 && !quad) {
                            ++failures;
                            printf("FAIL L=%d K=%d T=%lld: best-of-K has no kernel\n", L, K, (long long)T);
                        }
                    }
    line("one seed", 7, PK_EE_POSE, 0.01f, 1, false, 32768);
    line("three seeds", 7, PK_EE_POSE, 0.01f, 3, true, 512 * 63);
    line("a target per workgroup", 7, PK_EE_POSE, 0.01f, 33, true, 512 * 33);
    line("the same, best-of-K apart", 7, PK_EE_POSE, 0.01f, 33, false, 32736);
    line("8 joints", 8, PK_EE_POSE, 0.01f, 1, false, 16384);
    line("8 joints, FP64 steps", 8, PK_EE_POSE, 0.f, 1, false, 32768);
    line("8 joints, position", 8, PK_EE_POSITION, 0.01f, 1, false, 32768);
    line("9 joints", 9, PK_EE_POSE, 0.f, 1, false, 16384);
    // parts of a launch: every workgroup once, each part under 2^32 threads
    const int64_t big = (int64_t)1 << 31;
    for (int64_t n : {(int64_t)1, (int64_t)64, (int64_t)65, big / 2, big / 2 + 1, big - 1, 4 * big + 3})
        for (int per_block : {1, 33, 64})
            for (int threads : {64, 256}) {
                const int64_t all = (n + per_block - 1) / per_block;
                int64_t next = 0;
                bool ok = true;
                const hipError_t e = launch_parts(all, threads, [&](int64_t b, unsigned blocks) {
                    ok = ok && b == next && blocks > 0 && (int64_t)blocks * threads < ((int64_t)1 << 32);
                    next = b + blocks;
                    return hipSuccess;
                });
                if (!ok || e != hipSuccess || next != all) {
                    ++failures;
                    printf("FAIL parts of %lld workgroups of %d threads\n", (long long)all, threads);
                }
            }
    // parts of a batch with a wavefront per problem: a problem's target in its part
    // is its target in the batch
    for (int64_t K : {(int64_t)1, (int64_t)3, (int64_t)64, (int64_t)99, (int64_t)100, (int64_t)101, (int64_t)250, (int64_t)1000})
        for (int64_t N = K; N <= 2000; N += K) {
            int64_t p0 = 0, n;
            for (; p0 < N; p0 += n) {
                n = part_size(N, K, p0, 100);
                bool ok = n > 0 && n <= 100;
                for (int64_t p = 0; ok && p < n; ++p) ok = p0 / K + p / K == (p0 + p) / K;
                if (!ok) {
                    ++failures;
                    printf("FAIL part at %lld of %lld, K=%lld: %lld\n", (long long)p0, (long long)N, (long long)K, (long long)n);
                    break;
                }
            }
            if (p0 != N) ++failures;
        }
    SolveParams P = batch(10, 2, 0.f);
    P.target_exit = 1;
    if (lane::takes_quad(1, 7, PK_EE_POSE, P, false) || lane::takes_star(4, 4, P)) {
        ++failures;
        printf("FAIL target_exit\n");
    }
    printf("%d failures\n", failures);
    return failures ? 1 : 0;
}
