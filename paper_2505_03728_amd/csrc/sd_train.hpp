// Training step of the learned seeder in three launches: (1) the whole pass
// over the batch's rows, forward, loss and backward, (2) weight gradients
// with Adam, (3) bias gradients with Adam, the loss and the weight copies the
// next step reads.
//
// Every sum is taken in the order of the layer-by-layer pass (sd_gemm.hpp and
// the reductions of seeder.hip): the same MFMA on the same fragments with K
// ascending, the same split of the weight gradients' reduction with its
// slices added in order, the same row chains of the bias gradients and the
// loss.  The parameters after a step are the same bit for bit.
//
// Bound: the layer-by-layer step was 26 launches that moved every activation
// several times and read the weight gradients' operands across their leading
// dimension (bank conflicts in the transposing LDS stores).  7-512-512-512-56
// with a batch of 8192: 335 us a step -> 137.
#pragma once

#include "sd_mlp.hpp"

namespace pk {
namespace sd {

constexpr int TR_MAX_LAYERS = 4;    // weight matrices (depth 3 and the output)
constexpr int TR_ROWS = 32;         // rows per workgroup of the row pass

// Weight and bias tables of a network, padded as everywhere: layer l is
// W [lout][lin] at woff[l], b [lout] at boff[l].
struct TrainNet {
    int depth;                      // hidden layers; weight matrices 0 .. depth
    int lin[TR_MAX_LAYERS], lout[TR_MAX_LAYERS];
    int64_t woff[TR_MAX_LAYERS], boff[TR_MAX_LAYERS], foff[TR_MAX_LAYERS];
    float *P, *G, *M, *V;           // parameters, gradients, Adam moments (FP32)
    __bf16 *Pb;                     // BF16 parameters
    __bf16 *Wf, *Wt;                // fragment-order copies at foff[l]: for x W^T, for dz W
};

// Operands of the weight gradients in MFMA fragment order, K = the rows of
// the batch: column block cb (16 columns), row block kb (32 rows) of a
// matrix at (cb * rows/32 + kb) * 512, lane l = (c = l % 16, g = l / 16)
// holding rows 32 kb + 8 g .. + 7 of column 16 cb + c.
struct TrainActs {
    int64_t rows;
    __bf16 *in[TR_MAX_LAYERS];      // input of layer l
    __bf16 *dz[TR_MAX_LAYERS];      // gradient at layer l's output (before SiLU), BF16
    float *dz32[TR_MAX_LAYERS];     // the same in FP32, row-major
    float *colpart;                 // bias partials: layer l's [rows/128][lout] at cpoff[l]
    int64_t cpoff[TR_MAX_LAYERS];
    float *losspart;                // one per 16 rows
};

// Where the row pass takes its batch from: row i is sample perm[pos0 + i] (or
// pos0 + i) of x [..][7] (encoded inputs) and q (joint j of sample s at
// s * qs + j * qj).
struct TrainBatch {
    const float *x, *q;
    int64_t qs, qj, samples, pos0;
    const int *perm;
    int n, K;
};

// Column c (16 per block) of a 32-row BF16 tile in LDS as a fragment.
template <class At>
PK_DEV bf16x8 column_fragment(At at, int lane, int col)
{
    u16x8 v;
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = *(const unsigned short *)at(8 * (lane >> 4) + e, col);
    return __builtin_bit_cast(bf16x8, v);
}

template <int H>
struct RowGeo {
    static constexpr int NW = H >= 256 ? 8 : 4;      // wavefronts
    static constexpr int NT = H / (16 * NW);         // column blocks per wavefront
    static constexpr int KB = H / 32;
    static constexpr int RING = KB < 4 ? KB : 4;     // K steps of weights in flight
};

// acc[i][j] += A x B over KB steps of 32: A fragments ld_a(i, kb), B blocks
// wb + (j * KB + kb) * 512.  b holds the first RING steps' blocks on entry.
template <int NI, int NT, int KB, int RING, class LoadA>
PK_DEV void row_kloop(f32x4 (&acc)[NI][NT], bf16x8 (&b)[RING][NT], const __bf16 *__restrict__ wb, LoadA ld_a)
{
    bf16x8 a[2][NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) a[0][i] = ld_a(i, 0);
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
            if (kb + 1 < KB) a[(kb + 1) & 1][i] = ld_a(i, kb + 1);
#pragma unroll
        for (int j = 0; j < NT; ++j) {
#pragma unroll
            for (int i = 0; i < NI; ++i)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[kb % RING][j], a[kb & 1][i], acc[i][j], 0, 0, 0);
            if (kb + RING < KB) b[kb % RING][j] = *(const bf16x8 *)&wb[((size_t)j * KB + kb + RING) * 512];
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

template <int NT, int KB, int RING>
PK_DEV void row_prefetch(bf16x8 (&b)[RING][NT], const __bf16 *__restrict__ wb)
{
#pragma unroll
    for (int k = 0; k < RING && k < KB; ++k)
#pragma unroll
        for (int j = 0; j < NT; ++j) b[k][j] = *(const bf16x8 *)&wb[((size_t)j * KB + k) * 512];
}

// The row pass: 32 rows per workgroup, all layers.  The activation tile
// (later the gradient tile) stays in LDS and the pre-activations in
// registers; weights stream from L2 in fragment order, a layer's first steps
// fetched before the previous layer's epilogue.  Rows are independent, so
// only the weight stream (2.3 MB per workgroup at width 512) and the stores
// for the weight gradients leave the CU.
template <int H, int DEPTH>
__global__ __launch_bounds__(64 * RowGeo<H>::NW) void train_rows_kernel(TrainNet net, TrainActs A, TrainBatch T)
{
    using G = RowGeo<H>;
    constexpr int NW = G::NW, NT = G::NT, KB = G::KB, RING = G::RING;
    constexpr int THREADS = 64 * NW;
    constexpr int LD = H + 8;   // the 16 rows of a fragment read start 4 banks apart
    __shared__ __attribute__((aligned(16))) __bf16 act[TR_ROWS * LD];
    __shared__ __attribute__((aligned(16))) __bf16 x0[TR_ROWS * 32];
    __shared__ __attribute__((aligned(16))) __bf16 dyb[TR_ROWS * 64];
    __shared__ __attribute__((aligned(16))) float yt[TR_ROWS * 64];
    __shared__ float qs[TR_ROWS * 64], red[8];
    const int tid = threadIdx.x, wn = tid >> 6, lane = tid & 63, r16 = lane & 15, g = lane >> 4;
    const int64_t kbr = blockIdx.x, row0 = kbr * TR_ROWS, nkb = A.rows / 32;
    auto act_at = [&](int R, int ch) { return &act[R * LD + 8 * ch]; };
    auto act_el = [&](int R, int c) { return &act[R * LD + c]; };
    auto frag_out = [&](__bf16 *base, int cb) { return (bf16x8 *)&base[((int64_t)cb * nkb + kbr) * 512 + lane * 8]; };

    const __bf16 *wf[DEPTH + 1], *wt[DEPTH + 1];
#pragma unroll
    for (int l = 0; l <= DEPTH; ++l) {
        wf[l] = net.Wf + net.foff[l] + lane * 8;
        wt[l] = net.Wt + net.foff[l] + lane * 8;
    }
    bf16x8 b0[1][NT], b[RING][NT];
    row_prefetch<NT, 1, 1>(b0, wf[0] + (size_t)wn * NT * 512);

    // the batch's rows
    for (int e = tid; e < TR_ROWS * 32; e += THREADS) {
        const int r = e >> 5, u = e & 31;
        const int64_t pos = T.pos0 + row0 + r, s = T.perm ? T.perm[pos] : pos;
        const bool ok = s >= 0 && s < T.samples;
        x0[e] = (__bf16)(ok && u < 7 ? T.x[s * 7 + u] : 0.f);
    }
    for (int e = tid; e < TR_ROWS * 64; e += THREADS) {
        const int r = e >> 6, j = e & 63;
        if (j >= T.n) continue;
        const int64_t pos = T.pos0 + row0 + r, s = T.perm ? T.perm[pos] : pos;
        qs[r * T.n + j] = s >= 0 && s < T.samples ? T.q[s * T.qs + j * T.qj] : 0.f;
    }
    __syncthreads();
    if (wn < 2)
        *frag_out(A.in[0], wn) = column_fragment([&](int R, int c) { return &x0[R * 32 + c]; }, lane, 16 * wn + r16);

    f32x4 acc[2][NT], Z[DEPTH][2][NT];
    auto zero = [&]() {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    auto from_act = [&](int i, int kb) { return *(const bf16x8 *)act_at(16 * i + r16, 4 * kb + g); };

    // forward, hidden layers
    constexpr int NO = NW == 8 ? 1 : 2;     // row blocks per wavefront of the output layer
    bf16x8 bo[RING][1];
    const __bf16 *wo = wf[DEPTH] + (size_t)(NW == 8 ? wn >> 1 : wn) * KB * 512;
#pragma unroll
    for (int l = 0; l < DEPTH; ++l) {
        zero();
        const __bf16 *wl = wf[l] + (size_t)wn * NT * KB * 512;
        if (l == 0)
            row_kloop<2, NT, 1, 1>(acc, b0, wf[0] + (size_t)wn * NT * 512,
                                   [&](int i, int) { return *(const bf16x8 *)&x0[(16 * i + r16) * 32 + 8 * g]; });
        else
            row_kloop<2, NT, KB, RING>(acc, b, wl, from_act);
        if (l + 1 < DEPTH)
            row_prefetch<NT, KB, RING>(b, wf[l + 1] + (size_t)wn * NT * KB * 512);
        else
            row_prefetch<1, KB, RING>(bo, wo);
        const float *bias = net.P + net.boff[l];
        if (l > 0) __syncthreads();   // every wavefront has read the layer input
#pragma unroll
        for (int p = 0; p < NT / 2; ++p) {
            const f32x4 cv[2] = {*(const f32x4 *)&bias[frag_col(wn * NT + 2 * p, 4 * g, true)],
                                 *(const f32x4 *)&bias[frag_col(wn * NT + 2 * p + 1, 4 * g, true)]};
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const f32x4 z0 = acc[i][2 * p] + cv[0], z1 = acc[i][2 * p + 1] + cv[1];
                Z[l][i][2 * p] = z0;
                Z[l][i][2 * p + 1] = z1;
                const bf16x8 h = {(__bf16)silu(z0[0]), (__bf16)silu(z0[1]), (__bf16)silu(z0[2]),
                                  (__bf16)silu(z0[3]), (__bf16)silu(z1[0]), (__bf16)silu(z1[1]),
                                  (__bf16)silu(z1[2]), (__bf16)silu(z1[3])};
                *(bf16x8 *)act_at(16 * i + r16, 4 * (wn * NT / 2 + p) + g) = h;
            }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < NT; ++j)
            *frag_out(A.in[l + 1], wn * NT + j) = column_fragment(act_el, lane, 16 * (wn * NT + j) + r16);
    }
    // output layer: y = acc + b
    {
        f32x4 ao[NO][1];
#pragma unroll
        for (int i = 0; i < NO; ++i) ao[i][0] = f32x4{0.f, 0.f, 0.f, 0.f};
        const int i0 = NW == 8 ? wn & 1 : 0, jb = NW == 8 ? wn >> 1 : wn;
        row_kloop<NO, 1, KB, RING>(ao, bo, wo, [&](int i, int kb) { return from_act(i0 + i, kb); });
        const f32x4 co = *(const f32x4 *)&net.P[net.boff[DEPTH] + 16 * jb + 4 * g];
#pragma unroll
        for (int i = 0; i < NO; ++i) *(f32x4 *)&yt[(16 * (i0 + i) + r16) * 64 + 16 * jb + 4 * g] = ao[i][0] + co;
    }
    bf16x8 bd[2][NT];
    row_prefetch<NT, 2, 2>(bd, wt[DEPTH] + (size_t)wn * NT * 2 * 512);
    __syncthreads();

    // loss: loss_kernel's arithmetic, one wavefront per row, four rows each
    {
        const int n = T.n, K = T.K, kn = K * n;
        const float sc = 2.f / (float)A.rows;
        for (int pass = 0; pass < TR_ROWS / (4 * NW); ++pass) {
            float wl = 0.f;
            for (int rr = 0; rr < 4; ++rr) {
                const int r = 16 * (NW == 8 ? wn >> 2 : pass) + 4 * (wn & 3) + rr;
                float diff = 0.f;
                if (lane < kn) diff = yt[r * 64 + lane] - qs[r * n + lane % n];
                const float s2 = diff * diff;
                float dk = 0.f;
                for (int j = 0; j < n; ++j) dk += __shfl(s2, (lane < K ? lane : 0) * n + j, 64);
                float bdist = lane < K ? dk : INFINITY;
                int bi = lane;
#pragma unroll
                for (int o = 32; o >= 1; o >>= 1) {
                    const float od = __shfl_xor(bdist, o, 64);
                    const int oi = __shfl_xor(bi, o, 64);
                    if (od < bdist || (od == bdist && oi < bi)) {
                        bdist = od;
                        bi = oi;
                    }
                }
                const float gr = (lane < kn && lane / n == bi) ? sc * diff : 0.f;
                A.dz32[DEPTH][(row0 + r) * 64 + lane] = gr;
                dyb[r * 64 + lane] = (__bf16)gr;
                wl += bdist;
            }
            if (lane == 0) red[wn + 4 * pass] = wl;
        }
    }
    __syncthreads();
    if (tid < 2) {
        const float *rp = red + 4 * tid;
        A.losspart[kbr * 2 + tid] = ((rp[0] + rp[1]) + rp[2]) + rp[3];
    }
    if (wn < 4)
        *frag_out(A.dz[DEPTH], wn) = column_fragment([&](int R, int c) { return &dyb[R * 64 + c]; }, lane, 16 * wn + r16);

    // backward: dZ_l = (dZ_{l+1} W_{l+1}) SiLU'(Z_l)
#pragma unroll
    for (int l = DEPTH - 1; l >= 0; --l) {
        zero();
        if (l == DEPTH - 1)
            row_kloop<2, NT, 2, 2>(acc, bd, wt[DEPTH] + (size_t)wn * NT * 2 * 512,
                                   [&](int i, int kb) { return *(const bf16x8 *)&dyb[(16 * i + r16) * 64 + 32 * kb + 8 * g]; });
        else
            row_kloop<2, NT, KB, RING>(acc, b, wt[l + 1] + (size_t)wn * NT * KB * 512, from_act);
        if (l > 0) row_prefetch<NT, KB, RING>(b, wt[l] + (size_t)wn * NT * KB * 512);
        __syncthreads();   // every wavefront has read the tile
#pragma unroll
        for (int p = 0; p < NT / 2; ++p)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                f32x4 d[2];
                bf16x8 h;
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const f32x4 v = acc[i][2 * p + q], z = Z[l][i][2 * p + q];
                    d[q] = f32x4{v[0] * silu_grad(z[0]), v[1] * silu_grad(z[1]), v[2] * silu_grad(z[2]),
                                 v[3] * silu_grad(z[3])};
                }
                h = bf16x8{(__bf16)d[0][0], (__bf16)d[0][1], (__bf16)d[0][2], (__bf16)d[0][3],
                           (__bf16)d[1][0], (__bf16)d[1][1], (__bf16)d[1][2], (__bf16)d[1][3]};
                float *o = A.dz32[l] + (row0 + 16 * i + r16) * H + frag_col(wn * NT + 2 * p, 4 * g, true);
                *(f32x4 *)o = d[0];
                *(f32x4 *)(o + 4) = d[1];
                *(bf16x8 *)act_at(16 * i + r16, 4 * (wn * NT / 2 + p) + g) = h;
            }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < NT; ++j)
            *frag_out(A.dz[l], wn * NT + j) = column_fragment(act_el, lane, 16 * (wn * NT + j) + r16);
    }
}

// Adam (Kingma & Ba 2015) with bias correction on one value: adam_kernel's
// arithmetic.
struct AdamStep {
    float lr, b1, b2, eps, c1, c2;
    PK_DEV void operator()(float g, float &p, float &m, float &v) const
    {
        m = b1 * m + (1.f - b1) * g;
        v = b2 * v + (1.f - b2) * g * g;
        p = p - lr * (m / c1) / (sqrtf(v / c2) + eps);
    }
};

struct AdamArgs {
    int on;                 // 0: gradients only
    int step;               // t = step + 1
    float lr, b1, b2, eps;
    PK_DEV AdamStep at() const
    {
        const float t = (float)(step + 1);
        return AdamStep{lr, b1, b2, eps, 1.f - powf(b1, t), 1.f - powf(b2, t)};
    }
};

constexpr int DW_M = 32, DW_N = 64, DW_WAVES = 8;

// Tiles of a layer's weight gradient: 32 x 64 (32 x 32 for the 32-wide input).
PK_DEV int dw_tiles(int M, int N) { return (M / DW_M) * (N >= DW_N ? N / DW_N : 1); }

// One tile of dW [M][N] = dZ^T X: wavefront w takes slices w, w + 8, .. of
// the `splits` slices of the rows on its own (its fragments come straight
// from memory in fragment order, no LDS and no barrier in the reduction);
// after each round the slices are added in order, and at the end the tile's
// owner applies Adam.  One workgroup sees the whole reduction, so the slices'
// partial products never go through memory.
template <int NJ>
PK_DEV void dw_tile(const TrainNet &net, const TrainActs &A, int l, int mt, int nt, int splits,
                    const AdamArgs &ad, f32x4 *red)
{
    constexpr int NI = DW_M / 16, RING = 4;
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
    const int N = net.lin[l];
    const int64_t nkb = A.rows / 32;
    const int steps = (int)(nkb / splits);
    const __bf16 *pa = A.dz[l] + (int64_t)mt * NI * nkb * 512 + lane * 8;
    const __bf16 *pb = A.in[l] + (int64_t)nt * NJ * nkb * 512 + lane * 8;
    f32x4 total = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < splits; s0 += DW_WAVES) {
        const int s = s0 + w;
        if (s < splits) {
            f32x4 acc[NI][NJ];
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            const int64_t k0 = (int64_t)s * steps;
            bf16x8 a[RING][NI], b[RING][NJ];
            auto load = [&](int u, int k) {
                const int64_t kk = (k0 + (k < steps ? k : steps - 1)) * 512;
#pragma unroll
                for (int i = 0; i < NI; ++i) a[u][i] = *(const bf16x8 *)&pa[i * nkb * 512 + kk];
#pragma unroll
                for (int j = 0; j < NJ; ++j) b[u][j] = *(const bf16x8 *)&pb[j * nkb * 512 + kk];
            };
#pragma unroll
            for (int u = 0; u < RING; ++u) load(u, u);
            for (int k = 0; k < steps; k += RING) {
#pragma unroll
                for (int u = 0; u < RING; ++u) {
                    if (k + u < steps) {
#pragma unroll
                        for (int j = 0; j < NJ; ++j)
#pragma unroll
                            for (int i = 0; i < NI; ++i)
                                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[u][j], a[u][i], acc[i][j], 0, 0, 0);
                    }
                    load(u, k + u + RING);
                }
            }
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j) red[(w * NI * NJ + i * NJ + j) * 64 + lane] = acc[i][j];
        }
        __syncthreads();
        if (w < NI * NJ) {
            const int n = splits - s0 < DW_WAVES ? splits - s0 : DW_WAVES;
            for (int z = 0; z < n; ++z) {
                const f32x4 p = red[(z * NI * NJ + w) * 64 + lane];
                total = splits == 1 ? p : total + p;
            }
        }
        __syncthreads();
    }
    if (w >= NI * NJ) return;
    const int m = mt * DW_M + 16 * (w / NJ) + (lane & 15), n = nt * 16 * NJ + 16 * (w % NJ) + 4 * (lane >> 4);
    const int64_t at = net.woff[l] + (int64_t)m * N + n;
    *(f32x4 *)&net.G[at] = total;
    if (!ad.on) return;
    const AdamStep st = ad.at();
    f32x4 p = *(const f32x4 *)&net.P[at], mo = *(const f32x4 *)&net.M[at], v = *(const f32x4 *)&net.V[at];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float pe = p[e], me = mo[e], ve = v[e];
        st(total[e], pe, me, ve);
        p[e] = pe;
        mo[e] = me;
        v[e] = ve;
    }
    *(f32x4 *)&net.P[at] = p;
    *(f32x4 *)&net.M[at] = mo;
    *(f32x4 *)&net.V[at] = v;
    *(bf16x4 *)&net.Pb[at] = bf16x4{(__bf16)p[0], (__bf16)p[1], (__bf16)p[2], (__bf16)p[3]};
}

struct DwPlan {
    int first[TR_MAX_LAYERS + 1];    // workgroups of layer l's weight tiles: first[l] .. first[l + 1]
    int splits[TR_MAX_LAYERS];
    int cfirst[TR_MAX_LAYERS + 1];   // workgroups of layer l's bias partials, after the tiles
};

// Bias partials (colsum_pass1's sums): 128 rows of up to 512 columns per
// workgroup, thread = (row phase, 4 columns).
PK_DEV void bias_partial(const TrainNet &net, const TrainActs &A, int l, int item, f32x4 *red)
{
    const int C = net.lout[l], qc = min(C / 4, 128), groups = C / (4 * qc);
    const int chunk = item / groups, c0 = (item % groups) * 4 * qc;
    const int per = qc * 4, tid = threadIdx.x;       // threads in use per pass: 4 phases x qc
    if (tid < per) {
        const int ph = tid / qc, c = c0 + 4 * (tid % qc);
        const float *x = A.dz32[l] + ((int64_t)chunk * 128 + ph) * C + c;
        f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
        for (int r = 0; r < 32; ++r) s += *(const f32x4 *)&x[(int64_t)4 * r * C];
        red[tid] = s;
    }
    __syncthreads();
    if (tid < qc)
        *(f32x4 *)&A.colpart[A.cpoff[l] + (int64_t)chunk * C + c0 + 4 * tid] =
            ((red[tid] + red[qc + tid]) + red[2 * qc + tid]) + red[3 * qc + tid];
}

__global__ __launch_bounds__(64 * DW_WAVES) void train_dw_kernel(TrainNet net, TrainActs A, DwPlan plan, AdamArgs ad)
{
    __shared__ f32x4 red[DW_WAVES * (DW_M / 16) * (DW_N / 16) * 64];
    const int b = blockIdx.x, tiles = plan.first[net.depth + 1];
    if (b >= tiles) {
        int l = 0;
        while (b >= plan.cfirst[l + 1]) ++l;
        bias_partial(net, A, l, b - plan.cfirst[l], red);
        return;
    }
    int l = 0;
    while (b >= plan.first[l + 1]) ++l;
    int t = b - plan.first[l];
    const int M = net.lout[l], N = net.lin[l], tm = M / DW_M, tn = N >= DW_N ? N / DW_N : 1;
    // Workgroups go to the 8 XCDs in turn: give each a compact part of the
    // tile grid, so that its L2 serves the operands' column blocks again.
    if (tm % 4 == 0 && tn % 2 == 0) {
        const int x = t % 8, i = t / 8, pm = tm / 4, pn = tn / 2;
        t = ((x >> 1) * pm + i / pn) * tn + (x & 1) * pn + i % pn;
    }
    if (N >= DW_N)
        dw_tile<DW_N / 16>(net, A, l, t / tn, t % tn, plan.splits[l], ad, red);
    else
        dw_tile<2>(net, A, l, t, 0, plan.splits[l], ad, red);
}

// Fragment-order copies of layer l's BF16 weights, 16 bytes per thread: for
// x W^T as frag_layout_kernel, and for dz W: column block nb of W (paired, as
// frag_col), row block kb of 32 outputs at (nb * lout/32 + kb) * 512, lane
// (c, g) holding rows 32 kb + 8 g .. + 7 of column frag_col(nb, c).
PK_DEV void weight_fragments(const TrainNet &net, int l, int64_t p)
{
    const int N = net.lout[l], K = net.lin[l], lane = (int)(p % 64), c = lane & 15, g = lane >> 4;
    const __bf16 *W = net.Pb + net.woff[l];
    {
        const int KBf = K / 32, kb = (int)(p / 64 % KBf), nb = (int)(p / 64 / KBf);
        const int col = frag_col(nb, c, l < net.depth);
        *(uint4 *)&net.Wf[net.foff[l] + p * 8] = *(const uint4 *)&W[(size_t)col * K + 32 * kb + 8 * g];
    }
    if (l > 0) {
        const int KBt = N / 32, kb = (int)(p / 64 % KBt), nb = (int)(p / 64 / KBt);
        const int col = frag_col(nb, c, true);
        u16x8 v;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = *(const unsigned short *)&W[(size_t)(32 * kb + 8 * g + e) * K + col];
        *(u16x8 *)&net.Wt[net.foff[l] + p * 8] = v;
    }
}

__global__ void fragments_kernel(TrainNet net, int l)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < (int64_t)net.lin[l] * net.lout[l] / 8) weight_fragments(net, l, p);
}

struct FinishPlan {
    int bfirst[TR_MAX_LAYERS + 1];   // workgroups of layer l's biases (64 columns each)
    int ffirst[TR_MAX_LAYERS + 1];   // workgroups of layer l's fragments (256 threads)
    int loss_wg;                     // the loss's workgroup, -1: none
};

// Bias gradients (colsum_pass2's sums) with Adam, the batch's loss
// (loss_finish_kernel's sums), the step counter and the weight copies.
__global__ __launch_bounds__(256) void train_finish_kernel(TrainNet net, TrainActs A, FinishPlan plan, AdamArgs ad,
                                                           int *dstep, float *loss_out)
{
    __shared__ float red[256];
    const int b = blockIdx.x, tid = threadIdx.x, nb = plan.bfirst[net.depth + 1];
    if (b == plan.loss_wg) {
        const int nparts = (int)(A.rows / 16);
        float s = 0.f;
        for (int i = tid; i < nparts; i += 256) s += A.losspart[i];
        red[tid] = s;
        __syncthreads();
        for (int o = 128; o > 0; o >>= 1) {
            if (tid < o) red[tid] += red[tid + o];
            __syncthreads();
        }
        if (tid == 0) {
            if (loss_out) *loss_out = red[0] / (float)A.rows;
            if (ad.on) *dstep = ad.step + 1;
        }
        return;
    }
    if (b >= nb) {
        int l = 0;
        while (b >= plan.ffirst[l + 1]) ++l;
        const int64_t p = (int64_t)(b - plan.ffirst[l]) * 256 + tid;
        if (p < (int64_t)net.lin[l] * net.lout[l] / 8) weight_fragments(net, l, p);
        return;
    }
    int l = 0;
    while (b >= plan.bfirst[l + 1]) ++l;
    const int C = net.lout[l], cl = tid & 63, ph = tid >> 6, c = (b - plan.bfirst[l]) * 64 + cl;
    const int nchunk = (int)(A.rows / 128);
    const float *part = A.colpart + A.cpoff[l];
    float s = 0.f;
    for (int i = ph; i < nchunk; i += 4) s += part[(int64_t)i * C + c];
    red[tid] = s;
    __syncthreads();
    if (ph) return;
    const float g = ((red[cl] + red[64 + cl]) + red[128 + cl]) + red[192 + cl];
    const int64_t at = net.boff[l] + c;
    net.G[at] = g;
    if (!ad.on) return;
    const AdamStep st = ad.at();
    float p = net.P[at], m = net.M[at], v = net.V[at];
    st(g, p, m, v);
    net.P[at] = p;
    net.M[at] = m;
    net.V[at] = v;
    net.Pb[at] = (__bf16)p;
}

}  // namespace sd
}  // namespace pk
