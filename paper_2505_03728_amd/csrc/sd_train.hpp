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
// with a batch of 8192: 335 us a step -> 98 (row pass 50, weight gradients 38, the rest 9).
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

// What the row pass leaves for the gradients, all row-major over the batch.
struct TrainActs {
    int64_t rows;
    __bf16 *in[TR_MAX_LAYERS];      // [rows][lin] input of layer l
    __bf16 *dz[TR_MAX_LAYERS];      // [rows][lout] gradient at layer l's output (before SiLU)
    float *colpart;                 // bias partials: layer l's [rows/128][4][lout] at cpoff[l]
    int64_t cpoff[TR_MAX_LAYERS];
    float *rowloss;                 // [rows]
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

template <int H>
struct RowGeo {
    static constexpr int NW = H / 32;                // wavefronts, 32 columns each
    static constexpr int NT = H / (16 * NW);         // column blocks per wavefront
    static constexpr int KB = H / 32;
    static constexpr int RING = KB < 2 ? KB : 2;     // K steps of weights in flight
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
// (later the gradient tile) and the last hidden layer's pre-activations stay
// in LDS, the other pre-activations in registers (with 128 of them 19 values of
// the widest and deepest net go through scratch memory); weights stream from L2 in
// fragment order, a layer's first steps fetched before the previous layer's
// epilogue.
//
// A workgroup's rows are every fourth row of a 128-row chunk, r0 + 4 k: the
// bias gradients add exactly these rows one after the other, so each column
// is summed here, in FP32 from LDS, and the FP32 gradients (50 MB a step at
// width 512 and 8192 rows) never go to memory.
template <int H, int DEPTH>
__global__ __launch_bounds__(64 * RowGeo<H>::NW) void train_rows_kernel(TrainNet net, TrainActs A, TrainBatch T)
{
    using G = RowGeo<H>;
    constexpr int NW = G::NW, NT = G::NT, KB = G::KB, RING = G::RING;
    constexpr int THREADS = 64 * NW;
    constexpr int LD = H + 8, LZ = H + 4;   // 16 consecutive rows start 4 banks apart
    __shared__ __attribute__((aligned(16))) __bf16 act[TR_ROWS * LD];
    __shared__ __attribute__((aligned(16))) __bf16 x0[TR_ROWS * 32];
    __shared__ __attribute__((aligned(16))) __bf16 dyb[TR_ROWS * 64];
    __shared__ __attribute__((aligned(16))) float yt[TR_ROWS * 64];
    __shared__ __attribute__((aligned(16))) float zt[TR_ROWS * LZ];   // a layer's pre-activations, FP32 gradients
    __shared__ float qs[TR_ROWS * 64];
    const int tid = threadIdx.x, wn = tid >> 6, lane = tid & 63, r16 = lane & 15, g = lane >> 4;
    const int64_t row0 = (int64_t)(blockIdx.x >> 2) * 128 + (blockIdx.x & 3);   // row r: row0 + 4 r
    auto act_at = [&](int R, int ch) { return &act[R * LD + 8 * ch]; };
    // a BF16 tile of C columns (row stride ld in LDS) -> rows of base [rows][C]
    auto store_rows = [&](__bf16 *base, const __bf16 *tile, int ld, int C) {
        for (int e = tid; e < TR_ROWS * C / 8; e += THREADS) {
            const int r = e / (C / 8), ch = e % (C / 8);
            *(bf16x8 *)&base[(row0 + 4 * r) * C + 8 * ch] = *(const bf16x8 *)&tile[r * ld + 8 * ch];
        }
    };
    // column sums of an FP32 tile, rows in order -> the layer's bias partials
    auto column_sums = [&](int l, const float *tile, int ld, int C) {
        for (int c = tid; c < C; c += THREADS) {
            float s = 0.f;
#pragma unroll
            for (int r = 0; r < TR_ROWS; ++r) s += tile[r * ld + c];
            A.colpart[A.cpoff[l] + (int64_t)blockIdx.x * C + c] = s;
        }
    };

    const __bf16 *wf[DEPTH + 1], *wt[DEPTH + 1];
#pragma unroll
    for (int l = 0; l <= DEPTH; ++l) {
        wf[l] = net.Wf + net.foff[l] + lane * 8;
        wt[l] = net.Wt + net.foff[l] + lane * 8;
    }
    bf16x8 b0[1][NT], b[RING][NT];
    row_prefetch<NT, 1, 1>(b0, wf[0] + (size_t)wn * NT * 512);

    // the batch's rows: all sample numbers first, then all values, so that a
    // thread waits for memory twice and not twice per value
    {
        constexpr int NX = TR_ROWS * 32 / THREADS, NQ = TR_ROWS * 64 / THREADS;
        auto sample = [&](int r) -> int64_t {
            const int64_t pos = T.pos0 + row0 + 4 * r;
            return T.perm ? T.perm[pos] : pos;
        };
        int64_t sx[NX], sq[NQ];
        float vx[NX], vq[NQ];
#pragma unroll
        for (int i = 0; i < NX; ++i) sx[i] = sample((tid + i * THREADS) >> 5);
#pragma unroll
        for (int i = 0; i < NQ; ++i) sq[i] = sample((tid + i * THREADS) >> 6);
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            const int u = (tid + i * THREADS) & 31;
            vx[i] = sx[i] >= 0 && sx[i] < T.samples && u < 7 ? T.x[sx[i] * 7 + u] : 0.f;
        }
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            const int j = (tid + i * THREADS) & 63;
            vq[i] = sq[i] >= 0 && sq[i] < T.samples && j < T.n ? T.q[sq[i] * T.qs + j * T.qj] : 0.f;
        }
#pragma unroll
        for (int i = 0; i < NX; ++i) x0[tid + i * THREADS] = (__bf16)vx[i];
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            const int e = tid + i * THREADS, j = e & 63;
            if (j < T.n) qs[(e >> 6) * T.n + j] = vq[i];
        }
    }
    __syncthreads();
    store_rows(A.in[0], x0, 32, 32);

    f32x4 acc[2][NT], Z[DEPTH][2][NT];      // (Z[DEPTH - 1] is zt)
    auto zero = [&]() {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    auto from_act = [&](int i, int kb) { return *(const bf16x8 *)act_at(16 * i + r16, 4 * kb + g); };

    // forward, hidden layers
    constexpr int NO = NW >= 8 ? 1 : 2;     // row blocks per wavefront of the output layer
    bf16x8 bo[RING][1];
    const int i0 = NW >= 8 ? wn & 1 : 0, jb = NW >= 8 ? wn >> 1 & 3 : wn;   // its tile (16 x 16 each)
    const __bf16 *wo = wf[DEPTH] + (size_t)jb * KB * 512;
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
                if (l == DEPTH - 1) {
                    float *z = &zt[(16 * i + r16) * LZ + frag_col(wn * NT + 2 * p, 4 * g, true)];
                    *(f32x4 *)z = z0;
                    *(f32x4 *)(z + 4) = z1;
                } else {
                    Z[l][i][2 * p] = z0;
                    Z[l][i][2 * p + 1] = z1;
                }
                const bf16x8 h = {(__bf16)silu(z0[0]), (__bf16)silu(z0[1]), (__bf16)silu(z0[2]),
                                  (__bf16)silu(z0[3]), (__bf16)silu(z1[0]), (__bf16)silu(z1[1]),
                                  (__bf16)silu(z1[2]), (__bf16)silu(z1[3])};
                *(bf16x8 *)act_at(16 * i + r16, 4 * (wn * NT / 2 + p) + g) = h;
            }
        }
        __syncthreads();
        store_rows(A.in[l + 1], act, LD, H);
    }
    // output layer: y = acc + b
    if (wn < 8) {
        f32x4 ao[NO][1];
#pragma unroll
        for (int i = 0; i < NO; ++i) ao[i][0] = f32x4{0.f, 0.f, 0.f, 0.f};
        row_kloop<NO, 1, KB, RING>(ao, bo, wo, [&](int i, int kb) { return from_act(i0 + i, kb); });
        const f32x4 co = *(const f32x4 *)&net.P[net.boff[DEPTH] + 16 * jb + 4 * g];
#pragma unroll
        for (int i = 0; i < NO; ++i) *(f32x4 *)&yt[(16 * (i0 + i) + r16) * 64 + 16 * jb + 4 * g] = ao[i][0] + co;
    }
    bf16x8 bd[2][NT];
    row_prefetch<NT, 2, 2>(bd, wt[DEPTH] + (size_t)wn * NT * 2 * 512);
    __syncthreads();

    // loss: loss_kernel's arithmetic, one wavefront per row
    {
        const int n = T.n, K = T.K, kn = K * n;
        const float sc = 2.f / (float)A.rows;
#pragma unroll
        for (int rr = 0; rr < TR_ROWS / NW; ++rr) {
            const int r = rr * NW + wn;
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
            yt[r * 64 + lane] = gr;
            dyb[r * 64 + lane] = (__bf16)gr;
            if (lane == 0) A.rowloss[row0 + 4 * r] = bdist;
        }
    }
    __syncthreads();
    column_sums(DEPTH, yt, 64, 64);
    store_rows(A.dz[DEPTH], dyb, 64, 64);

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
                float *zp = &zt[(16 * i + r16) * LZ + frag_col(wn * NT + 2 * p, 4 * g, true)];
                f32x4 d[2];
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const f32x4 v = acc[i][2 * p + q];
                    const f32x4 z = l == DEPTH - 1 ? *(const f32x4 *)(zp + 4 * q) : Z[l][i][2 * p + q];
                    d[q] = f32x4{v[0] * silu_grad(z[0]), v[1] * silu_grad(z[1]), v[2] * silu_grad(z[2]),
                                 v[3] * silu_grad(z[3])};
                    *(f32x4 *)(zp + 4 * q) = d[q];
                }
                const bf16x8 h = {(__bf16)d[0][0], (__bf16)d[0][1], (__bf16)d[0][2], (__bf16)d[0][3],
                                  (__bf16)d[1][0], (__bf16)d[1][1], (__bf16)d[1][2], (__bf16)d[1][3]};
                *(bf16x8 *)act_at(16 * i + r16, 4 * (wn * NT / 2 + p) + g) = h;
            }
        __syncthreads();
        column_sums(l, zt, LZ, H);
        store_rows(A.dz[l], act, LD, H);
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
constexpr int DW_LD = DW_M + DW_N + 8;      // LDS row of a wavefront's slab: 32 columns of dZ, 64 of X

// MFMA fragment of 16 columns (at col) of a 32-row slab in LDS: lane (c, g)
// gets rows 8 g .. 8 g + 7 of column c.  The transposing read hands lane i of
// each 16 the i-th column of a 4 x 16 block whose row j lanes 4 j .. 4 j + 3
// address, four columns each.
PK_DEV bf16x8 slab_fragment(const __bf16 *slab, int lane, int col)
{
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    const int i = lane & 15;
    const __bf16 *p = slab + (8 * (lane >> 4) + (i >> 2)) * DW_LD + col + 4 * (i & 3);
    const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)p);
    const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(p + 4 * DW_LD));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

// Block and row (nb, c) of an output column under frag_col's pairing.
PK_DEV void frag_pos(int col, bool pair, int &nb, int &c)
{
    nb = pair ? 2 * (col >> 5) + ((col >> 2) & 1) : col >> 4;
    c = pair ? 4 * ((col >> 3) & 3) + (col & 3) : col & 15;
}

// Gradients of the weights (m, n .. n + 3) of layer l: G and, with ad.on,
// Adam and the BF16 copies (row-major and both fragment orders, laid out as
// in weight_fragments).
PK_DEV void take_gradient(const TrainNet &net, int l, int m, int n, f32x4 grad, const AdamArgs &ad)
{
    const int N = net.lin[l], M = net.lout[l];
    const int64_t at = net.woff[l] + (int64_t)m * N + n;
    *(f32x4 *)&net.G[at] = grad;
    if (!ad.on) return;
    const AdamStep st = ad.at();
    f32x4 p = *(const f32x4 *)&net.P[at], mo = *(const f32x4 *)&net.M[at], v = *(const f32x4 *)&net.V[at];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float pe = p[e], me = mo[e], ve = v[e];
        st(grad[e], pe, me, ve);
        p[e] = pe;
        mo[e] = me;
        v[e] = ve;
    }
    *(f32x4 *)&net.P[at] = p;
    *(f32x4 *)&net.M[at] = mo;
    *(f32x4 *)&net.V[at] = v;
    const bf16x4 h = {(__bf16)p[0], (__bf16)p[1], (__bf16)p[2], (__bf16)p[3]};
    *(bf16x4 *)&net.Pb[at] = h;
    int nb, c;
    frag_pos(m, l < net.depth, nb, c);
    *(bf16x4 *)&net.Wf[net.foff[l] + ((int64_t)nb * (N / 32) + n / 32) * 512 + (16 * (n % 32 / 8) + c) * 8 + n % 8] = h;
    if (l == 0) return;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        frag_pos(n + e, true, nb, c);
        net.Wt[net.foff[l] + ((int64_t)nb * (M / 32) + m / 32) * 512 + (16 * (m % 32 / 8) + c) * 8 + m % 8] = h[e];
    }
}

// dW [M][N] = dZ^T X of a 32 x 64 tile (NJ = 4; 32 x 32 with NJ = 2) over
// slice s of the rows, by one wavefront through its own slab of LDS, 32 rows
// at a time.
template <int NJ>
PK_DEV void dw_slice(const TrainNet &net, const TrainActs &A, int l, int mt, int nt, int s, int splits,
                     __bf16 *slab, f32x4 (&acc)[DW_M / 16][NJ])
{
    constexpr int NI = DW_M / 16, LA = 2, LB = NJ;   // 16-byte loads per lane and 32 rows: dZ, X
    constexpr int CB = 2 * NJ;                       // 16-byte chunks per slab row of X
    const int lane = threadIdx.x & 63, M = net.lout[l], N = net.lin[l];
    const int steps = (int)(A.rows / 32 / splits);
    const __bf16 *pa = A.dz[l] + (int64_t)(lane >> 2) * M + mt * DW_M + 8 * (lane & 3);
    const __bf16 *pb = A.in[l] + (int64_t)(lane / CB) * N + nt * 16 * NJ + 8 * (lane % CB);
    __bf16 *sa = slab + (lane >> 2) * DW_LD + 8 * (lane & 3);
    __bf16 *sb = slab + (lane / CB) * DW_LD + DW_M + 8 * (lane % CB);
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x8 a[2][LA], b[2][LB];
    auto load = [&](int u, int k) {
        const int64_t r = ((int64_t)s * steps + (k < steps ? k : steps - 1)) * 32;
#pragma unroll
        for (int i = 0; i < LA; ++i) a[u][i] = *(const bf16x8 *)&pa[(r + 16 * i) * M];
#pragma unroll
        for (int j = 0; j < LB; ++j) b[u][j] = *(const bf16x8 *)&pb[(r + 64 / CB * j) * N];
    };
    load(0, 0);
    load(1, 1);
    for (int k = 0; k < steps; k += 2) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (k + u < steps) {
#pragma unroll
                for (int i = 0; i < LA; ++i) *(bf16x8 *)&sa[16 * i * DW_LD] = a[u][i];
#pragma unroll
                for (int j = 0; j < LB; ++j) *(bf16x8 *)&sb[64 / CB * j * DW_LD] = b[u][j];
                load(u, k + u + 2);
                bf16x8 fa[NI];
#pragma unroll
                for (int i = 0; i < NI; ++i) fa[i] = slab_fragment(slab, lane, 16 * i);
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    const bf16x8 fb = slab_fragment(slab, lane, DW_M + 16 * j);
#pragma unroll
                    for (int i = 0; i < NI; ++i)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb, fa[i], acc[i][j], 0, 0, 0);
                }
            }
        }
    }
}

// Work of the weight-gradient launch.  A hidden layer's 32 x 64 tile is one
// workgroup's: its wavefronts take slices w, w + 8, .. of the rows and the
// slices are added in order after each round, so their partial products never
// go through memory.  The first and the last layer are too narrow to give
// every CU a tile of its own: their slices go one per wavefront on top of the
// tiles and their partial products (6 MB a step at width 512) to `part`,
// added in the next launch.  Taken as tiles too, they put a second workgroup
// on an eighth of the CUs, and the launch took 52.8 us against 38.3.
struct DwPlan {
    int tiles, tile_first[TR_MAX_LAYERS + 1];   // hidden layer l's tiles: tile_first[l] .. tile_first[l + 1]
    int units;                                  // slices of tiles of layers `depth`, then 0
    int splits[TR_MAX_LAYERS];
    float *part;                                // [splits][M * N] of layer depth, then of layer 0
    int64_t part0;                              // offset of layer 0's
};

// Bound: the operands' way through L1 (1.5 MB per tile at 8192 rows).  Each
// of the 8 XCDs takes a contiguous run of the tile list, and a layer's tiles
// are listed by quadrant, so that an XCD's L2 serves about half of the
// columns of one layer's operands and not an eighth of every layer's.
__global__ __launch_bounds__(64 * DW_WAVES) __attribute__((amdgpu_waves_per_eu(4))) void train_dw_kernel(
    TrainNet net, TrainActs A, DwPlan plan, AdamArgs ad)
{
    constexpr int NI = DW_M / 16, NJ = DW_N / 16;
    constexpr int RED = DW_WAVES * NI * NJ * 64 * 16, SLABS = DW_WAVES * 32 * DW_LD * 2;
    __shared__ __attribute__((aligned(16))) char lds[RED > SLABS ? RED : SLABS];
    f32x4 *red = (f32x4 *)lds;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    __bf16 *slab = (__bf16 *)lds + w * 32 * DW_LD;
    // slices of the narrow layers
    for (int u = w * gridDim.x + blockIdx.x; u < plan.units; u += DW_WAVES * gridDim.x) {
        const int L = net.depth, nout = plan.splits[L] * (net.lout[L] / DW_M) * (net.lin[L] / DW_N);
        if (u < nout) {
            const int tn = net.lin[L] / DW_N, tiles = net.lout[L] / DW_M * tn, s = u / tiles, t = u % tiles;
            f32x4 acc[NI][NJ];
            dw_slice<NJ>(net, A, L, t / tn, t % tn, s, plan.splits[L], slab, acc);
            float *o = plan.part + (int64_t)s * net.lout[L] * net.lin[L];
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
                    *(f32x4 *)&o[(int64_t)(t / tn * DW_M + 16 * i + (lane & 15)) * net.lin[L] + t % tn * DW_N + 16 * j +
                                 4 * (lane >> 4)] = acc[i][j];
        } else {
            const int v = u - nout, tiles = net.lout[0] / DW_M, s = v / tiles, t = v % tiles;
            f32x4 acc[NI][2];
            dw_slice<2>(net, A, 0, t, 0, s, plan.splits[0], slab, acc);
            float *o = plan.part + plan.part0 + (int64_t)s * net.lout[0] * 32;
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    *(f32x4 *)&o[(int64_t)(t * DW_M + 16 * i + (lane & 15)) * 32 + 16 * j + 4 * (lane >> 4)] = acc[i][j];
        }
    }
    // this workgroup's tile (workgroups go to the XCDs in turn)
    int t = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    if (t >= plan.tiles) return;
    int l = 1;
    while (t >= plan.tile_first[l + 1]) ++l;
    t -= plan.tile_first[l];
    // quadrants of the tile grid (both sides even: widths are multiples of 128)
    const int hm = net.lout[l] / DW_M / 2, hn = net.lin[l] / DW_N / 2, q = t / (hm * hn), i0 = t % (hm * hn);
    const int mt = (q >> 1) * hm + i0 / hn, nt = (q & 1) * hn + i0 % hn, splits = plan.splits[l];
    f32x4 total = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < splits; s0 += DW_WAVES) {
        f32x4 acc[NI][NJ];
        if (s0 + w < splits) dw_slice<NJ>(net, A, l, mt, nt, s0 + w, splits, slab, acc);
        __syncthreads();   // red overlays the slabs
        if (s0 + w < splits) {
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
    if (w < NI * NJ)
        take_gradient(net, l, mt * DW_M + 16 * (w / NJ) + (lane & 15), nt * DW_N + 16 * (w % NJ) + 4 * (lane >> 4),
                      total, ad);
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
    int wfirst, w0first;             // workgroups of the weights of layers depth and 0 (1024 each)
    int loss_wg;                     // the loss's workgroup
};

// Bias gradients (the column sums' last two levels) with Adam, the narrow
// layers' slices added in order with Adam, the batch's loss
// (loss_finish_kernel's sums) and the step counter.
__global__ __launch_bounds__(256) void train_finish_kernel(TrainNet net, TrainActs A, DwPlan dw, FinishPlan plan,
                                                           AdamArgs ad, int *dstep, float *loss_out)
{
    __shared__ float red[256];
    const int b = blockIdx.x, tid = threadIdx.x, nb = plan.bfirst[net.depth + 1];
    if (b == plan.loss_wg) {
        const int nparts = (int)(A.rows / 16);
        float s = 0.f;
        for (int i = tid; i < nparts; i += 256) {   // 16 rows, as loss_kernel's workgroups add them
            float w[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                w[j] = 0.f;
#pragma unroll
                for (int r = 0; r < 4; ++r) w[j] += A.rowloss[16 * i + 4 * j + r];
            }
            s += ((w[0] + w[1]) + w[2]) + w[3];
        }
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
        const int l = b >= plan.w0first ? 0 : net.depth, M = net.lout[l], N = net.lin[l], splits = dw.splits[l];
        const int64_t cnt = (int64_t)M * N, e = ((int64_t)(b - (l ? plan.wfirst : plan.w0first)) * 256 + tid) * 4;
        if (e >= cnt) return;
        const float *p = dw.part + (l ? 0 : dw.part0) + e;
        f32x4 g = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
        for (int z = 0; z < splits; ++z) {
            const f32x4 v = *(const f32x4 *)&p[z * cnt];
            g = splits == 1 ? v : g + v;
        }
        take_gradient(net, l, (int)(e / N), (int)(e % N), g, ad);
        return;
    }
    int l = 0;
    while (b >= plan.bfirst[l + 1]) ++l;
    const int C = net.lout[l], cl = tid & 63, ph = tid >> 6, c = (b - plan.bfirst[l]) * 64 + cl;
    const int nchunk = (int)(A.rows / 128);
    const float *part = A.colpart + A.cpoff[l];
    float s = 0.f;
    for (int i = ph; i < nchunk; i += 4) {   // colsum_pass1's chunk sum from its four phases
        const float *x = part + (int64_t)4 * i * C + c;
        s += ((x[0] + x[C]) + x[2 * C]) + x[3 * C];
    }
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
