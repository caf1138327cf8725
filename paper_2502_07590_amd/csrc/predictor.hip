// Predictor side (paper Sec. "Low-Rank based Sparsity Prediction"): the approximation loss
//     0.95 * CosLoss + 0.05 * NormLoss   between  Ahat = (Q_s Wq)(K Wk)^T  and  A = Q_s K^T
// on a sample of query rows, and its gradients for Wq and Wk -- without ever forming a row of A or Ahat.
//
// Every quantity the loss needs is a quadratic form in the key Gram matrix M = K^T K [d, d]:
//     |a_i|^2 = q_i^T M q_i,   <ahat_i, a_i> = qlr_i^T (Wk^T M q_i),   |ahat_i|^2 = qlr_i^T (Wk^T M Wk) qlr_i,
//     sum_j (ahat_ij - a_ij)^2 = |ahat_i|^2 - 2 <ahat_i, a_i> + |a_i|^2,
// and with dAhat_i = ca_i a_i + ch_i ahat_i (the chain rule of the two terms; coefficients below)
//     dWq = Q_s^T G,           G_i  = ca_i (Wk^T M q_i) + ch_i (Wk^T M Wk) qlr_i        (= dAhat_i Klr)
//     dWk = M (N1 + Wk N2),    N1 = sum_i ca_i q_i qlr_i^T,  N2 = sum_i ch_i qlr_i qlr_i^T   (= K^T dAhat^T Qlr).
// So the only pass over all L keys is the Gram matrix (K is read once: HBM-bound); the rest is small dense
// algebra on [d, d], [d, r] and the n sampled rows, done in fp64 (the norm term cancels to a small difference
// of large sums when the predictor is good).  The paper's point -- no [n, L] intermediate is stored -- holds in
// the strongest form: none is computed.
//
// Both kinds of contraction run on the matrix cores: the Gram matrix in the storage type with fp32 sums over at most
// 512 tokens (v_mfma_f32_32x32x16_bf16 / 32x32x2_f32), everything behind it in fp64 (v_mfma_f64_16x16x4_f64).
// L = 131072, 6 heads, 8192 rows each, bf16, r = 16: 143 us in all, of them gram_partial 48 (K at 4.2 TB/s), rows 41, accum 18; 167 with
// the weights' products and the loss in kernels and loops of their own, all of M in the rows' forms and half the blocks in accum.
// L = 3000, one head, 250 rows, d = 64: 66 -> 35 us.
#include <algorithm>

#include "common.h"

namespace dsv {

typedef __attribute__((__vector_size__(4 * sizeof(double)))) double doublex4_t;

// v_mfma_f64_16x16x4_f64: lane l holds A[l % 16][l / 16] and B[l / 16][l % 16]; element v of the result is
// C[4 v + l / 16][l % 16].
__device__ __forceinline__ doublex4_t mfma_f64(double a, double b, doublex4_t c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ double sum16(double x)  // over the 16 lanes that share l / 16
{
    for (int o = 8; o; o >>= 1) x += __shfl_xor(x, o);
    return x;
}

// ---- M = K^T K, partial sums over token blocks ---------------------------------------------------------
// A block takes tok_per_block tokens, kGramTok at a time through LDS.  The product's two operands are the same: 32
// channels by some tokens, tokens the contraction, so a fragment is a transposing LDS read of the parked rows (bf16) or
// a plain one (fp32).  D = 128: wave w forms rows 32 w .. 32 w + 31 of M; D = 64: one 32 x 32 tile per wave.
// Bound by reading K: 8 bytes per CU and clock against 128 clocks of matrix work per 4 KB.
constexpr int kGramTok = 64;     // tokens per LDS tile
constexpr int kGramFlush = 512;  // tokens summed in one chain of fp32 additions

template <typename T, int D>
__global__ __launch_bounds__(256) void gram_partial_kernel(const T *__restrict__ K, int L, int tok_per_block,
                                                           float *__restrict__ part)
{
    constexpr int NB = D / 32;
    constexpr int TW = NB == 4 ? 4 : 1;                    // tiles per wave
    constexpr int PITCH = D * (int)sizeof(T) + 16;         // bytes from one parked row to the next
    constexpr int PPR = D * (int)sizeof(T) / 16;           // 16-byte pieces per row
    constexpr int NP = kGramTok * PPR / 256;               // pieces per thread and tile
    __shared__ __align__(16) unsigned char tile[2][kGramTok * PITCH];
    const int bh = blockIdx.y;
    const int t0 = blockIdx.x * tok_per_block, t1 = min(t0 + tok_per_block, L);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = lane & 31, half = lane >> 5;
    const int rb = NB == 4 ? wave : wave >> 1;             // row block of this wave
    const int cb0 = NB == 4 ? 0 : wave & 1;                // first column block
    const unsigned char *Kh = reinterpret_cast<const unsigned char *>(K + (int64_t)bh * L * D);
    uint4 next[NP];
    auto request = [&](int tb) {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int e = threadIdx.x + 256 * i;
            const int t = tb + e / PPR;
            next[i] = make_uint4(0u, 0u, 0u, 0u);
            if (t < t1) next[i] = *reinterpret_cast<const uint4 *>(Kh + ((int64_t)t * PPR + e % PPR) * 16);
        }
    };
    floatx16_t acc[TW], sum[TW];
#pragma unroll
    for (int j = 0; j < TW; ++j)
#pragma unroll
        for (int i = 0; i < 16; ++i) { acc[j][i] = 0.f; sum[j][i] = 0.f; }
    request(t0);
    int buf = 0, since = 0;
    for (int tb = t0; tb < t1; tb += kGramTok, buf ^= 1) {
        unsigned char *ts = tile[buf];
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int e = threadIdx.x + 256 * i;
            *reinterpret_cast<uint4 *>(ts + (e / PPR) * PITCH + (e % PPR) * 16) = next[i];
        }
        __syncthreads();  // two tiles in turn: the one written next was last read before this barrier
        if (tb + kGramTok < t1) request(tb + kGramTok);
        if constexpr (sizeof(T) == 2) {
            const int c16 = lane & 15, g4 = lane >> 4;
            // rows 4 (c16 / 4) + 2 half (+ 1 in the second read) of 16: 64-byte stretches 16 banks apart
            const unsigned char *src = ts + (4 * (c16 >> 2) + 2 * half) * PITCH + (g4 & 1) * 32 + (c16 & 3) * 8;
#pragma unroll
            for (int s = 0; s < kGramTok / 16; ++s) {
                const unsigned char *p = src + s * 16 * PITCH;
                const bf16x8_t a = tr_frag(p + rb * 64, p + PITCH + rb * 64);
#pragma unroll
                for (int j = 0; j < TW; ++j)
                    acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, tr_frag(p + (cb0 + j) * 64, p + PITCH + (cb0 + j) * 64), acc[j], 0, 0, 0);
            }
        } else {
#pragma unroll 8
            for (int s = 0; s < kGramTok / 2; ++s) {
                const float *p = reinterpret_cast<const float *>(ts + (2 * s + half) * PITCH) + n;
                const float a = p[rb * 32];
#pragma unroll
                for (int j = 0; j < TW; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, p[(cb0 + j) * 32], acc[j], 0, 0, 0);
            }
        }
        if ((since += kGramTok) >= kGramFlush || tb + kGramTok >= t1) {
            since = 0;
#pragma unroll
            for (int j = 0; j < TW; ++j)
#pragma unroll
                for (int i = 0; i < 16; ++i) { sum[j][i] += acc[j][i]; acc[j][i] = 0.f; }
        }
    }
    float *out = part + ((int64_t)bh * gridDim.x + blockIdx.x) * D * D;
#pragma unroll
    for (int j = 0; j < TW; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) out[(32 * rb + 8 * (v / 4) + 4 * half + v % 4) * D + 32 * (cb0 + j) + n] = sum[j][v];
}

// M[bh] = sum of the partials, in fp64, in block order; of the 256 / D rows of M that a block forms also T1 = M Wk [D, R].
template <typename T, int D, int R>
__global__ __launch_bounds__(256) void gram_sum_kernel(const float *__restrict__ part, int nblk, const T *__restrict__ Wk, int H, double *__restrict__ M,
                                                       double *__restrict__ T1)
{
    constexpr int ROWS = 256 / D, TPE = 256 / (ROWS * R);  // threads that share an entry of T1
    __shared__ double m[256];
    const int e = blockIdx.x * 256 + threadIdx.x;
    const int64_t bh = blockIdx.y;
    const float *p = part + bh * nblk * (D * D) + e;
    double s = 0.0;
#pragma unroll 16
    for (int b = 0; b < nblk; ++b) s += (double)p[(int64_t)b * (D * D)];
    M[bh * (D * D) + e] = s;
    m[threadIdx.x] = s;
    __syncthreads();
    const int row = threadIdx.x / (TPE * R), t = threadIdx.x / TPE % R;
    const T *W = Wk + (bh % H) * D * R + t;
    double x = 0.0;
#pragma unroll 16
    for (int c = threadIdx.x % TPE; c < D; c += TPE) x += m[row * D + c] * (double)to_f32<T>(W[c * R]);
#pragma unroll
    for (int o = TPE / 2; o; o >>= 1) x += __shfl_xor(x, o);
    if (threadIdx.x % TPE == 0) T1[(bh * D + blockIdx.x * ROWS + row) * R + t] = x;
}

// T2 = Wk^T T1 [R, R], a thread per entry: for R = 64; below, every block of the rows' kernel forms its own.
template <typename T, int D, int R>
__global__ __launch_bounds__(256) void gram_weights2_kernel(const T *__restrict__ Wk, int H, const double *__restrict__ T1,
                                                            double *__restrict__ T2)
{
    const int64_t bh = blockIdx.y;
    const int e = blockIdx.x * 256 + threadIdx.x;
    const int a = e / R, b = e % R;
    const T *W = Wk + (bh % H) * D * R;
    double s = 0.0;
#pragma unroll 16
    for (int c = 0; c < D; ++c) s += (double)to_f32<T>(W[c * R + a]) * T1[(bh * D + c) * R + b];
    T2[bh * R * R + e] = s;
}

// ---- per sampled row ------------------------------------------------------------------------------------
// One wave per 16 sampled rows; U = Q_s M, Q_lr = Q_s Wq, V = Q_s T1 and W = Q_lr T2 as fp64 matrix products.  Writes, per
// row: qlr [R], G [R] (= dAhat_i Klr), the coefficients ca_i, ch_i and the loss terms {1 - cos_i, sum_j (ahat_ij - a_ij)^2}.
//   ca_i = -0.95 / (n |ahat_i| |a_i|) - 0.1 / (n L),   ch_i = 0.95 <ahat_i, a_i> / (n |ahat_i|^3 |a_i|) + 0.1 / (n L)
// Bound by the fp64 multiplications, 3 D^2 / 4 per row and more (64 clocks per 16 x 16 x 4 product); with few rows, by the way to M, T1 and Wq.  A lane group
// takes channels side by side: in steps of four rows of these every load has an address of its own (six heads, 57 rows each, R = 64: 64 -> 55 us; R = 16, 8192 rows:
// 44 -> 41).
template <typename T, int D, int R>
__global__ __launch_bounds__(256) void predictor_rows_kernel(const T *__restrict__ Q, const T *__restrict__ Wq, const T *__restrict__ Wk,
                                                             const int32_t *__restrict__ rows, int n, int L, int H,
                                                             const double *__restrict__ M, const double *__restrict__ T1,
                                                             const double *__restrict__ T2, double *__restrict__ qlr_out,
                                                             double *__restrict__ g_out, double2 *__restrict__ coef,
                                                             double2 *__restrict__ terms)
{
    constexpr int CPL = D / 4, RPL = R / 4, NT = R / 16;   // contraction steps: lane group g takes CPL / 2 channels in a row of either half
    constexpr bool OWN_T2 = R < 64;                        // (at R = 64 it would take the LDS of a second block)
    __shared__ float xq_all[4][16][D + 1];
    __shared__ double ql_all[4][16][R + 1];
    __shared__ double t2[OWN_T2 ? R * R : 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r16 = lane & 15, g = lane >> 4;
    const int i0 = (blockIdx.x * 4 + wave) * 16;
    const int64_t bh = blockIdx.y;
    const T *Wh = Wq + (bh % H) * D * R;
    const double *Mh = M + bh * D * D, *T1h = T1 + bh * D * R;
    if constexpr (OWN_T2) {  // T2 = Wk^T T1: a tile per wave (R = 32), or a quarter of the contraction (R = 16)
        const T *Wkh = Wk + (bh % H) * D * R;
        const int ta = NT == 1 ? 0 : wave / NT, tb = NT == 1 ? 0 : wave % NT, s0 = NT == 1 ? wave * (CPL / 4) : 0;
        doublex4_t x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < (NT == 1 ? CPL / 4 : CPL); ++s) {
            const int c = (4 * (s0 + s) + g) * R + r16;
            x = mfma_f64((double)to_f32<T>(Wkh[c + 16 * ta]), T1h[c + 16 * tb], x);
        }
        if constexpr (NT == 1) {
            double *quarter = &ql_all[0][0][0];  // free until the rows' Q_lr come
#pragma unroll
            for (int v = 0; v < 4; ++v) quarter[wave * 256 + (4 * v + g) * 16 + r16] = x[v];
            __syncthreads();
            t2[threadIdx.x] = (quarter[threadIdx.x] + quarter[256 + threadIdx.x]) + (quarter[512 + threadIdx.x] + quarter[768 + threadIdx.x]);
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v) t2[(16 * ta + 4 * v + g) * R + 16 * tb + r16] = x[v];
        }
        __syncthreads();
    }
    const double *T2h = OWN_T2 ? t2 : T2 + bh * R * R;
    if (i0 >= n) return;  // whole wave; nothing below synchronises across waves
    float (*xq)[D + 1] = xq_all[wave];
    double (*ql)[R + 1] = ql_all[wave];
    const int row = min(max(rows[min(i0 + r16, n - 1)], 0), L - 1);
    const int c0 = g * (CPL / 2);
    auto channel = [&](int s) __attribute__((always_inline)) { return c0 + (s < CPL / 2 ? s : D / 2 + s - CPL / 2); };
    const T *qrow = Q + (bh * L + row) * D;
    double q[CPL];
#pragma unroll
    for (int s = 0; s < CPL; ++s) {
        const float x = to_f32<T>(qrow[channel(s)]);
        xq[r16][channel(s)] = x;
        q[s] = (double)x;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    double aa[4] = {0.0, 0.0, 0.0, 0.0}, ah[4] = {0.0, 0.0, 0.0, 0.0}, hh[4] = {0.0, 0.0, 0.0, 0.0};
    // |a|^2 = q^T M q by four blocks of D / 2 x D / 2 channels: the one above the diagonal twice, the one below it not at all.  (By blocks of 16 the
    // products are fewer still, but those loops come out slower, with four-row steps of channels: 8192 rows of six heads, D = 128, R = 16: 44 us, by blocks of 16 39 with loads where they
    // are used -- and 61 for 24 where few rows leave a wave alone with them -- or 68 with a column's loads ahead of its products.)
    const double *col = Mh + c0 * D + r16;  // rows s and D / 2 + s from there
#pragma unroll 1
    for (int nt = 0; nt < D / 32; ++nt) {
        doublex4_t u = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < CPL / 2; ++s) u = mfma_f64(q[s], col[s * D + 16 * nt], u);
#pragma unroll
        for (int v = 0; v < 4; ++v) aa[v] += u[v] * (double)xq[4 * v + g][16 * nt + r16];
    }
#pragma unroll 1
    for (int nt = D / 32; nt < D / 16; ++nt) {
        doublex4_t u = {0.0, 0.0, 0.0, 0.0}, w = u;
#pragma unroll
        for (int s = 0; s < CPL / 2; ++s) {
            u = mfma_f64(q[s], col[s * D + 16 * nt], u);
            w = mfma_f64(q[s + CPL / 2], col[(D / 2 + s) * D + 16 * nt], w);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) aa[v] += (2.0 * u[v] + w[v]) * (double)xq[4 * v + g][16 * nt + r16];
    }
    doublex4_t a[NT], b[NT];  // Q_lr and V
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        a[nt] = doublex4_t{0.0, 0.0, 0.0, 0.0};
        b[nt] = a[nt];
#pragma unroll
        for (int s = 0; s < CPL; ++s) {
            const int e = channel(s) * R + 16 * nt + r16;
            a[nt] = mfma_f64(q[s], (double)to_f32<T>(Wh[e]), a[nt]);
            b[nt] = mfma_f64(q[s], T1h[e], b[nt]);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) ql[4 * v + g][16 * nt + r16] = a[nt][v];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    doublex4_t w[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        w[nt] = doublex4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < RPL; ++s) w[nt] = mfma_f64(ql[r16][g * RPL + s], T2h[(g * RPL + s) * R + 16 * nt + r16], w[nt]);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            ah[v] += a[nt][v] * b[nt][v];
            hh[v] += a[nt][v] * w[nt][v];
        }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const double saa = sum16(aa[v]), sah = sum16(ah[v]), shh = sum16(hh[v]);
        const double na = sqrt(saa), nh = sqrt(shh);
        const double ca = -0.95 / ((double)n * nh * na) - 0.1 / ((double)n * (double)L);
        const double ch = 0.95 * sah / ((double)n * nh * nh * nh * na) + 0.1 / ((double)n * (double)L);
        const int i = i0 + 4 * v + g;
        if (i < n) {
            const int64_t o = (bh * n + i) * R + r16;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                qlr_out[o + 16 * nt] = a[nt][v];
                g_out[o + 16 * nt] = ca * b[nt][v] + ch * w[nt][v];
            }
            if (r16 == 0) {
                coef[bh * n + i] = make_double2(ca, ch);
                terms[bh * n + i] = make_double2(1.0 - sah / (na * nh), shh - 2.0 * sah + saa);
            }
        }
    }
}

// ---- sums over the sampled rows ---------------------------------------------------------------------------
// dWq = Q_s^T G [D, R],  N1 = Q_s^T (ca Q_lr) [D, R],  N2 = Q_lr^T (ch Q_lr) [R, R] and the two loss terms: every block takes kAccRows sampled rows
// (their Q rows in LDS) and writes its partial sums; predictor_sum_kernel adds them in block order (deterministic).
// Waves take the 16-channel row tiles of dWq and N1 (and of N2) in turn.
constexpr int kAccRows = 64;  // a lane per row for the loss terms
template <typename T, int D, int R>
__global__ __launch_bounds__(256) void predictor_accum_kernel(const T *__restrict__ Q, const int32_t *__restrict__ rows,
                                                              int n, int L, const double *__restrict__ qlr,
                                                              const double *__restrict__ gm, const double2 *__restrict__ coef,
                                                              const double2 *__restrict__ terms, double *__restrict__ part)
{
    constexpr int NT = R / 16, CT = D / 64;                 // column tiles; row tiles of dWq and N1 per wave
    __shared__ float xq[kAccRows][D + 1];
    const int64_t bh = blockIdx.y;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r16 = lane & 15, g = lane >> 4;
    doublex4_t s1[CT][NT], s2[CT][NT], s3[NT];
    const doublex4_t zero = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        s3[nt] = zero;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) { s1[ct][nt] = zero; s2[ct][nt] = zero; }
    }
    const int i0 = blockIdx.x * kAccRows, i1 = min(i0 + kAccRows, n);
    constexpr int EPP = 16 / (int)sizeof(T), PPR = D / EPP;  // elements per 16-byte piece, pieces per row
#pragma unroll
    for (int u = 0; u < kAccRows * PPR / 256; ++u) {
        const int e = threadIdx.x + 256 * u;
        const int i = e / PPR, c = e % PPR * EPP;
        const int row = min(max(rows[min(i0 + i, i1 - 1)], 0), L - 1);
        const RowChunk<T, EPP> x = load_chunk<T, EPP>(Q + (bh * L + row) * D + c);  // rows past the end meet zero weights
#pragma unroll
        for (int m = 0; m < EPP; ++m) {
            if constexpr (sizeof(T) == 4) xq[i][c + m] = __uint_as_float(x.w[m]);
            else xq[i][c + m] = __uint_as_float(m & 1 ? x.w[m / 2] & 0xFFFF0000u : x.w[m / 2] << 16);
        }
    }
    __syncthreads();
#pragma unroll 4
    for (int s = 0; s < kAccRows / 4; ++s) {
        const int i = i0 + 4 * s + g;
        const bool ok = i < i1;
        const int64_t r = bh * n + (ok ? i : i1 - 1);
        const double2 cf = ok ? coef[r] : make_double2(0.0, 0.0);
        double vg[NT], vl[NT], x[CT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            vg[nt] = ok ? gm[r * R + 16 * nt + r16] : 0.0;
            vl[nt] = qlr[r * R + 16 * nt + r16];
        }
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) x[ct] = (double)xq[4 * s + g][16 * (wave + 4 * ct) + r16];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                s1[ct][nt] = mfma_f64(x[ct], vg[nt], s1[ct][nt]);
                s2[ct][nt] = mfma_f64(x[ct], ok ? cf.x * vl[nt] : 0.0, s2[ct][nt]);
            }
        if (wave < NT) {  // row tile `wave` of N2
            const double xl = qlr[r * R + 16 * wave + r16];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) s3[nt] = mfma_f64(xl, ok ? cf.y * vl[nt] : 0.0, s3[nt]);
        }
    }
    double *o = part + (bh * gridDim.x + blockIdx.x) * (2 * D * R + R * R + 2);
    if (wave == 0) {  // the loss terms of the block's rows
        const int i = i0 + lane;
        double2 x = i < i1 ? terms[bh * n + i] : make_double2(0.0, 0.0);
        for (int d = 32; d; d >>= 1) {
            x.x += __shfl_xor(x.x, d);
            x.y += __shfl_xor(x.y, d);
        }
        if (lane == 0) {
            o[2 * D * R + R * R] = x.x;
            o[2 * D * R + R * R + 1] = x.y;
        }
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                const int e = (16 * (wave + 4 * ct) + 4 * v + g) * R + 16 * nt + r16;
                o[e] = s1[ct][nt][v];
                o[D * R + e] = s2[ct][nt][v];
            }
            if (wave < NT) o[2 * D * R + (16 * wave + 4 * v + g) * R + 16 * nt + r16] = s3[nt][v];
        }
}

// sums [2 D R + R R + 2] = dWq, N1, N2, loss terms over the blocks' partials; dWq is final.
__global__ __launch_bounds__(256) void predictor_sum_kernel(const double *__restrict__ part, int nchunk, int DR, int count,
                                                            double *__restrict__ sums, float *__restrict__ dWq)
{
    const int e = blockIdx.x * 256 + threadIdx.x;
    const int64_t bh = blockIdx.y;
    if (e >= count) return;
    const double *p = part + bh * nchunk * count + e;
    double s = 0.0;
#pragma unroll 16
    for (int c = 0; c < nchunk; ++c) s += p[(int64_t)c * count];
    if (e < DR) dWq[bh * DR + e] = (float)s;
    else sums[bh * count + e] = s;
}

// dWk = M (N1 + Wk N2) = M N1 + T1 N2; block 0 of a head also writes the loss {0.95 cos + 0.05 norm, cos, norm}.
template <int D, int R>
__global__ __launch_bounds__(256) void predictor_finish_kernel(const double *__restrict__ M, const double *__restrict__ T1,
                                                               const double *__restrict__ sums, int n, int L, float *__restrict__ loss,
                                                               float *__restrict__ dWk)
{
    const int64_t bh = blockIdx.y;
    const double *N1 = sums + bh * (2 * D * R + R * R + 2) + D * R, *N2 = N1 + D * R, *terms = N2 + R * R;
    const int e = blockIdx.x * 256 + threadIdx.x;
    const int c = e / R, t = e % R;
    double s = 0.0;
#pragma unroll 32
    for (int c2 = 0; c2 < D; ++c2) s += M[(bh * D + c) * D + c2] * N1[c2 * R + t];
#pragma unroll 16
    for (int t2 = 0; t2 < R; ++t2) s += T1[(bh * D + c) * R + t2] * N2[t2 * R + t];
    dWk[bh * D * R + e] = (float)s;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        const double lc = terms[0] / (double)n, lm = terms[1] / ((double)n * (double)L);
        loss[bh * 3 + 0] = (float)(0.95 * lc + 0.05 * lm);
        loss[bh * 3 + 1] = (float)lc;
        loss[bh * 3 + 2] = (float)lm;
    }
}

// ------------------------------------------------------------------------------------ host
PredictorLayout predictor_layout(const dsv_problem &p, int n)
{
    const size_t nbh = (size_t)p.B * p.H, D = p.d, R = p.r;
    PredictorLayout w{};
    // about three blocks per CU, of 256 to 2048 tokens: every block leaves a [D, D] partial to be written and read again
    const size_t want = (nbh * p.L + 767) / 768;
    w.tok_per_block = (int)std::min<size_t>(2048, std::max<size_t>(256, align_up(want, 64)));
    w.nblk = (p.L + w.tok_per_block - 1) / w.tok_per_block;
    w.nchunk = (n + kAccRows - 1) / kAccRows;
    size_t o = 0;
    w.part = o; o = align_up(o + nbh * w.nblk * D * D * 4, 256);
    w.M = o; o = align_up(o + nbh * D * D * 8, 256);
    w.T1 = o; o = align_up(o + nbh * D * R * 8, 256);
    w.T2 = o; o = align_up(o + nbh * R * R * 8, 256);
    w.qlr = o; o = align_up(o + nbh * n * R * 8, 256);
    w.g = o; o = align_up(o + nbh * n * R * 8, 256);
    w.coef = o; o = align_up(o + nbh * n * 16, 256);
    w.terms = o; o = align_up(o + nbh * n * 16, 256);
    w.acc = o; o = align_up(o + nbh * w.nchunk * (2 * D * R + R * R + 2) * 8, 256);
    w.sums = o; o = align_up(o + nbh * (2 * D * R + R * R + 2) * 8, 256);
    w.total = o;
    return w;
}

template <typename T, int D, int R>
static dsv_status predictor_t(const dsv_problem &p, const void *Q, const void *K, const void *Wq, const void *Wk,
                              const int32_t *rows, int n, float *loss, float *dWq, float *dWk, char *ws,
                              const PredictorLayout &w, hipStream_t st)
{
    const int nbh = p.B * p.H;
    float *part = reinterpret_cast<float *>(ws + w.part);
    auto f64 = [&](size_t at) { return reinterpret_cast<double *>(ws + at); };
    double2 *coef = reinterpret_cast<double2 *>(ws + w.coef), *terms = reinterpret_cast<double2 *>(ws + w.terms);
    constexpr int kSums = 2 * D * R + R * R + 2;
    hipLaunchKernelGGL((gram_partial_kernel<T, D>), dim3(w.nblk, nbh), dim3(256), 0, st, (const T *)K, p.L, w.tok_per_block, part);
    hipLaunchKernelGGL((gram_sum_kernel<T, D, R>), dim3(D * D / 256, nbh), dim3(256), 0, st, part, w.nblk, (const T *)Wk, p.H, f64(w.M), f64(w.T1));
    if (R == 64)
        hipLaunchKernelGGL((gram_weights2_kernel<T, D, R>), dim3(R * R / 256, nbh), dim3(256), 0, st, (const T *)Wk, p.H, f64(w.T1), f64(w.T2));
    DSV_LAUNCH_CHECK();
    hipLaunchKernelGGL((predictor_rows_kernel<T, D, R>), dim3((n + 63) / 64, nbh), dim3(256), 0, st, (const T *)Q, (const T *)Wq, (const T *)Wk, rows,
                       n, p.L, p.H, f64(w.M), f64(w.T1), f64(w.T2), f64(w.qlr), f64(w.g), coef, terms);
    hipLaunchKernelGGL((predictor_accum_kernel<T, D, R>), dim3(w.nchunk, nbh), dim3(256), 0, st, (const T *)Q, rows, n, p.L, f64(w.qlr),
                       f64(w.g), coef, terms, f64(w.acc));
    hipLaunchKernelGGL(predictor_sum_kernel, dim3((kSums + 255) / 256, nbh), dim3(256), 0, st, f64(w.acc), w.nchunk, D * R, kSums,
                       f64(w.sums), dWq);
    hipLaunchKernelGGL((predictor_finish_kernel<D, R>), dim3(D * R / 256, nbh), dim3(256), 0, st, f64(w.M), f64(w.T1), f64(w.sums), n, p.L, loss, dWk);
    DSV_LAUNCH_CHECK();
    return DSV_OK;
}

dsv_status launch_predictor_loss(const dsv_problem &p, const void *Q, const void *K, const void *Wq, const void *Wk,
                                 const int32_t *rows, int n, float *loss, float *dWq, float *dWk, char *ws,
                                 const PredictorLayout &w, hipStream_t st)
{
#define DSV_CASE(TT, DD, RR) \
    if (p.d == DD && p.r == RR) return predictor_t<TT, DD, RR>(p, Q, K, Wq, Wk, rows, n, loss, dWq, dWk, ws, w, st)
    if (p.dtype == DSV_BF16) {
        DSV_CASE(bf16_t, 64, 16); DSV_CASE(bf16_t, 64, 32); DSV_CASE(bf16_t, 64, 64);
        DSV_CASE(bf16_t, 128, 16); DSV_CASE(bf16_t, 128, 32); DSV_CASE(bf16_t, 128, 64);
    } else if (p.dtype == DSV_F32) {
        DSV_CASE(float, 64, 16); DSV_CASE(float, 64, 32); DSV_CASE(float, 64, 64);
        DSV_CASE(float, 128, 16); DSV_CASE(float, 128, 32); DSV_CASE(float, 128, 64);
    }
#undef DSV_CASE
    return DSV_EUNSUPPORTED;
}

}  // namespace dsv
