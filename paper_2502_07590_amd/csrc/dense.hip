// Stage 2 forward over dense tiles with a selection mask (paper Sec. "Sparse Attention with Query Grouping", per-query form),
// bf16: the same sums as the gathering kernels, for heads that keep enough of their keys.
//
// A gathered (query, key) pair costs 18.5 ps at d = 128 -- 512 bytes through the vector memory path, whatever the density --;
// a pair of a dense tile costs 0.7 ps on the matrix cores, selected or not, because the tile's K and V rows cross that path
// once for 128 queries.  So from about one key in 25 on it is cheaper to form every pair and mask the others out (the
// rule, with the sizes that fill the chip, stands with dense_fwd_min_k).  L = 32768, four heads, k = 2048: 4.92 -> 3.40 ms,
// 0.4 of them the mask.
// The mask is a bit matrix [queries, keys] built from the index rows (bits_build_kernel: any order), some queries at a time.
//
//   S^T = K Q^T       v_mfma_f32_32x32x16_bf16, A = K rows out of LDS, B = the wave's 32 queries (registers).  A lane holds
//                     one query against 16 keys of the tile, so that masking, maximum, exponentials and sums stay in the
//                     lane; the two lanes of a query only meet when its maximum moves.
//   O^T += V^T P^T    B = the probabilities, which those lanes hold in the B layout already (which keys a lane group
//                     contracts is free: 16 s + 4 half + e % 4 + 8 (e / 4)), A = V transposed out of LDS (tr_frag).
//                     The probabilities go in as bf16 head and tail, 16 significant bits: the result is then as far from the
//                     64-bit one as its rounding to bf16 puts it (1.66e-3).  One bf16 word saves a fifth of the time
//                     (2.85 ms) and leaves 1.74e-3, further off than the gathering kernels over ranges (1.68e-3).
// Per 64 keys and wave: 1536 clocks of matrix work beside about 1450 of vector work, a third of those the exponentials: two waves
// per SIMD overlap them little (the sum, at the 2 GHz that such work runs at, is the time measured).
#include <algorithm>

#include "stage2_core.h"

namespace dsv {

constexpr int kDenseKeys = 64;      // keys per LDS tile
constexpr int kDenseQueries = 128;  // queries per block, 32 per wave

__device__ __forceinline__ float mask_or_neg_inf(float s, uint32_t word, int bit)
{
    const uint32_t keep = (uint32_t)__builtin_amdgcn_sbfe((int)word, (unsigned)bit, 1u);  // all ones or zero
    return __uint_as_float((__float_as_uint(s) & keep) | (0xFF800000u & ~keep));
}

// A masked pair has weight zero, and zero times a row of V that is not finite is no number: a query whose sum came out not
// finite is formed once more, by its wave, from its selected keys alone.
template <int D>
__device__ __forceinline__ void dense_fwd_exact(const bf16_t *__restrict__ qrow, const bf16_t *__restrict__ Kh, const bf16_t *__restrict__ Vh,
                                             const uint32_t *__restrict__ mrow, bf16_t *__restrict__ orow, int L, float c2, float mc, float l)
{
    constexpr int CH = D / 64;
    const int lane = threadIdx.x & 63;
    float acc[CH], q[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        acc[c] = 0.f;
        q[c] = bf16_to_f32(qrow[lane * CH + c]);
    }
    for (int wd = 0; wd * 32 < L; ++wd)
        for (uint32_t word = mrow[wd]; word; word &= word - 1) {
            const int64_t at = (int64_t)(wd * 32 + __ffs(word) - 1) * D + lane * CH;
            float s = 0.f;
#pragma unroll
            for (int c = 0; c < CH; ++c) s = fmaf(q[c], bf16_to_f32(Kh[at + c]), s);
            const float p = fast_exp2(fmaf(group_sum<1>(s), c2, -mc));
#pragma unroll
            for (int c = 0; c < CH; ++c) acc[c] = fmaf(p, bf16_to_f32(Vh[at + c]), acc[c]);
        }
#pragma unroll
    for (int c = 0; c < CH; ++c) orow[lane * CH + c] = f32_to_bf16(acc[c] / l);
}

template <int D>
__global__ __launch_bounds__(256, 2) void dense_fwd_kernel(const bf16_t *__restrict__ Q, const bf16_t *__restrict__ K,
                                                           const bf16_t *__restrict__ V, const uint32_t *__restrict__ bits,
                                                           int pitch, bf16_t *__restrict__ O, float *__restrict__ lse, int L,
                                                           float scale, HeadTable tab, int slot0, int row0, int nrows)
{
    constexpr int NM = D / 16, NB = D / 32;
    constexpr int KP = D * 2 + 16, VP = D * 2 + 64;   // bytes from one parked row to the next: K read by rows, V transposed
    constexpr int PPR = D / 8;                        // 16-byte pieces per row
    constexpr int NP = kDenseKeys * PPR / 256;        // pieces per thread and matrix
    __shared__ __align__(16) unsigned char ks[2][kDenseKeys * KP];
    __shared__ __align__(16) unsigned char vs[2][kDenseKeys * VP];
    const int bh = tab.bh[slot0 + blockIdx.y];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = lane & 31, half = lane >> 5;
    const int r = blockIdx.x * kDenseQueries + wave * 32 + n;  // row of this lane's query in this piece
    const bool live = r < nrows;
    const int64_t hb = (int64_t)bh * L * D;
    const int64_t qi = row0 + (live ? r : nrows - 1);
    const uint32_t *mrow = bits + ((int64_t)blockIdx.y * nrows + (live ? r : nrows - 1)) * pitch;
    const unsigned char *Kh = reinterpret_cast<const unsigned char *>(K + hb), *Vh = reinterpret_cast<const unsigned char *>(V + hb);

    bf16x8_t qf[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) qf[m] = *reinterpret_cast<const bf16x8_t *>(Q + hb + qi * D + m * 16 + half * 8);
    floatx16_t o[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[nb][v] = 0.f;
    float mx = -INFINITY, mc = 0.f, l = 0.f;  // running maximum (score units), the same times c2 (0 while there is none), sum
    const float c2 = scale * kLog2e;          // > 0

    bf16x8_t kn[NP], vn[NP];
    auto request = [&](int j0) {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int e = threadIdx.x + 256 * i;
            const int64_t off = ((int64_t)min(j0 + e / PPR, L - 1) * PPR + e % PPR) * 16;  // rows past the end are masked
            kn[i] = *reinterpret_cast<const bf16x8_t *>(Kh + off);
            vn[i] = *reinterpret_cast<const bf16x8_t *>(Vh + off);
        }
    };
    // this lane's addresses: K row n of a 32-key half tile; V rows for the transposing reads
    const int ka = n * KP + half * 16;
    const int va = (4 * half + ((lane & 15) >> 2)) * VP + ((lane >> 4) & 1) * 32 + (lane & 3) * 8;
    request(0);
    uint2 wn = *reinterpret_cast<const uint2 *>(mrow);
    int buf = 0;
    for (int j0 = 0; j0 < L; j0 += kDenseKeys, buf ^= 1) {
        unsigned char *kt = ks[buf], *vt = vs[buf];
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int e = threadIdx.x + 256 * i;
            *reinterpret_cast<bf16x8_t *>(kt + (e / PPR) * KP + (e % PPR) * 16) = kn[i];
            *reinterpret_cast<bf16x8_t *>(vt + (e / PPR) * VP + (e % PPR) * 16) = vn[i];
        }
        __syncthreads();  // two tiles in turn: what is written next was last read before this barrier
        const uint32_t w[2] = {wn.x >> (4 * half), wn.y >> (4 * half)};
        const bool some = __any((wn.x | wn.y) != 0u);
        if (j0 + kDenseKeys < L) {
            request(j0 + kDenseKeys);
            wn = *reinterpret_cast<const uint2 *>(mrow + (j0 + kDenseKeys) / 32);
        }
        if (!some) continue;  // nothing selected by these 32 queries: wave-uniform, and the barrier lies behind
        floatx16_t s[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
#pragma unroll
            for (int v = 0; v < 16; ++v) s[t][v] = 0.f;
#pragma unroll
            for (int m = 0; m < NM; ++m)
                s[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8_t *>(kt + t * 32 * KP + ka + m * 32), qf[m], s[t], 0, 0, 0);
        }
        float top = -INFINITY;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                s[t][v] = mask_or_neg_inf(s[t][v], w[t], 8 * (v / 4) + v % 4);
                top = fmaxf(top, s[t][v]);
            }
        if (__any(top > mx)) {
            const float to = fmaxf(mx, fmaxf(top, __shfl_xor(top, 32)));
            const float f = to > mx ? fast_exp2((mx - to) * c2) : 1.f;  // from -inf: 0
            mx = to;
            mc = to > -INFINITY ? to * c2 : 0.f;
            l *= f;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int v = 0; v < 16; ++v) o[nb][v] *= f;
        }
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int h = 0; h < 2; ++h) {  // 16 keys: a lane holds 8 of them
                float p[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) p[e] = fast_exp2(fmaf(s[t][8 * h + e], c2, -mc));
                l += ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
                const SplitWeights w0 = split_weights(p[0], p[1]), w1 = split_weights(p[2], p[3]);
                const SplitWeights w2 = split_weights(p[4], p[5]), w3 = split_weights(p[6], p[7]);
                const bf16x8_t ph = __builtin_bit_cast(bf16x8_t, make_uint4(w0.head, w1.head, w2.head, w3.head));
                const bf16x8_t pt = __builtin_bit_cast(bf16x8_t, make_uint4(w0.tail, w1.tail, w2.tail, w3.tail));
                const unsigned char *v0 = vt + va + (32 * t + 16 * h) * VP;
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    const bf16x8_t vf = tr_frag(v0 + nb * 64, v0 + 8 * VP + nb * 64);
                    o[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pt, o[nb], 0, 0, 0);
                    o[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, ph, o[nb], 0, 0, 0);
                }
            }
    }
    l += __shfl_xor(l, 32);
    float zero = 0.f;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int v = 0; v < 16; ++v) zero = fmaf(o[nb][v], 0.f, zero);
    const bool finite = zero + __shfl_xor(zero, 32) == 0.f;
    for (unsigned long long todo = __ballot(live && !finite && half == 0); todo; todo &= todo - 1) {
        const int q = __ffsll(todo) - 1, rq = blockIdx.x * kDenseQueries + wave * 32 + q;
        const int64_t at = hb + (int64_t)(row0 + rq) * D;
        dense_fwd_exact<D>(Q + at, K + hb, V + hb, bits + ((int64_t)blockIdx.y * nrows + rq) * pitch, O + at, L, c2, __shfl(mc, q), __shfl(l, q));
    }
    if (half == 0 && live) lse[(int64_t)bh * L + qi] = (mc + log2f(l)) * kLn2;
    if (!live || !finite) return;
    const float inv = 1.f / l;
    bf16_t *orow = O + hb + qi * D + 4 * half;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *reinterpret_cast<uint2 *>(orow + 32 * nb + 8 * g) =
                make_uint2(pack_bf16x2(o[nb][4 * g] * inv, o[nb][4 * g + 1] * inv), pack_bf16x2(o[nb][4 * g + 2] * inv, o[nb][4 * g + 3] * inv));
}

// ------------------------------------------------------------------------------------ host
// Scratch of the mask: as many heads and rows at a time as fit `bytes`.
size_t dense_row_bytes(int L) { return (size_t)bits_pitch(L) * 4; }

template <int D>
static dsv_status dense_fwd_t(const dsv_problem &p, const HeadTable &tab, const void *Q, const void *K, const void *V,
                              const int32_t *idx, void *O, float *lse, char *ws, size_t ws_bytes, hipStream_t st)
{
    const int pitch = bits_pitch(p.L);
    uint32_t *bits = reinterpret_cast<uint32_t *>(ws);
    const size_t fit = ws_bytes / dense_row_bytes(p.L);  // rows of the mask
    const int heads = (int)std::min<size_t>(std::max<size_t>(fit / p.L, 1), (size_t)tab.n);
    const int rows = fit >= (size_t)p.L ? p.L : (int)(fit / kDenseQueries * kDenseQueries);
    if (rows < 1) return DSV_EWORKSPACE;
    for (int s0 = 0; s0 < tab.n; s0 += heads) {
        const int nh = std::min(heads, tab.n - s0);
        for (int r0 = 0; r0 < p.L; r0 += rows) {
            const int nr = std::min(rows, p.L - r0);
            const dsv_status rc = launch_bits_build(p, tab, s0, nh, idx, r0, nr, bits, st);
            if (rc != DSV_OK) return rc;
            hipLaunchKernelGGL((dense_fwd_kernel<D>), dim3((nr + kDenseQueries - 1) / kDenseQueries, nh), dim3(256), 0, st,
                               (const bf16_t *)Q, (const bf16_t *)K, (const bf16_t *)V, bits, pitch, (bf16_t *)O, lse, p.L, p.scale, tab,
                               s0, r0, nr);
            DSV_LAUNCH_CHECK();
        }
    }
    return DSV_OK;
}

dsv_status launch_dense_fwd(const dsv_problem &p, const HeadTable &tab, const void *Q, const void *K, const void *V,
                            const int32_t *idx, void *O, float *lse, char *ws, size_t ws_bytes, hipStream_t st)
{
    if (p.dtype == DSV_BF16 && p.d == 64) return dense_fwd_t<64>(p, tab, Q, K, V, idx, O, lse, ws, ws_bytes, st);
    if (p.dtype == DSV_BF16 && p.d == 128) return dense_fwd_t<128>(p, tab, Q, K, V, idx, O, lse, ws, ws_bytes, st);
    return DSV_EUNSUPPORTED;
}

}  // namespace dsv
