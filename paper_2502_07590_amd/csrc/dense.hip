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
// Per 64 keys and wave: 1536 clocks of matrix work beside about 1450 of vector work, a third of those the exponentials.
#include <algorithm>
#include <type_traits>

#include "dense_tile.h"

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

// The larger of two numbers, as the middle one of three.  (fmaxf first makes quiet what might be a signalling NaN, an instruction per operand, and
// the compiler makes fmaxf of a middle one with an infinity that it can see.  A NaN loses here too.)
__device__ __forceinline__ float larger(float a, float b, float infinity) { return __builtin_amdgcn_fmed3f(a, b, infinity); }

// The same on sparse products, for heads that keep few pairs of a tile, as in the backward (dense_bwd.hip): every lane takes the first two
// selected of a group of four keys, only those become weights, and v_smfmac_f32_32x32x32_bf16 adds up twice the keys in the time of a
// dense product; where some group has a third the wave goes over the tile again.  A sum's rows are queries then, its lanes
// channels: what is known per query goes there through LDS, which the maximum does rarely, as it may lag by 2^8.
// What bounds it is power: at 1.7 to 1.8 of 2.4 GHz more waves or fewer waits change nothing, fewer operations do.  Per 32 keys and wave 512 clocks
// of matrix work (768 on dense products) and about 520 of vector work, those of second rounds aside.  L = 32768, four heads, k = 2048, with the
// mask: 3.28 -> 2.90 ms.  Setting the pairs of second rounds aside for products of their own, sixteen at a time, cost what it gave.
template <int D, int NW>
__global__ __launch_bounds__(64 * NW, 2) void dense_fwd_pairs_kernel(const bf16_t *__restrict__ Q, const bf16_t *__restrict__ K,
                                                                     const bf16_t *__restrict__ V, const uint32_t *__restrict__ bits,
                                                                     int pitch, bf16_t *__restrict__ O, float *__restrict__ lse, int L,
                                                                     float scale, HeadTable tab, int slot0, int row0, int nrows)
{
    typedef TileLayout<D> TL;
    constexpr int NM = D / 16, NB = D / 32, CT = 2;
    // two pairs of tiles in turn, each array a variable of its own: reads of one then need not wait for the loads into the other
    __shared__ __align__(16) unsigned char t1a[CT * TL::BYTES], t1b[CT * TL::BYTES], t2a[CT * TL::BYTES], t2b[CT * TL::BYTES];
    __shared__ __align__(16) float by_row[NW * 32];           // a factor per query, from its lanes to the rows of the sums
    const int bh = tab.bh[slot0 + blockIdx.y];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 31, half = lane >> 5;
    const int first = blockIdx.x * (32 * NW) + wave * 32;  // the wave's first row in this piece
    const bool live = first + n < nrows;
    const int rc = live ? first + n : nrows - 1;
    const int64_t hb = (int64_t)bh * L * D;
    const int64_t qi = row0 + rc;
    // the wave's rows of the mask from its first one on; all masks of a launch together may pass 2^32 words
    const uint32_t *mask = bits + ((int64_t)blockIdx.y * nrows + min(first, nrows - 1)) * pitch;
    const uint32_t mrow = (uint32_t)((rc - min(first, nrows - 1)) * pitch);
    const unsigned char *m1 = reinterpret_cast<const unsigned char *>(K + hb), *m2 = reinterpret_cast<const unsigned char *>(V + hb);
    const int tile1 = (L + kTile - 1) / kTile;

    bf16x8_t qf[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) qf[m] = *reinterpret_cast<const bf16x8_t *>(Q + hb + qi * D + m * 16 + half * 8);
    floatx16_t o[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[nb][v] = 0.f;
    float mx = -INFINITY, mc = 0.f, l = 0.f;  // maximum that weights are taken against (score units), the same times c2, sum
    const float c2 = scale * kLog2e;          // > 0
    float infinity = INFINITY;
    asm("" : "+v"(infinity));
    const float lag = 8.f / c2;               // weights reach 2^8 before the maximum follows: head and tail do not depend on it

    const int ar = 4 * (n & 3) + ((n >> 2) & 3) + 16 * (n >> 4);
    const int ae = TL::base(ar) + ((half ^ (ar & 3)) << 4), ao = TL::base(ar) + (((2 + half) ^ (ar & 3)) << 4);
    int tr[4];
#pragma unroll
    for (int c = 0; c < 4; ++c)
        tr[c] = TL::base(16 * half + 4 * ((lane & 15) >> 2) + c) + (((2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) ^ c) << 4) + (lane & 1) * 8;
    float *mine = by_row + 32 * wave;
    auto spread = [&](float f, float (&g)[16]) __attribute__((always_inline)) {  // g[v]: the value of query 8 (v / 4) + 4 half + v % 4
        if (half == 0) mine[n] = f;
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float4 f4 = *reinterpret_cast<const float4 *>(mine + 8 * i + 4 * half);
            g[4 * i] = f4.x; g[4 * i + 1] = f4.y; g[4 * i + 2] = f4.z; g[4 * i + 3] = f4.w;
        }
        __builtin_amdgcn_wave_barrier();
    };

    const TileLoads<D, NW, CT> loads(L, wave, lane);
    uint2 words;  // the masks of the next tiles
    auto request = [&](int t, unsigned char *p1, unsigned char *p2) __attribute__((always_inline)) {
        loads.request(m1, t, p1);
        loads.request(m2, t, p2);
        words = *reinterpret_cast<const uint2 *>(mask + mrow + t);
    };
    request(0, t1a, t2a);
    auto tile = [&](uint32_t word, const unsigned char *p1, const unsigned char *p2) __attribute__((always_inline)) {
        if (!__any(word != 0u)) return;  // wave-uniform
        // Fragments are read four products before the one that needs them; the order of reads and products is pinned, for left alone the
        // reads sink to their uses.
        constexpr int AHEAD = 4;
        bf16x8_t f1[AHEAD];
        auto fetch = [&](int m) __attribute__((always_inline)) { f1[m % AHEAD] = *reinterpret_cast<const bf16x8_t *>(p1 + (m & 1 ? ao : ae) + (m >> 1) * 64); };
#pragma unroll
        for (int m = 0; m < AHEAD; ++m) fetch(m);
        __builtin_amdgcn_sched_barrier(0x406);
        floatx16_t s;
#pragma unroll
        for (int v = 0; v < 16; ++v) s[v] = 0.f;
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f1[m % AHEAD], qf[m], s, 0, 0, 0);
            if (m + AHEAD < NM) fetch(m + AHEAD);
            __builtin_amdgcn_sched_barrier(0x406);
        }
        const PairSlots ps(word >> half);
        const float none = -INFINITY;
        float x[8], top = none;
        auto first_two = [&](auto group) __attribute__((always_inline)) {
            constexpr int g = decltype(group)::value, bit = 2 * (g & 1) + 16 * (g >> 1);
            const uint32_t k0 = bit_mask<bit>(ps.b0), k1 = bit_mask<bit>(ps.b1), k2 = bit_mask<bit>(ps.n2), k3 = bit_mask<bit>(ps.n3);
            x[2 * g] = pick(bit_mask<bit>(ps.v0), pick(k0, s[4 * g], pick(k1, s[4 * g + 1], s[4 * g + 2])), none);
            x[2 * g + 1] = pick(bit_mask<bit>(ps.v1), pick(k3, pick(k2, s[4 * g + 1], s[4 * g + 2]), s[4 * g + 3]), none);
            top = larger(top, larger(x[2 * g], x[2 * g + 1], infinity), infinity);
        };
        first_two(std::integral_constant<int, 0>{});
        first_two(std::integral_constant<int, 1>{});
        first_two(std::integral_constant<int, 2>{});
        first_two(std::integral_constant<int, 3>{});
        const bool again = __any((ps.r1 | ps.r2) != 0u);  // a third or fourth pair of some group: a second round
        float y[8];
        if (again) {
            auto others = [&](auto group) __attribute__((always_inline)) {
                constexpr int g = decltype(group)::value, bit = 2 * (g & 1) + 16 * (g >> 1);
                const uint32_t k1 = bit_mask<bit>(ps.r1), k2 = bit_mask<bit>(ps.r2);
                y[2 * g] = pick(k1 | k2, pick(k1, s[4 * g + 1], s[4 * g + 2]), none);
                y[2 * g + 1] = pick(k1 & k2, s[4 * g + 2], none);
                top = larger(top, larger(y[2 * g], y[2 * g + 1], infinity), infinity);
            };
            others(std::integral_constant<int, 0>{});
            others(std::integral_constant<int, 1>{});
            others(std::integral_constant<int, 2>{});
            others(std::integral_constant<int, 3>{});
        }
        if (__any(top > mx + lag)) {
            const float to = fmaxf(mx, fmaxf(top, __shfl_xor(top, 32)));
            const float f = to > mx ? fast_exp2((mx - to) * c2) : 1.f;  // from -inf: 0
            mx = to;
            mc = to > -INFINITY ? to * c2 : 0.f;
            l *= f;
            float g[16];
            spread(f, g);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int v = 0; v < 16; ++v) o[nb][v] *= g[v];
        }
        bf16x16_t f2[2];
        auto fetch_rows = [&](int nb) __attribute__((always_inline)) {
            const unsigned char *p = p2 + nb * 64;
            const bf16x8_t lo = tr_frag(p + tr[0], p + tr[2]), hi = tr_frag(p + tr[1], p + tr[3]);
            f2[nb & 1] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15);
        };
        auto add = [&](const float (&z)[8], uint32_t index) __attribute__((always_inline)) {
            fetch_rows(0);
            fetch_rows(1);
            __builtin_amdgcn_sched_barrier(0);
            uint32_t ph[4], pt[4];
            float sum = 0.f;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float q0 = fast_exp2(fmaf(z[2 * g], c2, -mc)), q1 = fast_exp2(fmaf(z[2 * g + 1], c2, -mc));
                sum += q0 + q1;
                const SplitWeights w = split_weights(q0, q1);
                ph[g] = w.head;
                pt[g] = w.tail;
            }
            l += sum;
            const bf16x8_t fh = __builtin_bit_cast(bf16x8_t, make_uint4(ph[0], ph[1], ph[2], ph[3]));
            const bf16x8_t ft = __builtin_bit_cast(bf16x8_t, make_uint4(pt[0], pt[1], pt[2], pt[3]));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                o[nb] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(ft, f2[nb & 1], o[nb], (int)index, 0, 0);
                o[nb] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(fh, f2[nb & 1], o[nb], (int)index, 0, 0);
                if (nb + 2 < NB) fetch_rows(nb + 2);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        add(x, ps.index);
        if (again) add(y, ps.index_left());
    };
    auto pair = [&](int t, const unsigned char *p1, const unsigned char *p2, unsigned char *n1, unsigned char *n2) __attribute__((always_inline)) {
        const uint32_t word = live ? words.x : 0u, then = live ? words.y : 0u;
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): a barrier alone does not wait for loads into LDS
        __syncthreads();                     // these tiles are there, and the other buffer is no longer read
        if (t + CT < tile1) request(t + CT, n1, n2);
        tile(word, p1, p2);
        tile(then, p1 + TL::BYTES, p2 + TL::BYTES);
    };
    for (int t = 0; t < tile1; t += 2 * CT) {
        pair(t, t1a, t2a, t1b, t2b);
        if (t + CT < tile1) pair(t + CT, t1b, t2b, t1a, t2a);
    }
    l += __shfl_xor(l, 32);
    if (half == 0 && live) lse[(int64_t)bh * L + qi] = (mc + log2f(l)) * kLn2;
    float inv[16];
    spread(1.f / l, inv);
    uint32_t bad = 0;  // queries with a sum that is not finite: formed once more, below
    bf16_t *Oh = O + hb + (int64_t)(row0 + first) * D;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int at = 8 * (v / 4) + v % 4;
        float zero = 0.f;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) zero = fmaf(o[nb][v], 0.f, zero);
        const unsigned long long off = __ballot(zero != 0.f);
        const uint32_t here = ((uint32_t)off ? 1u << at : 0u) | ((uint32_t)(off >> 32) ? 16u << at : 0u);
        bad |= here;
        if (first + at + 4 * half < nrows && !(here >> (at + 4 * half) & 1u)) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) Oh[(at + 4 * half) * D + 32 * nb + n] = f32_to_bf16(o[nb][v] * inv[v]);
        }
    }
    for (; bad; bad &= bad - 1) {
        const int q = __ffs(bad) - 1;
        if (first + q >= nrows) continue;
        dense_fwd_exact<D>(Q + hb + (int64_t)(row0 + first + q) * D, K + hb, V + hb, bits + ((int64_t)blockIdx.y * nrows + first + q) * pitch,
                           Oh + q * D, L, c2, __shfl(mc, q), __shfl(l, q));
    }
}

// ------------------------------------------------------------------------------------ host
// Scratch of the mask: as many heads and rows at a time as fit `bytes`.
size_t dense_row_bytes(int L) { return (size_t)bits_pitch(L) * 4; }

// Queries per block of the form on sparse products, 0 for the one on dense products.  Second rounds over tiles cost more than sparse products
// save where more than one key in 14 is kept, and with one block per CU and fewer the 64 keys between two barriers of the dense form
// count more.  ms, dense : sparse with 128 : with 256 queries, four heads of 32768, one key in 22: 3.17 : 2.78 : 2.67, in 16: 3.28 : 3.01 :
// 2.90, in 12: 3.43 : 3.43 : 3.33, in 10: 3.51 : 3.72 : 3.64; d = 64, in 16: 2.16 : 2.04 : 1.98, in 12: 2.29 : 2.35 : 2.29; three heads of 9000, one in 13: 0.288 :
// 0.298 : 0.386.  Blocks of 256 (one per CU) where they leave their last round nearly full: four heads of 20280, one in 16, 1.25 rounds: 1.51 :
// 1.43 : 1.68; one head of 131072, two rounds: 13.8 : 12.8 : 12.0.  Where heads differ their mean decides: of 31 mixes none was slower than on dense products
// alone (eight heads of 32768, one key in 4 in one of them and in 26 in seven: 6.39 -> 5.85).
static int dense_fwd_form(int L, int heads, int rows, int64_t kept)
{
    if (kept * 14 > (int64_t)L * heads || (int64_t)heads * ((rows + 127) / 128) <= 256) return 0;
    const int64_t blocks = (int64_t)heads * ((rows + 255) / 256), rounds = (blocks + 255) / 256;
    return blocks * 100 >= rounds * 256 * 85 ? 256 : 128;
}

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
            auto run = [&](auto kernel, int queries) {
                hipLaunchKernelGGL(kernel, dim3((nr + queries - 1) / queries, nh), dim3(2 * queries), 0, st, (const bf16_t *)Q, (const bf16_t *)K,
                                   (const bf16_t *)V, bits, pitch, (bf16_t *)O, lse, p.L, p.scale, tab, s0, r0, nr);
            };
            int64_t kept = 0;
            for (int s = s0; s < s0 + nh; ++s) kept += tab.k[s];
            switch (dense_fwd_form(p.L, nh, nr, kept)) {
            case 256: run(dense_fwd_pairs_kernel<D, 8>, 256); break;
            case 128: run(dense_fwd_pairs_kernel<D, 4>, 128); break;
            default: run(dense_fwd_kernel<D>, kDenseQueries);
            }
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
