// Stage 2 backward over dense tiles with a selection mask, bf16: the partial sums of the ranged kernels (stage2_split.hip) for
// heads that keep enough of their keys.
//
// The gathering sweeps read 512 bytes per selected pair through the vector memory path, 0.7 to 0.8 of what that path carries.
// Here a wave owns 32 rows (queries in the dq step, keys in the dkdv step), walks the other axis of a range in tiles of 32
// rows that four waves share in LDS, and forms every pair:
//   S, dP      v_mfma_f32_32x32x16_bf16, A = the tile's rows out of LDS, B = the wave's rows; a lane holds one own row against
//              16 tile rows, in groups of four consecutive accumulators.
//   sums       v_smfmac_f32_32x32x32_bf16, which forms a contraction over twice the depth in the same time if of every four
//              elements of A at most two are not zero.  Selected pairs are few: every lane takes the first two selected of a
//              group, turns only those into weights (half the exponentials too), and where some lane has a third (a group in
//              a thousand at 6 % kept) the wave goes over the tile a second time with what is left; two rounds hold any mask.
//              Weights enter as bf16 head and tail, 16 significant bits, as in the gathering sweeps.
// The tile's row of accumulator m = 8 g + 4 half + i is pi(m) = 4 i + 2 (g % 2) + half + 16 (g / 2): the rows of a group lie
// four apart, and with the tile laid out as tile_addr says both kinds of reads -- 16 bytes of eight rows, transposing ones of
// four -- are free of bank conflicts.  Tiles come by direct loads into LDS, two in turn.
//
// Measured, L = 32768, four heads, k = 2048 (6 % kept), with the mask (0.43 ms): dq 5.09 ms by gathers -> 4.70, dkdv 5.68 -> 5.77 (which
// therefore gathers there); L = 20280, two of four heads at one key in 10 and in 5: whole backward 7.63 -> 4.78 ms, 0.4 of that the ascending copy that they no longer need.  Matrix cores are busy for
// 0.44 to 0.48 of the cycles and the vector units for 0.48 to 0.52: a wave's products and weights wait for each other, and two waves per SIMD --
// all that 256 registers allow -- overlap them little.  Weights laid beside the products inside a wave gave nothing (dq) or spilled
// (dkdv, 6.5 ms); fragment reads left to the compiler's order, which puts each right before its use, cost 0.5 ms of dq.
#include <algorithm>
#include <type_traits>

#include "dense_tile.h"

namespace dsv {

constexpr int kOwn = 128;          // own rows per block, 32 per wave

// Zero times a row that is not finite is no number, and the products above multiply rows that are not selected by zero: an own row whose
// sums came out not finite is formed once more, by its wave, from its selected pairs alone.  16 lanes per pair, eight pairs at a
// time.  One such row of K sends about half of its range's queries through here, and every key that such a query selects: L = 20280, four
// heads, k = 2028, the whole backward 5.1 ms on finite rows, 8.6 with one NaN row in a head's K (15.7 with one pair at a time), 11.0 with a head
// of them (23.1); by gathers 6.9 whatever the rows hold.
template <int D, bool KEYS>
__device__ __forceinline__ void exact_row(const bf16_t *__restrict__ xr, const bf16_t *__restrict__ yr, const bf16_t *__restrict__ R1,
                                          const bf16_t *__restrict__ R2, const uint32_t *__restrict__ mr, int tile0, int tile1, float c2, float l2,
                                          float dd, const float2 *__restrict__ stat, float *__restrict__ oa, float *__restrict__ ob,
                                          float *__restrict__ odelta)
{
    constexpr int CH = D / 16, U = 2;
    const int lane = threadIdx.x & 63, grp = lane >> 4, at = (lane & 15) * CH;
    const RowChunk<bf16_t, CH> x = load_chunk<bf16_t, CH>(xr + at), y = load_chunk<bf16_t, CH>(yr + at);
    float sa[CH], sb[CH], dsum = 0.f;
#pragma unroll
    for (int c = 0; c < CH; ++c) sa[c] = sb[c] = 0.f;
    auto words = [&](int t) -> uint64_t { return (t < tile1 ? mr[t] : 0u) | (uint64_t)(t + 1 < tile1 ? mr[t + 1] : 0u) << 32; };
    uint64_t next = words(tile0);
    for (int t = tile0; t < tile1; t += 2) {
        uint64_t w = next;
        next = words(t + 2);
        while (w) {  // wave-uniform
            int j[U];
            bool has[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {  // group g: the g-th of the next four
                uint64_t mine = w;
#pragma unroll
                for (int i = 0; i < 3; ++i) mine = i < grp ? mine & (mine - 1) : mine;
                has[u] = mine != 0;
                j[u] = t * kTile + (has[u] ? __ffsll((unsigned long long)mine) - 1 : 0);
#pragma unroll
                for (int i = 0; i < 4; ++i) w &= w - 1;
            }
            RowChunk<bf16_t, CH> r1[U], r2[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                r1[u] = load_chunk<bf16_t, CH>(R1 + (int64_t)j[u] * D + at);
                r2[u] = load_chunk<bf16_t, CH>(R2 + (int64_t)j[u] * D + at);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float s = row_sum<16>(dot_chunk<bf16_t, CH>(x, r1[u])), e = row_sum<16>(dot_chunk<bf16_t, CH>(y, r2[u]));
                float q, wgt;
                if constexpr (KEYS) {
                    const float2 rs = stat[j[u]];
                    q = fast_exp2(fmaf(s, c2, -rs.x));
                    wgt = q * (e - rs.y);
                } else {
                    q = fast_exp2(fmaf(s, c2, -l2));
                    wgt = q * (e - dd);
                }
                if (has[u]) {
                    if constexpr (!KEYS) dsum = fmaf(q, e, dsum);
#pragma unroll
                    for (int c = 0; c < CH; ++c) {
                        const uint32_t v1 = r1[u].w[c / 2], v2 = KEYS ? r2[u].w[c / 2] : v1;
                        sa[c] = fmaf(wgt, __uint_as_float(c & 1 ? v1 & 0xFFFF0000u : v1 << 16), sa[c]);
                        sb[c] = fmaf(q, __uint_as_float(c & 1 ? v2 & 0xFFFF0000u : v2 << 16), sb[c]);
                    }
                }
            }
        }
    }
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        sa[c] = group_sum<16>(sa[c]);
        sb[c] = group_sum<16>(sb[c]);
        if (grp == 0) {
            oa[at + c] = sa[c];
            ob[at + c] = sb[c];
        }
    }
    if constexpr (!KEYS) {
        dsum = group_sum<16>(dsum);
        if (lane == 0) *odelta = dsum;
    }
}

// KEYS: own rows are keys (X, Y = K, V; R1, R2 = Q, dO): a = dK = sum dS q, b = dV = sum p dO, with row statistics stat[query] =
// {lse * log2(e), Delta}.  Else own rows are queries (X, Y = Q, dO; R1, R2 = K, V): a = C = sum p (dP - D0) k, b = B = sum p k, and
// Delta (dq_sweep in stage2_core.h says what they are).
// The own rows' second operand stays in LDS: with both in registers a wave would need more than the 256 that let two run per SIMD.
template <int D, bool KEYS>
__global__ __launch_bounds__(256, 2) void dense_bwd_kernel(const bf16_t *__restrict__ X, const bf16_t *__restrict__ Y,
                                                           const bf16_t *__restrict__ R1, const bf16_t *__restrict__ R2,
                                                           const uint32_t *__restrict__ bits, int pitch, const bf16_t *__restrict__ O,
                                                           const float *__restrict__ lse, const float2 *__restrict__ stat,
                                                           float *__restrict__ pa, float *__restrict__ pb, float *__restrict__ pdelta,
                                                           int L, float scale, HeadTable tab, SplitPlan pl, int slot0, int row0, int nrows)
{
    typedef TileLayout<D> TL;
    constexpr int NM = D / 16, NB = D / 32;
    constexpr int XR = D == 128 ? NM - 3 : NM;  // fragments of X in registers; the others stay in LDS
    // two tiles in turn, each array a variable of its own: reads of one tile then need not wait for the loads into the other
    __shared__ __align__(16) unsigned char t1a[TL::BYTES], t1b[TL::BYTES], t2a[TL::BYTES], t2b[TL::BYTES];
    __shared__ __align__(16) unsigned char own[4 * (2 * NM - XR) * 1024];
    __shared__ __align__(16) float sta[2 * kTile], stb[2 * kTile];  // KEYS: -lse / scale, then -Delta, of the tile's queries by half, group, i
    int slot, range, rb;
    if (!decode_range_item(pl.S, pl.S_pad, pl.nqb, blockIdx.x, slot, range, rb)) return;
    const int bh = tab.bh[slot0 + slot];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 31, half = lane >> 5;
    const int r = rb * kOwn + wave * 32 + n;  // own row in this piece
    const bool live = r < nrows;
    const int rc = live ? r : nrows - 1;
    const int64_t hb = (int64_t)bh * L * D, own_row = (int64_t)bh * L + row0 + rc;
    const int tiles = (L + kTile - 1) / kTile, per = (tiles + pl.S - 1) / pl.S;
    const int tile0 = range * per, tile1 = min(tiles, tile0 + per);
    const uint32_t mrow = ((uint32_t)slot * nrows + rc) * pitch;  // a launch's masks hold less than 2^32 words (checked on the host)
    const unsigned char *m1 = reinterpret_cast<const unsigned char *>(R1 + hb), *m2 = reinterpret_cast<const unsigned char *>(R2 + hb);

    const int own_at = wave * ((2 * NM - XR) * 1024) + lane * 16;
    bf16x8_t xf[XR];
#pragma unroll
    for (int m = 0; m < NM; ++m) {
        const bf16x8_t x = *reinterpret_cast<const bf16x8_t *>(X + own_row * D + m * 16 + half * 8);
        if (m < XR) xf[m] = x;
        else *reinterpret_cast<bf16x8_t *>(own + own_at + (NM + m - XR) * 1024) = x;
        *reinterpret_cast<bf16x8_t *>(own + own_at + m * 1024) = *reinterpret_cast<const bf16x8_t *>(Y + own_row * D + m * 16 + half * 8);
    }
    const float c2 = scale * kLog2e;
    float lse2 = 0.f, d0 = 0.f;
    if constexpr (!KEYS) {
        lse2 = lse[own_row] * kLog2e;
        for (int m = 0; m < NM; ++m) {
            const RowChunk<bf16_t, 8> g = load_chunk<bf16_t, 8>(Y + own_row * D + m * 16 + half * 8), o = load_chunk<bf16_t, 8>(O + own_row * D + m * 16 + half * 8);
            d0 += dot_chunk<bf16_t, 8>(g, o);
        }
        d0 += __shfl_xor(d0, 32);
    }
    floatx16_t a[NB], b[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int v = 0; v < 16; ++v) a[nb][v] = b[nb][v] = 0.f;
    float delta = 0.f;  // sum p dP of this lane's pairs

    // this lane's addresses: row pi(n) of a tile by pieces (even and odd 16-channel steps); rows for the transposing reads
    const int ar = 4 * (n & 3) + ((n >> 2) & 3) + 16 * (n >> 4);
    const int ae = TL::base(ar) + ((half ^ (ar & 3)) << 4), ao = TL::base(ar) + (((2 + half) ^ (ar & 3)) << 4);
    int tr[4];
#pragma unroll
    for (int c = 0; c < 4; ++c)
        tr[c] = TL::base(16 * half + 4 * ((lane & 15) >> 2) + c) + (((2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) ^ c) << 4) + (lane & 1) * 8;

    const int sr = threadIdx.x & 31;  // KEYS: query of the tile whose statistics this thread (of the first 32) brings, and its place
    const int sp = (sr & 1) * 16 + (((sr >> 1) & 1) + 2 * (sr >> 4)) * 4 + ((sr >> 2) & 3);
    float2 sn = make_float2(0.f, 0.f);
    const TileLoads<D, 4, 1> loads(L, wave, lane);
    auto request = [&](int t, unsigned char *p1, unsigned char *p2) {
        loads.request(m1, t, p1);
        loads.request(m2, t, p2);
        if (KEYS && threadIdx.x < kTile) sn = stat[(int64_t)bh * L + min(t * kTile + sr, L - 1)];
    };
    auto park = [&](float *st) {
        if (KEYS && threadIdx.x < kTile) {
            st[sp] = -sn.x / c2;
            st[kTile + sp] = -sn.y;
        }
    };
    uint32_t next = 0;
    if (tile0 < tile1) {
        request(tile0, t1a, t2a);
        next = bits[mrow + tile0];
        park(sta);
    }
    auto step = [&](int t, const unsigned char *p1, const unsigned char *p2, const float *st, unsigned char *n1, unsigned char *n2,
                    float *stn) __attribute__((always_inline)) {
        const uint32_t word = live ? next : 0u;
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): a barrier alone does not wait for loads into LDS
        __syncthreads();                     // this tile is there, and the other buffer is no longer read
        if (t + 1 < tile1) {
            request(t + 1, n1, n2);
            next = bits[mrow + t + 1];
        }
        if (__any(word != 0u)) {  // wave-uniform
            floatx16_t s, dp;
            if constexpr (KEYS) {
                // (the additions of the products round at the size of lse / scale and Delta; against 64 bits the gradients are as far off as by
                // gathers, scales of 1e-6 to 1)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const float4 l4 = *reinterpret_cast<const float4 *>(st + half * 16 + g * 4);
                    const float4 d4 = *reinterpret_cast<const float4 *>(st + kTile + half * 16 + g * 4);
                    s[4 * g] = l4.x; s[4 * g + 1] = l4.y; s[4 * g + 2] = l4.z; s[4 * g + 3] = l4.w;
                    dp[4 * g] = d4.x; dp[4 * g + 1] = d4.y; dp[4 * g + 2] = d4.z; dp[4 * g + 3] = d4.w;
                }
            } else {
#pragma unroll
                for (int v = 0; v < 16; ++v) s[v] = dp[v] = 0.f;
            }
            // Fragments are read two steps before the products that need them; the order is pinned, for left alone the reads sink
            // to their uses.
            bf16x8_t f1[2], f2[2], fy[2], fx[2];
            auto fetch = [&](int m) __attribute__((always_inline)) {
                const int at = (m & 1 ? ao : ae) + (m >> 1) * 64;
                f1[m & 1] = *reinterpret_cast<const bf16x8_t *>(p1 + at);
                f2[m & 1] = *reinterpret_cast<const bf16x8_t *>(p2 + at);
                fy[m & 1] = *reinterpret_cast<const bf16x8_t *>(own + own_at + m * 1024);
                fx[m & 1] = m < XR ? xf[m < XR ? m : 0] : *reinterpret_cast<const bf16x8_t *>(own + own_at + (NM + m - XR) * 1024);
            };
            fetch(0);
            fetch(1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f1[m & 1], fx[m & 1], s, 0, 0, 0);
                dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f2[m & 1], fy[m & 1], dp, 0, 0, 0);
                if (m + 2 < NM) fetch(m + 2);
                __builtin_amdgcn_sched_barrier(0);
            }
            // the weights of two pairs of a group from their scores and dP, zero where v0, v1 are
            uint32_t wh[4], wt[4], ph[4], pt[4];
            auto weigh = [&](int g, float s0, float s1, float e0, float e1, uint32_t v0, uint32_t v1) __attribute__((always_inline)) {
                const float q0 = keep(v0, fast_exp2(KEYS ? s0 * c2 : fmaf(s0, c2, -lse2)));
                const float q1 = keep(v1, fast_exp2(KEYS ? s1 * c2 : fmaf(s1, c2, -lse2)));
                const float w0 = keep(v0, q0 * (KEYS ? e0 : e0 - d0)), w1 = keep(v1, q1 * (KEYS ? e1 : e1 - d0));
                const SplitWeights w = split_weights(w0, w1);
                wh[g] = w.head;
                wt[g] = w.tail;
                if constexpr (KEYS) {
                    const SplitWeights q = split_weights(q0, q1);
                    ph[g] = q.head;
                    pt[g] = q.tail;
                } else {
                    ph[g] = pack_bf16x2(q0, q1);
                    delta = fmaf(q0 + q1, d0, delta + (w0 + w1));
                }
            };
            auto sums = [&](uint32_t index) __attribute__((always_inline)) {
                const bf16x8_t fwh = __builtin_bit_cast(bf16x8_t, make_uint4(wh[0], wh[1], wh[2], wh[3]));
                const bf16x8_t fwt = __builtin_bit_cast(bf16x8_t, make_uint4(wt[0], wt[1], wt[2], wt[3]));
                const bf16x8_t fph = __builtin_bit_cast(bf16x8_t, make_uint4(ph[0], ph[1], ph[2], ph[3]));
                bf16x16_t f[2];
                auto fetch_rows = [&](int i) __attribute__((always_inline)) {  // KEYS: rows of Q and dO in turn
                    const unsigned char *p = (KEYS && (i & 1) ? p2 : p1) + (KEYS ? i >> 1 : i) * 64;
                    const bf16x8_t lo = tr_frag(p + tr[0], p + tr[2]), hi = tr_frag(p + tr[1], p + tr[3]);
                    f[i & 1] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15);
                };
                constexpr int NF = KEYS ? 2 * NB : NB;
                fetch_rows(0);
                fetch_rows(1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < NF; ++i) {
                    const int nb = KEYS ? i >> 1 : i;
                    if constexpr (KEYS) {
                        if (i & 1) {
                            const bf16x8_t fpt = __builtin_bit_cast(bf16x8_t, make_uint4(pt[0], pt[1], pt[2], pt[3]));
                            b[nb] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(fpt, f[1], b[nb], (int)index, 0, 0);
                            b[nb] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(fph, f[1], b[nb], (int)index, 0, 0);
                        } else {
                            a[nb] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(fwt, f[0], a[nb], (int)index, 0, 0);
                            a[nb] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(fwh, f[0], a[nb], (int)index, 0, 0);
                        }
                    } else {
                        a[nb] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(fwt, f[i & 1], a[nb], (int)index, 0, 0);
                        b[nb] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(fph, f[i & 1], b[nb], (int)index, 0, 0);
                        a[nb] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(fwh, f[i & 1], a[nb], (int)index, 0, 0);
                    }
                    if (i + 2 < NF) fetch_rows(i + 2);
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            const PairSlots ps(word >> half);
            auto first_two = [&](auto group) __attribute__((always_inline)) {
                constexpr int g = decltype(group)::value, bit = 2 * (g & 1) + 16 * (g >> 1);
                const uint32_t k0 = bit_mask<bit>(ps.b0), k1 = bit_mask<bit>(ps.b1), k2 = bit_mask<bit>(ps.n2), k3 = bit_mask<bit>(ps.n3);
                weigh(g, pick(k0, s[4 * g], pick(k1, s[4 * g + 1], s[4 * g + 2])), pick(k3, pick(k2, s[4 * g + 1], s[4 * g + 2]), s[4 * g + 3]),
                      pick(k0, dp[4 * g], pick(k1, dp[4 * g + 1], dp[4 * g + 2])), pick(k3, pick(k2, dp[4 * g + 1], dp[4 * g + 2]), dp[4 * g + 3]),
                      bit_mask<bit>(ps.v0), bit_mask<bit>(ps.v1));
            };
            first_two(std::integral_constant<int, 0>{});
            first_two(std::integral_constant<int, 1>{});
            first_two(std::integral_constant<int, 2>{});
            first_two(std::integral_constant<int, 3>{});
            sums(ps.index);
            if (__any((ps.r1 | ps.r2) != 0u)) {  // a third or fourth pair of some group: number 1, 2 or both
                auto others = [&](auto group) __attribute__((always_inline)) {
                    constexpr int g = decltype(group)::value, bit = 2 * (g & 1) + 16 * (g >> 1);
                    wh[g] = wt[g] = ph[g] = pt[g] = 0u;
                    if (!__any(((ps.r1 | ps.r2) & (1u << bit)) != 0u)) return;
                    const uint32_t k1 = bit_mask<bit>(ps.r1), k2 = bit_mask<bit>(ps.r2);
                    weigh(g, pick(k1, s[4 * g + 1], s[4 * g + 2]), s[4 * g + 2], pick(k1, dp[4 * g + 1], dp[4 * g + 2]), dp[4 * g + 2], k1 | k2, k1 & k2);
                };
                others(std::integral_constant<int, 0>{});
                others(std::integral_constant<int, 1>{});
                others(std::integral_constant<int, 2>{});
                others(std::integral_constant<int, 3>{});
                sums(ps.index_left());
            }
        }
        if (t + 1 < tile1) park(stn);
    };
    for (int t = tile0; t < tile1; t += 2) {
        step(t, t1a, t2a, sta, t1b, t2b, stb);
        if (t + 1 < tile1) step(t + 1, t1b, t2b, stb, t1a, t2a, sta);
    }

    // Accumulator v of a lane: own row 8 (v / 4) + 4 half + v % 4, channel 32 nb + n.
    const int64_t first = (int64_t)bh * L + row0 + rb * kOwn + wave * 32;
    uint32_t bad = 0;  // own rows with a sum that is not finite: they are stored below, once
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int o = 8 * (v / 4) + v % 4;
        float zero = 0.f;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) zero = fmaf(a[nb][v], 0.f, fmaf(b[nb][v], 0.f, zero));
        const unsigned long long off = __ballot(zero != 0.f);
        const uint32_t here = ((uint32_t)off ? 1u << o : 0u) | ((uint32_t)(off >> 32) ? 16u << o : 0u);
        bad |= here;
        if (rb * kOwn + wave * 32 + o + 4 * half < nrows && !(here >> (o + 4 * half) & 1u)) {
            const int64_t at = ((first + o + 4 * half) * pl.S + range) * D + n;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                pa[at + 32 * nb] = a[nb][v];
                pb[at + 32 * nb] = b[nb][v];
            }
        }
    }
    if constexpr (!KEYS) {
        const float all = delta + __shfl_xor(delta, 32);
        if (live && half == 0 && !(bad >> n & 1u)) pdelta[own_row * pl.S + range] = all;
    }
    for (; bad; bad &= bad - 1) {
        const int o = __ffs(bad) - 1;
        if (rb * kOwn + wave * 32 + o >= nrows) continue;
        const int64_t row = first + o;
        const uint32_t *mr = bits + ((int64_t)slot * nrows + rb * kOwn + wave * 32 + o) * pitch;
        exact_row<D, KEYS>(X + row * D, Y + row * D, R1 + hb, R2 + hb, mr, tile0, tile1, c2, __shfl(lse2, o), __shfl(d0, o),
                           KEYS ? stat + (int64_t)bh * L : nullptr, pa + (row * pl.S + range) * D, pb + (row * pl.S + range) * D,
                           KEYS ? nullptr : pdelta + row * pl.S + range);
    }
}

// ------------------------------------------------------------------------------------ host
// One step over the heads of a table, as many heads and rows at a time as masks fit the scratch.  keys: the dkdv step, on
// key-major lists.
template <int D>
static dsv_status dense_bwd_t(const dsv_problem &p, const HeadTable &tab, bool keys, const void *Q, const void *K, const void *V, const int32_t *index,
                              const int64_t *col, const void *O, const float *lse, const void *dO, const SplitPlan &plan,
                              const BwdSplitWorkspace &w, const DenseHeads &dense, hipStream_t st)
{
    const int pitch = bits_pitch(p.L);
    const size_t fit = dense.bits ? (size_t)tab.n * p.L : dense.mask_bytes / ((size_t)pitch * 4);  // rows of the mask
    const int heads = (int)std::min<size_t>(std::max<size_t>(fit / p.L, 1), (size_t)tab.n);
    // pieces of a head: whole rounds of blocks (two per CU) where that much fits
    const size_t unit = (size_t)kOwn * std::max(1, 512 / plan.S_pad);
    const int rows = fit >= (size_t)p.L ? p.L : (int)(fit >= unit ? fit / unit * unit : fit / kOwn * kOwn);
    if (rows < 1) return DSV_EWORKSPACE;
    SplitPlan pl = plan;
    for (int s0 = 0; s0 < tab.n; s0 += heads) {
        const int nh = std::min(heads, tab.n - s0);
        for (int r0 = 0; r0 < p.L; r0 += rows) {
            const int nr = std::min(rows, p.L - r0);
            const uint32_t *bits = dense.bits;
            if (!bits) {
                uint32_t *mask = reinterpret_cast<uint32_t *>(dense.mask);
                const dsv_status rc = launch_bits_build(p, tab, s0, nh, index, r0, nr, mask, st, col);
                if (rc != DSV_OK) return rc;
                bits = mask;
            }
            pl.nqb = (nr + kOwn - 1) / kOwn;
            const int64_t blocks = nh * range_items(pl.S_pad, pl.nqb);
            if (blocks > 0x7FFFFFFF || ((uint64_t)nh * nr * pitch) >> 32) return DSV_EUNSUPPORTED;  // never: masks take 2 GB at most
            if (keys)
                hipLaunchKernelGGL((dense_bwd_kernel<D, true>), dim3((unsigned)blocks), dim3(256), 0, st, (const bf16_t *)K, (const bf16_t *)V,
                                   (const bf16_t *)Q, (const bf16_t *)dO, bits, pitch, (const bf16_t *)nullptr, (const float *)nullptr,
                                   (const float2 *)w.rowstat, w.pa, w.pb, (float *)nullptr, p.L, p.scale, tab, pl, s0, r0, nr);
            else
                hipLaunchKernelGGL((dense_bwd_kernel<D, false>), dim3((unsigned)blocks), dim3(256), 0, st, (const bf16_t *)Q, (const bf16_t *)dO,
                                   (const bf16_t *)K, (const bf16_t *)V, bits, pitch, (const bf16_t *)O, lse, (const float2 *)nullptr, w.pa, w.pb,
                                   w.pdelta, p.L, p.scale, tab, pl, s0, r0, nr);
            DSV_LAUNCH_CHECK();
        }
    }
    return DSV_OK;
}

dsv_status launch_dense_bwd(const dsv_problem &p, const HeadTable &tab, bool keys, const void *Q, const void *K, const void *V, const int32_t *index,
                            const int64_t *col, const void *O, const float *lse, const void *dO, const SplitPlan &plan,
                            const BwdSplitWorkspace &w, const DenseHeads &dense, hipStream_t st)
{
    if (p.dtype == DSV_BF16 && p.d == 64) return dense_bwd_t<64>(p, tab, keys, Q, K, V, index, col, O, lse, dO, plan, w, dense, st);
    if (p.dtype == DSV_BF16 && p.d == 128) return dense_bwd_t<128>(p, tab, keys, Q, K, V, index, col, O, lse, dO, plan, w, dense, st);
    return DSV_EUNSUPPORTED;
}

}  // namespace dsv
