// Query grouping, backward: dK and dV of the grouped attention (paper Sec. "Sparse Attention with Query Grouping"), bf16,
// d = 128, groups of up to 32 queries.
//
// Key-major, and dense where the selection is: a wave owns 16 consecutive keys and walks the UNION of their lists of groups;
// every group of the union brings its G queries' Q and dO rows once, and all four products of 32 queries x 16 keys run on
// the matrix cores with a mask for the (group, key) pairs that are not selected.  Neighbouring keys of the token grid are
// selected by much the same groups: on spatially smooth inputs the union of 16 keys is 3.2 times a single list, so that
// a step of 512 (query, key) pairs holds 160 selected ones.  Keys chosen independently of their neighbours (10 times at 6 % kept)
// are better served by the per-query sweep on the lists of groups; union_prepare_kernel looks.
//
//   S^T = Q_u K^T, dP^T = dO_u V^T   v_mfma_f32_16x16x32_bf16, A = 16 gathered rows as they come from memory (lane = row
//        l % 16, channels 32 m + 8 (l / 16): one load instruction touches whole 64-byte sectors), B = the keys' K and V rows,
//        kept in registers.  Lane l then holds key l % 16 against queries 4 (l / 16) + 0..3 of either half of the step.
//   dK += dS^T Q_u, dV += P^T dO_u   A = the weights, which those lanes hold in the A layout already (which queries a lane
//        group contracts is free: slots 16 (e / 4) + 4 (l / 16) + e % 4), as bf16 head + tail -- 16 significant bits of every
//        fp32 weight, as in the per-query sweep --, B = the gathered rows transposed out of LDS (tr_frag).
//
// Work item = (head, query range, 4 x 16 keys): the rows of a range (at most 8192 queries, 4 MB) stay in an XCD's L2, and
// every XCD walks its ranges one after the other.  A range leaves partial sums for the per-query merge; a single range
// writes the result.  L = 32768, four heads, k = 2048, 2 x 2 x 2 cubes, smooth inputs: 3.5 ms, with the
// merge 3.6 (the per-query key-major sweep on the lists of groups: 5.75 + 0.45), a sixth of it matrix work: a step is a
// chain of loads, LDS, two products and the queue that eight waves per CU only partly hide.  One wave per block instead of
// four neighbouring ones measured 7 % slower (neighbours share rows in the L1).
#include <algorithm>

#include "stage2_core.h"

namespace dsv {

typedef uint32_t __attribute__((may_alias)) u32m;

constexpr int kUnionKeys = 16;        // keys per wave
constexpr int kUnionGroups = 1024;    // groups whose key masks a wave holds at a time
constexpr int kUnionRow = 128 * 2 + 16;  // bytes from one parked row to the next
constexpr int kUnionQueue = 128;      // queued (group, mask) entries, a power of two

struct UnionWave {
    unsigned char q[32 * kUnionRow], g[32 * kUnionRow];  // the step's 32 Q and dO rows
    uint32_t mask[kUnionGroups / 2];                     // 16-bit key masks of the groups in the window, two per word
    uint32_t queue[kUnionQueue];                         // group - first of the range << 16 | mask
    float2 stat[32];                                     // {lse log2 e, Delta} of the step's queries
    uint32_t smask[32];                                  // key mask of every slot
};
static_assert(4 * sizeof(UnionWave) <= 80 * 1024, "two blocks per CU");

struct UnionPlan {
    int S, S_pad;      // ranges, as the gathering sweep has them
    int groups;        // groups per range
    int nkb;           // blocks of 64 keys
};

// Place of slot s among the parked rows: the eight rows that one pass of a transposing read serves (two lane groups) lie
// two apart, i.e. in disjoint LDS banks.
__device__ __forceinline__ int union_row(int s) { return (s & 16) + 2 * (s & 7) + ((s >> 3) & 1); }

__device__ __forceinline__ void union_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A pair that is not selected has weight zero, and zero times a row of Q or dO that is not finite is no number: a key whose
// sums came out not finite is formed once more, by its wave, from its own list (n groups of G queries) alone.  A lane takes
// channels 2 lane and 2 lane + 1.
__device__ __forceinline__ void grouped_dkdv_exact(const bf16_t *__restrict__ Qr, const bf16_t *__restrict__ Gr, const float2 *__restrict__ stat,
                                                const bf16_t *__restrict__ krow, const bf16_t *__restrict__ vrow,
                                                const int32_t *__restrict__ list, int n, int gb, int ge, int G, float c2,
                                                float (&dk)[2], float (&dv)[2])
{
    const int lane = threadIdx.x & 63;
    auto pair = [&](const bf16_t *row, float (&x)[2]) {
        const uint32_t w = *reinterpret_cast<const uint32_t *>(row + 2 * lane);
        x[0] = __uint_as_float(w << 16);
        x[1] = __uint_as_float(w & 0xFFFF0000u);
    };
    float k[2], v[2];
    pair(krow, k);
    pair(vrow, v);
    dk[0] = dk[1] = dv[0] = dv[1] = 0.f;
    for (int t = 0; t < n; ++t) {
        const int g = list[t];
        if (g < gb || g >= ge) continue;
        for (int m = 0; m < G; ++m) {
            const int64_t row = (int64_t)(g - gb) * G + m;
            float q[2], o[2];
            pair(Qr + row * 128, q);
            pair(Gr + row * 128, o);
            const float s = group_sum<1>(fmaf(q[0], k[0], q[1] * k[1])), dp = group_sum<1>(fmaf(o[0], v[0], o[1] * v[1]));
            const float2 st = stat[row];
            const float p = fast_exp2(s * c2 - st.x), ds = p * (dp - st.y);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                dk[c] = fmaf(ds, q[c], dk[c]);
                dv[c] = fmaf(p, o[c], dv[c]);
            }
        }
    }
}

// Q, dO, rowstat: queries in group-major order (group g = queries g G .. g G + G - 1).
__global__ __launch_bounds__(256, 2) void grouped_dkdv_kernel(const bf16_t *__restrict__ Q, const bf16_t *__restrict__ K,
                                                              const bf16_t *__restrict__ V, const bf16_t *__restrict__ dO,
                                                              const int32_t *__restrict__ lists, const int64_t *__restrict__ col,
                                                              const float2 *__restrict__ rowstat, bf16_t *__restrict__ dK,
                                                              bf16_t *__restrict__ dV, float *__restrict__ pdk,
                                                              float *__restrict__ pdv, int L, int G, float scale, HeadTable tab,
                                                              UnionPlan pl, const int32_t *__restrict__ use)
{
    constexpr int D = 128;
    __shared__ __align__(16) UnionWave sh_all[4];
    int slot, range, kb;
    if (!decode_range_item(pl.S, pl.S_pad, pl.nkb, blockIdx.x, slot, range, kb)) return;
    const int bh = tab.bh[slot];
    if (use && !use[bh]) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c16 = lane & 15, g4 = lane >> 4;
    UnionWave &sh = sh_all[wave];
    const int j0 = (kb * 4 + wave) * kUnionKeys;
    if (j0 >= L) return;  // whole wave; nothing below synchronises across waves
    const int Lq = L / G;
    const int gb = min(range * pl.groups, Lq), ge = min(gb + pl.groups, Lq);  // this range's groups
    const int64_t hb = (int64_t)bh * L * D;
    const bf16_t *Qr = Q + hb + (int64_t)gb * G * D, *Gr = dO + hb + (int64_t)gb * G * D;  // rows of the range
    const float2 *stat = rowstat + (int64_t)bh * L + (int64_t)gb * G;

    // B operands: the keys' rows (past the end: the last key, never selected)
    bf16x8_t kf[4], vf[4];
    {
        const int64_t row = hb + (int64_t)min(j0 + c16, L - 1) * D + g4 * 8;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            kf[m] = *reinterpret_cast<const bf16x8_t *>(K + row + m * 32);
            vf[m] = *reinterpret_cast<const bf16x8_t *>(V + row + m * 32);
        }
    }
    // list pointers: four lanes per key, each takes every fourth entry from its first on
    const int32_t *list;
    int pos, end;
    {
        const int j = j0 + (lane >> 2);
        const int64_t *cp = col + (int64_t)bh * (L + 1) + min(j, L - 1);
        const int64_t first = cp[0];
        end = j < L ? (int)(cp[1] - first) : 0;
        list = lists + tab.off[slot] + first;
        int lo = 0, hi = end;  // first entry of this range
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (list[mid] < gb) lo = mid + 1; else hi = mid;
        }
        pos = lo + (lane & 3);
    }
    floatx4_t dk[8], dv[8];  // [channel block]: channel 16 nb + l % 16, keys 4 (l / 16) + v
#pragma unroll
    for (int nb = 0; nb < 8; ++nb) { dk[nb] = floatx4_t{0.f, 0.f, 0.f, 0.f}; dv[nb] = dk[nb]; }
    const float c2 = scale * kLog2e;
    const int NG = 32 / G;                                   // groups per step
    const int ga = c16 / G, gc = (16 + c16) / G;             // this lane's two load slots: group of the step ...
    const int ma = c16 - ga * G, mc = 16 + c16 - gc * G;     // ... and member (a group >= NG: an unused slot)
    const int gs = (lane & 31) / G, ms = (lane & 31) - gs * G;  // slot lane % 32, for row statistics and mask
    const int rowa = union_row(c16) * kUnionRow + g4 * 16, rowc = union_row(16 + c16) * kUnionRow + g4 * 16;
    const int tr0 = union_row(4 * g4 + (c16 >> 2)) * kUnionRow + (c16 & 3) * 8, tr1 = tr0 + 16 * kUnionRow;

    int head = 0, count = 0;          // queue: ring positions head .. head + count - 1
    int win = gb, scan = kUnionGroups;  // window of masks [win, win + kUnionGroups); groups of it already queued
    bool fresh = false;               // no window built yet
    // Fills the queue up to a step's groups, or as far as the range goes.
    auto refill = [&]() {
        while (count < NG) {
            if (scan >= kUnionGroups) {
                if (fresh) win += kUnionGroups;
                fresh = true;
                if (win >= ge) { win = ge; scan = kUnionGroups; fresh = false; return; }
                const int lim = min(win + kUnionGroups, ge);
#pragma unroll
                for (int e = 0; e < kUnionGroups / 2 / 64; ++e) sh.mask[lane + 64 * e] = 0u;
                union_sync();
                const uint32_t bit = 1u << (lane >> 2);
                bool more = true;
                while (more) {
                    int e[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) e[u] = pos + 4 * u < end ? list[pos + 4 * u] : 0x7FFFFFFF;
                    int took = 0;
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (e[u] < lim) {  // ascending: a prefix of the four
                            const int r = max(e[u] - win, 0);
                            atomicOr(&sh.mask[r >> 1], bit << (16 * (r & 1)));
                            ++took;
                        }
                    pos += 4 * took;
                    more = __any(took == 4);
                }
                union_sync();
                scan = 0;
            }
            const uint32_t w = sh.mask[(scan + lane) >> 1];
            const uint32_t m = (w >> (16 * (lane & 1))) & 0xFFFFu;
            const unsigned long long some = __ballot(m != 0u);
            if (m) {
                const int at = head + count + __popcll(some & ((1ull << lane) - 1ull));
                sh.queue[at & (kUnionQueue - 1)] = (uint32_t)(win - gb + scan + lane) << 16 | m;
            }
            count += __popcll(some);
            scan += 64;
        }
    };
    bf16x8_t qa[2][4], oa[2][4];  // A operands: rows of slots l % 16 and 16 + l % 16
    float2 st = make_float2(0.f, 0.f);
    uint32_t sm = 0u;
    // Takes the next step's groups off the queue and requests their rows; false at the end of the range.
    auto fetch = [&]() -> bool {
        refill();
        if (count == 0) return false;
        union_sync();
        const int n = min(NG, count);
        const uint32_t first = sh.queue[head & (kUnionQueue - 1)];
        auto entry = [&](int gi) { return gi < n ? sh.queue[(head + gi) & (kUnionQueue - 1)] : (first & 0xFFFF0000u); };
        const uint32_t ea = entry(ga), ec = entry(gc), es = entry(gs);
        const int64_t ra = (int64_t)((int)(ea >> 16) * G + ma) * D + g4 * 8;
        const int64_t rc = (int64_t)((int)(ec >> 16) * G + mc) * D + g4 * 8;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            qa[0][m] = *reinterpret_cast<const bf16x8_t *>(Qr + ra + m * 32);
            qa[1][m] = *reinterpret_cast<const bf16x8_t *>(Qr + rc + m * 32);
            oa[0][m] = *reinterpret_cast<const bf16x8_t *>(Gr + ra + m * 32);
            oa[1][m] = *reinterpret_cast<const bf16x8_t *>(Gr + rc + m * 32);
        }
        st = stat[(int)(es >> 16) * G + ms];
        sm = es & 0xFFFFu;
        head += n;
        count -= n;
        return true;
    };
    bool have = fetch();
    while (have) {  // wave-uniform
        // park the rows, the row statistics and the masks
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            *reinterpret_cast<bf16x8_t *>(sh.q + rowa + m * 64) = qa[0][m];
            *reinterpret_cast<bf16x8_t *>(sh.q + rowc + m * 64) = qa[1][m];
            *reinterpret_cast<bf16x8_t *>(sh.g + rowa + m * 64) = oa[0][m];
            *reinterpret_cast<bf16x8_t *>(sh.g + rowc + m * 64) = oa[1][m];
        }
        if (lane < 32) {
            sh.stat[lane] = st;
            sh.smask[lane] = sm;
        }
        floatx4_t as[2], ap[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            as[t] = floatx4_t{0.f, 0.f, 0.f, 0.f};
            ap[t] = as[t];
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                as[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qa[t][m], kf[m], as[t], 0, 0, 0);
                ap[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(oa[t][m], vf[m], ap[t], 0, 0, 0);
            }
        }
        union_sync();
        have = fetch();  // the next step's rows travel while this one is finished
        uint32_t ph[4], pt[4], sh_[4], st_[4];  // A operands of the second products: two queries per word
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const uint4 mk = *reinterpret_cast<const uint4 *>(&sh.smask[16 * t + 4 * g4]);
            const float4 s01 = *reinterpret_cast<const float4 *>(&sh.stat[16 * t + 4 * g4]);
            const float4 s23 = *reinterpret_cast<const float4 *>(&sh.stat[16 * t + 4 * g4 + 2]);
            const uint32_t mm[4] = {mk.x, mk.y, mk.z, mk.w};
            const float l2[4] = {s01.x, s01.z, s23.x, s23.z}, dl[4] = {s01.y, s01.w, s23.y, s23.w};
            float p[4], ds[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                p[v] = (mm[v] >> c16) & 1u ? fast_exp2(as[t][v] * c2 - l2[v]) : 0.f;
                ds[v] = p[v] * (ap[t][v] - dl[v]);
            }
#pragma unroll
            for (int v = 0; v < 4; v += 2) {
                const SplitWeights wp = split_weights(p[v], p[v + 1]), ws = split_weights(ds[v], ds[v + 1]);
                ph[2 * t + v / 2] = wp.head; pt[2 * t + v / 2] = wp.tail;
                sh_[2 * t + v / 2] = ws.head; st_[2 * t + v / 2] = ws.tail;
            }
        }
        auto frag = [](const uint32_t (&w)[4]) { return __builtin_bit_cast(bf16x8_t, make_uint4(w[0], w[1], w[2], w[3])); };
        const bf16x8_t fph = frag(ph), fpt = frag(pt), fsh = frag(sh_), fst = frag(st_);
#pragma unroll
        for (int nb = 0; nb < 8; ++nb) {
            const bf16x8_t qt = tr_frag(sh.q + tr0 + nb * 32, sh.q + tr1 + nb * 32);
            const bf16x8_t ot = tr_frag(sh.g + tr0 + nb * 32, sh.g + tr1 + nb * 32);
            dk[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fst, qt, dk[nb], 0, 0, 0);
            dv[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fpt, ot, dv[nb], 0, 0, 0);
            dk[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fsh, qt, dk[nb], 0, 0, 0);
            dv[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fph, ot, dv[nb], 0, 0, 0);
        }
        union_sync();  // the next step overwrites the parked rows
    }
    unsigned finite = 0u;  // bit v: key 4 g4 + v
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        float zero = 0.f;
#pragma unroll
        for (int nb = 0; nb < 8; ++nb) zero = fmaf(dk[nb][v], 0.f, fmaf(dv[nb][v], 0.f, zero));
        const unsigned long long bad = __ballot(!(zero == 0.f));
        finite |= (((bad >> (16 * g4)) & 0xFFFFull) == 0ull) << v;
        for (int g = 0; g < 4; ++g) {
            const int j = j0 + 4 * g + v;
            if (((bad >> (16 * g)) & 0xFFFFull) == 0ull || j >= L) continue;
            const int64_t *cp = col + (int64_t)bh * (L + 1) + j;
            const int64_t row = hb + (int64_t)j * D;
            float xk[2], xv[2];
            grouped_dkdv_exact(Qr, Gr, stat, K + row, V + row, lists + tab.off[slot] + cp[0], (int)(cp[1] - cp[0]), gb, ge, G, c2, xk, xv);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                if (pl.S == 1) {
                    dK[row + 2 * lane + c] = f32_to_bf16(scale * xk[c]);
                    dV[row + 2 * lane + c] = f32_to_bf16(xv[c]);
                } else {
                    const int64_t o = (((int64_t)bh * L + j) * pl.S + range) * D + 2 * lane + c;
                    pdk[o] = xk[c];
                    pdv[o] = xv[c];
                }
            }
        }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int j = j0 + 4 * g4 + v;
        if (j < L && (finite >> v & 1u)) {
            if (pl.S == 1) {
                bf16_t *ok = dK + hb + (int64_t)j * D + c16, *ov = dV + hb + (int64_t)j * D + c16;
#pragma unroll
                for (int nb = 0; nb < 8; ++nb) {
                    ok[16 * nb] = f32_to_bf16(scale * dk[nb][v]);
                    ov[16 * nb] = f32_to_bf16(dv[nb][v]);
                }
            } else {
                const int64_t o = (((int64_t)bh * L + j) * pl.S + range) * D + c16;
#pragma unroll
                for (int nb = 0; nb < 8; ++nb) {
                    pdk[o + 16 * nb] = dk[nb][v];
                    pdv[o + 16 * nb] = dv[nb][v];
                }
            }
        }
    }
}

// Which heads go by unions: use[bh] = 1 where the union of 16 neighbouring lists, measured on kChoiceSamples blocks of 16 keys (of
// long lists the groups of one window), is at most `limit` times a list -- in queries per step, of which a group size that does not
// divide 32 leaves some unused.  limit == 0: head by head, each against its own limit, a block per head of the table.  Else
// one answer for all `heads`, from samples of the table's, in block 0.  A wave per sample, four lanes per key; the other blocks
// pack the row statistics meanwhile.
constexpr int kChoiceSamples = 16;
constexpr int kChoiceGroups = 8192;
__host__ __device__ inline float union_limit_of(float k, float fixed)
{
    return (1.5e-5f * k + 0.0066f + fixed) / (3.1e-6f * (k + 118));
}
__global__ __launch_bounds__(64 * kChoiceSamples) void union_prepare_kernel(const int32_t *__restrict__ lists, const int64_t *__restrict__ col,
                                                                            int L, int G, HeadTable tab, float limit, int heads,
                                                                            const float *__restrict__ lse,
                                                                            const float *__restrict__ delta,
                                                                            float2 *__restrict__ rowstat, int64_t rows,
                                                                            int32_t *__restrict__ use)
{
    __shared__ uint32_t bm_all[kChoiceSamples][kChoiceGroups / 32];
    __shared__ int32_t sums[2];  // entries, groups in the unions
    const int choosers = !use ? 0 : limit == 0.f ? tab.n : 1;
    if ((int)blockIdx.x >= choosers) {
        const int64_t e = (int64_t)(blockIdx.x - choosers) * (64 * kChoiceSamples) + threadIdx.x;
        if (e < rows) rowstat[e] = make_float2(lse[e] * kLog2e, delta[e]);
        return;
    }
    const int lane = threadIdx.x & 63, sample = threadIdx.x >> 6;
    const int slot = limit == 0.f ? blockIdx.x : sample % tab.n, bh = tab.bh[slot];
    const int Lq = L / G, blocks = (L + kUnionKeys - 1) / kUnionKeys;
    uint32_t *bm = bm_all[sample];
    for (int w = lane; w < kChoiceGroups / 32; w += 64) bm[w] = 0u;
    if (threadIdx.x < 2) sums[threadIdx.x] = 0;
    __syncthreads();
    const int j = (int)((int64_t)sample * blocks / kChoiceSamples) * kUnionKeys + (lane >> 2);
    const int w0 = Lq > kChoiceGroups ? (int)((int64_t)(Lq - kChoiceGroups) * sample / (kChoiceSamples - 1)) : 0;
    int entries = 0;
    if (j < L) {
        const int64_t *cp = col + (int64_t)bh * (L + 1) + j;
        const int32_t *list = lists + tab.off[slot] + cp[0];
        const int n = (int)(cp[1] - cp[0]);
        int lo = 0;
        if (w0 > 0)
            for (int hi = n; lo < hi;) {
                const int mid = (lo + hi) >> 1;
                if (list[mid] < w0) lo = mid + 1; else hi = mid;
            }
        for (int t = lo + (lane & 3); t < n; t += 32) {
            int e[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) e[u] = list[min(t + 4 * u, n - 1)] - w0;
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (t + 4 * u < n && e[u] >= 0 && e[u] < kChoiceGroups) {
                    atomicOr(&bm[e[u] >> 5], 1u << (e[u] & 31));
                    ++entries;
                }
            if (e[7] >= kChoiceGroups) break;  // ascending
        }
    }
    union_sync();
    int groups = 0;
    for (int w = lane; w < kChoiceGroups / 32; w += 64) groups += __popc(bm[w]);
    if (entries) atomicAdd(&sums[0], entries);
    if (groups) atomicAdd(&sums[1], groups);
    __syncthreads();
    const int slots = 32 / G * G;  // queries of a step that are used
    const float most = limit == 0.f ? union_limit_of((float)tab.k[slot], 0.f) : limit;
    const int32_t by_unions = (float)sums[1] * 16.f * 32.f <= most * (float)sums[0] * (float)slots;
    if (limit == 0.f) {
        if (threadIdx.x == 0) use[bh] = by_unions;
    } else {
        for (int h = threadIdx.x; h < heads; h += 64 * kChoiceSamples) use[h] = by_unions;
    }
}

// Times of the two forms in us, for P pairs and R rows: unions 3.1e-6 (P + 118 R) per list that a union is long, the sweep 1.5e-5 P +
// 0.0066 R + 39 (segments, row order, more launches).  Fitted to 462 problems (1 to 12 heads of 2048 to 32768 keys, 1 to 16 % kept,
// groups of 4, 8 and 32, smooth and independent inputs, unions 2.3 to 15 lists long), and a little to the sweep's side of the fit.
// L = 32768, k = 2730, 2 x 2 x 2, four heads, the whole backward: unions of 3 lists 6.9 ms, sweep 11.0; of 9 lists (keys chosen
// independently) 13.4, 9.6; L = 16384, 5.7 lists: 4.94, 4.95; one head of 4096, k = 102, 5.8 lists: 125 us, 207; 13.4 lists: 123, 165.  Where
// any union pays (16 lists), nothing is measured and the sweep is not launched: 25 us.
static double pairs_of(const dsv_problem &p)
{
    double pairs = 0;
    for (int h = 0; h < p.H; ++h) pairs += (double)p.B * p.L * p.k_per_head[h];
    return pairs;
}
double union_limit(const dsv_problem &p)
{
    const double pairs = pairs_of(p), rows = (double)p.B * p.H * p.L;
    auto limit = [&](double fixed) { return union_limit_of((float)(pairs / rows), (float)(fixed / rows)); };
    return limit(39 + 25) >= 16 ? 16 : limit(39);
}

// Whether heads are chosen one by one: from 5e7 pairs on.  Below, two forms side by side leave each other's launches short.
// Measured over 169 problems with heads of unlike k (2 to 16 heads of 2048 to 65536 keys, keys chosen independently), one by one against one
// answer: below 3e6 pairs 1.03 (1.36 at worst), 3e6 to 2e7 1.06 (1.40), 2e7 to 4e8 1.00 (0.95 to 1.06), above 0.975 (0.92 to 1.005).
static bool choose_by_head(const dsv_problem &p) { return pairs_of(p) >= 5e7; }

dsv_status launch_union_prepare(const dsv_problem &p, int G, const HeadTable *tabs, int n_tabs, const int32_t *lists, const int64_t *col,
                                const float *lse, const float *delta, float2 *rowstat, int32_t *use, hipStream_t st)
{
    const bool by_head = choose_by_head(p);
    const int block = 64 * kChoiceSamples;
    for (int t = 0; t < (use && by_head ? n_tabs : 1); ++t) {
        const int64_t rows = t ? 0 : (int64_t)p.B * p.H * p.L;
        const int choosers = !use ? 0 : by_head ? tabs[t].n : 1;
        hipLaunchKernelGGL(union_prepare_kernel, dim3((unsigned)((rows + block - 1) / block) + choosers), dim3(block), 0, st, lists, col, p.L, G,
                           tabs[t], by_head ? 0.f : (float)union_limit(p), p.B * p.H, lse, delta, rowstat, rows, use);
        DSV_LAUNCH_CHECK();
    }
    return DSV_OK;
}

dsv_status launch_grouped_dkdv(const dsv_problem &p, int G, const HeadTable *tabs, int n_tabs, const void *Q, const void *K,
                               const void *V, const int32_t *lists, const int64_t *col, const void *dO, void *dK, void *dV,
                               const SplitPlan &plan, const BwdSplitWorkspace &w, const int32_t *use, hipStream_t st)
{
    if (p.dtype != DSV_BF16 || p.d != 128 || G > 32) return DSV_EUNSUPPORTED;
    UnionPlan pl;
    pl.S = plan.S;
    pl.S_pad = plan.S_pad;
    pl.groups = (p.L / G + pl.S - 1) / pl.S;  // of at most 8192 queries and a group: group numbers inside a range fit 16 bits
    pl.nkb = (p.L + 4 * kUnionKeys - 1) / (4 * kUnionKeys);
    for (int t = 0; t < n_tabs; ++t) {
        const int64_t blocks = tabs[t].n * range_items(pl.S_pad, pl.nkb);
        if (blocks > 0x7FFFFFFF) return DSV_EUNSUPPORTED;
        hipLaunchKernelGGL(grouped_dkdv_kernel, dim3((unsigned)blocks), dim3(256), 0, st, (const bf16_t *)Q, (const bf16_t *)K,
                           (const bf16_t *)V, (const bf16_t *)dO, lists, col, (const float2 *)w.rowstat, (bf16_t *)dK, (bf16_t *)dV,
                           w.pa, w.pb, p.L, G, p.scale, tabs[t], pl, use);
        DSV_LAUNCH_CHECK();
    }
    return DSV_OK;
}

}  // namespace dsv
