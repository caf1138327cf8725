// Stage 1 for short sequences: threshold search and query-major emission in one kernel (paper Sec. "Critical KV Estimation
// with Kernel Fusion").  A block of 16 waves takes 32 queries of one head; its waves score up to NT key tiles each ONCE and
// keep the scores in registers through the search and the emission, so that a call is two launches -- projection and
// this -- instead of six, and no score is formed five times by blocks that the few tiles of a short sequence leave waiting
// for one another.
//   search   256 equal bins between each query's smallest and largest score (bins of equal width in the VALUE: a few scores
//            each, where the leading bits of the float patterns put hundreds into each of a handful of counters); the
//            scores of the bin that holds the k-th largest go to LDS and are ranked against each other.  Exact: the map
//            from score to bin is monotone.  If a query of the block finds more than kSmallCap scores in its bin (massive
//            ties), the block takes the four 8-bit digits of the radix search (stage1.hip) instead.
//
// What bounds it: barriers and LDS round trips, about ten in a row.  L = 1024, two heads, fp32, per call with the projection:
// 128 us in six launches, 32 with the digits, 28.6 with the bins, 22 since fragments come in 16-byte pieces (before, the sixteen waves'
// loads alone took ten of them).  Outputs are those of the radix search and of the
// emission (stage1_emit.hip), bit for bit.
#include "stage1_core.h"

namespace dsv {

constexpr int kSmallWaves = 16;
constexpr int kSmallMaxTiles = 4;  // score tiles a wave keeps: 64 accumulators of the 128 registers that 16 waves leave it, some of them in scratch
constexpr int kSmallCap = 64;      // scores of a query's bin that are ranked in LDS
constexpr int kSmallMaxKeys = kSmallWaves * kSmallMaxTiles * 32;

template <typename T, int R, int NT>
__global__ __launch_bounds__(64 * kSmallWaves) void select_small_kernel(const T *__restrict__ Qlr, const T *__restrict__ Klr, int Lq,
                                                                        int L, HeadTable tab, uint32_t *__restrict__ prefix,
                                                                        int32_t *__restrict__ idx, int32_t *__restrict__ jcut,
                                                                        int32_t *__restrict__ tile_flag)
{
    constexpr int TILES = kSmallWaves * NT;
    __shared__ uint32_t hist[256 * 32];
    __shared__ uint32_t gt[TILES][33], eq[TILES][33];  // per key tile and query: scores above (or at) the threshold, ties
    __shared__ BucketScratch<64 * kSmallWaves> scratch;
    __shared__ uint32_t cand[32][kSmallCap + 1];
    __shared__ uint32_t lo_s[32], hi_s[32];            // smallest and largest score of every query (order-preserving keys)
    __shared__ int32_t ccnt[32], rem[32], ties[32];
    __shared__ uint32_t tau_s[32];
    __shared__ int32_t eq_s[32];
    const int slot = blockIdx.y;
    const int bh = tab.bh[slot];
    const int k = tab.k[slot];
    const int q0 = blockIdx.x * 32;
    const T *Qb = Qlr + (int64_t)bh * Lq * R;
    const T *Kb = Klr + (int64_t)bh * L * R;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = lane & 31, half = lane >> 5;
    const int ntiles = (L + 31) >> 5;

    const Frag<T, R> qf = load_frag<T, R>(Qb, q0, Lq, lane);
    floatx16_t acc[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) acc[i] = score_tile<T, R>(load_frag<T, R>(Kb, (wave + kSmallWaves * i) * 32, L, lane), qf);

    uint32_t pre = 0;
    int want = k, count = 0;
    auto valid_key = [&](int i, int v) { return tile_pos(v) < L - (wave + kSmallWaves * i) * 32 - 4 * half; };
    auto clear_hist = [&]() {
#pragma unroll
        for (int e = 0; e < 256 * 32 / (64 * kSmallWaves); ++e) hist[threadIdx.x + e * 64 * kSmallWaves] = 0u;
    };
    if (threadIdx.x < 32) {
        lo_s[n] = 0xFFFFFFFFu;
        hi_s[n] = 0u;
        ccnt[n] = 0;
    }
    clear_hist();
    uint32_t lo = 0xFFFFFFFFu, hi = 0u;
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v)
            if (valid_key(i, v)) {
                const uint32_t key = score_key(acc[i][v]);
                lo = min(lo, key);
                hi = max(hi, key);
            }
    __syncthreads();
    if (lo <= hi) {
        atomicMin(&lo_s[n], lo);
        atomicMax(&hi_s[n], hi);
    }
    __syncthreads();
    const float least = key_score(lo_s[n]);
    const float span = key_score(hi_s[n]) - least;
    const float per = span > 0.f ? 255.9f / span : 0.f;  // all alike (or a span beyond the floats): one bin
    auto bin = [&](float x) { return (uint32_t)fminf(fmaxf((x - least) * per, 0.f), 255.f); };  // not a number (infinite scores): 0
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v)
            if (valid_key(i, v)) atomicAdd(&hist[bin(acc[i][v]) * 32 + n], 1u);
    __syncthreads();
    const Bucket top = find_bucket(hist, scratch, [](int b) { return b; }, k);
    if (__all(top.count <= kSmallCap)) {  // the same 32 queries in every wave: the whole block
        if (threadIdx.x < 32) rem[n] = k - top.above;
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                if (valid_key(i, v) && (int)bin(acc[i][v]) == top.digit) {
                    const int at = atomicAdd(&ccnt[n], 1);
                    if (at < kSmallCap) cand[n][at] = score_key(acc[i][v]);
                }
        __syncthreads();
        // the r-th largest of a query's scores in the bin: the key x with #(y > x) < r <= #(y >= x)
        const int q = threadIdx.x >> 5, c = min(ccnt[q], kSmallCap), r = rem[q];
        for (int i = n; i < c; i += 32) {
            const uint32_t x = cand[q][i];
            int above = 0, same = 0;
            for (int y = 0; y < c; ++y) {
                const uint32_t other = cand[q][y];
                above += other > x;
                same += other == x;
            }
            if (above < r && r <= above + same) {  // every thread that finds it writes the same values
                tau_s[q] = x;
                ties[q] = r - above;
                eq_s[q] = same;
            }
        }
        __syncthreads();
        pre = tau_s[n];
        want = ties[n];
        count = eq_s[n];
    } else {
#pragma unroll
        for (int pass = 0; pass < 4; ++pass) {
            const int shift = 24 - 8 * pass;
#pragma unroll
            for (int e = 0; e < 256 * 32 / (64 * kSmallWaves); ++e) hist[threadIdx.x + e * 64 * kSmallWaves] = 0u;
            __syncthreads();
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                const int left = L - (wave + kSmallWaves * i) * 32 - 4 * half;  // keys of the tile from this half's first on
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const uint32_t key = score_key(acc[i][v]);
                    if (tile_pos(v) < left && (pass == 0 || (key >> ((shift + 8) & 31)) == (pre >> ((shift + 8) & 31))))
                        atomicAdd(&hist[((key >> shift) & 255u) * 32 + n], 1u);
                }
            }
            __syncthreads();
            const Bucket f = find_bucket(hist, scratch, [](int b) { return b; }, want);
            pre |= (uint32_t)f.digit << shift;
            want -= f.above;
            count = f.count;
        }
    }
    const float tau = key_score(pre);
    const bool all_simple = __all(want == count);  // every query takes all its ties: "score >= tau" decides
    if (threadIdx.x < 32) ties[n] = want;
#pragma unroll
    for (int i = 0; i < NT; ++i) {
        const int tile = wave + kSmallWaves * i;
        const int j0 = tile * 32;
        const uint32_t valid = j0 + 32 <= L ? 0xFFFFFFFFu : (j0 < L ? (1u << (L - j0)) - 1u : 0u);
        uint32_t g, e;
        threshold_words(acc[i], tau, all_simple, valid, half, g, e);
        if (half == 0) {
            gt[tile][n] = g;
            eq[tile][n] = e;
        }
    }
    __syncthreads();

    const int q = 2 * wave + half;
    const bool live = q0 + q < Lq;
    RowOut ro{0, ties[q], -1};
    for (int t0 = 0; t0 < ntiles; t0 += 32) {
        const bool in = t0 + n < ntiles;
        emit_row_words(ro, in ? gt[t0 + n][q] : 0u, in ? eq[t0 + n][q] : 0u, all_simple, t0 + n, half, live,
                       idx + tab.off[slot] + (int64_t)min(q0 + q, Lq - 1) * k, k);
    }
    const int64_t g0 = (int64_t)bh * padded_len(Lq) + q0;
    if (threadIdx.x < 32 && q0 + n < Lq) prefix[g0 + n] = __float_as_uint(tau);
    if (jcut && live && n == 0) jcut[g0 + q] = all_simple ? kAllTies : ro.last_tie;
    if (tile_flag && threadIdx.x == 0) tile_flag[(int64_t)bh * gridDim.x + blockIdx.x] = all_simple ? 1 : 0;
}

// ------------------------------------------------------------------------------------ host
// Up to 1024 keys always; up to 2048 (four tiles per wave, of which 68 registers' worth goes through scratch memory) where
// each CU has one block, or where scores cost most.  Against the four passes and the emission, with the projection, us, k = L / 16:
// bf16, r = 16, L = 1024, 1 head 18.9 : 30.5, 24 heads 46 : 51, 96 heads 161 : 158; L = 2048, 4 heads (256 blocks) 30 : 40, 12 heads 73 : 69,
// 96 heads 506 : 388; r = 64, 96 heads 763 : 1120; fp32, r = 16, 1 head 42 : 104, 96 heads 873 : 1936.
bool small_select(const dsv_problem &p, int Lq)
{
    if (p.L <= kSmallMaxKeys / 2 || p.L > kSmallMaxKeys) return p.L <= kSmallMaxKeys;
    return p.dtype == DSV_F32 || p.r == 64 || (int64_t)p.B * p.H * ((Lq + 31) / 32) <= 256;
}

template <typename T, int R>
static dsv_status select_small_t(const dsv_problem &p, int Lq, const HeadTable &tab, const void *Qlr, const void *Klr,
                                 const SelectBuffers &b, hipStream_t st)
{
    const dim3 grid((Lq + 31) / 32, tab.n), block(64 * kSmallWaves);
    auto launch = [&](auto kern) {
        hipLaunchKernelGGL(kern, grid, block, 0, st, (const T *)Qlr, (const T *)Klr, Lq, p.L, tab, b.prefix, b.idx, b.jcut, b.tile_flag);
    };
    if (p.L <= kSmallMaxKeys / 4) launch(select_small_kernel<T, R, 1>);
    else if (p.L <= kSmallMaxKeys / 2) launch(select_small_kernel<T, R, 2>);
    else launch(select_small_kernel<T, R, 4>);
    DSV_LAUNCH_CHECK();
    return DSV_OK;
}

dsv_status launch_select_small(const dsv_problem &p, int Lq, const HeadTable &tab, const void *Qlr, const void *Klr,
                               const SelectBuffers &b, hipStream_t st)
{
#define DSV_CASE(TT, RR) return select_small_t<TT, RR>(p, Lq, tab, Qlr, Klr, b, st)
    if (p.dtype == DSV_BF16) {
        if (p.r == 16) DSV_CASE(bf16_t, 16);
        if (p.r == 32) DSV_CASE(bf16_t, 32);
        if (p.r == 64) DSV_CASE(bf16_t, 64);
    } else if (p.dtype == DSV_F32) {
        if (p.r == 16) DSV_CASE(float, 16);
        if (p.r == 32) DSV_CASE(float, 32);
        if (p.r == 64) DSV_CASE(float, 64);
    }
#undef DSV_CASE
    return DSV_EUNSUPPORTED;
}

}  // namespace dsv
