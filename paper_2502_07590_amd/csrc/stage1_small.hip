// Stage 1 for short sequences: threshold search and query-major emission in one kernel (paper Sec. "Critical KV Estimation
// with Kernel Fusion").  A block of 16 waves takes 32 queries of one head; its waves score up to NT key tiles each ONCE and
// keep the scores in registers through the four digits of the radix search (stage1.hip) and the emission, so that a
// call is two launches -- projection and this -- instead of six, and no score is formed five times by blocks that the
// few tiles of a short sequence leave waiting for one another.  What bounds it: the barriers and LDS round trips of the
// four digits -- 10 us of the first, whose counters are few and hot, 3 us of each of the others.  L = 1024, two heads, fp32:
// 128 -> 32 us per call.  Outputs are those of the radix search and of the emission (stage1_emit.hip), bit for bit.
#include "stage1_core.h"

namespace dsv {

constexpr int kSmallWaves = 16;
constexpr int kSmallMaxTiles = 4;  // score tiles a wave keeps: 64 accumulators of the 128 registers that 16 waves leave it
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
    __shared__ int32_t ties[32];
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
// 4 tiles per wave is what the registers hold.
bool small_select(int L) { return L <= kSmallMaxKeys; }

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
