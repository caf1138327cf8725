// Stage 1: critical-KV estimation (paper Sec. "Low-Rank based Sparsity Prediction" and
// Sec. "Critical KV Estimation with Kernel Fusion"; two-pass threshold form of Appendix
// "Implementation details").
//
//   project      Q_lr = Q Wq, K_lr = K Wk            (fp32 accumulate, rounded to the storage type)
//   select       per (head, query): exact value of the k-th largest score by a radix search on the
//                order-preserving bit pattern of the fp32 score (four 8-bit digits, one pass over
//                all keys per digit, histograms in LDS), then
//   emit         (stage1_emit.hip) one more pass that writes every key above the threshold plus the
//                lowest-index ties, in ascending key order; optionally the same key-major.
// Scores are recomputed in every pass on the matrix cores (one 32x32 MFMA tile = 32 keys x 32
// queries); the L x L matrix never exists in memory.  Every pass uses the same instruction
// sequence for a score, so a score has the same bits in every pass.
#include <algorithm>
#include <atomic>

#include "stage1_core.h"

namespace dsv {

// ------------------------------------------------------------------------------------ projection
// Q holds Lq rows per head and K holds Lk (equal for per-query selection; with query grouping only the
// groups' centre queries are projected and scored).  A lane projects one token: its row comes out of LDS 16 bytes at a
// time (the wave's rows were loaded whole), the weights are the same for all lanes and so come through the scalar unit, and
// every output is a plain ascending-c fp32 FMA chain.  A lane forms OPL of its token's outputs.  Bound by those D * R
// multiplications per token.  L = 32768, four heads, bf16, r = 16: 118 -> 36 us (weights and elements of the rows read from
// LDS one by one before).
template <typename T> __device__ __forceinline__ float piece_elem(const uint4 &x, int e)
{
    const uint32_t w = sizeof(T) == 4 ? (e == 0 ? x.x : e == 1 ? x.y : e == 2 ? x.z : x.w)
                                      : (e < 2 ? x.x : e < 4 ? x.y : e < 6 ? x.z : x.w);
    if (sizeof(T) == 4) return __uint_as_float(w);
    return __uint_as_float(e & 1 ? w & 0xFFFF0000u : w << 16);
}

template <typename T, int D, int R, int OPL>
__global__ __launch_bounds__(256) void project_kernel(const T *__restrict__ Q, const T *__restrict__ K,
                                                      const T *__restrict__ Wq, const T *__restrict__ Wk,
                                                      T *__restrict__ Qlr, T *__restrict__ Klr, int Lq, int Lk, int H)
{
    constexpr int EPP = 16 / (int)sizeof(T), PPR = D / EPP;  // elements per 16-byte piece, pieces per row
    constexpr int WPE = (int)sizeof(T) / 2;                  // 16-bit halves per weight
    // elements whose weights (64 words at most) wait in scalar registers
    constexpr int GE = 256 / (OPL * (int)sizeof(T)) < EPP ? 256 / (OPL * (int)sizeof(T)) : EPP;
    constexpr int CP = 8;                                    // pieces of every row in LDS at a time
    __shared__ uint4 xs_all[4][64][CP + 1];                  // padded: rows 36 words apart
    const int bh = blockIdx.y;
    const int h = bh % H;
    const bool side = blockIdx.z & 1;
    const int o0 = (blockIdx.z >> 1) * OPL;                  // first output
    const int L = side ? Lk : Lq;                            // tokens on this side (the grid covers the longer side)
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int t0 = (blockIdx.x * 4 + wave) * 64;
    if (t0 >= L) return;                                     // whole wave; nothing below synchronises across waves
    const uint4 *X = reinterpret_cast<const uint4 *>((side ? K : Q) + (int64_t)bh * L * D);
    // weights: read-only and the same for the whole wave, so constant address space (scalar loads, scalar conversions)
    typedef const __attribute__((address_space(4))) uint32_t scalar_u32;
    const scalar_u32 *W = (const scalar_u32 *)(uintptr_t)((side ? Wk : Wq) + (int64_t)h * D * R + o0);
    T *out = (side ? Klr : Qlr) + ((int64_t)bh * L + t0) * R + o0;
    const int ntok = min(64, L - t0);
    uint4 (*xs)[CP + 1] = xs_all[wave];
    float acc[OPL];
#pragma unroll
    for (int t = 0; t < OPL; ++t) acc[t] = 0.f;
    for (int p0 = 0; p0 < PPR; p0 += CP) {
#pragma unroll
        for (int i = 0; i < CP; ++i) {  // 8 lanes per row and load: 128 contiguous bytes
            const int tok = 8 * i + (lane >> 3);
            xs[tok][lane & 7] = X[(int64_t)(t0 + min(tok, ntok - 1)) * PPR + p0 + (lane & 7)];
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll 1
        for (int p = 0; p < CP; ++p) {
            const uint4 x = xs[lane][p];
#pragma unroll
            for (int e0 = 0; e0 < EPP; e0 += GE) {
                const scalar_u32 *w = W + ((p0 + p) * EPP + e0) * (R * WPE / 2);
                uint32_t word[GE][OPL * WPE / 2];
#pragma unroll
                for (int e = 0; e < GE; ++e)
#pragma unroll
                    for (int t = 0; t < OPL * WPE / 2; ++t) word[e][t] = w[e * (R * WPE / 2) + t];
#pragma unroll
                for (int e = 0; e < GE; ++e) {
                    const float xv = piece_elem<T>(x, e0 + e);
#pragma unroll
                    for (int t = 0; t < OPL; ++t) {
                        const uint32_t wt = word[e][t * WPE / 2];
                        acc[t] = fmaf(xv, __uint_as_float(WPE == 2 ? wt : (t & 1 ? wt & 0xFFFF0000u : wt << 16)), acc[t]);
                    }
                    __builtin_amdgcn_sched_barrier(0);  // the converted weights of one element at a time: scalar registers
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    if (lane < ntok) store_chunk<T, OPL>(out + (int64_t)lane * R, acc);
}

// ------------------------------------------------------------------------------------ radix pass
// One digit of the search for the k-th largest score of each query.  Block = 32 queries of one
// head, kRadixWaves waves striding over the key tiles, one shared histogram in LDS laid out [256 digits][32
// queries]: the bank of a counter depends on the query alone, so the 32 lanes of a half-wave (32
// different queries) never collide, whatever their digits are.
//   PASS 0 counts every key by the top digit; PASS p counts only keys whose higher digits equal
//   the prefix found so far.  Afterwards: the digit whose bucket holds the k_rem-th largest
//   remaining key is appended to the prefix and k_rem is reduced by the keys in higher buckets.
// After pass 3 the prefix is the full key of the k-th largest score and |k_rem| is the number of
// keys equal to it that belong to the top-k (at least 1); k_rem < 0 marks "all of them".

// One 32-query tile (queries q0 .. q0+31 of head slot `slot`); hist: the block's 256 x 32 counters.
template <typename T, int R, int PASS>
__device__ __forceinline__ void radix_pass_tile(uint32_t *hist, BucketScratch<64 * kRadixWaves> &scratch, const T *__restrict__ Qlr, const T *__restrict__ Klr, int Lq,
                                                int L, const HeadTable &tab, int slot, int q0, uint32_t *__restrict__ prefix,
                                                int32_t *__restrict__ krem)
{
    constexpr int SHIFT = 24 - 8 * PASS;
    const int bh = tab.bh[slot];
    const T *Qb = Qlr + (int64_t)bh * Lq * R;   // Lq query rows (all L tokens, or one proxy per query group)
    const T *Kb = Klr + (int64_t)bh * L * R;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = lane & 31, half = lane >> 5;

    for (int e = threadIdx.x; e < 256 * 32; e += 64 * kRadixWaves) hist[e] = 0;
    __syncthreads();

    const int qi = min(q0 + n, Lq - 1);
    uint32_t pre = 0;
    if constexpr (PASS > 0) pre = prefix[(int64_t)bh * padded_len(Lq) + qi];
    const Frag<T, R> qf = load_frag<T, R>(Qb, q0, Lq, lane);
    const int ntiles = (L + 31) >> 5;
    const int nfull = L >> 5;  // tiles with all 32 keys in range
    uint32_t *hcol_mine = hist + n;  // counter of digit b: hcol_mine[32 * b]
    // When every query of the tile has a threshold prefix in the positive floats (the usual case:
    // k < L/2), a score matches the prefix iff its RAW bits do: negative scores have the sign bit
    // set and can never match, and for positive floats the raw pattern is already monotone.  That
    // drops the key transform from the hot loop: one xor + one compare per score, digits are only
    // extracted for the few matches.
    bool fast = false;
    if constexpr (PASS > 0) fast = __all((pre & 0x80000000u) != 0u);
    if (fast) {
        const uint32_t raw_pre = pre ^ 0x80000000u;
        Frag<T, R> kf_next = load_frag<T, R>(Kb, wave * 32, L, lane);
        for (int tile = wave; tile < nfull; tile += kRadixWaves) {
            // the next tile's fragment is requested before this tile is scored (rows past the end clamp)
            const Frag<T, R> kf = kf_next;
            kf_next = load_frag<T, R>(Kb, (tile + kRadixWaves) * 32, L, lane);
            const floatx16_t acc = score_tile<T, R>(kf, qf);
            constexpr uint32_t kLimit = 1u << ((SHIFT + 8) & 31);
            if constexpr (PASS >= 2) {
                // Matches are rare from the third digit on (a 16-bit prefix leaves about one score in a
                // thousand): look at four scores at a time with plain xor / min, and only enter the
                // masked histogram update for a group in which some lane has a match.
#pragma unroll
                for (int v0 = 0; v0 < 16; v0 += 4) {
                    uint32_t x[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) x[u] = __float_as_uint(acc[v0 + u]) ^ raw_pre;
                    const uint32_t lo = min(min(x[0], x[1]), min(x[2], x[3]));
                    if (__any(lo < kLimit)) {
#pragma unroll
                        for (int u = 0; u < 4; ++u)
                            if (x[u] < kLimit) atomicAdd(&hcol_mine[((x[u] >> SHIFT) & 255u) * 32], 1u);
                    }
                }
            } else {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const uint32_t bits = __float_as_uint(acc[v]);
                    if ((bits ^ raw_pre) < kLimit) atomicAdd(&hcol_mine[((bits >> SHIFT) & 255u) * 32], 1u);
                }
            }
        }
    } else {
        Frag<T, R> kf_next = load_frag<T, R>(Kb, wave * 32, L, lane);
        for (int tile = wave; tile < nfull; tile += kRadixWaves) {
            const Frag<T, R> kf = kf_next;
            kf_next = load_frag<T, R>(Kb, (tile + kRadixWaves) * 32, L, lane);
            const floatx16_t acc = score_tile<T, R>(kf, qf);
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                if constexpr (PASS == 0) {
                    // first digit: counted by the RAW top byte (no key transform in the loop); the scan
                    // below visits the raw buckets in key order
                    atomicAdd(&hcol_mine[(__float_as_uint(acc[v]) >> 24) * 32], 1u);
                } else {
                    const uint32_t key = score_key(acc[v]);
                    if ((key >> (SHIFT + 8)) == (pre >> (SHIFT + 8))) atomicAdd(&hcol_mine[((key >> SHIFT) & 255u) * 32], 1u);
                }
            }
        }
    }
    if (nfull < ntiles && wave == nfull % kRadixWaves) {  // the ragged last tile
        const int j0 = nfull * 32;
        const Frag<T, R> kf = load_frag<T, R>(Kb, j0, L, lane);
        const floatx16_t acc = score_tile<T, R>(kf, qf);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const uint32_t key = score_key(acc[v]);
            bool ok = j0 + tile_pos(v) + 4 * half < L;
            if constexpr (PASS > 0) ok = ok && ((key >> (SHIFT + 8)) == (pre >> (SHIFT + 8)));
            const uint32_t bucket = PASS == 0 ? __float_as_uint(acc[v]) >> 24 : (key >> SHIFT) & 255u;
            if (ok) atomicAdd(&hcol_mine[bucket * 32], 1u);
        }
    }
    __syncthreads();

    const int64_t g = (int64_t)bh * padded_len(Lq) + qi;  // every thread of a query (they share n)
    const int kr = PASS == 0 ? tab.k[slot] : krem[g];
    // bucket of key digit b: the digit itself, except in pass 0, whose buckets are raw top bytes
    // (positive floats: key digit = raw ^ 0x80; negative floats: key digit = ~raw)
    const Bucket f = find_bucket(hist, scratch, [](int b) { return PASS == 0 ? (b >= 128 ? b ^ 0x80 : b ^ 0xFF) : b; }, kr);
    if (threadIdx.x < 32 && q0 + n < Lq) {
        prefix[g] = (PASS == 0 ? 0u : pre) | ((uint32_t)f.digit << SHIFT);
        // after the last digit the bucket holds exactly the keys equal to the threshold: a negative
        // k_rem tells the emission that all of them are taken (then "score >= threshold" decides)
        const int want = kr - f.above;
        krem[g] = (PASS == 3 && want == f.count) ? -want : want;
    }
}

template <typename T, int R, int PASS>
__global__ __launch_bounds__(64 * kRadixWaves) void radix_pass_kernel(const T *__restrict__ Qlr, const T *__restrict__ Klr, int Lq, int L,
                                                         HeadTable tab, uint32_t *__restrict__ prefix,
                                                         int32_t *__restrict__ krem)
{
    __shared__ uint32_t hist[256 * 32];
    __shared__ BucketScratch<64 * kRadixWaves> scratch;
    radix_pass_tile<T, R, PASS>(hist, scratch, Qlr, Klr, Lq, L, tab, blockIdx.y, blockIdx.x * 32, prefix, krem);
}

// The same digit pass for the query tiles on a list (todo[0] = their number, todo[1 + i] = slot * qtiles +
// tile): the tiles the windowed search (stage1_window.hip) could not settle.  The grid is fixed; an empty
// list costs a launch.
template <typename T, int R, int PASS>
__global__ __launch_bounds__(64 * kRadixWaves) void radix_pass_list_kernel(const T *__restrict__ Qlr, const T *__restrict__ Klr,
                                                              int Lq, int L, HeadTable tab, uint32_t *__restrict__ prefix,
                                                              int32_t *__restrict__ krem, const int32_t *__restrict__ todo,
                                                              int qtiles)
{
    __shared__ uint32_t hist[256 * 32];
    __shared__ BucketScratch<64 * kRadixWaves> scratch;
    const int n = min(todo[0], tab.n * qtiles);
    for (int i = blockIdx.x; i < n; i += gridDim.x) {
        const int id = todo[1 + i];
        const int slot = id / qtiles;
        if (slot >= 0 && slot < tab.n)  // an id outside the table can only come from a corrupted list
            radix_pass_tile<T, R, PASS>(hist, scratch, Qlr, Klr, Lq, L, tab, slot, (id - slot * qtiles) * 32, prefix, krem);
        __syncthreads();  // the tile's last readers of hist are done before the next tile clears it
    }
}

// ------------------------------------------------------------------------------------ debug scores
// fp32 scores of chosen query rows against every key, through the same tile routine.
template <typename T, int R>
__global__ __launch_bounds__(64) void scores_rows_kernel(const T *__restrict__ Qlr, const T *__restrict__ Klr, int L,
                                                         const int32_t *__restrict__ rows, int n_rows,
                                                         float *__restrict__ scores)
{
    const int lane = threadIdx.x;
    const int n = lane & 31, half = lane >> 5;
    const int r0 = blockIdx.y * 32;
    const int rsel = min(r0 + n, n_rows - 1);
    const Frag<T, R> qf = load_frag_row<T, R>(Qlr, rows[rsel], lane);
    const int j0 = blockIdx.x * 32;
    const Frag<T, R> kf = load_frag<T, R>(Klr, j0, L, lane);
    const floatx16_t acc = score_tile<T, R>(kf, qf);
    if (r0 + n < n_rows) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int j = j0 + tile_pos(v) + 4 * half;
            if (j < L) scores[(int64_t)(r0 + n) * L + j] = acc[v];
        }
    }
}

// ------------------------------------------------------------------------------------ host
template <typename T, int D, int R>
static dsv_status project_t(const dsv_problem &p, int Lq, const void *Q, const void *K, const void *Wq, const void *Wk,
                            void *Qlr, void *Klr, hipStream_t st)
{
    const int64_t tokens = (int64_t)std::max(p.L, Lq) * p.B * p.H;
    // outputs per lane: all of them up to 32; few tokens: 4, for more waves (L = 1024, two heads, fp32: 7.1 us against 8.9)
    constexpr int kMost = R < 32 ? R : 32;
    const bool few = tokens < 32768;
    const int opl = few ? 4 : kMost;
    dim3 grid((std::max(p.L, Lq) + 255) / 256, p.B * p.H, 2 * (R / opl));
    const auto kern = few ? &project_kernel<T, D, R, 4> : &project_kernel<T, D, R, kMost>;
    hipLaunchKernelGGL(kern, grid, dim3(256), 0, st, (const T *)Q, (const T *)K, (const T *)Wq,
                       (const T *)Wk, (T *)Qlr, (T *)Klr, Lq, p.L, p.H);
    DSV_LAUNCH_CHECK();
    return DSV_OK;
}

template <typename T, int D>
static dsv_status project_r(const dsv_problem &p, int Lq, const void *Q, const void *K, const void *Wq, const void *Wk,
                            void *Qlr, void *Klr, hipStream_t st)
{
    switch (p.r) {
    case 16: return project_t<T, D, 16>(p, Lq, Q, K, Wq, Wk, Qlr, Klr, st);
    case 32: return project_t<T, D, 32>(p, Lq, Q, K, Wq, Wk, Qlr, Klr, st);
    case 64: return project_t<T, D, 64>(p, Lq, Q, K, Wq, Wk, Qlr, Klr, st);
    default: return DSV_EUNSUPPORTED;
    }
}

dsv_status launch_project(const dsv_problem &p, int Lq, const void *Q, const void *K, const void *Wq, const void *Wk,
                          void *Qlr, void *Klr, hipStream_t st)
{
    if (p.dtype == DSV_BF16) {
        if (p.d == 64) return project_r<bf16_t, 64>(p, Lq, Q, K, Wq, Wk, Qlr, Klr, st);
        if (p.d == 128) return project_r<bf16_t, 128>(p, Lq, Q, K, Wq, Wk, Qlr, Klr, st);
    } else if (p.dtype == DSV_F32) {
        if (p.d == 64) return project_r<float, 64>(p, Lq, Q, K, Wq, Wk, Qlr, Klr, st);
        if (p.d == 128) return project_r<float, 128>(p, Lq, Q, K, Wq, Wk, Qlr, Klr, st);
    }
    return DSV_EUNSUPPORTED;
}

template <typename T, int R>
static dsv_status scores_rows_t(const dsv_problem &p, const void *Qlr, const void *Klr, int bh, const int32_t *rows,
                                int n_rows, float *scores, hipStream_t st)
{
    const T *Qb = (const T *)Qlr + (int64_t)bh * p.L * R;
    const T *Kb = (const T *)Klr + (int64_t)bh * p.L * R;
    dim3 grid((p.L + 31) / 32, (n_rows + 31) / 32);
    hipLaunchKernelGGL((scores_rows_kernel<T, R>), grid, dim3(64), 0, st, Qb, Kb, p.L, rows, n_rows, scores);
    DSV_LAUNCH_CHECK();
    return DSV_OK;
}

dsv_status launch_scores_rows(const dsv_problem &p, const void *Qlr, const void *Klr, int bh, const int32_t *rows,
                              int n_rows, float *scores, hipStream_t st)
{
#define DSV_CASE(TT, RR) return scores_rows_t<TT, RR>(p, Qlr, Klr, bh, rows, n_rows, scores, st)
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

static std::atomic<int> g_threshold_search{0};
int set_threshold_search(int mode) { return mode < 0 ? g_threshold_search.load() : g_threshold_search.exchange(mode); }

// Which head slots take the windowed search (mode: see set_threshold_search).
static bool slot_takes_window(const dsv_problem &p, int k, int mode)
{
    return mode != 1 && window_sample_keys(p.L, k, mode == 2) > 0;
}

template <typename T, int R>
static dsv_status select_t(const dsv_problem &p, int Lq, const HeadTable *tabs, int n_tabs, const void *Qlr, const void *Klr,
                           const SelectBuffers &b, hipStream_t st)
{
    const T *Ql = (const T *)Qlr;
    const T *Kl = (const T *)Klr;
    const int qtiles = (Lq + 31) / 32;
    const int asked = g_threshold_search.load();
    const int mode = b.win && b.todo ? asked : 1;
    if (asked != 1 && small_select(p, Lq)) {  // asked for the radix search: short sequences take it too
        {
            KernelSpan search(DSV_KERNEL_THRESHOLD, st), emission(DSV_KERNEL_EMIT, st);  // one kernel does both
            for (int t = 0; t < n_tabs; ++t) {
                const dsv_status rc = launch_select_small(p, Lq, tabs[t], Qlr, Klr, b, st);
                if (rc != DSV_OK) return rc;
            }
        }
        return launch_emit(p, Lq, tabs, n_tabs, Qlr, Klr, b, true, st);
    }
    {
        KernelSpan span(DSV_KERNEL_THRESHOLD, st);
        for (int t = 0; t < n_tabs; ++t) {
            HeadTable radix{}, window{};  // the table's slots by search method
            for (int s = 0; s < tabs[t].n; ++s) {
                HeadTable &dst = slot_takes_window(p, tabs[t].k[s], mode) ? window : radix;
                dst.bh[dst.n] = tabs[t].bh[s];
                dst.k[dst.n] = tabs[t].k[s];
                dst.off[dst.n] = tabs[t].off[s];
                ++dst.n;
            }
            const dim3 block(64 * kRadixWaves);
            if (radix.n) {
                dim3 grid(qtiles, radix.n);
                hipLaunchKernelGGL((radix_pass_kernel<T, R, 0>), grid, block, 0, st, Ql, Kl, Lq, p.L, radix, b.prefix, b.krem);
                hipLaunchKernelGGL((radix_pass_kernel<T, R, 1>), grid, block, 0, st, Ql, Kl, Lq, p.L, radix, b.prefix, b.krem);
                hipLaunchKernelGGL((radix_pass_kernel<T, R, 2>), grid, block, 0, st, Ql, Kl, Lq, p.L, radix, b.prefix, b.krem);
                hipLaunchKernelGGL((radix_pass_kernel<T, R, 3>), grid, block, 0, st, Ql, Kl, Lq, p.L, radix, b.prefix, b.krem);
                DSV_LAUNCH_CHECK();
            }
            if (window.n) {
                const dsv_status rc = launch_window_search(p, Lq, window, Qlr, Klr, b, st);
                if (rc != DSV_OK) return rc;
                // the tiles it listed (normally none): the grid is fixed, the blocks walk the list
                const dim3 grid((unsigned)std::min<int64_t>((int64_t)qtiles * window.n, 2048));
                hipLaunchKernelGGL((radix_pass_list_kernel<T, R, 0>), grid, block, 0, st, Ql, Kl, Lq, p.L, window, b.prefix, b.krem, (const int32_t *)b.todo, qtiles);
                hipLaunchKernelGGL((radix_pass_list_kernel<T, R, 1>), grid, block, 0, st, Ql, Kl, Lq, p.L, window, b.prefix, b.krem, (const int32_t *)b.todo, qtiles);
                hipLaunchKernelGGL((radix_pass_list_kernel<T, R, 2>), grid, block, 0, st, Ql, Kl, Lq, p.L, window, b.prefix, b.krem, (const int32_t *)b.todo, qtiles);
                hipLaunchKernelGGL((radix_pass_list_kernel<T, R, 3>), grid, block, 0, st, Ql, Kl, Lq, p.L, window, b.prefix, b.krem, (const int32_t *)b.todo, qtiles);
                DSV_LAUNCH_CHECK();
            }
        }
    }
    return launch_emit(p, Lq, tabs, n_tabs, Qlr, Klr, b, false, st);
}

dsv_status launch_select(const dsv_problem &p, int Lq, const HeadTable *tabs, int n_tabs, const void *Qlr, const void *Klr,
                         const SelectBuffers &b, hipStream_t st)
{
#define DSV_CASE(TT, RR) return select_t<TT, RR>(p, Lq, tabs, n_tabs, Qlr, Klr, b, st)
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
