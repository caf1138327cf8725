// Score tiles of stage 1 (paper Sec. "Critical KV Estimation with Kernel Fusion"): one 32x32 block of
// the low-rank product Q_lr K_lr^T per MFMA (bf16: v_mfma_f32_32x32x16_bf16, one per 16 ranks; fp32:
// v_mfma_f32_32x32x2_f32, one per 2 ranks), recomputed wherever it is needed -- never stored.
//
// Every kernel of stage 1 forms a score through score_tile() below from the same two fragments, so a
// given (query, key) pair has the same fp32 bits in every pass.  That also holds when the two
// operands trade places (rows <-> columns): the matrix cores form each output element from the same
// products in the same order either way, which the key-major emission relies on and the parity tests
// check (the transposed index must equal the transpose of the index, bit for bit).
#pragma once

#include "common.h"

namespace dsv {

// MFMA operand fragment of 32 rows of a [*, R] low-rank matrix.  Lane l holds row (l % 32) and the
// K-slice selected by (l / 32).  With fragments `rows` (A operand) and `cols` (B operand),
// acc[v] of lane l is the score of column (l % 32) against row 8*(v/4) + 4*(l/32) + (v%4).
template <typename T, int R> struct Frag;
template <int R> struct Frag<bf16_t, R> { bf16x8_t v[R / 16]; };
template <int R> struct Frag<float, R> { float v[R / 2]; };

// The lane's share of the row at p.  fp32: a lane needs every other channel, but reading them one by one is an access to the vector cache per
// lane and channel, four times what the products of a sweep take (L = 16384, four heads, r = 16, selection and transpose: 4160 -> 2140 us); so each
// half reads half of the row in 16-byte pieces, and the halves exchange.
template <typename T, int R> __device__ __forceinline__ Frag<T, R> load_frag_at(const T *__restrict__ p, int half)
{
    Frag<T, R> f;
    if constexpr (sizeof(T) == 2) {
#pragma unroll
        for (int m = 0; m < R / 16; ++m) f.v[m] = *reinterpret_cast<const bf16x8_t *>(p + m * 16 + half * 8);
    } else {
#pragma unroll
        for (int i = 0; i < R / 8; ++i) {
            const uint4 x = *reinterpret_cast<const uint4 *>(p + half * (R / 2) + 4 * i);
            // (lower half's register, its partner's): even channels stay below, odd ones above
            const auto a = __builtin_amdgcn_permlane32_swap(x.x, x.y, false, false), b = __builtin_amdgcn_permlane32_swap(x.z, x.w, false, false);
            f.v[2 * i] = __uint_as_float(a[0]);
            f.v[2 * i + 1] = __uint_as_float(b[0]);
            f.v[R / 4 + 2 * i] = __uint_as_float(a[1]);
            f.v[R / 4 + 2 * i + 1] = __uint_as_float(b[1]);
        }
    }
    return f;
}

template <typename T, int R>
__device__ __forceinline__ Frag<T, R> load_frag_row(const T *__restrict__ base, int64_t row, int lane)
{
    return load_frag_at<T, R>(base + row * R, lane >> 5);
}

// Rows row0 .. row0+31 of the matrix; rows past the end are clamped (callers mask their results).
template <typename T, int R>
__device__ __forceinline__ Frag<T, R> load_frag(const T *__restrict__ base, int row0, int L, int lane)
{
    return load_frag_row<T, R>(base, min(row0 + (lane & 31), L - 1), lane);
}

// The rows of a matrix as a sweep walks them, 32 at a time.  Row operands come in the order that gives a lane 16 rows side by side
// (accumulator v of half h: row 16 h + v of the tile): its 16 predicates are a halfword then, in order.  Two vector instructions
// per tile for the address (a head's matrix has less than 2^32 bytes); rows past the end repeat the last one.
template <typename T, int R> struct TileWalk {
    uint32_t at, last;
    __device__ __forceinline__ TileWalk(int L, int lane)
    {
        const int r = lane & 31;
        at = (uint32_t)(16 * ((r >> 2) & 1) + 4 * (r >> 3) + (r & 3)) * (R * (uint32_t)sizeof(T));
        last = (uint32_t)(L - 1) * (R * (uint32_t)sizeof(T));
    }
    __device__ __forceinline__ Frag<T, R> load(const T *__restrict__ base, int tile, int half) const
    {
        return load_frag_at<T, R>(reinterpret_cast<const T *>(reinterpret_cast<const char *>(base) +
                                                              min(at + (uint32_t)tile * (32u * R * (uint32_t)sizeof(T)), last)), half);
    }
};

template <typename T, int R>
__device__ __forceinline__ floatx16_t score_tile(const Frag<T, R> &rows, const Frag<T, R> &cols)
{
    floatx16_t acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
    if constexpr (sizeof(T) == 2) {
#pragma unroll
        for (int m = 0; m < R / 16; ++m)
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rows.v[m], cols.v[m], acc, 0, 0, 0);
    } else {
#pragma unroll
        for (int m = 0; m < R / 2; ++m)
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(rows.v[m], cols.v[m], acc, 0, 0, 0);
    }
    return acc;
}

// Row inside a 32-row tile of accumulator v for a lane in half 0 (half 1 adds 4).
__device__ __forceinline__ constexpr int tile_pos(int v) { return 8 * (v / 4) + (v % 4); }

// Order-preserving map fp32 -> uint32 (larger float <=> larger key), and its inverse.
__device__ __forceinline__ uint32_t score_key(float s)
{
    uint32_t u = __float_as_uint(s);
    return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}
__device__ __forceinline__ float key_score(uint32_t key)
{
    return __uint_as_float((key & 0x80000000u) ? (key ^ 0x80000000u) : ~key);
}

// 16 predicate bits of a lane, bit tile_pos(v) <- pred(v); the caller shifts by 4*half and merges.
#define DSV_MASK16(m, pred_expr)                                   \
    do {                                                           \
        (m) = 0u;                                                  \
        _Pragma("unroll") for (int v = 0; v < 16; ++v)             \
            (m) |= (uint32_t)(pred_expr) << tile_pos(v);           \
    } while (0)

// Same, for predicates of the form "d(v) < 0" with d a float expression (NaN-free): the sign bits
// are shifted into a register with one v_alignbit each (no compare, no condition-code traffic),
// then put in tile order: bit-reverse, and spread the four nibbles to the low nibbles of four bytes.
#define DSV_SIGNMASK16(m, d_expr)                                                          \
    do {                                                                                   \
        uint32_t acc_ = 0u;                                                                \
        _Pragma("unroll") for (int v = 0; v < 16; ++v)                                     \
            acc_ = __builtin_amdgcn_alignbit(acc_, __float_as_uint(d_expr), 31);           \
        acc_ = __builtin_bitreverse32(acc_) >> 16; /* bit v = sign of d(v) */              \
        acc_ = (acc_ | (acc_ << 8)) & 0x00FF00FFu;                                         \
        (m) = (acc_ | (acc_ << 4)) & 0x0F0F0F0Fu;  /* bit tile_pos(v) */                   \
    } while (0)

// Bits v of a lane for rows in the order of TileWalk: predicates, and signs (above).
#define DSV_PRED16(m, pred_expr)                                                             \
    do {                                                                                   \
        (m) = 0u;                                                                          \
        _Pragma("unroll") for (int v = 0; v < 16; ++v) (m) |= (uint32_t)(pred_expr) << v;  \
    } while (0)
#define DSV_SIGNS16(m, d_expr)                                                             \
    do {                                                                                   \
        uint32_t acc_ = 0u;                                                                \
        _Pragma("unroll") for (int v = 15; v >= 0; --v)                                    \
            acc_ = __builtin_amdgcn_alignbit(acc_, __float_as_uint(d_expr), 31);           \
        (m) = acc_;                                                                        \
    } while (0)

__device__ __forceinline__ uint32_t merge_halves(uint32_t m, int half)
{
    m <<= 4 * half;
    return m | (uint32_t)__shfl_xor((int)m, 32);
}

// Waves per block of the threshold-search kernels (one block = 32 queries, the waves stride over the key
// tiles); their 32 KB histogram allows 4 blocks per CU.
#ifndef DSV_RADIX_WAVES
#define DSV_RADIX_WAVES 8
#endif
constexpr int kRadixWaves = DSV_RADIX_WAVES;

// The bucket of an LDS histogram that holds each query's want-th largest count.  hist: [256 buckets][32 queries]; bucket_of
// maps key order (0 = smallest) to buckets.  All THREADS threads of the block call it, thread t with the `want` of query
// t % 32; each sums 256 / (THREADS / 32) buckets of its query, so that the search is a few dozen LDS reads deep instead
// of 256 (the four radix passes over two heads of L = 20280, r = 32: 355 -> 301 us; the sample of four heads: 236 -> 157 us).  digit: in key order, -1 when the query's counts do not reach want;
// above: counts in higher buckets; count: in the bucket itself.
struct Bucket {
    int digit, above, count;
};
template <int THREADS> struct BucketScratch {
    int part[THREADS / 32][32];
    Bucket found[32];
};
template <int THREADS, typename F>
__device__ __forceinline__ Bucket find_bucket(const uint32_t *hist, BucketScratch<THREADS> &sh, F bucket_of, int want)
{
    constexpr int G = THREADS / 32, C = 256 / G;
    const int q = threadIdx.x & 31, t = threadIdx.x >> 5;
    int c[C], sum = 0;
#pragma unroll
    for (int i = 0; i < C; ++i) {
        c[i] = (int)hist[32 * bucket_of(t * C + i) + q];
        sum += c[i];
    }
    sh.part[t][q] = sum;
    if (t == 0) sh.found[q] = Bucket{-1, 0, 0};
    __syncthreads();
    int above = 0;
#pragma unroll
    for (int u = 1; u < G; ++u) above += u > t ? sh.part[u][q] : 0;
    if (above < want && want <= above + sum) {
        int digit = -1, count = 0;
#pragma unroll
        for (int i = C - 1; i >= 0; --i) {
            if (digit < 0) {
                if (above + c[i] >= want) { digit = t * C + i; count = c[i]; }
                else above += c[i];
            }
        }
        sh.found[q] = Bucket{digit, above, count};
    }
    __syncthreads();
    const Bucket found = sh.found[q];
    __syncthreads();  // the scratch and the histogram are free again
    return found;
}

// Per-query selection state (threshold, tie budget, jcut) is stored [B*H, padded_len(L)]: rows padded
// to whole 32-query tiles, so that a tile's 32 values can be fetched with aligned vector loads.
__host__ __device__ __forceinline__ constexpr int padded_len(int L) { return (L + 31) & ~31; }

// jcut value of a query all of whose threshold-equal keys are selected: "score >= tau" decides.
constexpr int32_t kAllTies = 0x7FFFFFFF;

// Block-wide emission: a half-wave per query, its lanes a word (32 keys) each, in ascending order.  gt: the lane's keys above
// the threshold (all_simple: at or above it); eq: its keys equal to it, of which the query takes the lowest `room`.
struct RowOut {
    int at, room, last_tie;  // entries written, ties still to take, highest tie taken (the same in the half-wave)
};
__device__ __forceinline__ void emit_row_words(RowOut &ro, uint32_t gt, uint32_t eq, bool all_simple, int tile, int half, bool live,
                                               int32_t *__restrict__ row, int k)
{
    uint32_t m = gt;
    if (!all_simple) {
        const int c = __popc(eq);
        const int incl = half_scan(c);
        const int take = max(0, min(c, ro.room - (incl - c)));
        while (__popc(eq) > take) eq &= ~(0x80000000u >> __clz(eq));
        int tie = eq ? tile * 32 + 31 - __clz(eq) : -1;
        for (int o = 16; o; o >>= 1) tie = max(tie, __shfl_xor(tie, o));
        ro.last_tie = max(ro.last_tie, tie);
        ro.room = max(0, ro.room - __shfl(incl, 31 + 32 * half));
        m |= eq;
    }
    const int c = __popc(m);
    const int incl = half_scan(c);
    const int pos = ro.at + incl - c;
    ro.at += __shfl(incl, 31 + 32 * half);
    if (live) {
        if (pos + c > k) {  // a correct threshold fills the row exactly
            const int fits = max(k - pos, 0);
            while (__popc(m) > fits) m &= ~(0x80000000u >> __clz(m));
        }
        int32_t *dst = row + pos;
        while (m) {
            *dst++ = tile * 32 + (__ffs(m) - 1);
            m &= m - 1;
        }
    }
}

// The two words of a 32 x 32 score tile for this lane's query (both lanes of a query get them).
__device__ __forceinline__ void threshold_words(const floatx16_t &acc, float tau, bool all_simple, uint32_t valid, int half,
                                                uint32_t &gt, uint32_t &eq)
{
    eq = 0u;
    if (all_simple) {
        DSV_SIGNMASK16(gt, acc[v] - tau);
        gt = ~merge_halves(gt, half) & valid;
    } else {
        DSV_MASK16(gt, acc[v] > tau);
        DSV_MASK16(eq, acc[v] == tau);
        gt = merge_halves(gt, half) & valid;
        eq = merge_halves(eq, half) & valid;
    }
}

}  // namespace dsv
