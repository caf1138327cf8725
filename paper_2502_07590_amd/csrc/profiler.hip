// Sparsity profiler (paper Sec. "Sparsity Profiling"; definition of critical KV and head sparsity in Sec.
// "Exploiting Dynamic Sparsity"): on a sample of query rows, how many of the highest-probability keys hold
// `mass` (the paper: 90 %) of each query's softmax; the head's sparsity is the mean fraction of the other keys.
//
// Same machinery as the selection of stage 1, on the TRUE scores (contraction over all d channels, matrix
// cores) and with probability MASS in place of counts: a first sweep gives every sampled query its softmax
// normaliser (running maximum and sum); four sweeps then find, digit by digit on the order-preserving bit
// pattern of the score, the score at which the cumulative probability -- taken from the top -- reaches the
// target, histogramming count and mass per digit in LDS; the last bucket holds keys of one score, of which
// ceil(missing mass / their probability) are needed.  Scores are recomputed in every sweep, never stored.
// Count and mass share one 64-bit integer counter, the mass in units of 2^-38: one LDS atomic per score instead of two,
// and integer ones -- LDS float additions retire about one wave per 44 clocks and CU, which was half of the whole call
// (L = 32768, four heads, 2048 rows each: the first digit's sweep 1364 us, 270 now; the call 2660 -> 1230) --, and sums that
// do not depend on the order of arrival.  Every sweep requests a wave's next key tile before it scores this one.
#include <algorithm>

#include "stage1_core.h"

namespace dsv {

// Waves per block: 16 where the registers allow it (the fragments of two key tiles and a query tile beside the scores).
template <typename T, int D> struct ProfWaves { static constexpr int n = sizeof(T) == 2 ? 16 : 8; };

constexpr int kMassBits = 39;  // low bits of a counter: mass in units of 2^-38 (at most 1 + rounding); above them the count
                               // (L < 2^25 wherever a head's matrix is below 4 GB)
__device__ __forceinline__ unsigned long long count_and_mass(float p)
{
    const float x = p * 0x1p31f;           // p <= 1 up to rounding
    const uint32_t hi = (uint32_t)x;
    const uint32_t lo = (uint32_t)fmaf(x - (float)hi, 128.f, 0.5f);
    return (1ull << kMassBits) + ((unsigned long long)hi << 7) + lo;
}
__device__ __forceinline__ unsigned long long mass_of(unsigned long long c) { return c & ((1ull << kMassBits) - 1ull); }
__device__ __forceinline__ int count_of(unsigned long long c) { return (int)(c >> kMassBits); }

template <typename T, int D>
__device__ __forceinline__ Frag<T, D> load_query_frag(const T *__restrict__ Qh, const int32_t *__restrict__ rows, int q0,
                                                      int n, int L, int lane)
{
    const int i = min(q0 + (lane & 31), n - 1);
    return load_frag_row<T, D>(Qh, (int64_t)min(max(rows[i], 0), L - 1), lane);
}

// ---- sweep 0: softmax normaliser of every sampled query -------------------------------------------------
// stat[bh, i] = {m2, 1 / z}: m2 = max_j (s_ij * c2) (log2 domain, c2 = scale * log2 e), z = sum_j 2^(s_ij c2 - m2).
template <typename T, int D>
__global__ __launch_bounds__((64 * ProfWaves<T, D>::n)) void profile_norm_kernel(const T *__restrict__ Q, const T *__restrict__ K,
                                                                       const int32_t *__restrict__ rows, int n, int L,
                                                                       float c2, float2 *__restrict__ stat)
{
    constexpr int kProfWaves = ProfWaves<T, D>::n;
    __shared__ float red_m[kProfWaves][64], red_z[kProfWaves][64];
    const int bh = blockIdx.y;
    const int q0 = blockIdx.x * 32;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int half = lane >> 5;
    const T *Qh = Q + (int64_t)bh * L * D;
    const T *Kh = K + (int64_t)bh * L * D;
    const Frag<T, D> qf = load_query_frag<T, D>(Qh, rows, q0, n, L, lane);
    const int ntiles = (L + 31) >> 5;
    float m = -INFINITY, z = 0.f;
    Frag<T, D> kf_next = load_frag<T, D>(Kh, wave * 32, L, lane);
    for (int tile = wave; tile < ntiles; tile += kProfWaves) {
        const int j0 = tile * 32;
        const Frag<T, D> kf = kf_next;
        kf_next = load_frag<T, D>(Kh, (tile + kProfWaves) * 32, L, lane);
        const floatx16_t acc = score_tile<T, D>(kf, qf);
        float s[16], mt = -INFINITY;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            s[v] = j0 + tile_pos(v) + 4 * half < L ? acc[v] * c2 : -INFINITY;
            mt = fmaxf(mt, s[v]);
        }
        const float mn = fmaxf(m, mt);
        if (mn > -INFINITY) {  // a lane whose 16 keys all lie past the end has seen nothing yet
            float add = 0.f;
#pragma unroll
            for (int v = 0; v < 16; ++v) add += __builtin_amdgcn_exp2f(s[v] - mn);
            z = z * __builtin_amdgcn_exp2f(m - mn) + add;   // m = -inf on the first tile: factor 0
            m = mn;
        }
    }
    red_m[wave][lane] = m;
    red_z[wave][lane] = z;
    __syncthreads();
    if (threadIdx.x < 32 && q0 + (int)threadIdx.x < n) {
        float mm = -INFINITY;
        for (int w = 0; w < kProfWaves; ++w) mm = fmaxf(mm, fmaxf(red_m[w][threadIdx.x], red_m[w][threadIdx.x + 32]));
        float zz = 0.f;
        for (int w = 0; w < kProfWaves; ++w)
            for (int h = 0; h < 2; ++h) {
                const float mw = red_m[w][threadIdx.x + 32 * h];
                if (mw > -INFINITY) zz += red_z[w][threadIdx.x + 32 * h] * __builtin_amdgcn_exp2f(mw - mm);
            }
        stat[(int64_t)bh * padded_len(n) + q0 + threadIdx.x] = make_float2(mm, 1.f / zz);
    }
}

// ---- sweeps 1-4: one digit of the threshold score ---------------------------------------------------------
// Per sampled query: prefix (digits found so far), mass_above (units of 2^-38) / count_above (probability and number of keys
// in the buckets above the prefix's).  PASS 3 also writes the count of critical keys.
template <typename T, int D, int PASS>
__global__ __launch_bounds__((64 * ProfWaves<T, D>::n)) void profile_pass_kernel(const T *__restrict__ Q, const T *__restrict__ K,
                                                                       const int32_t *__restrict__ rows, int n, int L,
                                                                       float c2, float target,
                                                                       const float2 *__restrict__ stat,
                                                                       uint32_t *__restrict__ prefix,
                                                                       unsigned long long *__restrict__ mass_above,
                                                                       int32_t *__restrict__ count_above,
                                                                       int32_t *__restrict__ counts)
{
    constexpr int SHIFT = 24 - 8 * PASS;
    constexpr int kProfWaves = ProfWaves<T, D>::n, THREADS = 64 * kProfWaves;
    constexpr int G = THREADS / 32, C = 256 / G;       // threads per query in the search, buckets of each
    extern __shared__ unsigned long long hist[];       // [256 digits][32 queries], then the search's scratch [G][32]
    unsigned long long *part = hist + 256 * 32;
    const int bh = blockIdx.y;
    const int q0 = blockIdx.x * 32;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nq = lane & 31, half = lane >> 5;
    const T *Qh = Q + (int64_t)bh * L * D;
    const T *Kh = K + (int64_t)bh * L * D;
    for (int e = threadIdx.x; e < 256 * 32; e += THREADS) hist[e] = 0ull;
    __syncthreads();
    const int64_t g = (int64_t)bh * padded_len(n) + min(q0 + nq, n - 1);
    const float2 st = stat[g];
    uint32_t pre = 0;
    if constexpr (PASS > 0) pre = prefix[g];
    const Frag<T, D> qf = load_query_frag<T, D>(Qh, rows, q0, n, L, lane);
    const int ntiles = (L + 31) >> 5;
    Frag<T, D> kf_next = load_frag<T, D>(Kh, wave * 32, L, lane);
    for (int tile = wave; tile < ntiles; tile += kProfWaves) {
        const int left = L - tile * 32 - 4 * half;     // keys from this half's first on
        const Frag<T, D> kf = kf_next;
        kf_next = load_frag<T, D>(Kh, (tile + kProfWaves) * 32, L, lane);
        const floatx16_t acc = score_tile<T, D>(kf, qf);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const uint32_t key = score_key(acc[v]);
            bool ok = tile_pos(v) < left;
            if constexpr (PASS > 0) ok = ok && ((key >> (SHIFT + 8)) == (pre >> (SHIFT + 8)));
            if (ok) atomicAdd(&hist[((key >> SHIFT) & 255u) * 32 + nq], count_and_mass(__builtin_amdgcn_exp2f(acc[v] * c2 - st.x) * st.y));
        }
    }
    __syncthreads();
    // the bucket in which the cumulative mass, from the top, reaches the target; thread t of a query adds up C buckets
    const unsigned long long want = (unsigned long long)((double)target * 0x1p38);
    const unsigned long long above0 = PASS == 0 ? 0ull : mass_above[g];
    const int t = threadIdx.x >> 5;
    unsigned long long c[C], sum = 0ull;
#pragma unroll
    for (int i = 0; i < C; ++i) {
        c[i] = hist[(t * C + i) * 32 + nq];
        sum += c[i];                                   // counts and masses add up side by side
    }
    part[t * 32 + nq] = sum;
    __syncthreads();
    unsigned long long above = 0ull;
    for (int u = t + 1; u < G; ++u) above += part[u * 32 + nq];
    // the thread whose buckets cross the target; the lowest one also where rounding left the total a hair short
    const bool reached = above0 + mass_of(above) + mass_of(sum) >= want, before = above0 + mass_of(above) >= want;
    if (!before && (reached || t == 0) && q0 + nq < n) {
        int digit = t * C;
#pragma unroll
        for (int i = C - 1; i > 0; --i) {
            if (digit == t * C) {
                if (above0 + mass_of(above + c[i]) >= want) digit = t * C + i;
                else above += c[i];
            }
        }
        const int64_t gq = (int64_t)bh * padded_len(n) + q0 + nq;
        const unsigned long long ma = above0 + mass_of(above);
        const int ca = (PASS == 0 ? 0 : count_above[gq]) + count_of(above);
        const uint32_t full = pre | ((uint32_t)digit << SHIFT);
        prefix[gq] = full;
        mass_above[gq] = ma;
        count_above[gq] = ca;
        if constexpr (PASS == 3) {
            // every key of this bucket has the score `full` decodes to, hence the same probability
            const int cb = max(count_of(hist[digit * 32 + nq]), 1);
            const float p = __builtin_amdgcn_exp2f(key_score(full) * c2 - st.x) * st.y;
            const float missing = (float)((double)(want > ma ? want - ma : 0ull) * 0x1p-38);
            const int need = p > 0.f ? (int)fminf(ceilf(missing / p), (float)cb) : cb;
            counts[(int64_t)bh * n + q0 + nq] = ca + min(max(need, 1), cb);
        }
    }
}

// sparsity[bh] = mean_i (1 - counts_i / L); ema[bh] = alpha * sparsity + (1 - alpha) * ema[bh] when ema is given.
__global__ __launch_bounds__(256) void profile_finish_kernel(const int32_t *__restrict__ counts, int n, int L,
                                                             float *__restrict__ sparsity, float *__restrict__ ema,
                                                             float alpha)
{
    __shared__ double part[256];
    const int bh = blockIdx.x;
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += 256) s += 1.0 - (double)counts[(int64_t)bh * n + i] / (double)L;
    part[threadIdx.x] = s;
    __syncthreads();
    for (int step = 128; step; step >>= 1) {
        if ((int)threadIdx.x < step) part[threadIdx.x] += part[threadIdx.x + step];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const float p = (float)(part[0] / (double)n);
        sparsity[bh] = p;
        if (ema) ema[bh] = alpha * p + (1.f - alpha) * ema[bh];
    }
}

// ------------------------------------------------------------------------------------ host
template <typename T, int D>
static dsv_status profile_t(const dsv_problem &p, const void *Q, const void *K, const int32_t *rows, int n, float mass,
                            int32_t *counts, float *sparsity, float *ema, float alpha, char *ws, hipStream_t st)
{
    const int nbh = p.B * p.H;
    const size_t np_ = (size_t)nbh * padded_len(n);
    float2 *stat = reinterpret_cast<float2 *>(ws);
    uint32_t *prefix = reinterpret_cast<uint32_t *>(ws + align_up(np_ * 8, 256));
    unsigned long long *mabove = reinterpret_cast<unsigned long long *>(reinterpret_cast<char *>(prefix) + align_up(np_ * 4, 256));
    int32_t *cabove = reinterpret_cast<int32_t *>(reinterpret_cast<char *>(mabove) + align_up(np_ * 8, 256));
    const float c2 = p.scale * 1.4426950408889634f;
    constexpr int threads = 64 * ProfWaves<T, D>::n;
    const size_t lds = (256 * 32 + threads / 32 * 32) * 8;  // counters and the search's scratch: above the default of 64 KB
    const void *kernels[] = {reinterpret_cast<const void *>(&profile_pass_kernel<T, D, 0>), reinterpret_cast<const void *>(&profile_pass_kernel<T, D, 1>),
                             reinterpret_cast<const void *>(&profile_pass_kernel<T, D, 2>), reinterpret_cast<const void *>(&profile_pass_kernel<T, D, 3>)};
    for (const void *k : kernels) DSV_HIP_CHECK(hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    dim3 grid((n + 31) / 32, nbh), block(threads);
    hipLaunchKernelGGL((profile_norm_kernel<T, D>), grid, block, 0, st, (const T *)Q, (const T *)K, rows, n, p.L, c2, stat);
    DSV_LAUNCH_CHECK();
    hipLaunchKernelGGL((profile_pass_kernel<T, D, 0>), grid, block, lds, st, (const T *)Q, (const T *)K, rows, n, p.L, c2, mass, stat, prefix, mabove, cabove, counts);
    hipLaunchKernelGGL((profile_pass_kernel<T, D, 1>), grid, block, lds, st, (const T *)Q, (const T *)K, rows, n, p.L, c2, mass, stat, prefix, mabove, cabove, counts);
    hipLaunchKernelGGL((profile_pass_kernel<T, D, 2>), grid, block, lds, st, (const T *)Q, (const T *)K, rows, n, p.L, c2, mass, stat, prefix, mabove, cabove, counts);
    hipLaunchKernelGGL((profile_pass_kernel<T, D, 3>), grid, block, lds, st, (const T *)Q, (const T *)K, rows, n, p.L, c2, mass, stat, prefix, mabove, cabove, counts);
    DSV_LAUNCH_CHECK();
    hipLaunchKernelGGL(profile_finish_kernel, dim3(nbh), dim3(256), 0, st, counts, n, p.L, sparsity, ema, alpha);
    DSV_LAUNCH_CHECK();
    return DSV_OK;
}

size_t profile_workspace_bytes(const dsv_problem &p, int n)
{
    const size_t np_ = (size_t)p.B * p.H * padded_len(n);
    return 2 * align_up(np_ * 8, 256) + 2 * align_up(np_ * 4, 256);
}

dsv_status launch_profile_sparsity(const dsv_problem &p, const void *Q, const void *K, const int32_t *rows, int n,
                                   float mass, int32_t *counts, float *sparsity, float *ema, float alpha, char *ws,
                                   hipStream_t st)
{
    if (p.dtype == DSV_BF16) {
        if (p.d == 64) return profile_t<bf16_t, 64>(p, Q, K, rows, n, mass, counts, sparsity, ema, alpha, ws, st);
        if (p.d == 128) return profile_t<bf16_t, 128>(p, Q, K, rows, n, mass, counts, sparsity, ema, alpha, ws, st);
    } else if (p.dtype == DSV_F32) {
        if (p.d == 64) return profile_t<float, 64>(p, Q, K, rows, n, mass, counts, sparsity, ema, alpha, ws, st);
        if (p.d == 128) return profile_t<float, 128>(p, Q, K, rows, n, mass, counts, sparsity, ema, alpha, ws, st);
    }
    return DSV_EUNSUPPORTED;
}

}  // namespace dsv
