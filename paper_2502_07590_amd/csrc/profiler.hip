// Sparsity profiler (paper Sec. "Sparsity Profiling"; definition of critical KV and head sparsity in Sec.
// "Exploiting Dynamic Sparsity"): on a sample of query rows, how many of the highest-probability keys hold
// `mass` (the paper: 90 %) of each query's softmax; the head's sparsity is the mean fraction of the other keys.
//
// One kernel, a block per 32 sampled queries of a head; the TRUE scores (contraction over all d channels, matrix cores) are
// recomputed in every sweep over the keys, never stored:
//   sweep 1   smallest and largest score and the sum of the exponentials of every query;
//   sweep 2   count and probability mass in 256 bins of equal width between the smallest and the largest score: the bin in
//             which the cumulative mass, from the top, reaches the target (equal widths in the VALUE: the bin holds L / 100
//             scores or so, where the leading eight bits of the float pattern name an octave and a sign);
//   sweep 3   the scores of that bin go to LDS, where one more histogram and a comparison of the few that share its bin find
//             the score that crosses; of keys with that very score, ceil(missing mass / their probability) are needed.
// A bin of more than kProfCap scores is divided again by 256 (a sweep each, twice at most); what is then still too many
// are ties or nearly so, and four sweeps over the order-preserving bit pattern of the score decide.
// Count and mass share one 64-bit integer counter, the mass in units of 2^-38: one LDS atomic per score instead of two,
// and integer ones -- LDS float additions retire about one wave per 44 clocks and CU --, and sums that do not depend on the
// order of arrival.  Every sweep requests a wave's next key tile before it scores this one; fragment loads bound the sweeps (32 rows
// x 32 bytes each).  L = 32768, four heads, 2048 rows each: 2660 us with float counters and five sweeps, 1176 with
// integer ones, 796 with three sweeps.
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

constexpr int kProfCap = 512;  // scores of a query's bin that fit LDS

template <int G> struct ProfShared {
    unsigned long long hist[256 * 32];   // [bin][query]
    unsigned long long part[G * 32];     // the search's partial sums
    float cand[32][kProfCap + 1];
    int ncand[32];
    float lo[32], hi[32], m2[32], rz[32];
    struct { uint32_t digit; int count; unsigned long long above; } found[32];
};

// The bin in which the cumulative mass, from the top, reaches `want`: above0 (count and mass) lies above all of them.  All
// threads of the block; thread t of a query (32 t + query) adds up C bins.
template <int G>
__device__ __forceinline__ void cross_bin(ProfShared<G> &sh, unsigned long long above0, unsigned long long want)
{
    constexpr int C = 256 / G;
    const int q = threadIdx.x & 31, t = threadIdx.x >> 5;
    __syncthreads();
    unsigned long long c[C], sum = 0ull;
#pragma unroll
    for (int i = 0; i < C; ++i) {
        c[i] = sh.hist[(t * C + i) * 32 + q];
        sum += c[i];                                   // counts and masses add up side by side
    }
    sh.part[t * 32 + q] = sum;
    __syncthreads();
    unsigned long long above = above0;
    for (int u = t + 1; u < G; ++u) above += sh.part[u * 32 + q];
    // the thread whose bins cross the target; the lowest one also where rounding left the total a hair short
    if (mass_of(above) < want && (mass_of(above + sum) >= want || t == 0)) {
        int digit = t * C;
        unsigned long long mine = c[0];
#pragma unroll
        for (int i = C - 1; i > 0; --i) {
            if (digit == t * C) {
                if (mass_of(above + c[i]) >= want) { digit = t * C + i; mine = c[i]; }
                else above += c[i];
            }
        }
        sh.found[q].digit = (uint32_t)digit;
        sh.found[q].count = count_of(mine);
        sh.found[q].above = above;
    }
    __syncthreads();
}

template <typename T, int D>
__global__ __launch_bounds__((64 * ProfWaves<T, D>::n)) void profile_kernel(const T *__restrict__ Q, const T *__restrict__ K,
                                                                  const int32_t *__restrict__ rows, int n, int L,
                                                                  float c2, float target, int32_t *__restrict__ counts)
{
    constexpr int WAVES = ProfWaves<T, D>::n, THREADS = 64 * WAVES, G = THREADS / 32;
    extern __shared__ __align__(16) unsigned char lds[];
    ProfShared<G> &sh = *reinterpret_cast<ProfShared<G> *>(lds);
    const int bh = blockIdx.y;
    const int q0 = blockIdx.x * 32;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nq = lane & 31, half = lane >> 5;      // in the sweeps; the searches below take query threadIdx.x % 32 too
    const T *Kh = K + (int64_t)bh * L * D;
    const Frag<T, D> qf = load_query_frag<T, D>(Q + (int64_t)bh * L * D, rows, q0, n, L, lane);
    const int ntiles = (L + 31) >> 5;
    // f(score of key j0 + tile_pos(v), whether there is such a key), 16 a tile
    auto sweep = [&](auto f) {
        Frag<T, D> kf_next = load_frag<T, D>(Kh, wave * 32, L, lane);
        for (int tile = wave; tile < ntiles; tile += WAVES) {
            const int left = L - tile * 32 - 4 * half;  // keys from this half's first on
            const Frag<T, D> kf = kf_next;
            kf_next = load_frag<T, D>(Kh, (tile + WAVES) * 32, L, lane);
            f(score_tile<T, D>(kf, qf), left);
        }
    };

    // ---- softmax normaliser (log2 domain: m2 = max_j s_ij c2, z = sum_j 2^(s_ij c2 - m2)) and range of the scores
    float lo = INFINITY, hi = -INFINITY, m = -INFINITY, z = 0.f;
    sweep([&](const floatx16_t &acc, int left) {
        float s[16], mt = -INFINITY;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const bool ok = tile_pos(v) < left;
            lo = fminf(lo, ok ? acc[v] : INFINITY);
            hi = fmaxf(hi, ok ? acc[v] : -INFINITY);
            s[v] = ok ? acc[v] * c2 : -INFINITY;
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
    });
    {
        float (*red)[4][64] = reinterpret_cast<float (*)[4][64]>(sh.hist);
        red[wave][0][lane] = m;
        red[wave][1][lane] = z;
        red[wave][2][lane] = lo;
        red[wave][3][lane] = hi;
        __syncthreads();
        if (threadIdx.x < 32) {
            float mm = -INFINITY, l = INFINITY, h = -INFINITY;
            for (int w = 0; w < WAVES; ++w)
                for (int x = 0; x < 64; x += 32) {
                    mm = fmaxf(mm, red[w][0][nq + x]);
                    l = fminf(l, red[w][2][nq + x]);
                    h = fmaxf(h, red[w][3][nq + x]);
                }
            float zz = 0.f;
            for (int w = 0; w < WAVES; ++w)
                for (int x = 0; x < 64; x += 32) {
                    const float mw = red[w][0][nq + x];
                    if (mw > -INFINITY) zz += red[w][1][nq + x] * __builtin_amdgcn_exp2f(mw - mm);
                }
            sh.m2[nq] = mm;
            sh.rz[nq] = 1.f / zz;
            sh.lo[nq] = l;
            sh.hi[nq] = h;
            sh.ncand[nq] = 0;
        }
        __syncthreads();
    }
    const float m2 = sh.m2[nq], rz = sh.rz[nq], least = sh.lo[nq], span = sh.hi[nq] - least;
    const float per = span > 0.f ? 0x1p32f / span : 0.f;
    // at least one unit: a target below 2^-38 is met by the most probable key (nothing would reach a target of zero)
    const unsigned long long want = max((unsigned long long)((double)target * 0x1p38), 1ull);
    auto mass = [&](float x) { return count_and_mass(__builtin_amdgcn_exp2f(x * c2 - m2) * rz); };
    // the score's place between the smallest and the largest, in 2^-32 (not a number: 0), or its order-preserving pattern
    auto code = [&](float x, bool pattern) {
        return pattern ? score_key(x) : (uint32_t)fminf(fmaxf((x - least) * per, 0.f), 0x1.fffffep31f);
    };
    auto clear = [&]() {
        for (int e = threadIdx.x; e < 256 * 32; e += THREADS) sh.hist[e] = 0ull;
        __syncthreads();
    };

    // ---- bins, by eight bits of the code at a time, until the crossing bin of every query fits LDS
    bool pattern = false;
    uint32_t pre = 0u;
    unsigned long long above = 0ull;
    int known = 0, count = 0;  // leading bits found; scores that share them
    for (;;) {
        clear();
        const int shift = 24 - known;
        sweep([&](const floatx16_t &acc, int left) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const uint32_t x = code(acc[v], pattern);
                if (tile_pos(v) < left && (known == 0 || (x ^ pre) >> (shift + 8) == 0u))
                    atomicAdd(&sh.hist[((x >> shift) & 255u) * 32 + nq], mass(acc[v]));
            }
        });
        cross_bin(sh, above, want);
        pre |= sh.found[nq].digit << shift;
        above = sh.found[nq].above;
        count = sh.found[nq].count;
        known += 8;
        if (!pattern && __all(count <= kProfCap)) break;  // the same 32 queries in every wave: the whole block
        if (known == 32) break;
        if (!pattern && known == 24) {
            pattern = true;
            pre = 0u;
            above = 0ull;
            known = 0;
        }
    }
    const bool mine = q0 + nq < n;
    int32_t *out = counts + (int64_t)bh * n + q0 + nq;
    // of `same` keys of score x, below `above`, as many as the missing mass takes
    auto write = [&](float x, unsigned long long over, int same) {
        const float p = __builtin_amdgcn_exp2f(x * c2 - m2) * rz;
        const float missing = (float)((double)(want > mass_of(over) ? want - mass_of(over) : 0ull) * 0x1p-38);
        const int need = p > 0.f ? (int)fminf(ceilf(missing / p), (float)same) : same;
        // the total may fall short of a target next to 1: then every key counts, and no more
        *out = min(count_of(over) + min(max(need, 1), same), L);
    };
    if (pattern) {  // every key of the bin has the score that `pre` decodes to
        if (threadIdx.x < 32 && mine) write(key_score(pre), above, max(count, 1));
        return;
    }
    // ---- the crossing bin's scores, in LDS
    clear();
    sweep([&](const floatx16_t &acc, int left) {
#pragma unroll
        for (int v = 0; v < 16; ++v)
            if (tile_pos(v) < left && (code(acc[v], false) ^ pre) >> (32 - known) == 0u) {
                const int at = atomicAdd(&sh.ncand[nq], 1);
                if (at < kProfCap) sh.cand[nq][at] = acc[v];
            }
    });
    __syncthreads();
    const int t = threadIdx.x >> 5, c = min(sh.ncand[nq], kProfCap);
    const int shift = 24 - known;
    auto bin = [&](float x) { return (code(x, false) >> shift) & 255u; };
    for (int i = t; i < c; i += G) atomicAdd(&sh.hist[bin(sh.cand[nq][i]) * 32 + nq], mass(sh.cand[nq][i]));
    cross_bin(sh, above, want);
    above = sh.found[nq].above;
    const uint32_t digit = sh.found[nq].digit;
    for (int i = t; i < c; i += G) {
        const float x = sh.cand[nq][i];
        if (bin(x) != digit) continue;
        const uint32_t key = score_key(x);
        unsigned long long over = above, with = 0ull;
        bool lowest = true;
        for (int j = 0; j < c; ++j) {
            const float y = sh.cand[nq][j];
            if (bin(y) != digit) continue;
            const uint32_t other = score_key(y);
            if (other > key) over += mass(y);
            else if (other == key) with += mass(y);
            else lowest = false;
        }
        // every thread that finds the crossing score writes the same count
        if (mine && mass_of(over) < want && (mass_of(over + with) >= want || lowest)) write(x, over, count_of(with));
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
                            int32_t *counts, float *sparsity, float *ema, float alpha, hipStream_t st)
{
    const int nbh = p.B * p.H;
    constexpr int threads = 64 * ProfWaves<T, D>::n;
    constexpr size_t lds = sizeof(ProfShared<threads / 32>);  // above the default of 64 KB
    static_assert(lds <= 160 * 1024, "LDS of a CU");
    DSV_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void *>(&profile_kernel<T, D>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL((profile_kernel<T, D>), dim3((n + 31) / 32, nbh), dim3(threads), lds, st, (const T *)Q, (const T *)K, rows, n, p.L,
                       p.scale * 1.4426950408889634f, mass, counts);
    DSV_LAUNCH_CHECK();
    hipLaunchKernelGGL(profile_finish_kernel, dim3(nbh), dim3(256), 0, st, counts, n, p.L, sparsity, ema, alpha);
    DSV_LAUNCH_CHECK();
    return DSV_OK;
}

dsv_status launch_profile_sparsity(const dsv_problem &p, const void *Q, const void *K, const int32_t *rows, int n,
                                   float mass, int32_t *counts, float *sparsity, float *ema, float alpha, hipStream_t st)
{
    if (p.dtype == DSV_BF16) {
        if (p.d == 64) return profile_t<bf16_t, 64>(p, Q, K, rows, n, mass, counts, sparsity, ema, alpha, st);
        if (p.d == 128) return profile_t<bf16_t, 128>(p, Q, K, rows, n, mass, counts, sparsity, ema, alpha, st);
    } else if (p.dtype == DSV_F32) {
        if (p.d == 64) return profile_t<float, 64>(p, Q, K, rows, n, mass, counts, sparsity, ema, alpha, st);
        if (p.d == 128) return profile_t<float, 128>(p, Q, K, rows, n, mass, counts, sparsity, ema, alpha, st);
    }
    return DSV_EUNSUPPORTED;
}

}  // namespace dsv
