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
// order of arrival.
// Sweeps were bound by accesses to the vector cache, one per 16 bytes where lanes read an operand's rows: key tiles go through LDS now, whole
// lines at a time, and the sweeps are vector work (the exponentials and a bin per score) and matrix work again.  L = 32768, four heads, 2048
// rows each, bf16: 800 -> 515 us; two heads of 20280, 1000 rows: 490 -> 315; fp32, d = 128, two heads of 10000, 700 rows (4-byte loads of 32 rows
// before, 16-byte ones of 16 rows now): 1750 -> 700.  A count differs from that in 64 bits in 25 of 82000 rows (37 before the sum of
// exponentials kept what its additions lose), by one.
#include <algorithm>
#include <type_traits>

#include "grid.h"
#include "stage1_core.h"

namespace dsv {

// Waves per block (a block per CU): as many as LDS holds key tiles for, and the registers the operands of a tile.
constexpr int kProfWaves = 8;
template <typename T, int D> constexpr int kProfWavesMost = D * sizeof(T) <= 128 ? 16 : kProfWaves;

constexpr int kMassBits = 39;  // low bits of a counter: mass in units of 2^-38 (at most 1 + rounding); above them the count
                               // (L < 2^25 wherever a head's matrix is below 4 GB)
// p38: the probability times 2^38.  Added to 2^52 in 64 bits it is rounded to a whole number in the low bits; what is left of the exponent
// makes room for the count.
__device__ __forceinline__ unsigned long long count_and_mass(float p38)
{
    const unsigned long long x = __builtin_bit_cast(unsigned long long, (double)p38 + 0x1p52);
    return x + ((1ull << kMassBits) - (0x433ull << 52));
}
__device__ __forceinline__ unsigned long long mass_of(unsigned long long c) { return c & ((1ull << kMassBits) - 1ull); }
__device__ __forceinline__ int count_of(unsigned long long c) { return (int)(c >> kMassBits); }

// Operand of 16 rows of a [*, D] matrix for products of 16 x 16: lane l holds row l % 16, of every 64 bytes of it the l / 16-th quarter.
// Which channels a lane's piece holds is free as long as both operands agree.
template <typename T, int D> struct Rows16 {
    static constexpr int N = D * (int)sizeof(T) / 64;
    uint4 v[N];
};
template <typename T, int D>
__device__ __forceinline__ Rows16<T, D> load_rows16(const T *__restrict__ base, int row, int lane)
{
    Rows16<T, D> f;
    const char *p = reinterpret_cast<const char *>(base) + (uint32_t)row * (D * (uint32_t)sizeof(T)) + 16u * (lane >> 4);
#pragma unroll
    for (int j = 0; j < Rows16<T, D>::N; ++j) f.v[j] = *reinterpret_cast<const uint4 *>(p + 64 * j);
    return f;
}
// Element v of lane l: the score of column row l % 16 against row 4 (l / 16) + v.
template <typename T, int D>
__device__ __forceinline__ floatx4_t scores16(const Rows16<T, D> &rows, const Rows16<T, D> &cols)
{
    floatx4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < Rows16<T, D>::N; ++j) {
        if constexpr (sizeof(T) == 2) {
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, rows.v[j]), __builtin_bit_cast(bf16x8_t, cols.v[j]), acc, 0, 0, 0);
        } else {
            const floatx4_t a = __builtin_bit_cast(floatx4_t, rows.v[j]), b = __builtin_bit_cast(floatx4_t, cols.v[j]);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], acc, 0, 0, 0);
        }
    }
    return acc;
}

constexpr int kProfCap = 512;  // scores of a query's bin that fit LDS

template <int G> struct ProfShared {
    unsigned long long hist[256 * 32];   // [bin][query]; while scores of a bin are collected: key tiles
    unsigned long long part[G * 32];     // the search's partial sums
    alignas(16) float cand[32][kProfCap + 1];  // before: key tiles
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

template <typename T, int D, int WAVES>
__global__ __launch_bounds__((64 * WAVES)) void profile_kernel(const T *__restrict__ Q, const T *__restrict__ K,
                                                                  const int32_t *__restrict__ rows, int n, int L, int nbh,
                                                                  float c2, float target, int32_t *__restrict__ counts)
{
    constexpr int THREADS = 64 * WAVES, G = THREADS / 32;
    extern __shared__ __align__(16) unsigned char lds[];
    ProfShared<G> &sh = *reinterpret_cast<ProfShared<G> *>(lds);
    // consecutive blocks land on consecutive XCDs: each takes a stretch of the (head, queries) pairs, so that its L2 sees one head or two
    const int nblk = (n + 31) >> 5;
    // (less than 2^32 of them: every 32 sampled rows come with K rows of 4096 bytes and more)
    const uint32_t block = blockIdx.y * gridDim.x + blockIdx.x, per_xcd = gridDim.x * gridDim.y >> 3, item = (block & 7u) * per_xcd + (block >> 3);
    const int bh = (int)(item / (uint32_t)nblk), q0 = (int)(item - (uint32_t)bh * nblk) * 32;
    if (bh >= nbh) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nq = lane & 31;                        // the query that a thread searches for
    const int ql = lane & 15, g = lane >> 4;         // in the sweeps: a lane's queries are ql and 16 + ql
    const T *Kh = K + (int64_t)bh * L * D;
    Rows16<T, D> qf[2];
#pragma unroll
    for (int b = 0; b < 2; ++b)
        qf[b] = load_rows16<T, D>(Q + (int64_t)bh * L * D, min(max(rows[min(q0 + 16 * b + ql, n - 1)], 0), L - 1), lane);
    const int ntiles = (L + 31) >> 5;
    // f(scores [keys 16 a + 4 g + v of the tile][queries 16 b + ql], keys from 4 g on, whether all 32 keys of the tile exist).
    // Operands read from memory lane by lane are an access to the cache per 16 bytes, 0.86 per clock and CU and the sweeps' bound.  So a wave
    // brings its tile into LDS, whole lines at a time (`stage`: 8 KB per wave), and the next one while it works on this one's operands.  Pieces of a
    // row lie in an order of the row's own, so that neither side meets bank conflicts.  (Rows of 512 bytes do not fit.)
    constexpr int RB = D * (int)sizeof(T), PPR = RB / 16;
    constexpr bool STAGED = RB <= 256;
    static_assert(!STAGED || WAVES * 32 * RB <= (int)std::min(sizeof(sh.cand), sizeof(sh.hist)), "a tile per wave");
    auto sweep = [&](void *stage, auto f) {
        auto visit = [&](int tile, const Rows16<T, D> (&kf)[2]) __attribute__((always_inline)) {
            floatx4_t acc[2][2];
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b) acc[a][b] = scores16<T, D>(kf[a], qf[b]);
            if (tile * 32 + 32 <= L) f(acc, 32, std::true_type{});  // wave-uniform
            else f(acc, L - tile * 32 - 4 * g, std::false_type{});
        };
        if constexpr (STAGED) {
            constexpr int CH = 32 * RB / 1024;
            unsigned char *mine = static_cast<unsigned char *>(stage) + wave * (32 * RB);
            uint32_t from[CH], last[CH];
            int at[Rows16<T, D>::N];
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                const int row = (64 * i + lane) / PPR;
                const uint32_t piece = 16u * ((lane & (PPR - 1)) ^ (row & (PPR - 1)));
                from[i] = row * RB + piece;
                last[i] = (uint32_t)(L - 1) * RB + piece;
            }
#pragma unroll
            for (int j = 0; j < Rows16<T, D>::N; ++j) at[j] = ql * RB + 16 * ((4 * j + g) ^ (ql & (PPR - 1)));
            auto request = [&](int tile) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < CH; ++i)
                    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(reinterpret_cast<const char *>(Kh) +
                                                                                                     min(from[i] + (uint32_t)tile * (32u * RB), last[i])),
                                                     (__attribute__((address_space(3))) void *)(mine + 1024 * i), 16, 0, 0);
            };
            if (wave < ntiles) request(wave);
            for (int tile = wave; tile < ntiles; tile += WAVES) {
                Rows16<T, D> kf[2];
                __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this tile is there
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int j = 0; j < Rows16<T, D>::N; ++j) kf[a].v[j] = *reinterpret_cast<const uint4 *>(mine + 16 * a * RB + at[j]);
                __builtin_amdgcn_sched_barrier(0);
                __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): it has been read
                __builtin_amdgcn_sched_barrier(0);
                if (tile + WAVES < ntiles) request(tile + WAVES);
                visit(tile, kf);
            }
        } else {
            Rows16<T, D> next[2];
            auto request = [&](int tile) __attribute__((always_inline)) {
#pragma unroll
                for (int a = 0; a < 2; ++a) next[a] = load_rows16<T, D>(Kh, min(tile * 32 + 16 * a + ql, L - 1), lane);
            };
            request(wave);
            for (int tile = wave; tile < ntiles; tile += WAVES) {
                const Rows16<T, D> kf[2] = {next[0], next[1]};
                request(tile + WAVES);
                visit(tile, kf);
            }
        }
    };
    // f(score, which of the lane's queries) for the keys that exist
    auto each = [&](const floatx4_t (&acc)[2][2], int left, auto full, auto f) __attribute__((always_inline)) {
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (decltype(full)::value || 16 * a + v < left) {
                    f(acc[a][0][v], 0);
                    f(acc[a][1][v], 1);
                }
    };

    // ---- softmax normaliser (log2 domain: m2 = max_j s_ij c2, z = sum_j 2^(s_ij c2 - m2)) and range of the scores: the largest s c2 seen is
    // that of the largest or of the smallest score
    // (what an addition to z loses goes into the next one: a lane adds up hundreds of tiles)
    float lo[2], hi[2], m[2], z[2], lost[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        lo[b] = INFINITY;
        hi[b] = m[b] = -INFINITY;
        z[b] = lost[b] = 0.f;
    }
    float infinity = INFINITY;  // out of the compiler's sight, which would make middle ones of three minima and maxima with an instruction more per operand
    asm("" : "+v"(infinity));
    sweep(sh.cand, [&](const floatx4_t (&acc)[2][2], int left, auto full) {
        each(acc, left, full, [&](float x, int b) __attribute__((always_inline)) {
            lo[b] = __builtin_amdgcn_fmed3f(lo[b], x, -infinity);
            hi[b] = __builtin_amdgcn_fmed3f(hi[b], x, infinity);
        });
        if (decltype(full)::value || left > 0) {  // a lane whose keys all lie past the end has seen nothing yet
            float mn[2], add[2] = {0.f, 0.f};
#pragma unroll
            for (int b = 0; b < 2; ++b) mn[b] = fmaxf(lo[b] * c2, hi[b] * c2);
            each(acc, left, full, [&](float x, int b) __attribute__((always_inline)) { add[b] += __builtin_amdgcn_exp2f(fmaf(x, c2, -mn[b])); });
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const float f = __builtin_amdgcn_exp2f(m[b] - mn[b]);   // m = -inf on the first tile: factor 0
                const float old = z[b] * f, more = add[b] - lost[b] * f;
                z[b] = old + more;
                lost[b] = (z[b] - old) - more;
                m[b] = mn[b];
            }
        }
    });
    {
        float (*red)[4][4][32] = reinterpret_cast<float (*)[4][4][32]>(sh.hist);  // [wave][figure][lane group][query]
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            red[wave][0][g][16 * b + ql] = m[b];
            red[wave][1][g][16 * b + ql] = z[b];
            red[wave][2][g][16 * b + ql] = lo[b];
            red[wave][3][g][16 * b + ql] = hi[b];
        }
        __syncthreads();
        if (threadIdx.x < 32) {
            float mm = -INFINITY, l = INFINITY, h = -INFINITY;
            for (int w = 0; w < WAVES; ++w)
                for (int x = 0; x < 4; ++x) {
                    mm = fmaxf(mm, red[w][0][x][nq]);
                    l = fminf(l, red[w][2][x][nq]);
                    h = fmaxf(h, red[w][3][x][nq]);
                }
            double zz = 0.0;
            for (int w = 0; w < WAVES; ++w)
                for (int x = 0; x < 4; ++x) {
                    const float mw = red[w][0][x][nq];
                    if (mw > -INFINITY) zz += (double)(red[w][1][x][nq] * __builtin_amdgcn_exp2f(mw - mm));
                }
            sh.m2[nq] = mm;
            sh.rz[nq] = (float)(1.0 / zz);
            sh.lo[nq] = l;
            sh.hi[nq] = h;
            sh.ncand[nq] = 0;
        }
        __syncthreads();
    }
    // at least one unit: a target below 2^-38 is met by the most probable key (nothing would reach a target of zero)
    const unsigned long long want = max((unsigned long long)((double)target * 0x1p38), 1ull);
    struct Query {
        float m2, rz38, least, per;
        __device__ __forceinline__ unsigned long long mass(float x, float c2) const
        {
            return count_and_mass(__builtin_amdgcn_exp2f(fmaf(x, c2, -m2)) * rz38);
        }
        // the score's place between the smallest and the largest, in 2^-32 (not a number: 0), or its order-preserving pattern
        __device__ __forceinline__ uint32_t code(float x, bool pattern) const
        {
            return pattern ? score_key(x) : (uint32_t)(__builtin_amdgcn_fmed3f((x - least) * per, 0.f, 0x1.fffffep-1f) * 0x1p32f);
        }
    };
    auto query = [&](int q) {
        const float span = sh.hi[q] - sh.lo[q];
        return Query{sh.m2[q], sh.rz[q] * 0x1p38f, sh.lo[q], span > 0.f ? 1.f / span : 0.f};
    };
    const Query of[2] = {query(ql), query(16 + ql)};
    auto clear = [&]() {
        for (int e = threadIdx.x; e < 256 * 32; e += THREADS) sh.hist[e] = 0ull;
        __syncthreads();
    };

    // ---- bins, by eight bits of the code at a time, until the crossing bin of every query fits LDS
    bool pattern = false;
    uint32_t pre = 0u, pre_of[2] = {0u, 0u};
    unsigned long long above = 0ull;
    int known = 0, count = 0;  // leading bits found; scores that share them
    for (;;) {
        clear();
        const int shift = 24 - known;
        if (known == 0 && !pattern)  // the eight highest bits of all scores
            sweep(sh.cand, [&](const floatx4_t (&acc)[2][2], int left, auto full) {
                each(acc, left, full, [&](float x, int b) __attribute__((always_inline)) {
                    atomicAdd(&sh.hist[(of[b].code(x, false) >> 24) * 32 + 16 * b + ql], of[b].mass(x, c2));
                });
            });
        else
            sweep(sh.cand, [&](const floatx4_t (&acc)[2][2], int left, auto) {
                each(acc, left, std::false_type{}, [&](float s, int b) __attribute__((always_inline)) {
                    const uint32_t x = of[b].code(s, pattern);
                    if (known == 0 || (x ^ pre_of[b]) >> (shift + 8) == 0u)
                        atomicAdd(&sh.hist[((x >> shift) & 255u) * 32 + 16 * b + ql], of[b].mass(s, c2));
                });
            });
        cross_bin(sh, above, want);
        pre |= sh.found[nq].digit << shift;
#pragma unroll
        for (int b = 0; b < 2; ++b) pre_of[b] |= sh.found[16 * b + ql].digit << shift;
        above = sh.found[nq].above;
        count = sh.found[nq].count;
        known += 8;
        if (!pattern && __all(count <= kProfCap)) break;  // the same 32 queries in every wave: the whole block
        if (known == 32) break;
        if (!pattern && known == 24) {
            pattern = true;
            pre = pre_of[0] = pre_of[1] = 0u;
            above = 0ull;
            known = 0;
        }
    }
    const bool mine = q0 + nq < n;
    int32_t *out = counts + (int64_t)bh * n + q0 + nq;
    // of `same` keys of score x, below `above`, as many as the missing mass takes
    auto write = [&](float x, unsigned long long over, int same) {
        const float p = __builtin_amdgcn_exp2f(fmaf(x, c2, -sh.m2[nq])) * sh.rz[nq];
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
    __syncthreads();  // nobody brings key tiles there any more
    sweep(sh.hist, [&](const floatx4_t (&acc)[2][2], int left, auto full) {
        each(acc, left, full, [&](float x, int b) __attribute__((always_inline)) {
            if ((of[b].code(x, false) ^ pre_of[b]) >> (32 - known) == 0u) {
                const int at = atomicAdd(&sh.ncand[16 * b + ql], 1);
                if (at < kProfCap) sh.cand[16 * b + ql][at] = x;
            }
        });
    });
    __syncthreads();
    clear();
    const int t = threadIdx.x >> 5, c = min(sh.ncand[nq], kProfCap);
    const int shift = 24 - known;
    const Query mine_of = query(nq);
    auto bin = [&](float x) { return (mine_of.code(x, false) >> shift) & 255u; };
    auto mass = [&](float x) { return mine_of.mass(x, c2); };
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
template <typename T, int D, int WAVES>
static dsv_status profile_waves(const dsv_problem &p, const void *Q, const void *K, const int32_t *rows, int n, float mass,
                                int32_t *counts, hipStream_t st)
{
    const int nbh = p.B * p.H;
    constexpr int threads = 64 * WAVES;
    constexpr size_t lds = sizeof(ProfShared<threads / 32>);  // above the default of 64 KB
    static_assert(lds <= 160 * 1024, "LDS of a CU");
    DSV_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void *>(&profile_kernel<T, D, WAVES>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    const GridXY grid = grid_of((int64_t)((n + 31) / 32) * nbh);
    hipLaunchKernelGGL((profile_kernel<T, D, WAVES>), dim3(grid.x, grid.y), dim3(threads), lds, st, (const T *)Q, (const T *)K, rows, n, p.L, nbh,
                       p.scale * 1.4426950408889634f, mass, counts);
    DSV_LAUNCH_CHECK();
    return DSV_OK;
}

// Sixteen waves spill a few registers: they pay where each has a few tiles.  bf16, d = 64, us before tiles went through LDS, with 8, with 16 waves: four heads of 800,
// 60 rows each: 30.1, 25.6, 28.4; of 1200, 100 rows: 36.0, 32.5, 32.8; of 2000, 160: 49.9, 44.7, 41.6; five of 30134, 893: 711, 866, 564.
template <typename T, int D>
static dsv_status profile_t(const dsv_problem &p, const void *Q, const void *K, const int32_t *rows, int n, float mass,
                            int32_t *counts, float *sparsity, float *ema, float alpha, hipStream_t st)
{
    const int nbh = p.B * p.H;
    const dsv_status rc = p.L > 1280 ? profile_waves<T, D, kProfWavesMost<T, D>>(p, Q, K, rows, n, mass, counts, st)
                                     : profile_waves<T, D, kProfWaves>(p, Q, K, rows, n, mass, counts, st);
    if (rc != DSV_OK) return rc;
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
