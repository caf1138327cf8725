// Stage 1, emission: once every query's threshold score tau and its tie budget are known
// (stage1.hip), write the selected keys of every query (idx, query-major) and, on request, the
// selecting queries of every key (idx_t, key-major).  Both are pure re-evaluations of
//   selected(i, j)  <=>  s_ij > tau_i  or  (s_ij == tau_i and j <= jcut_i)
// over recomputed score tiles; jcut_i is the index of the last threshold-equal key query i takes
// (lowest index first), or kAllTies when it takes all of them -- then "s_ij >= tau_i" decides, which
// is the case for every query unless scores tie exactly at the threshold.
//
// Layout of both kernels: a block owns 32 "owners" (queries for idx, keys for idx_t) as the MFMA column operand and walks the other
// axis in tiles of 32, ascending, its waves a batch of tiles each in turn.  Lanes l and l+32 hold the same owner; each has 16 predicate
// bits, neighbours on the other axis, and parks them as its half of the tile's word in LDS.  The words are expanded into index
// entries a batch at a time (below), in tile order, so every row / list comes out ascending without any sorting.
// What bounds both is vector-instruction issue and, with few tiles, waves in flight: one wave per 32 owners left four per SIMD at L = 32768 and four
// heads (2.9 on the mean), half of them waiting for LDS or memory.  Four waves per block, words parked by halves in place of being
// reordered and shuffled, addresses in 32 bits, up to four entries per store: L = 32768, four heads, r = 16, k = 2048, us: idx 1137 -> 715, list
// lengths 471 -> 321, idx_t 1081 -> 770 (stores about 200 of that, 1.07 GB; without them it is the 16 differences and signs of a tile, 100 clocks).
#include "stage1_core.h"

namespace dsv {

// ---- output: masks parked per tile, expanded in batches -------------------------------------------
// A selected entry is 4 bytes and consecutive entries of one owner are produced ~16 tiles apart, so
// writing them as they appear makes every store a partial cache line (measured: 5x write
// amplification), and appending them one by one to a per-owner buffer costs a serial loop per tile
// that runs as long as the fullest of the 32 owners needs.  Instead a wave parks each tile's 32-bit
// mask per owner in LDS and, every batch of tiles, expands owner by owner: lanes side by side take the owner's
// parked words (one tile each), a prefix sum of their popcounts gives every lane its
// place in the owner's row, and the lanes write their entries side by side -- one store instruction
// covers a contiguous stretch of the row.  Query-major a wave has 32 owners and up to 32 tiles a batch, and expands two owners at a time (one
// per half-wave); key-major it has 64 and up to 16, and expands four (one per 16 lanes).
constexpr int kBatch = 32;  // words of an owner's batch in the block form below (= lanes of a half-wave)
constexpr int kWaves = 4;   // waves of a block, a batch each in turn

// OT: owner tiles per wave.  Where a wave's batch goes: per owner the next place and the end of its row or list (a correct threshold
// fills it exactly; the clamp keeps a wrong one from writing out of bounds), in entries after the start of its tile's first owner.
template <int OT> struct EmitShared {
    static constexpr int TILES = 32 / OT;                // of a batch, at most
    uint32_t mask[kWaves][TILES][32 * OT + 1];           // [tile in batch][owner], padded: conflict-free both ways
    int32_t count[2][kWaves][OT][64];                    // entries of a batch by owner tile and lane (owner and half), two rounds in turn
    int2 place[kWaves][32 * OT];
};

typedef uint16_t __attribute__((may_alias)) halfword_t;  // half of a parked word, which is read whole

// Tiles per batch: full rounds of the block's waves.
__device__ __forceinline__ int batch_tiles(int ntiles, int most)
{
    const int rounds = (ntiles + kWaves * most - 1) / (kWaves * most);
    return (ntiles + kWaves * rounds - 1) / (kWaves * rounds);
}

typedef int32_t entries4_t __attribute__((ext_vector_type(4), aligned(4)));
typedef int32_t entries2_t __attribute__((ext_vector_type(2), aligned(4)));

// One word's entries, base_val + its bits, at entries pos on from `to`; no more of them than fit before `end`.
__device__ __forceinline__ void write_word(char *to, uint32_t m, int c, int pos, int end, int base_val)
{
    if (pos + c > end) {  // entries past the row's capacity are dropped, highest first
        const int room = max(end - pos, 0);
        while (__popc(m) > room) m &= ~(0x80000000u >> __clz(m));
        c = __popc(m);
    }
    uint32_t off = (uint32_t)pos * 4u;
    auto take = [&]() __attribute__((always_inline)) {
        const int e = base_val + (__ffs(m) - 1);
        m &= m - 1;
        return e;
    };
    for (; c >= 4; c -= 4, off += 16) {
        entries4_t e;
#pragma unroll
        for (int i = 0; i < 4; ++i) e[i] = take();
        *reinterpret_cast<entries4_t *>(to + off) = e;
    }
    if (c & 2) {
        entries2_t e;
        e[0] = take();
        e[1] = take();
        *reinterpret_cast<entries2_t *>(to + off) = e;
        off += 8;
    }
    if (c & 1) *reinterpret_cast<int32_t *>(to + off) = take();
}

// Expand the parked masks of tiles tile0 .. tile0 + nfilled - 1 for all owners: 64 words at a time, of 2 OT owners.  out, out_last: where the
// rows or lists of the first and of the last owner tile begin.  Offsets from there have 32 bits: 32 lists of every query are less than 2^32 bytes (64 are not).
// (Compacting an owner's entries in LDS first and writing them out with consecutive lanes on consecutive
// entries was measured slower -- 24.2 against 21.2 ms for the query-major emission at L = 128k, k = 8192.)
template <int OT>
__device__ __forceinline__ void expand_batch(const EmitShared<OT> &sh, int wave, int32_t *out, int32_t *out_last, int tile0, int nfilled, int lane)
{
    static_assert(32 * kMaxKeys * (int64_t)sizeof(int32_t) < 1ll << 32, "offsets inside an owner tile's rows or lists");
    constexpr int TILES = EmitShared<OT>::TILES, STEP = 64 / TILES;
    const int t = lane & (TILES - 1), sub = lane / TILES;
    const int base_val = (tile0 + t) * 32;
    uint32_t next = t < nfilled ? sh.mask[wave][t][sub] : 0u;
    int2 next_at = sh.place[wave][sub];
#pragma unroll 2
    for (int i = 0; i < 16; ++i) {
        const uint32_t m = next;
        const int2 at = next_at;
        const int o = STEP * min(i + 1, 15) + sub;
        next = t < nfilled ? sh.mask[wave][t][o] : 0u;
        next_at = sh.place[wave][o];
        const int c = __popc(m);
        write_word(reinterpret_cast<char *>(STEP * i < 32 ? out : out_last), m, c, at.x + (OT == 1 ? half_scan(c) : row_scan(c)) - c, at.y, base_val);
    }
}

// The same where one round is not full and all there is: a wave takes 16 of the 64 owners and the words that all waves have parked, 16 tiles
// at a time, in 4 steps for every 16 tiles where its own tiles' words take 16 (few queries to a head, as where they come in groups: 24 heads of 3360 keys, 210
// groups, k = L / 14: 17.1 -> 10.4 us; a wave per 32 keys that takes all tiles: 13.4).
constexpr int kFewTiles = 48;
__device__ __forceinline__ void expand_few(const EmitShared<2> &sh, int wave, int32_t *out, int32_t *out_last, int batch, int ntiles, int lane)
{
    static_assert(kFewTiles <= kWaves * EmitShared<2>::TILES, "one round");
    const uint32_t per = 65536u / (uint32_t)batch + 1u;  // tile / batch for tiles below 64
    char *to = reinterpret_cast<char *>(wave < 2 ? out : out_last);
#pragma unroll 1
    for (int o = 16 * wave + (lane >> 4); o < 16 * wave + 16; o += 4) {
        int2 at = sh.place[wave][o];
#pragma unroll 1
        for (int t = lane & 15; t < ntiles + (lane & 15); t += 16) {  // the same steps for all lanes
            const int w = (int)((uint32_t)t * per >> 16);
            const uint32_t m = t < ntiles ? sh.mask[w][t - w * batch][o] : 0u;
            const int c = __popc(m), sum = row_scan(c);
            write_word(to, m, c, at.x + sum - c, at.y, t * 32);
            at.x += __shfl(sum, lane | 15);
        }
    }
}

// After a round's words are parked and its counts written: the batch's place in its owners' rows.  at, end: of this lane's owners.
template <int OT>
__device__ __forceinline__ void place_batch(EmitShared<OT> &sh, int buf, int wave, int lane, int (&at)[OT], const int (&end)[OT])
{
#pragma unroll
    for (int i = 0; i < OT; ++i) {
        int before = 0, all = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const int c = sh.count[buf][w][i][lane & 31] + sh.count[buf][w][i][32 + (lane & 31)];
            before += w < wave ? c : 0;
            all += c;
        }
        if (lane < 32) sh.place[wave][32 * i + lane] = make_int2(min(at[i] + before, end[i]), end[i]);
        at[i] = min(at[i] + all, end[i]);
    }
    __builtin_amdgcn_wave_barrier();
}

// ------------------------------------------------------------------------------------ query-major
// Ties that a query does not take: a tile of queries one of which does not take all of its threshold-equal keys counts them beside the
// selected ones, and a batch that holds more of them than its query may still take (or the last of those) is scored once more to find which.
struct Ties {
    int32_t count[2][kWaves][64];
    int32_t last[32];  // the highest one taken
};

template <typename T, int R>
__device__ __forceinline__ uint32_t equal_word(const T *__restrict__ Kb, const TileWalk<T, R> &walk, const Frag<T, R> &kf, const Frag<T, R> &qf, int L, float tau, int t, int half)
{
    const floatx16_t acc = score_tile<T, R>(kf, qf);
    uint32_t m;
    DSV_PRED16(m, acc[v] == tau);
    const int left = L - t * 32 - 16 * half;
    m = (left >= 16 ? m : left > 0 ? m & ((1u << left) - 1u) : 0u) << (16 * half);
    return m | (uint32_t)__shfl_xor((int)m, 32);
}

// prefix[query] holds the order-preserving key of tau on entry and the fp32 bits of tau on exit.
// krem[query] = +-(number of threshold-equal keys to take); negative: that is all of them.
// jcut (optional) and tile_flag (optional; 1 when all 32 queries of the tile take all their ties)
// are what the key-major emission needs.
template <typename T, int R>
__global__ __launch_bounds__(64 * kWaves, 4) void emit_kernel(const T *__restrict__ Qlr, const T *__restrict__ Klr, int Lq, int L,
                                                           HeadTable tab, uint32_t *__restrict__ prefix,
                                                           const int32_t *__restrict__ krem, int32_t *__restrict__ idx,
                                                           int32_t *__restrict__ jcut, int32_t *__restrict__ tile_flag)
{
    __shared__ __align__(16) EmitShared<1> sh;
    __shared__ Ties ties;
    const int slot = blockIdx.y;
    const int bh = tab.bh[slot];
    const int k = tab.k[slot];
    const int q0 = blockIdx.x * 32;
    const T *Qb = Qlr + (int64_t)bh * Lq * R;
    const T *Kb = Klr + (int64_t)bh * L * R;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 31, half = lane >> 5;
    const bool live = q0 + n < Lq;
    const int64_t g = (int64_t)bh * padded_len(Lq) + min(q0 + n, Lq - 1);
    const float tau = key_score(prefix[g]);
    const int kr = krem[g];
    const bool all_simple = __all(kr < 0);
    int32_t *out = idx + tab.off[slot] + (int64_t)q0 * k;
    const Frag<T, R> qf = load_frag<T, R>(Qb, q0, Lq, lane);
    const TileWalk<T, R> walk(L, lane);
    if (!all_simple && threadIdx.x < 32) ties.last[n] = -1;

    const int ntiles = (L + 31) >> 5, batch = batch_tiles(ntiles, EmitShared<1>::TILES);
    const uint32_t whole = live ? 0xFFFFu : 0u;
    const int want = kr < 0 ? 0x7FFFFFFF : kr;  // ties to take; taken: those of earlier rounds, whether or not there was room
    int at[1] = {live ? n * k : 0}, taken = 0;
    const int end[1] = {live ? at[0] + k : 0};
    int buf = 0;
    for (int b0 = 0; b0 < ntiles; b0 += kWaves * batch, buf ^= 1) {
        const int t0 = min(b0 + wave * batch, ntiles), t1 = min(t0 + batch, ntiles);
        halfword_t *park = reinterpret_cast<halfword_t *>(sh.mask[wave][0]) + 2 * n + half;
        Frag<T, R> kf_next = walk.load(Kb, t0, half);
        int count = 0, equal = 0;
#pragma unroll 1
        for (int t = t0; t < t1; ++t, park += 66) {
            // the next tile's fragment is requested before this tile is scored (rows past the end clamp)
            const Frag<T, R> kf = kf_next;
            kf_next = walk.load(Kb, t + 1, half);
            const floatx16_t acc = score_tile<T, R>(kf, qf);
            uint32_t sel, in = whole;
            if (t + 1 == ntiles) {
                const int left = L - t * 32 - 16 * half;
                in &= left >= 16 ? 0xFFFFu : left > 0 ? (1u << left) - 1u : 0u;
            }
            DSV_SIGNS16(sel, acc[v] - tau);  // score < tau  <=>  (score - tau) is negative; equal scores give +0
            sel = ~sel & in;
            if (!all_simple) {
                uint32_t eq;
                DSV_PRED16(eq, acc[v] == tau);
                equal += __popc(eq & in);
            }
            *park = (uint16_t)sel;
            count += __popc(sel);
        }
        sh.count[buf][wave][0][lane] = count;
        if (!all_simple) ties.count[buf][wave][lane] = equal;
        __syncthreads();  // (two rounds in turn: what is written next was last read before this barrier)
        if (!all_simple) {
            // ties that do not fit leave the counts: those of this batch by this wave, for all to see
            int before = taken, here = 0;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                const int c = ties.count[buf][w][n] + ties.count[buf][w][32 + n];
                before += w < wave ? c : 0;
                here = w == wave ? c : here;
                taken += c;
            }
            const int fit = max(0, min(here, want - before));
            if (half == 0) sh.count[buf][wave][0][lane] -= here - fit;
            if (__any(live && here > 0 && before < want && want <= before + here) || __any(live && fit < here)) {
                int left = want - before;
                for (int t = t0; t < t1; ++t) {
                    const uint32_t eq = equal_word<T, R>(Kb, walk, walk.load(Kb, t, half), qf, L, tau, t, half);
                    const int c = __popc(eq);
                    uint32_t drop = eq;
                    for (int i = 0; i < min(left, c); ++i) drop &= drop - 1;
                    if (left > 0 && left <= c && half == 0) ties.last[n] = t * 32 + 31 - __clz(eq & ~drop);
                    if (half == 0 && live) sh.mask[wave][t - t0][n] &= ~drop;
                    left -= c;
                }
            }
            __syncthreads();
        }
        place_batch<1>(sh, buf, wave, lane, at, end);
        expand_batch<1>(sh, wave, out, out, t0, t1 - t0, lane);
    }
    if (!all_simple) __syncthreads();
    if (wave == 0 && live && half == 0) {
        prefix[g] = __float_as_uint(tau);
        if (jcut) jcut[g] = kr < 0 ? kAllTies : ties.last[n];
    }
    if (tile_flag && threadIdx.x == 0) tile_flag[(int64_t)bh * gridDim.x + blockIdx.x] = all_simple ? 1 : 0;
}

// The same by blocks of 16 waves per 32 queries, which form the words of 32 key tiles together and expand two queries each:
// for few queries, whose single waves (one per 32 of them, the whole key axis in turn) would leave most of the chip idle.
constexpr int kEmitWaves = 16;
template <typename T, int R>
__global__ __launch_bounds__(64 * kEmitWaves) void emit_block_kernel(const T *__restrict__ Qlr, const T *__restrict__ Klr, int Lq,
                                                                     int L, HeadTable tab, uint32_t *__restrict__ prefix,
                                                                     const int32_t *__restrict__ krem, int32_t *__restrict__ idx,
                                                                     int32_t *__restrict__ jcut, int32_t *__restrict__ tile_flag)
{
    constexpr int TPW = kBatch / kEmitWaves;       // tiles per wave and round
    __shared__ uint32_t gt[2][kBatch][33], eq[2][kBatch][33];
    const int slot = blockIdx.y;
    const int bh = tab.bh[slot];
    const int k = tab.k[slot];
    const int q0 = blockIdx.x * 32;
    const T *Qb = Qlr + (int64_t)bh * Lq * R;
    const T *Kb = Klr + (int64_t)bh * L * R;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = lane & 31, half = lane >> 5;
    const int64_t g0 = (int64_t)bh * padded_len(Lq) + q0;
    const int last = Lq - 1 - q0;                  // queries past the end repeat the last one
    const float tau = key_score(prefix[g0 + min(n, last)]);
    const bool all_simple = __all(krem[g0 + min(n, last)] < 0);
    const int q = 2 * wave + half;                 // the query this half-wave expands
    const bool live = q <= last;
    const int kr = krem[g0 + min(q, last)];
    RowOut ro{0, kr < 0 ? -kr : kr, -1};
    int32_t *row = idx + tab.off[slot] + (int64_t)(q0 + min(q, last)) * k;
    const Frag<T, R> qf = load_frag<T, R>(Qb, q0, Lq, lane);
    const int ntiles = (L + 31) >> 5;
    int buf = 0;
    for (int t0 = 0; t0 < ntiles; t0 += kBatch, buf ^= 1) {
#pragma unroll
        for (int i = 0; i < TPW; ++i) {
            const int at = TPW * wave + i, j0 = (t0 + at) * 32;
            const uint32_t valid = j0 + 32 <= L ? 0xFFFFFFFFu : (j0 < L ? (1u << (L - j0)) - 1u : 0u);
            uint32_t g, e;
            threshold_words(score_tile<T, R>(load_frag<T, R>(Kb, j0, L, lane), qf), tau, all_simple, valid, half, g, e);
            if (half == 0) {
                gt[buf][at][n] = g;
                if (!all_simple) eq[buf][at][n] = e;
            }
        }
        __syncthreads();  // two buffers in turn: the one written next was last read before this barrier
        emit_row_words(ro, gt[buf][n][q], all_simple ? 0u : eq[buf][n][q], all_simple, t0 + n, half, live, row, k);
    }
    __syncthreads();      // every wave has read the thresholds
    if (threadIdx.x < 32 && (int)threadIdx.x <= last) prefix[g0 + n] = __float_as_uint(tau);
    if (jcut && live && n == 0) jcut[g0 + q] = kr < 0 ? kAllTies : ro.last_tie;
    if (tile_flag && threadIdx.x == 0) tile_flag[(int64_t)bh * gridDim.x + blockIdx.x] = all_simple ? 1 : 0;
}

// ------------------------------------------------------------------------------------ key-major
// tau_f: the fp32 thresholds left in `prefix` by emit_kernel.  The tile is computed with the query
// fragment as the row operand and the key fragment as the column operand, so lane l owns key
// (l % 32) and accumulator v is query v + 16 * (l/32) of the tile; the thresholds of a lane's 16
// queries come from a chunk staged in LDS (state rows are padded to whole tiles; queries past the end get one that nothing reaches).
struct QueryChunk {
    static constexpr int kTiles = 8;  // one coalesced 16-byte load per lane
    float tau[kWaves][kTiles * 32];
    int32_t jcut[kWaves][kTiles * 32];
};

// Visits tiles t0 .. t1 - 1: f(the last ties that the lane's 16 queries take, key tile, its scores, the lane's 16 thresholds, whether all queries of the tile take all their ties).
// A wave owns two key tiles: reading the thresholds costs the LDS of a CU, which four SIMDs share, as much time as a SIMD needs for a tile.
// Thresholds and flags of eight tiles are requested while the eight before are worked on.
template <typename T, int R, typename F>
__device__ __forceinline__ void walk_queries(QueryChunk &qc, const T *__restrict__ Qb, const TileWalk<T, R> &walk, const Frag<T, R> (&kf)[2],
                                             const float *__restrict__ tau_b, const int32_t *__restrict__ jcut_b, const int32_t *__restrict__ flag_b, int Lq, int t0, int t1, int wave, int lane,
                                             F f)
{
    constexpr int C = QueryChunk::kTiles;
    const int half = lane >> 5, npad = padded_len(Lq), ntiles = npad >> 5;
    float *tau_s = qc.tau[wave];
    int32_t *jcut_s = qc.jcut[wave];
    auto thresholds = [&](int t) __attribute__((always_inline)) { return *reinterpret_cast<const float4 *>(tau_b + min(t * 32 + lane * 4, npad - 4)); };
    auto cuts = [&](int t) __attribute__((always_inline)) { return *reinterpret_cast<const int4 *>(jcut_b + min(t * 32 + lane * 4, npad - 4)); };
    auto flags = [&](int t) __attribute__((always_inline)) { return flag_b[min(t + (lane & (C - 1)), ntiles - 1)]; };
    if (t0 >= t1) return;
    float4 tau_next = thresholds(t0);
    int4 cut_next = cuts(t0);
    int32_t flag_next = flags(t0);
    Frag<T, R> qf_next = walk.load(Qb, t0, half);
    for (int c = t0; c < t1; c += C) {
        const int left = Lq - (c * 32 + lane * 4);  // of this lane's four thresholds
        float4 t4 = tau_next;
        if (left < 4) {
            if (left < 1) t4.x = INFINITY;
            if (left < 2) t4.y = INFINITY;
            if (left < 3) t4.z = INFINITY;
            t4.w = INFINITY;
        }
        __builtin_amdgcn_wave_barrier();
        *reinterpret_cast<float4 *>(tau_s + lane * 4) = t4;
        *reinterpret_cast<int4 *>(jcut_s + lane * 4) = cut_next;
        __builtin_amdgcn_wave_barrier();
        const uint32_t simple = (uint32_t)__ballot(flag_next != 0);
        tau_next = thresholds(c + C);
        cut_next = cuts(c + C);
        flag_next = flags(c + C);
        const int tn = min(C, t1 - c);
#pragma unroll 1
        for (int t = 0; t < tn; ++t) {
            const Frag<T, R> qf = qf_next;
            qf_next = walk.load(Qb, c + t + 1, half);
            float tq[16];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float4 v4 = *reinterpret_cast<const float4 *>(tau_s + t * 32 + 16 * half + 4 * i);
                tq[4 * i] = v4.x; tq[4 * i + 1] = v4.y; tq[4 * i + 2] = v4.z; tq[4 * i + 3] = v4.w;
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) f(jcut_s + t * 32 + 16 * half, i, score_tile<T, R>(qf, kf[i]), tq, (simple >> t & 1u) != 0u);
        }
    }
}

// The 16 predicates of a lane where some query of the tile does not take all its ties.
__device__ __forceinline__ uint32_t selected_with_ties(const floatx16_t &acc, const float (&tq)[16], const int32_t *jcut, int j)
{
    uint32_t m = 0u;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int4 c4 = *reinterpret_cast<const int4 *>(jcut + 4 * i);
        const int cut[4] = {c4.x, c4.y, c4.z, c4.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int v = 4 * i + e;
            m |= ((uint32_t)(acc[v] > tq[v]) | ((uint32_t)(acc[v] == tq[v]) & (uint32_t)(j <= cut[e]))) << v;
        }
    }
    return m;
}

// List lengths -> cnt[bh, j].  A pair costs three plain instructions (difference, sign, sum); each wave takes a stretch of the queries.
template <typename T, int R>
__global__ __launch_bounds__(64 * kWaves) void count_t_kernel(const T *__restrict__ Qlr, const T *__restrict__ Klr, int Lq, int L, HeadTable tab,
                                                              const float *__restrict__ tau_f, const int32_t *__restrict__ jcut,
                                                              const int32_t *__restrict__ tile_flag, int32_t *__restrict__ cnt)
{
    __shared__ __align__(16) QueryChunk qc;
    __shared__ int32_t sum[kWaves][2][64];
    const int bh = tab.bh[blockIdx.y], j0 = blockIdx.x * 64;
    const T *Qb = Qlr + (int64_t)bh * Lq * R;
    const T *Kb = Klr + (int64_t)bh * L * R;
    const float *tau_b = tau_f + (int64_t)bh * padded_len(Lq);
    const int32_t *jcut_b = jcut + (int64_t)bh * padded_len(Lq);
    const int ntiles = (Lq + 31) >> 5;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int half = lane >> 5, j = j0 + (lane & 31);
    const Frag<T, R> kf[2] = {load_frag<T, R>(Kb, j0, L, lane), load_frag<T, R>(Kb, j0 + 32, L, lane)};
    const TileWalk<T, R> walk(Lq, lane);
    constexpr int CHUNKS = kWaves * QueryChunk::kTiles;
    // few tiles: every wave some, unless the operands of the two key tiles, which each of them reads, are most of the work (24 heads of 3360 keys, 7 tiles,
    // r = 16: 7.2 -> 4.6 us; of 1536, 3 tiles, r = 64: 4.9, 6.6 by four waves)
    const int per = R * sizeof(T) != 128 && ntiles <= CHUNKS ? (ntiles + kWaves - 1) / kWaves : (ntiles + CHUNKS - 1) / CHUNKS * QueryChunk::kTiles;
    int taken[2] = {0, 0};
    walk_queries<T, R>(qc, Qb, walk, kf, tau_b, jcut_b, tile_flag + (int64_t)bh * ntiles, Lq, min(wave * per, ntiles), min((wave + 1) * per, ntiles), wave, lane,
                       [&](const int32_t *cuts, int i, const floatx16_t &acc, const float (&tq)[16], bool simple) __attribute__((always_inline)) {
                           int below = 0;  // scores under their threshold
                           if (simple) {
#pragma unroll
                               for (int v = 0; v < 16; ++v) below += (int)(__float_as_uint(acc[v] - tq[v]) >> 31);
                           } else {
                               below = 16 - __popc(selected_with_ties(acc, tq, cuts, j + 32 * i));
                           }
                           taken[i] += 16 - below;
                       });
#pragma unroll
    for (int i = 0; i < 2; ++i) sum[wave][i][lane] = taken[i];
    __syncthreads();
    if (threadIdx.x < 64 && j0 + (int)threadIdx.x < L) {
        int all = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) all += sum[w][threadIdx.x >> 5][threadIdx.x & 31] + sum[w][threadIdx.x >> 5][32 + (threadIdx.x & 31)];
        cnt[(int64_t)bh * L + j0 + threadIdx.x] = all;
    }
}

// The lists, starting at col[bh, j].
// FEW: at most kFewTiles query tiles.  (Rows of 128 bytes: a third wave per SIMD for 6 registers less; 24 heads of 2304, 6 query tiles, the selection
// 129 -> 124 us together with expand_few.)
template <typename T, int R, bool FEW>
__global__ __launch_bounds__(64 * kWaves, R * sizeof(T) == 128 ? 3 : 1) void emit_t_kernel(const T *__restrict__ Qlr, const T *__restrict__ Klr, int Lq, int L, HeadTable tab,
                                                             const float *__restrict__ tau_f, const int32_t *__restrict__ jcut,
                                                             const int32_t *__restrict__ tile_flag, const int64_t *__restrict__ col,
                                                             int32_t *__restrict__ idxT)
{
    __shared__ __align__(16) EmitShared<2> sh;
    __shared__ __align__(16) QueryChunk qc;
    const int slot = blockIdx.y;
    const int bh = tab.bh[slot];
    const int j0 = blockIdx.x * 64;
    const T *Qb = Qlr + (int64_t)bh * Lq * R;
    const T *Kb = Klr + (int64_t)bh * L * R;
    const float *tau_b = tau_f + (int64_t)bh * padded_len(Lq);
    const int32_t *jcut_b = jcut + (int64_t)bh * padded_len(Lq);
    const int ntiles = (Lq + 31) >> 5;  // query tiles: the axis this kernel walks
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 31, half = lane >> 5;

    const Frag<T, R> kf[2] = {load_frag<T, R>(Kb, j0, L, lane), load_frag<T, R>(Kb, j0 + 32, L, lane)};
    // col comes from the counting pass over the same predicate, so the lists fill the head's block of
    // L * k entries exactly; the clamps (to [0, cap], ascending, and a tile's 32 lists to 32 * Lq entries) only keep an
    // inconsistent col from sending writes out of it
    const int64_t cap = (int64_t)Lq * tab.k[slot];
    const int64_t *cp = col + (int64_t)bh * (L + 1);
    auto clamped = [&](int64_t x, int64_t lo, int64_t hi) { return x < lo ? lo : x < hi ? x : hi; };
    const int64_t origin[2] = {clamped(cp[j0], 0, cap), clamped(cp[min(j0 + 32, L)], 0, cap)};
    int32_t *out = idxT + tab.off[slot] + origin[0], *out_last = idxT + tab.off[slot] + origin[1];
    int at[2], end[2];
    uint32_t whole[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int j = min(j0 + 32 * i + n, L - 1);
        const bool live = j0 + 32 * i + n < L;
        const int64_t far = clamped(origin[i] + 32ll * Lq, 0, cap);
        const int64_t c0 = clamped(cp[j], origin[i], far), c1 = clamped(cp[j + 1], c0, far);
        at[i] = (int)(c0 - origin[i]);
        end[i] = live ? (int)(c1 - origin[i]) : at[i];
        whole[i] = live ? 0xFFFFu : 0u;
    }

    const TileWalk<T, R> walk(Lq, lane);
    const int batch = batch_tiles(ntiles, EmitShared<2>::TILES);
    int buf = 0;
    for (int b0 = 0; b0 < ntiles; b0 += kWaves * batch, buf ^= 1) {
        const int t0 = min(b0 + wave * batch, ntiles), t1 = min(t0 + batch, ntiles);
        halfword_t *park = reinterpret_cast<halfword_t *>(sh.mask[wave][0]) + 2 * n + half;
        int count[2] = {0, 0};
        walk_queries<T, R>(qc, Qb, walk, kf, tau_b, jcut_b, tile_flag + (int64_t)bh * ntiles, Lq, t0, t1, wave, lane,
                           [&](const int32_t *cuts, int i, const floatx16_t &acc, const float (&tq)[16], bool simple) __attribute__((always_inline)) {
                               uint32_t sel;
                               if (simple) {
                                   DSV_SIGNS16(sel, acc[v] - tq[v]);  // score < tau as the sign of (score - tau)
                                   sel = ~sel & whole[i];
                               } else {
                                   sel = selected_with_ties(acc, tq, cuts, j0 + 32 * i + n) & whole[i];
                               }
                               park[64 * i] = (uint16_t)sel;
                               if (i == 1) park += 130;
                               count[i] += __popc(sel);
                           });
#pragma unroll
        for (int i = 0; i < 2; ++i) sh.count[buf][wave][i][lane] = count[i];
        __syncthreads();  // (two rounds in turn: what is written next was last read before this barrier)
        if constexpr (FEW) {  // one round
#pragma unroll
            for (int i = 0; i < 2; ++i)
                if (lane < 32) sh.place[wave][32 * i + lane] = make_int2(at[i], end[i]);
            __builtin_amdgcn_wave_barrier();
            expand_few(sh, wave, out, out_last, batch, ntiles, lane);
            return;
        }
        place_batch<2>(sh, buf, wave, lane, at, end);
        expand_batch<2>(sh, wave, out, out_last, t0, t1 - t0, lane);
    }
}

// ------------------------------------------------------------------------------------ host
// Whether the query-major emission takes the form of 16 waves that write two queries each, instead of that of four that write batches:
// while there are few tiles of queries.  us, batches : two queries each, r = 16: L = 8192, k = L / 16, 256 tiles 121 : 90, 512 151 : 129, 1024 216 : 215,
// k = L / 64 106 : 111 and 208 : 202; L = 16384, 512 tiles 210 : 195, 1024 312 : 341, 2048 505 : 629; k = L / 64, 1024 337 : 364.  r = 64, L = 8192,
// 256 tiles 179 : 179, 512 364 : 345; L = 16384, 512 451 : 454, 1024 847 : 864.  fp32, r = 16, L = 8192, 256 tiles 216 : 181, 512 333 : 290, 1024 501 : 513;
// r = 64, 256 tiles 484 : 488, 512 1020 : 980, 1024 1803 : 1917.
// Short rows of keys pay for the barriers sooner (fp32, L = 2080, 520 tiles, 62 : 75).
template <typename T, int R>
static bool emit_by_blocks(int L, int qtiles, const HeadTable &tab)
{
    const int64_t tiles = (int64_t)qtiles * tab.n;
    if (sizeof(T) == 4) return tiles <= (int64_t)(R > 16 ? 512 : 768) * std::min(L, 5120) / 5120;
    return tiles < (R == 64 ? 512 : 1024);
}

template <typename T, int R>
static dsv_status emit_all_t(const dsv_problem &p, int Lq, const HeadTable *tabs, int n_tabs, const void *Qlr,
                             const void *Klr, const SelectBuffers &b, bool emitted, hipStream_t st)
{
    const T *Ql = (const T *)Qlr;
    const T *Kl = (const T *)Klr;
    const int tiles = (p.L + 31) / 32;    // key tiles
    const int qtiles = (Lq + 31) / 32;    // query (or query-group) tiles
    const float *tau_f = reinterpret_cast<const float *>(b.prefix);
    if (!emitted) {
        KernelSpan span(DSV_KERNEL_EMIT, st);
        for (int t = 0; t < n_tabs; ++t) {
            dim3 grid(qtiles, tabs[t].n);
            if (emit_by_blocks<T, R>(p.L, qtiles, tabs[t]))
                hipLaunchKernelGGL((emit_block_kernel<T, R>), grid, dim3(64 * kEmitWaves), 0, st, Ql, Kl, Lq, p.L, tabs[t], b.prefix, b.krem,
                                   b.idx, b.jcut, b.tile_flag);
            else
                hipLaunchKernelGGL((emit_kernel<T, R>), grid, dim3(64 * kWaves), 0, st, Ql, Kl, Lq, p.L, tabs[t], b.prefix, b.krem, b.idx,
                                   b.jcut, b.tile_flag);
            DSV_LAUNCH_CHECK();
        }
    }
    if (b.idx_t) {
        {
            KernelSpan span(DSV_KERNEL_EMIT_T_COUNT, st);
            for (int t = 0; t < n_tabs; ++t) {
                dim3 grid((tiles + 1) / 2, tabs[t].n);
                hipLaunchKernelGGL((count_t_kernel<T, R>), grid, dim3(64 * kWaves), 0, st, Ql, Kl, Lq, p.L, tabs[t], tau_f, b.jcut,
                                   b.tile_flag, b.cnt);
                DSV_LAUNCH_CHECK();
            }
        }
        for (int t = 0; t < n_tabs; ++t) {
            const dsv_status rc = launch_col_scan(b.cnt, b.col, p.L, tabs[t], st);
            if (rc != DSV_OK) return rc;
        }
        KernelSpan span(DSV_KERNEL_EMIT_T_WRITE, st);
        for (int t = 0; t < n_tabs; ++t) {
            dim3 grid((tiles + 1) / 2, tabs[t].n);
            auto lists = [&](auto kernel) {
                hipLaunchKernelGGL(kernel, grid, dim3(64 * kWaves), 0, st, Ql, Kl, Lq, p.L, tabs[t], tau_f, b.jcut, b.tile_flag, b.col, b.idx_t);
            };
            if (qtiles <= kFewTiles) lists(emit_t_kernel<T, R, true>);
            else lists(emit_t_kernel<T, R, false>);
            DSV_LAUNCH_CHECK();
        }
    }
    return DSV_OK;
}

dsv_status launch_emit(const dsv_problem &p, int Lq, const HeadTable *tabs, int n_tabs, const void *Qlr, const void *Klr,
                       const SelectBuffers &b, bool emitted, hipStream_t st)
{
#define DSV_CASE(TT, RR) return emit_all_t<TT, RR>(p, Lq, tabs, n_tabs, Qlr, Klr, b, emitted, st)
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
