// Transposed index: for every key, the ascending list of queries whose row holds it (dsv_idx_transpose; the first step of
// a backward that brings no key-major index), and the rewriting of rows in any order as ascending rows.
//
// Two forms, both a stable counting sort by key:
// (L = 20280, four heads keeping 507 .. 4056 keys: 0.75 ms by the bit matrix, 8.25 ms by the entry sort.)
//   bit matrix   rows become rows of a bit matrix [queries, keys] (an LDS bitmap per row, so any order inside a row will
//                do); column sums per 1024 queries and their scan give every list's place; 32 x 32 bit blocks are then
//                transposed inside the waves and expanded into entries, 1024 queries x 512 keys per block.  Costs about
//                two bits of traffic per (query, key) pair and a few instructions per 1024 pairs, whatever the order.
//   entry sort   one scattered request per entry and pass; cheaper only where rows keep very few of the keys.
#include <algorithm>

#include "common.h"

namespace dsv {

// ------------------------------------------------------------------------------------ bit matrix
// Bits of row i: pitch words, bit j % 32 of word j / 32 set when the row holds key j; pitch is a multiple of 16 words, so
// that the 512 keys of a block are whole 64-byte pieces of every row.
constexpr int kBitsKeys = 512;               // keys per block of the counting and filling kernels (16 words)
constexpr int kBitsRows = 1024;              // queries per block of those kernels: one segment of every list
constexpr size_t kBitsBytes = (size_t)2 << 30;  // bits of the matrix: larger problems go through it piece by piece

// One wave per row at a time: its entries are OR-ed into a bitmap in LDS, which is then written out and cleared.  col: the rows are
// key-major lists, whose bits are queries.  Bound by the memory: entries come in 16-byte pieces, eight kilobytes of a row in flight, and no
// wave waits for another.  L = 32768, four heads, k = 2048 (1.07 GB in, 0.54 out): 289 us, 5.6 TB/s; 408 with a block per row, an entry per lane
// and load, and three barriers.  Long rows leave a CU few bitmaps, and are faster that way too: the transposition of one head of 262144, k = 8192,
// 23.3 -> 16.2 ms; of 524288, two waves per CU, k = 1024 : 8192, 46.7 : 84.4 -> 43.5 : 61.5.
constexpr int kBitsWaves = 4;  // rows per block, at most
__global__ __launch_bounds__(64 * kBitsWaves) void bits_build_kernel(const int32_t *__restrict__ idx, const int64_t *__restrict__ col, int L, HeadTable tab,
                                                                     int slot0, int row0, int nrows, int pitch, uint32_t *__restrict__ bits)
{
    extern __shared__ __align__(16) uint32_t bm_all[];  // [waves][pitch]
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
    uint32_t *bm = bm_all + wave * pitch;
    const int slot = slot0 + blockIdx.y;
    const int32_t *base = idx + tab.off[slot];
    const int64_t *cp = col ? col + (int64_t)tab.bh[slot] * (L + 1) + row0 : nullptr;
    uint32_t *out = bits + (int64_t)blockIdx.y * nrows * pitch;
    for (int w = lane; w < (pitch >> 2); w += 64) reinterpret_cast<uint4 *>(bm)[w] = make_uint4(0u, 0u, 0u, 0u);
    __builtin_amdgcn_wave_barrier();
    auto mark = [&](int v) __attribute__((always_inline)) {
        if ((uint32_t)v < (uint32_t)L) atomicOr(&bm[v >> 5], 1u << (v & 31));
    };
    for (int i = blockIdx.x * waves + wave; i < nrows; i += gridDim.x * waves) {
        const int k = cp ? (int)(cp[i + 1] - cp[i]) : tab.k[slot];
        const int32_t *row = base + (cp ? cp[i] : (int64_t)(row0 + i) * k);
        const int head = min(k, (int)(-(reinterpret_cast<uintptr_t>(row) >> 2) & 3u));  // entries before the first whole piece
        if (lane < head) mark(row[lane]);
        const int4 *piece = reinterpret_cast<const int4 *>(row + head);
        const int pieces = (k - head) >> 2;
        constexpr int U = 8;
        if (pieces <= 64) {  // a path of few instructions: fetching those below takes longer than a short row (L = 511, two heads, k = 51: 4.0 -> 3.3 us; 2336, three, 116: 5.7 -> 4.5)
            if (lane < pieces) {
                const int4 v = piece[lane];
                mark(v.x);
                mark(v.y);
                mark(v.z);
                mark(v.w);
            }
        } else for (int p = lane; p < pieces; p += 64 * U) {
            int4 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = p + 64 * u < pieces ? piece[p + 64 * u] : make_int4(-1, -1, -1, -1);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                mark(v[u].x);
                mark(v[u].y);
                mark(v[u].z);
                mark(v[u].w);
            }
        }
        const int rest = head + 4 * pieces + lane;
        if (rest < k) mark(row[rest]);
        __builtin_amdgcn_wave_barrier();
        uint4 *dst = reinterpret_cast<uint4 *>(out + (int64_t)i * pitch);
        for (int w = lane; w < (pitch >> 2); w += 64) {
            dst[w] = reinterpret_cast<uint4 *>(bm)[w];
            reinterpret_cast<uint4 *>(bm)[w] = make_uint4(0u, 0u, 0u, 0u);
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// Carry-save adder on 32 columns at once: a + b + c = 2 h + l.
__device__ __forceinline__ void csa(uint32_t &h, uint32_t &l, uint32_t a, uint32_t b, uint32_t c)
{
    const uint32_t u = a ^ b;
    h = (a & b) | (u & c);
    l = u ^ c;
}

// cnt2[bh, segment, j] = number of the segment's kBitsRows rows that hold key j.  A thread adds up 64 words of one word
// column with bit-sliced counters (about five logical operations per 32 pairs), the 16 threads of a column meet in LDS.
__global__ __launch_bounds__(256) void bits_count_kernel(const uint32_t *__restrict__ bits, int pitch, int L, HeadTable tab,
                                                         int slot0, int row0, int nrows, int nseg, int32_t *__restrict__ cnt2)
{
    __shared__ int32_t cnt[16 * 33];
    const int bh = tab.bh[slot0 + blockIdx.z];
    const int r_first = blockIdx.y * kBitsRows;  // in this piece
    const int w = threadIdx.x & 15, rl = threadIdx.x >> 4;
    const uint32_t *src = bits + ((int64_t)blockIdx.z * nrows + r_first) * pitch + blockIdx.x * 16 + w;
    const int nr = min(kBitsRows, nrows - r_first);
    for (int e = threadIdx.x; e < 16 * 33; e += 256) cnt[e] = 0;
    __syncthreads();
    uint32_t p0 = 0, p1 = 0, p2 = 0, p3 = 0, p4 = 0, p5 = 0, p6 = 0;  // bit planes of 32 counters
#pragma unroll 2
    for (int g = 0; g < 8; ++g) {
        uint32_t x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int row = rl + 16 * (8 * g + u);
            x[u] = row < nr ? src[(int64_t)row * pitch] : 0u;
        }
        uint32_t a, b, c, d, e;
        csa(a, p0, p0, x[0], x[1]);
        csa(b, p0, p0, x[2], x[3]);
        csa(c, p1, p1, a, b);
        csa(a, p0, p0, x[4], x[5]);
        csa(b, p0, p0, x[6], x[7]);
        csa(d, p1, p1, a, b);
        csa(e, p2, p2, c, d);
        a = p3 & e; p3 ^= e;
        b = p4 & a; p4 ^= a;
        a = p5 & b; p5 ^= b;
        p6 ^= a;
    }
#pragma unroll
    for (int b = 0; b < 32; ++b) {
        const int n = (int)(((p0 >> b) & 1u) + 2u * ((p1 >> b) & 1u) + 4u * ((p2 >> b) & 1u) + 8u * ((p3 >> b) & 1u) +
                            16u * ((p4 >> b) & 1u) + 32u * ((p5 >> b) & 1u) + 64u * ((p6 >> b) & 1u));
        atomicAdd(&cnt[w * 33 + b], n);
    }
    __syncthreads();
    const int seg = (row0 + r_first) / kBitsRows;
    for (int e = threadIdx.x; e < kBitsKeys; e += 256) {
        const int j = blockIdx.x * kBitsKeys + e;
        if (j < L) cnt2[((int64_t)bh * nseg + seg) * L + j] = cnt[(e >> 5) * 33 + (e & 31)];
    }
}

// The 32 lanes of a half-wave hold the 32 rows of a bit block; afterwards lane n holds its column n (bit b from lane b).
struct BitTranspose {
    uint32_t keep[5];
    int amt[5];
    __device__ __forceinline__ explicit BitTranspose(int lane)
    {
        constexpr uint32_t low[5] = {0x0000FFFFu, 0x00FF00FFu, 0x0F0F0F0Fu, 0x33333333u, 0x55555555u};
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            const int s = 16 >> i;
            keep[i] = (lane & s) ? ~low[i] : low[i];
            amt[i] = (lane & s) ? s : 32 - s;
        }
    }
    __device__ __forceinline__ uint32_t step(uint32_t x, uint32_t y, int i) const
    {
        const uint32_t r = __builtin_amdgcn_alignbit(y, y, (uint32_t)amt[i]);
        return (x & keep[i]) | (r & ~keep[i]);
    }
    __device__ __forceinline__ uint32_t operator()(uint32_t x) const
    {
        x = step(x, (uint32_t)__builtin_amdgcn_ds_swizzle((int)x, 0x401F), 0);                              // lane ^ 16
        x = step(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xF, 0xF, false), 1);           // lane ^ 8: row_ror:8
        x = step(x, (uint32_t)__builtin_amdgcn_ds_swizzle((int)x, 0x101F), 2);                              // lane ^ 4
        x = step(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xF, 0xF, false), 3);            // lane ^ 2
        x = step(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xF, 0xF, false), 4);            // lane ^ 1
        return x;
    }
};

// The entries of kBitsRows queries in the lists of kBitsKeys keys.  The block's bits go to LDS (row r at r * 17 + r / 32
// words: both the rows of a 32 x 32 block and the words of one key over the 32 blocks are then 32 different banks apart);
// every wave transposes the blocks of its word columns in place and expands them two keys at a time: lane t of a
// half-wave takes the key's word of queries 32 t .. 32 t + 31, a prefix sum of the bit counts places it in the list.
__global__ __launch_bounds__(512) void bits_fill_kernel(const uint32_t *__restrict__ bits, int pitch, int L, HeadTable tab,
                                                        int slot0, int row0, int nrows, int nseg,
                                                        const int32_t *__restrict__ cnt2, const int32_t *__restrict__ tot,
                                                        const int64_t *__restrict__ col, int32_t *__restrict__ idxT)
{
    constexpr int P = 17;
    __shared__ uint32_t T[kBitsRows * P + kBitsRows / 32];
    __shared__ int64_t o_off[kBitsKeys];
    __shared__ int32_t o_lim[kBitsKeys];
    const int slot = slot0 + blockIdx.z;
    const int bh = tab.bh[slot];
    const int r_first = blockIdx.y * kBitsRows;
    const int nr = min(kBitsRows, nrows - r_first);
    const int seg = (row0 + r_first) / kBitsRows;
    const uint32_t *src = bits + ((int64_t)blockIdx.z * nrows + r_first) * pitch + blockIdx.x * 16;
#pragma unroll
    for (int it = 0; it < 8; ++it) {
        const int e = threadIdx.x + 512 * it;
        const int row = e >> 2, q = (e & 3) * 4;
        uint4 x = make_uint4(0u, 0u, 0u, 0u);
        if (row < nr) x = *reinterpret_cast<const uint4 *>(src + (int64_t)row * pitch + q);
        uint32_t *d = T + row * P + (row >> 5) + q;
        d[0] = x.x; d[1] = x.y; d[2] = x.z; d[3] = x.w;
    }
    {
        // a list's stretch of this segment, from the column sums of the same bits: the entries fill it exactly
        const int j = blockIdx.x * kBitsKeys + threadIdx.x;
        int64_t off = 0;
        int lim = 0;
        if (j < L) {
            const int32_t *c = cnt2 + ((int64_t)bh * nseg + seg) * L + j;
            const int first = c[0];
            const int next = seg + 1 < nseg ? c[L] : tot[(int64_t)bh * L + j];
            off = tab.off[slot] + col[(int64_t)bh * (L + 1) + j] + first;
            lim = next - first;
        }
        o_off[threadIdx.x] = off;
        o_lim[threadIdx.x] = lim;
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = lane & 31, half = lane >> 5;
    const BitTranspose tr(lane);
    const int base_val = row0 + r_first + 32 * n;
#pragma unroll 1
    for (int w = wave; w < 16; w += 8) {
#pragma unroll 4
        for (int i = 0; i < 16; ++i) {
            const int t = 2 * i + half;
            uint32_t *cell = T + (32 * t + n) * P + t + w;
            *cell = tr(*cell);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll 1
        for (int o0 = 0; o0 < 32; o0 += 2) {
            const int o = o0 + half;
            uint32_t m = T[(32 * n + o) * P + n + w];
            const int c = __popc(m);
            const int pos = half_scan(c) - c;
            const int lim = o_lim[w * 32 + o];
            if (pos + c > lim) {  // never with counts of the same bits; keeps anything else inside the list
                const int room = max(lim - pos, 0);
                while (__popc(m) > room) m &= ~(0x80000000u >> __clz(m));
            }
            int32_t *dst = idxT + o_off[w * 32 + o] + pos;
            while (m) {
                *dst++ = base_val + (__ffs(m) - 1);
                m &= m - 1;
            }
        }
    }
}

// Rows in any order -> the same rows in ascending order (one block per row: LDS bitmap, prefix sums of the bit counts,
// expansion).  Entries outside [0, L) and repeated ones, which the index contract excludes, leave the row short: it is
// then filled up with L - 1, so that whatever it held it ends as an ascending row of valid keys.  bits (or null): the bitmaps as
// the bit matrix of the transposition, [head, row][pitch] (L = 20280, four heads keeping 507 .. 4056 keys, the whole
// backward: 7799 -> 7618 us).
__global__ __launch_bounds__(256) void sort_rows_kernel(const int32_t *__restrict__ idx, int L, HeadTable tab,
                                                        int32_t *__restrict__ out, int pitch, uint32_t *__restrict__ bits)
{
    extern __shared__ __align__(16) uint32_t bm[];  // [quarters * 4]
    __shared__ int32_t part[4];
    const int slot = blockIdx.y;
    const int k = tab.k[slot];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int quarter = (((L + 31) / 32 + 3) / 4 + 63) / 64 * 64;  // words per wave, whole steps of 64
    const int32_t *base = idx + tab.off[slot];
    int32_t *obase = out + tab.off[slot];
    for (int w = threadIdx.x; w < 4 * quarter; w += 256) bm[w] = 0u;
    __syncthreads();
    for (int64_t i = blockIdx.x; i < L; i += gridDim.x) {
        const int32_t *row = base + i * k;
        for (int t = threadIdx.x; t < k; t += 256) {
            const int v = row[t];
            if (v >= 0 && v < L) atomicOr(&bm[v >> 5], 1u << (v & 31));
        }
        __syncthreads();
        uint32_t *mine = bm + wave * quarter;
        int sum = 0;
        for (int w = lane; w < quarter; w += 64) sum += __popc(mine[w]);
        for (int o = 32; o; o >>= 1) sum += __shfl_xor(sum, o);
        if (lane == 0) part[wave] = sum;
        __syncthreads();
        int at = 0;
        for (int w = 0; w < wave; ++w) at += part[w];
        int32_t *orow = obase + i * k;
        for (int w = lane; w < quarter; w += 64) {
            uint32_t m = mine[w];
            mine[w] = 0u;
            if (bits && wave * quarter + w < pitch) bits[((int64_t)slot * L + i) * pitch + wave * quarter + w] = m;
            const int c = __popc(m);
            int s = half_scan(c);
            const int low = __shfl(s, 31);
            if (lane >= 32) s += low;
            int32_t *dst = orow + at + s - c;  // at most k distinct entries: inside the row
            const int b0 = (wave * quarter + w) * 32 - 1;
            while (m) {
                *dst++ = b0 + __ffs(m);
                m &= m - 1;
            }
            at += __shfl(s, 63);
        }
        if (wave == 3)
            for (int t = at + lane; t < k; t += 64) orow[t] = L - 1;
        __syncthreads();  // the next row's entries and counts
    }
}

// ------------------------------------------------------------------------------------ scan of the list lengths
// col[bh, 0 .. L] = exclusive prefix sums of cnt[bh, 0 .. L - 1].  A block scans 4096 keys; what lies before them it adds
// up by itself (at most 4 L bytes from L2 per block), so one launch does.
constexpr int kScanKeys = 4096;
__global__ __launch_bounds__(1024) void col_scan_kernel(const int32_t *__restrict__ cnt, int64_t *__restrict__ col, int L,
                                                        HeadTable tab, int slot0)
{
    __shared__ int64_t wsum[16];
    const int64_t bh = tab.bh[slot0 + blockIdx.y];
    const int32_t *c = cnt + bh * L;
    int64_t *o = col + bh * (L + 1);
    const int j0 = blockIdx.x * kScanKeys;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int64_t before = 0;
#pragma unroll 4
    for (int j = threadIdx.x; j < j0; j += 1024) before += c[j];
    const int a = j0 + threadIdx.x * 4;
    int64_t v[4], s = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        v[u] = s;
        s += a + u < L ? c[a + u] : 0;
    }
    // block-wide: total of `before`, exclusive scan of s
    for (int d = 32; d; d >>= 1) before += __shfl_xor(before, d);
    int64_t incl = s;
    for (int d = 1; d < 64; d <<= 1) {
        const int64_t up = __shfl_up(incl, d);
        if (lane >= d) incl += up;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    int64_t run = incl - s;
    for (int w = 0; w < wave; ++w) run += wsum[w];
    __syncthreads();
    if (lane == 0) wsum[wave] = before;
    __syncthreads();
    for (int w = 0; w < 16; ++w) run += wsum[w];
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (a + u < L) o[a + u] = run + v[u];
    if (a < L && a + 4 >= L) o[L] = run + s;
}

dsv_status launch_col_scan(const int32_t *cnt, int64_t *col, int L, const HeadTable &tab, hipStream_t st)
{
    hipLaunchKernelGGL(col_scan_kernel, dim3((L + kScanKeys - 1) / kScanKeys, tab.n), dim3(1024), 0, st, cnt, col, L, tab, 0);
    DSV_LAUNCH_CHECK();
    return DSV_OK;
}

// ------------------------------------------------------------------------------------ entry sort
// A stable counting sort by key, so that every list comes out in ascending query order whatever the order inside the
// rows is (the L2-blocked key-major sweep needs ascending lists) and the result is the same from run to run:
//   count    the queries are cut into chunks of consecutive rows; cnt2[bh, chunk, j] = rows of the chunk holding j
//            (integer atomics: the counts do not depend on the order of arrival);
//   offsets  per key, an exclusive scan over the chunks (cnt2 becomes the chunk's first position inside the key's
//            list) and the key's total; the totals are scanned into col as before;
//   fill     one block per chunk walks its rows in ascending order, one row at a time; the entries of a row are
//            distinct keys, so the threads bump the chunk's cursors with plain loads and stores.
constexpr int kTransposeChunks = 256;  // at most this many query chunks per head (cnt2 holds chunks x L counters; 1024
                                       // chunks measured no faster: both passes are bound by scattered 4-byte requests)

__host__ __device__ __forceinline__ int transpose_chunk_rows(int L)
{
    const int r = (L + kTransposeChunks - 1) / kTransposeChunks;
    return r < 64 ? 64 : r;
}

__global__ __launch_bounds__(256) void tindex_count_kernel(const int32_t *__restrict__ idx, int L, int n_chunks,
                                                           HeadTable tab, int32_t *__restrict__ cnt2)
{
    const int slot = blockIdx.y;
    const int bh = tab.bh[slot];
    const int k = tab.k[slot];
    const int rc = transpose_chunk_rows(L);
    const int chunk = blockIdx.x;
    const int32_t *base = idx + tab.off[slot];
    int32_t *c = cnt2 + ((int64_t)bh * n_chunks + chunk) * L;
    const int i1 = min((chunk + 1) * rc, L);
    for (int64_t i = (int64_t)chunk * rc; i < i1; ++i) {
        const int32_t *row = base + i * k;
        for (int t = threadIdx.x; t < k; t += 256) {
            const int j = row[t];
            if (j >= 0 && j < L) atomicAdd(&c[j], 1);
        }
    }
}

// thread per key: cnt2[bh, c, j] <- number of rows in chunks before c holding j; tot[bh, j] <- all of them
__global__ __launch_bounds__(256) void tindex_offsets_kernel(int32_t *__restrict__ cnt2, int32_t *__restrict__ tot, int L,
                                                             int n_chunks, HeadTable tab, int slot0)
{
    const int64_t bh = tab.bh[slot0 + blockIdx.y];
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= L) return;
    int32_t *c = cnt2 + bh * n_chunks * L + j;
    int run = 0;
    for (int ch = 0; ch < n_chunks; ++ch) {
        const int v = c[(int64_t)ch * L];
        c[(int64_t)ch * L] = run;
        run += v;
    }
    tot[bh * L + j] = run;
}

__global__ __launch_bounds__(256) void tindex_fill_kernel(const int32_t *__restrict__ idx, int L, int n_chunks,
                                                          HeadTable tab, int32_t *__restrict__ cnt2,
                                                          const int64_t *__restrict__ col, int32_t *__restrict__ idxT)
{
    const int slot = blockIdx.y;
    const int bh = tab.bh[slot];
    const int k = tab.k[slot];
    const int rc = transpose_chunk_rows(L);
    const int chunk = blockIdx.x;
    const int32_t *base = idx + tab.off[slot];
    int32_t *out = idxT + tab.off[slot];
    int32_t *cur = cnt2 + ((int64_t)bh * n_chunks + chunk) * L;  // this chunk's next position inside every list
    const int64_t *cp = col + (int64_t)bh * (L + 1);
    const int i1 = min((chunk + 1) * rc, L);
    constexpr int U = 8;  // entries a thread has in flight: the loads of all U come before the first store
    for (int64_t i = (int64_t)chunk * rc; i < i1; ++i) {
        const int32_t *row = base + i * k;
        for (int t0 = threadIdx.x; t0 < k; t0 += 256 * U) {
            int j[U], pos[U];
            int64_t dst[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int t = t0 + u * 256;
                j[u] = t < k ? row[t] : -1;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool ok = j[u] >= 0 && j[u] < L;
                pos[u] = ok ? cur[j[u]] : 0;   // no other thread touches cur[j] during this row: a row's keys are distinct
                dst[u] = ok ? cp[j[u]] + pos[u] : -1;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (j[u] >= 0 && j[u] < L) {
                    cur[j[u]] = pos[u] + 1;
                    // col and the cursors come from the counting pass over the same idx, so dst stays inside the
                    // head's L * k entries; the bound keeps a broken idx (duplicates, changed between the passes)
                    // from sending the store anywhere else
                    if (dst[u] >= 0 && dst[u] < (int64_t)L * k) out[dst[u]] = (int32_t)i;
                }
            }
        }
        __syncthreads();  // the next row may bump the same cursors
    }
}

__global__ __launch_bounds__(256) void fill_zero_i32_kernel(int4 *__restrict__ p, int64_t n4)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n4; e += stride) p[e] = make_int4(0, 0, 0, 0);
}

// ------------------------------------------------------------------------------------ host
// Where rows would lie whole kilobytes apart, 64 bytes more: the words that the waves of the chip read together, one of every row, otherwise
// come from a few of the L2's channels (forward over dense tiles, L = 131072, one head, k = 8192: 12.43 -> 11.99 ms; L = 32768, four heads, k = 2048:
// 3.04 -> 2.91).  The largest rows stay as long as the bitmap in LDS may be.
static int bits_words(int L) { return (L + kBitsKeys - 1) / kBitsKeys * 16; }
int bits_pitch(int L)
{
    const int words = bits_words(L);
    return words % 256 == 0 && L <= kBitsMaxKeys / 2 ? words + 16 : words;
}
// Limits of scratch hold for the bits alone: rows with space between them are those of lengths that fill such a limit exactly (131072 keys
// and queries: 2 GB), and would come in a piece more.  That length, one head, transposed, k = 512 : 8192: 2.81 : 5.80 ms in two pieces, 2.30 : 4.51
// in one; its forward, d = 64, k = 8192: 10.8 ms in three, 7.9 in two.
size_t bits_rows(int L, size_t bytes) { return bytes / ((size_t)bits_words(L) * 4); }

dsv_status launch_bits_build(const dsv_problem &p, const HeadTable &tab, int slot0, int heads, const int32_t *idx, int row0,
                             int nrows, uint32_t *bits, hipStream_t st, const int64_t *col)
{
    const int pitch = bits_pitch(p.L);
    const int waves = std::max(1, std::min(kBitsWaves, (64 << 10) / (pitch * 4)));  // 64 KB of bitmaps
    hipLaunchKernelGGL(bits_build_kernel, dim3(std::min((nrows + waves - 1) / waves, 8192 / waves), heads), dim3(64 * waves), (size_t)waves * pitch * 4, st, idx,
                       col, p.L, tab, slot0, row0, nrows, pitch, bits);
    DSV_LAUNCH_CHECK();
    return DSV_OK;
}

struct TransposePlan {
    bool bits;
    int n_chunks;       // segments (bit matrix) or chunks (entry sort) of queries per head
    int pitch;          // words per row of the bit matrix
    int heads, rows;    // heads and rows per piece of the bit matrix
    size_t tot, cnt2, mat, total;
};

static TransposePlan transpose_plan(const dsv_problem &p)
{
    TransposePlan w{};
    const size_t nbh = (size_t)p.B * p.H;
    int64_t sum_k = 0;
    for (int h = 0; h < p.H; ++h) sum_k += p.k_per_head[h];
    // The bit matrix costs nearly the same whatever a row keeps, the entry sort 50 to 100 ps per entry: measured per head, bits
    // against entries, 168 : 284 us at L = 32768, k = 32; 2.4 : 2.1 ms at L = 131072, k = 128 and 2.4 : 3.7 ms at k = 256;
    // 2.7 : 11.8 ms at k = 1024; 3.7 : 49 ms at k = 4096.
    w.bits = p.L <= kBitsMaxKeys && sum_k * 768 >= (int64_t)p.H * p.L;
    const int rc = transpose_chunk_rows(p.L);
    w.n_chunks = w.bits ? (p.L + kBitsRows - 1) / kBitsRows : (p.L + rc - 1) / rc;
    size_t o = 0;
    w.tot = o; o = align_up(o + nbh * p.L * 4, 256);
    w.cnt2 = o; o = align_up(o + nbh * w.n_chunks * p.L * 4, 256);
    w.mat = o;
    if (w.bits) {
        w.pitch = bits_pitch(p.L);
        const size_t row = (size_t)w.pitch * 4;
        const size_t fit = bits_rows(p.L, kBitsBytes);
        if (fit >= (size_t)p.L) {
            w.heads = (int)std::min<size_t>({fit / p.L, nbh, (size_t)kMaxSlots});
            w.rows = p.L;
        } else {
            w.heads = 1;
            w.rows = (int)(fit / kBitsRows * kBitsRows);  // fit >= 32768 rows (row <= 64 KB)
        }
        o = align_up(o + row * w.heads * w.rows, 256);
    }
    w.total = o;
    return w;
}

size_t idx_transpose_bytes(const dsv_problem &p) { return transpose_plan(p).total; }

static dsv_status transpose_bits(const dsv_problem &p, const HeadTable &tab, const TransposePlan &w, const int32_t *idx, bool built,
                                 int32_t *idxT, int64_t *col, char *ws, hipStream_t st)
{
    int32_t *tot = reinterpret_cast<int32_t *>(ws + w.tot), *cnt2 = reinterpret_cast<int32_t *>(ws + w.cnt2);
    uint32_t *bits = reinterpret_cast<uint32_t *>(ws + w.mat);
    const unsigned kb = (p.L + kBitsKeys - 1) / kBitsKeys;
    const bool whole = w.rows >= p.L;        // the piece built for counting still stands when the lists are filled
    for (int s0 = 0; s0 < tab.n; s0 += w.heads) {
        const unsigned nh = std::min(w.heads, tab.n - s0);
        for (int fill = 0; fill < 2; ++fill) {
            for (int r0 = 0; r0 < p.L; r0 += w.rows) {
                const int nr = std::min(w.rows, p.L - r0);
                const dim3 grid(kb, (nr + kBitsRows - 1) / kBitsRows, nh);
                if (!built && (!fill || !whole)) {
                    const dsv_status rc = launch_bits_build(p, tab, s0, nh, idx, r0, nr, bits, st);
                    if (rc != DSV_OK) return rc;
                }
                if (!fill)
                    hipLaunchKernelGGL(bits_count_kernel, grid, dim3(256), 0, st, bits, w.pitch, p.L, tab, s0, r0, nr, w.n_chunks, cnt2);
                else
                    hipLaunchKernelGGL(bits_fill_kernel, grid, dim3(512), 0, st, bits, w.pitch, p.L, tab, s0, r0, nr, w.n_chunks, cnt2,
                                       tot, col, idxT);
                DSV_LAUNCH_CHECK();
            }
            if (!fill) {
                hipLaunchKernelGGL(tindex_offsets_kernel, dim3((p.L + 255) / 256, nh), dim3(256), 0, st, cnt2, tot, p.L, w.n_chunks,
                                   tab, s0);
                hipLaunchKernelGGL(col_scan_kernel, dim3((p.L + kScanKeys - 1) / kScanKeys, nh), dim3(1024), 0, st, tot, col, p.L, tab, s0);
                DSV_LAUNCH_CHECK();
            }
        }
    }
    return DSV_OK;
}

static dsv_status transpose_entries(const dsv_problem &p, const HeadTable *tabs, int n_tabs, const TransposePlan &w,
                                    const int32_t *idx, int32_t *idxT, int64_t *col, char *ws, hipStream_t st)
{
    int32_t *tot = reinterpret_cast<int32_t *>(ws + w.tot), *cnt2 = reinterpret_cast<int32_t *>(ws + w.cnt2);
    const int64_t ncnt4 = (int64_t)((w.total - w.cnt2) / 16);
    const int zero_blocks = (int)std::min<int64_t>((ncnt4 + 255) / 256, 4096);
    hipLaunchKernelGGL(fill_zero_i32_kernel, dim3(zero_blocks), dim3(256), 0, st, (int4 *)cnt2, ncnt4);
    DSV_LAUNCH_CHECK();
    for (int t = 0; t < n_tabs; ++t) {
        hipLaunchKernelGGL(tindex_count_kernel, dim3(w.n_chunks, tabs[t].n), dim3(256), 0, st, idx, p.L, w.n_chunks, tabs[t], cnt2);
        hipLaunchKernelGGL(tindex_offsets_kernel, dim3((p.L + 255) / 256, tabs[t].n), dim3(256), 0, st, cnt2, tot, p.L, w.n_chunks,
                           tabs[t], 0);
        DSV_LAUNCH_CHECK();
        const dsv_status rc = launch_col_scan(tot, col, p.L, tabs[t], st);
        if (rc != DSV_OK) return rc;
        hipLaunchKernelGGL(tindex_fill_kernel, dim3(w.n_chunks, tabs[t].n), dim3(256), 0, st, idx, p.L, w.n_chunks, tabs[t], cnt2,
                           col, idxT);
        DSV_LAUNCH_CHECK();
    }
    return DSV_OK;
}

uint32_t *transpose_matrix(const dsv_problem &p, void *ws)
{
    const TransposePlan w = transpose_plan(p);
    const size_t nbh = (size_t)p.B * p.H;
    return w.bits && w.rows >= p.L && (size_t)w.heads >= nbh ? reinterpret_cast<uint32_t *>(static_cast<char *>(ws) + w.mat) : nullptr;
}

dsv_status launch_idx_transpose(const dsv_problem &p, const HeadTable *tabs, int n_tabs, const int32_t *idx, bool built,
                                int32_t *idxT, int64_t *col, void *ws, size_t ws_bytes, hipStream_t st)
{
    const TransposePlan w = transpose_plan(p);
    if (ws_bytes < w.total) return DSV_EWORKSPACE;
    if (!w.bits) return transpose_entries(p, tabs, n_tabs, w, idx, idxT, col, static_cast<char *>(ws), st);
    for (int t = 0; t < n_tabs; ++t) {
        const dsv_status rc = transpose_bits(p, tabs[t], w, idx, built, idxT, col, static_cast<char *>(ws), st);
        if (rc != DSV_OK) return rc;
    }
    return DSV_OK;
}

bool can_sort_rows(const dsv_problem &p) { return p.L <= kBitsMaxKeys; }

dsv_status launch_sort_rows(const dsv_problem &p, const HeadTable *tabs, int n_tabs, const int32_t *idx, int32_t *out,
                            uint32_t *bits, hipStream_t st)
{
    const size_t lds = (size_t)((((p.L + 31) / 32 + 3) / 4 + 63) / 64 * 64) * 16;  // as in the kernel: at most 64 KB
    for (int t = 0; t < n_tabs; ++t) {
        hipLaunchKernelGGL(sort_rows_kernel, dim3(std::min(p.L, 4096), tabs[t].n), dim3(256), lds, st, idx, p.L, tabs[t], out,
                           bits_pitch(p.L), bits);
        DSV_LAUNCH_CHECK();
    }
    return DSV_OK;
}

}  // namespace dsv
