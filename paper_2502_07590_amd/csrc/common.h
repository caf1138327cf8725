// Shared device/host helpers of libdsv (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dsv.h"

namespace dsv {

// bf16 tensors are handled as raw 16-bit patterns.
typedef uint16_t bf16_t;

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4_t;

constexpr int kWave = 64;
constexpr int64_t kMaxKeys = (1 << 25) - 1;  // keys of a head: its matrix is below 4 GB, the shortest row (bf16, d = 64) has 128 bytes
constexpr int kMaxSlots = 64;  // (batch, head) pairs described by one kernel launch

// Per-launch table of the (batch, head) pairs a grid works on, passed by value as a kernel
// argument.  Slots are ordered by descending k so that the heaviest heads are dispatched first.
struct HeadTable {
    int32_t n;
    int32_t bh[kMaxSlots];   // b * H + h
    int32_t k[kMaxSlots];    // KV kept per query in that head
    int64_t off[kMaxSlots];  // element offset of the head's [L, k] block inside idx
};

__device__ __forceinline__ float bf16_to_f32(bf16_t v) { return __uint_as_float(((uint32_t)v) << 16); }

// Round-to-nearest-even fp32 -> bf16 for finite inputs.
__device__ __forceinline__ bf16_t f32_to_bf16(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (bf16_t)(u >> 16);
}

template <typename T> __device__ __forceinline__ float to_f32(T v);
template <> __device__ __forceinline__ float to_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ float to_f32<bf16_t>(bf16_t v) { return bf16_to_f32(v); }

template <typename T> __device__ __forceinline__ T from_f32(float v);
template <> __device__ __forceinline__ float from_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ bf16_t from_f32<bf16_t>(float v) { return f32_to_bf16(v); }

// Sum over the 16 lanes of a DPP row; every lane of the row ends with the total.
__device__ __forceinline__ float row16_sum(float x)
{
    // row_ror:8, :4, :2, :1 (rotations inside each group of 16 lanes)
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x128, 0xF, 0xF, false));
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x124, 0xF, 0xF, false));
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x122, 0xF, 0xF, false));
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x121, 0xF, 0xF, false));
    return x;
}

// Sum over the LPR (4, 8 or 16) consecutive lanes that share one row; every lane ends with the total.
template <int LPR> __device__ __forceinline__ float row_sum(float x)
{
    static_assert(LPR == 4 || LPR == 8 || LPR == 16, "lanes per row");
    if constexpr (LPR == 16) {
        return row16_sum(x);
    } else {
        if constexpr (LPR == 8)  // row_half_mirror: lane i <-> 7 - i inside each group of 8
            x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x141, 0xF, 0xF, false));
        x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xB1, 0xF, 0xF, false));  // quad_perm [1,0,3,2]
        x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x4E, 0xF, 0xF, false));  // quad_perm [2,3,0,1]
        return x;
    }
}

__device__ __forceinline__ float row16_max(float x)
{
    x = fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x128, 0xF, 0xF, false)));
    x = fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x124, 0xF, 0xF, false)));
    x = fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x122, 0xF, 0xF, false)));
    x = fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x121, 0xF, 0xF, false)));
    return x;
}

// Inclusive prefix sum inside each half-wave (lanes 0..31 and lanes 32..63 separately).
__device__ __forceinline__ int half_scan(int x)
{
    int s = x;
    s += __builtin_amdgcn_update_dpp(0, s, 0x111, 0xF, 0xF, false);  // row_shr:1 (rows of 16 lanes, zero fill)
    s += __builtin_amdgcn_update_dpp(0, s, 0x112, 0xF, 0xF, false);  // row_shr:2
    s += __builtin_amdgcn_update_dpp(0, s, 0x114, 0xF, 0xF, false);  // row_shr:4
    s += __builtin_amdgcn_update_dpp(0, s, 0x118, 0xF, 0xF, false);  // row_shr:8
    s += __builtin_amdgcn_update_dpp(0, s, 0x142, 0xA, 0xF, false);  // row_bcast15 into rows 1 and 3
    return s;
}

// The same inside each row of 16 lanes.
__device__ __forceinline__ int row_scan(int x)
{
    int s = x;
    s += __builtin_amdgcn_update_dpp(0, s, 0x111, 0xF, 0xF, false);
    s += __builtin_amdgcn_update_dpp(0, s, 0x112, 0xF, 0xF, false);
    s += __builtin_amdgcn_update_dpp(0, s, 0x114, 0xF, 0xF, false);
    s += __builtin_amdgcn_update_dpp(0, s, 0x118, 0xF, 0xF, false);
    return s;
}

// Transposing LDS read (ds_read_b64_tr_b16): inside every block of 16 lanes, lane i receives four halfwords, the
// e-th being halfword (i % 4) at the address passed by lane 4 e + i / 4 of the block.  So when lane 4 e + q
// passes the address of channels c0 + 4 q .. + 3 of parked row key(e), lane i ends up with channel c0 + i of rows
// key(0..3): a quarter of a matrix-core B fragment whose contraction runs over the parked rows.  Two reads
// (rows key(0..3), key(4..7)) make the 8-element fragment.
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;
__device__ __forceinline__ bf16x8_t tr_frag(const unsigned char *a0, const unsigned char *a1)
{
    const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t *)a0);
    const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t *)a1);
    typedef short s16x8_t __attribute__((ext_vector_type(8)));
    const s16x8_t f = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8_t, f);
}

// ---- a lane's share of one [d]-row: CH channels, kept as raw 32-bit words --------------------
template <typename T, int CH> struct RowChunk {
    static constexpr int NW = CH * (int)sizeof(T) / 4;
    uint32_t w[NW];
};

// How the LPR lanes of a group share a row of D elements.  A lane's chunk is made of 16-byte pieces;
// its i-th piece is the lane's slot in the row's i-th strip of LPR * 16 bytes, so that one load
// instruction of the whole group covers whole strips -- whole cache lines -- instead of every other
// 16 bytes of twice as many lines (the vector memory path charges by the lines an instruction touches).
// Chunks shorter than 16 bytes are a single piece and lie side by side.
template <typename T, int D, int LPR> struct LaneLayout {
    static constexpr int CH = D / LPR;
    static constexpr int BYTES = CH * (int)sizeof(T);
    static constexpr int PE = BYTES >= 16 ? 16 / (int)sizeof(T) : CH;  // elements per piece
    static constexpr int PIECES = CH / PE;
    static constexpr int PSB = BYTES >= 16 ? LPR * 16 : 16;            // bytes from one piece to the next
    // element offset of lane s's first piece inside the row
    __device__ __forceinline__ static constexpr int off(int s) { return s * PE; }
    // true channel of the lane's c-th chunk element
    __device__ __forceinline__ static constexpr int channel(int s, int c) { return (c / PE) * (LPR * PE) + s * PE + c % PE; }
};

// The chunks of a group's lanes must tile the row: every channel owned by exactly one (lane, element).
template <typename T, int D, int LPR> constexpr bool lane_layout_tiles_the_row()
{
    typedef LaneLayout<T, D, LPR> LL;
    bool seen[D] = {};
    for (int s = 0; s < LPR; ++s)
        for (int c = 0; c < LL::CH; ++c) {
            const int ch = (c / LL::PE) * (LPR * LL::PE) + s * LL::PE + c % LL::PE;  // = LL::channel(s, c)
            if (ch < 0 || ch >= D || seen[ch]) return false;
            seen[ch] = true;
        }
    return true;
}
static_assert(lane_layout_tiles_the_row<uint16_t, 128, 4>() && lane_layout_tiles_the_row<uint16_t, 128, 8>() &&
              lane_layout_tiles_the_row<uint16_t, 128, 16>() && lane_layout_tiles_the_row<uint16_t, 64, 4>() &&
              lane_layout_tiles_the_row<uint16_t, 64, 16>() && lane_layout_tiles_the_row<float, 128, 8>() &&
              lane_layout_tiles_the_row<float, 128, 16>() && lane_layout_tiles_the_row<float, 64, 4>() &&
              lane_layout_tiles_the_row<float, 64, 8>(), "LaneLayout must be a permutation of the row's channels");

// PSB: bytes between the chunk's consecutive 16-byte pieces (16 = contiguous).
template <typename T, int CH, int PSB = 16>
__device__ __forceinline__ RowChunk<T, CH> load_chunk(const T *p)
{
    RowChunk<T, CH> c;
    constexpr int NW = RowChunk<T, CH>::NW;
    if constexpr (NW == 2) {
        uint2 v = *reinterpret_cast<const uint2 *>(p);
        c.w[0] = v.x; c.w[1] = v.y;
    } else {
        static_assert(NW % 4 == 0, "row chunk must be 8 bytes or a multiple of 16 bytes");
#pragma unroll
        for (int i = 0; i < NW / 4; ++i) {
            uint4 v = *reinterpret_cast<const uint4 *>(reinterpret_cast<const char *>(p) + i * PSB);
            c.w[4 * i + 0] = v.x; c.w[4 * i + 1] = v.y; c.w[4 * i + 2] = v.z; c.w[4 * i + 3] = v.w;
        }
    }
    return c;
}

template <typename T, int CH, int PSB = 16>
__device__ __forceinline__ void store_chunk(T *p, const float (&f)[CH])
{
    constexpr int NW = RowChunk<T, CH>::NW;
    uint32_t w[NW];
    if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int i = 0; i < CH; ++i) w[i] = __float_as_uint(f[i]);
    } else {
#pragma unroll
        for (int i = 0; i < CH / 2; ++i)
            w[i] = (uint32_t)f32_to_bf16(f[2 * i]) | ((uint32_t)f32_to_bf16(f[2 * i + 1]) << 16);
    }
    if constexpr (NW == 2) {
        *reinterpret_cast<uint2 *>(p) = make_uint2(w[0], w[1]);
    } else {
#pragma unroll
        for (int i = 0; i < NW / 4; ++i)
            *reinterpret_cast<uint4 *>(reinterpret_cast<char *>(p) + i * PSB) =
                make_uint4(w[4 * i], w[4 * i + 1], w[4 * i + 2], w[4 * i + 3]);
    }
}

// fp32 accumulators of a lane whose chunk follows LaneLayout<T, D, LPR>, written to a plain [D] float
// row in true channel order (the partial results of the split kernels).
template <typename T, int D, int LPR>
__device__ __forceinline__ void store_acc(float *row, int s, const float (&f)[D / LPR])
{
    typedef LaneLayout<T, D, LPR> LL;
#pragma unroll
    for (int i = 0; i < LL::PIECES; ++i) {
        float *dst = row + LL::channel(s, i * LL::PE);
#pragma unroll
        for (int e = 0; e < LL::PE; e += 4)
            *reinterpret_cast<float4 *>(dst + e) = make_float4(f[i * LL::PE + e], f[i * LL::PE + e + 1], f[i * LL::PE + e + 2], f[i * LL::PE + e + 3]);
    }
}

// Partial dot product of two row chunks (this lane's CH channels), fp32 accumulation.
template <typename T, int CH>
__device__ __forceinline__ float dot_chunk(const RowChunk<T, CH> &a, const RowChunk<T, CH> &b)
{
    float acc = 0.f;
    if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int i = 0; i < CH; ++i) acc = fmaf(__uint_as_float(a.w[i]), __uint_as_float(b.w[i]), acc);
    } else {
#pragma unroll
        for (int i = 0; i < CH / 2; ++i)
            acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a.w[i]),
                                                  __builtin_bit_cast(bf16x2_t, b.w[i]), acc, false);
    }
    return acc;
}

// ---- host side ------------------------------------------------------------------------------
#define DSV_HIP_CHECK(expr)                         \
    do {                                            \
        hipError_t e_ = (expr);                     \
        if (e_ != hipSuccess) return DSV_EHIP;      \
    } while (0)

#define DSV_LAUNCH_CHECK()                                  \
    do {                                                    \
        if (hipGetLastError() != hipSuccess) return DSV_EHIP; \
    } while (0)

static inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Measurement aid behind dsv_kernel_timing / dsv_kernel_ms: when switched on, a KernelSpan records one
// HIP event on the launch stream before and one after the kernel launches it encloses.
struct KernelTimer {
    bool on = false;
    hipEvent_t ev[DSV_KERNEL_COUNT][2] = {};
    bool recorded[DSV_KERNEL_COUNT] = {};
    bool open[DSV_KERNEL_COUNT] = {};  // inside a span of that kind: a nested one is part of it
};
extern KernelTimer g_kernel_timer;
struct KernelSpan {
    int id;
    hipStream_t st;
    bool outer;
    KernelSpan(int id_, hipStream_t st_) : id(id_), st(st_), outer(g_kernel_timer.on && !g_kernel_timer.open[id_])
    {
        if (!outer) return;
        g_kernel_timer.open[id] = true;
        (void)hipEventRecord(g_kernel_timer.ev[id][0], st);
    }
    ~KernelSpan()
    {
        if (!outer) return;
        g_kernel_timer.open[id] = false;
        g_kernel_timer.recorded[id] = hipEventRecord(g_kernel_timer.ev[id][1], st) == hipSuccess;
    }
};

// Host: entry points of the per-stage translation units (called from api.hip).
// Lq: query rows per head in Q / Qlr (p.L for per-query selection; one proxy per group with query grouping);
// K / Klr always hold p.L rows.
dsv_status launch_project(const dsv_problem &p, int Lq, const void *Q, const void *K, const void *Wq, const void *Wk,
                          void *Qlr, void *Klr, hipStream_t st);
dsv_status launch_scores_rows(const dsv_problem &p, const void *Qlr, const void *Klr, int bh,
                              const int32_t *rows, int n_rows, float *scores, hipStream_t st);
// ---- L2-blocked (split-K) form of stage 2 -----------------------------------------------------
// Target bytes of K+V (or Q+dO) rows per key (query) range, against a 4 MB L2 per XCD.  Measured at
// L = 128k (bf16, d = 128): the forward runs best with 2 MB ranges (32 per head: 121 ms, 3 MB: 123,
// 4 MB: 124), the backward steps -- whose partial results are twice as large per range -- with 4 MB
// (dq 132 / 131 / 135 ms and dkdv 158 / 162 / 164 ms at 4 / 3 / 2 MB); 8 ranges per head are 20 % slower.
constexpr size_t kFwdRangeBytes = 2u << 20;
constexpr size_t kBwdRangeBytes = 4u << 20;
constexpr size_t kMaxRangeRows = 8192;  // rows of a range: 8 bytes of row statistics each fit 64 KB of LDS

// A key-major list of GROUPS standing for the per-query list it expands to (queries in group-major order: group g
// holds queries g G .. g G + G - 1): position pos of the expanded list is entry pos / G of the stored one, times G,
// plus pos % G.  G = 1: a plain list.  magic = floor(2^32 / G) + 1 divides positions below 2^32 / G exactly.
struct GroupExpand {
    int32_t G;
    uint32_t magic;
};
__host__ __device__ __forceinline__ GroupExpand no_expand() { return GroupExpand{1, 0u}; }
__host__ __forceinline__ GroupExpand make_expand(int G) { return GroupExpand{G, (uint32_t)((1ull << 32) / (uint64_t)G) + 1u}; }
__device__ __forceinline__ int32_t expanded_entry(const int32_t *__restrict__ list, int pos, const GroupExpand &ge)
{
    if (ge.G == 1) return list[pos];
    const int q = (int)__umulhi((uint32_t)pos, ge.magic);
    return list[q] * ge.G + (pos - q * ge.G);
}

struct SplitPlan {
    int range_len;  // keys (queries) per range
    int S;          // ranges
    int S_pad;      // ranges as laid out over the XCDs: 2, 4 or a multiple of 8, at least S
    int nqb;        // row blocks per range (each kernel sets it from its own rows per block)
};
SplitPlan make_split_plan(const dsv_problem &p, size_t range_bytes, bool few);
constexpr int64_t kFewRangesBlocks = 4096;
__host__ __forceinline__ int64_t row_blocks(const dsv_problem &p) { return (int64_t)p.B * p.H * ((p.L + 63) / 64); }

// Work items (row block, range) of a head: linear id -> range and row block, consecutive ids on consecutive XCDs.  Eight ranges or
// more: an XCD (one of eight) walks the blocks of its own ranges one range after the other.  One, two or four: the XCDs that
// share a range take its blocks in turn.
__host__ __device__ __forceinline__ int64_t range_items(int S_pad, int nqb)
{
    return S_pad < 8 ? 8ll * ((nqb * S_pad + 7) / 8) : (int64_t)S_pad * nqb;
}
__device__ __forceinline__ bool decode_range_item(int S, int S_pad, int nqb, int64_t b, int &slot, int &range, int &rb)
{
    const int64_t per_head = range_items(S_pad, nqb);
    slot = (int)(b / per_head);
    const int rem = (int)(b - (int64_t)slot * per_head);
    const int xcd = rem & 7, local = rem >> 3;
    if (S_pad < 8) {
        const int share = 8 / S_pad;
        range = xcd % S_pad;
        rb = local * share + xcd / S_pad;
    } else {
        const int t = local / nqb;
        rb = local - t * nqb;
        range = t * 8 + xcd;
    }
    return range < S && rb < nqb;
}

struct FwdSplitWorkspace {
    int32_t *seg;  // [B*H, L, S+1] segment pointers into every idx row
    float *pm;     // [B*H, L, S]    partial running max (log2 domain)
    float *pl;     // [B*H, L, S]    partial normaliser
    float *pacc;   // [B*H, L, S, d] partial unnormalised output
    int32_t *hist;   // [B*H, S, range_len + 1]  rows per segment length (then their start offsets)
    int32_t *order;  // [B*H, S, L]  rows of every (head, range) by descending segment length
};
dsv_status launch_sparse_fwd_split(const dsv_problem &p, const HeadTable *tabs, int n_tabs, const void *Q,
                                   const void *K, const void *V, const int32_t *idx, void *O, float *lse,
                                   const SplitPlan &pl, const FwdSplitWorkspace &w, hipStream_t st);

// Scratch of one split backward step (dq: A, B, Delta partials; dkdv: dK, dV partials).
struct BwdSplitWorkspace {
    int32_t *seg;   // [B*H, L, S+1]
    float *pa;      // [B*H, L, S, d]
    float *pb;      // [B*H, L, S, d]
    float *pdelta;  // [B*H, L, S]   (dq step only)
    int32_t *hist;  // [B*H, S, range_len + 1]  rows per segment length (then their start offsets)
    int32_t *order; // [B*H, S, L]   rows of every (head, range) by descending segment length
    float2 *rowstat;  // [B*H, L]    {lse * log2(e), Delta} per query (dkdv step only)
};
// Heads of a ranged backward step that form every pair of a tile (dense_bwd.hip; bf16, scale > 0, L <= kBitsMaxKeys): their
// partial results take the same places.  mask: scratch, at least kDenseMinRows rows of it.
struct DenseHeads {
    const HeadTable *tabs;
    int n_tabs;
    char *mask;
    size_t mask_bytes;
    const int32_t *rows;   // dq step: their index rows, in any order (null: those of the call)
    const uint32_t *bits;  // dq step: the masks of all of them [heads, L, bits_pitch(L)], in the order of the (one) table; null: to be built
};
dsv_status launch_dense_bwd(const dsv_problem &p, const HeadTable &tab, bool keys, const void *Q, const void *K, const void *V, const int32_t *index,
                            const int64_t *col, const void *O, const float *lse, const void *dO, const SplitPlan &plan,
                            const BwdSplitWorkspace &w, const DenseHeads &dense, hipStream_t st);
dsv_status launch_bwd_dq_split(const dsv_problem &p, const HeadTable *tabs, int n_tabs, const DenseHeads &dense, const void *Q, const void *K,
                               const void *V, const int32_t *idx, const void *O, const float *lse, const void *dO,
                               void *dQ, float *delta, const SplitPlan &pl, const BwdSplitWorkspace &w, hipStream_t st);
dsv_status launch_bwd_dkdv_split(const dsv_problem &p, const HeadTable *tabs, int n_tabs, const DenseHeads &dense, const void *Q,
                                 const void *K, const void *V, const int32_t *idxT, const int64_t *col,
                                 const float *lse, const float *delta, const void *dO, void *dK, void *dV,
                                 const SplitPlan &pl, const BwdSplitWorkspace &w, hipStream_t st, int expand_G = 1,
                                 const int32_t *skip = nullptr);
// expand_G > 1: idxT / col hold lists of groups of expand_G queries (tabs[].off the offsets of those lists); the sweep
// runs on the per-query lists they stand for.  Needs p.L < 2^32 / expand_G.  skip (device, [B*H], or null): heads that something else has
// swept, into the partial results (with a single range, into dK and dV); w.rowstat is then filled already.

// Device buffers of the selection.  idx_t == nullptr skips the key-major emission (then jcut, cnt,
// col may be null as well).
struct SelectBuffers {
    uint32_t *prefix;  // [B*H, L]   order-preserving key of each query's threshold score
    int32_t *krem;     // [B*H, L]   number of keys equal to the threshold that belong to the top-k
    int32_t *idx;      // out: ragged query-major index
    int32_t *jcut;     // [B*H, L]   index of the last tie taken
    int32_t *tile_flag;  // [B*H, ceil(L/32)]  1: every query of the tile takes all its threshold ties
    int32_t *cnt;      // [B*H, L]   list length of every key
    int64_t *col;      // out: [B*H, L+1]
    int32_t *idx_t;    // out: ragged key-major index
    uint32_t *win;     // [B*H, L]   windowed threshold search: upper end of the bracket, then the bin width
    int32_t *todo;     // [1 + B*H * ceil(L/32)]  windowed search: number and ids of the query tiles left to the radix search
};
// Lq index rows per head (state arrays are [B*H, padded_len(Lq)], tile_flag [B*H, ceil(Lq/32)], lists hold row
// numbers below Lq); tabs[].off must be the offsets of [Lq, k] blocks.
dsv_status launch_select(const dsv_problem &p, int Lq, const HeadTable *tabs, int n_tabs, const void *Qlr, const void *Klr,
                         const SelectBuffers &b, hipStream_t st);
// Threshold search in two sweeps (stage1_window.hip) for the head slots of one table; the tiles it lists in
// b.todo still need the radix passes.
dsv_status launch_window_search(const dsv_problem &p, int Lq, const HeadTable &tab, const void *Qlr, const void *Klr,
                                const SelectBuffers &b, hipStream_t st);
// Keys the search would sample for a head keeping k of L keys, 0 if it does not fit that head (forced: leave
// out the checks that only decide whether it pays).
int window_sample_keys(int L, int k, bool forced);
// 0: automatic; 1: always the four-pass radix search; 2: the windowed search wherever it fits.  Returns the old mode
// (mode < 0: only that).
int set_threshold_search(int mode);
// Threshold search and query-major emission of short sequences in one launch (stage1_small.hip): for problems that
// small_select accepts (Lq queries per head).  Leaves the same state behind as the search and launch_emit's first part.
bool small_select(const dsv_problem &p, int Lq);
dsv_status launch_select_small(const dsv_problem &p, int Lq, const HeadTable &tab, const void *Qlr, const void *Klr,
                               const SelectBuffers &b, hipStream_t st);
// emitted: the query-major index is there already.
dsv_status launch_emit(const dsv_problem &p, int Lq, const HeadTable *tabs, int n_tabs, const void *Qlr, const void *Klr,
                       const SelectBuffers &b, bool emitted, hipStream_t st);
// waves: a wave per row, else a lane group per row.
dsv_status launch_sparse_fwd(const dsv_problem &p, const HeadTable *tabs, int n_tabs, bool waves, const void *Q, const void *K,
                             const void *V, const int32_t *idx, void *O, float *lse, hipStream_t st);
dsv_status launch_bwd_dq(const dsv_problem &p, const HeadTable *tabs, int n_tabs, bool waves, const void *Q, const void *K,
                         const void *V, const int32_t *idx, const void *O, const float *lse, const void *dO, void *dQ,
                         float *delta, hipStream_t st);
dsv_status launch_bwd_dkdv(const dsv_problem &p, const HeadTable *tabs, int n_tabs, const void *Q, const void *K,
                           const void *V, const int32_t *idxT, const int64_t *col, const float *lse, const float *delta,
                           const void *dO, void *dK, void *dV, hipStream_t st);
// ---- query grouping (grouped.hip) -----------------------------------------------------------------------
struct GroupGeom {
    int F, Hh, Ww, gf, gh, gw;
    int nh, nw;  // cubes along height and width
    int G;       // queries per group
};
// mode 0: out [B*H, L/G, d] = the groups' centre query rows; 1: out [B*H, L, d] = rows in group-major order;
// 2: the inverse of 1.
dsv_status launch_group_rows(const dsv_problem &p, const dsv_grouping &gr, int mode, const void *in, void *out,
                             hipStream_t st);
dsv_status launch_group_scalar(const dsv_problem &p, const dsv_grouping &gr, const float *in, float *out, hipStream_t st,
                               bool inverse = false);
// tabs: built for L/G rows per head.  Writes the per-query form (group-major query order) of the key-major index
// (unless idx_t_x / col_x are null) and of the query-major index (unless idx_x is null).
dsv_status launch_group_expand(const dsv_problem &p, const dsv_grouping &gr, const HeadTable *tabs, int n_tabs,
                               const int32_t *idx_g, const int32_t *idx_t_g, const int64_t *col, int32_t *idx_x,
                               int32_t *idx_t_x, int64_t *col_x, hipStream_t st);
// Group-size profiling: overlap[bh] = share of the members' own rows (per-query idx, tabs for L rows per head) that the
// centre's row holds.  count: one 64-bit counter per (b, h).
dsv_status launch_group_overlap(const dsv_problem &p, const dsv_grouping &gr, const HeadTable *tabs, int n_tabs,
                                const int32_t *idx, unsigned long long *count, float *overlap, hipStream_t st);
// Scratch of the L2-blocked grouped kernels (null seg: plain form, rows in any order).
struct GroupedSplit {
    SplitPlan plan;
    int32_t *seg;   // [B*H, L/G, S+1]
    float *pa;      // forward: pm [rows, S];          dq: C partials [rows, S, d]
    float *pb;      // forward: pl [rows, S];          dq: B partials [rows, S, d]
    float *pc;      // forward: pacc [rows, S, d];     dq: Delta partials [rows, S]
};
dsv_status launch_grouped_fwd(const dsv_problem &p, const dsv_grouping &gr, const HeadTable *tabs, int n_tabs,
                              const void *Q, const void *K, const void *V, const int32_t *idx_g, void *O, float *lse,
                              const GroupedSplit *split, hipStream_t st);
dsv_status launch_grouped_dq(const dsv_problem &p, const dsv_grouping &gr, const HeadTable *tabs, int n_tabs,
                             const void *Q, const void *K, const void *V, const int32_t *idx_g, const void *O,
                             const float *lse, const void *dO, void *dQ, float *delta, const GroupedSplit *split,
                             hipStream_t st);
dsv_status launch_row_segments(const dsv_problem &p, int rows, const HeadTable *tabs, int n_tabs, const SplitPlan &pl,
                               const int32_t *index, int32_t *seg, hipStream_t st);
dsv_status launch_fwd_merge_bf16_128(const dsv_problem &p, const HeadTable *tabs, int n_tabs, const float *pm, const float *pl_, const float *pacc, void *O,
                                     float *lse, int S, hipStream_t st);
// dK, dV of the group kernels' cases over unions of lists (grouped_dkdv.hip): Q, dO, w.rowstat in group-major order, lists of groups
// (tabs built for L / G rows per head).  Writes the partial results of every range, or, with a single range, dK and dV.
// union_limit: the longest union, in lists, that is worth it (16: any).  launch_union_prepare fills rowstat and, below that, use
// [B*H]; launch_grouped_dkdv leaves out heads with use[bh] == 0 (use null: none).
double union_limit(const dsv_problem &p);
dsv_status launch_union_prepare(const dsv_problem &p, int G, const HeadTable *tabs, int n_tabs, const int32_t *lists, const int64_t *col,
                                const float *lse, const float *delta, float2 *rowstat, int32_t *use, hipStream_t st);
dsv_status launch_grouped_dkdv(const dsv_problem &p, int G, const HeadTable *tabs, int n_tabs, const void *Q, const void *K,
                               const void *V, const int32_t *lists, const int64_t *col, const void *dO, void *dK, void *dV,
                               const SplitPlan &plan, const BwdSplitWorkspace &w, const int32_t *use, hipStream_t st);
dsv_status launch_dkdv_merge_bf16_128(const dsv_problem &p, const HeadTable *tabs, int n_tabs, void *dK, void *dV, const SplitPlan &pl,
                                      const BwdSplitWorkspace &w, hipStream_t st);
dsv_status launch_dq_merge_bf16_128(const dsv_problem &p, const HeadTable *tabs, int n_tabs, const float *pa, const float *pb, const float *pdelta,
                                    const void *O, const void *dO, void *dQ, float *delta, int S, hipStream_t st);

// ---- predictor side (predictor.hip) ---------------------------------------------------------------------
struct PredictorLayout {
    int tok_per_block, nblk, nchunk;
    size_t part, M, T1, T2, qlr, g, coef, terms, acc, sums, total;
};
PredictorLayout predictor_layout(const dsv_problem &p, int n_rows);
dsv_status launch_predictor_loss(const dsv_problem &p, const void *Q, const void *K, const void *Wq, const void *Wk,
                                 const int32_t *rows, int n, float *loss, float *dWq, float *dWk, char *ws,
                                 const PredictorLayout &w, hipStream_t st);

// ---- sparsity profiler (profiler.hip) ----------------------------------------------------------------------
dsv_status launch_profile_sparsity(const dsv_problem &p, const void *Q, const void *K, const int32_t *rows, int n,
                                   float mass, int32_t *counts, float *sparsity, float *ema, float alpha, hipStream_t st);

// report_dev: two 64-bit counters in device memory; report_host: optional HOST int64 [3].  Waits for the stream.
dsv_status launch_idx_validate(const dsv_problem &p, const HeadTable *tabs, int n_tabs, const int32_t *idx,
                               unsigned long long *report_dev, int64_t *report_host, hipStream_t st);
// Stable transposition: every list ascending in the query index, the same result from run to run.
// ws: scratch of idx_transpose_bytes(p) bytes; col: [B*H, L+1] int64.
size_t idx_transpose_bytes(const dsv_problem &p);
dsv_status launch_idx_transpose(const dsv_problem &p, const HeadTable *tabs, int n_tabs, const int32_t *idx, bool built,
                                int32_t *idxT, int64_t *col, void *ws, size_t ws_bytes, hipStream_t st);
// Rows row0 .. row0 + nrows - 1 of `heads` head slots as a bit matrix [heads, nrows, bits_pitch(L) words]; L <= kBitsMaxKeys.
// col: the rows are key-major lists (idx: idx_t).
constexpr int kBitsMaxKeys = 524288;  // a row's bitmap fits 64 KB of LDS
int bits_pitch(int L);
size_t bits_rows(int L, size_t bytes);  // rows whose bits take that much, the space between rows (bits_pitch) not counted
dsv_status launch_bits_build(const dsv_problem &p, const HeadTable &tab, int slot0, int heads, const int32_t *idx, int row0,
                             int nrows, uint32_t *bits, hipStream_t st, const int64_t *col = nullptr);
// Forward of some heads over dense tiles with a mask (dense.hip; bf16, scale > 0, L <= kBitsMaxKeys); ws: scratch for the
// mask, at least kDenseMinRows rows of it.
constexpr int kDenseMinRows = 128;
dsv_status launch_dense_fwd(const dsv_problem &p, const HeadTable &tab, const void *Q, const void *K, const void *V,
                            const int32_t *idx, void *O, float *lse, char *ws, size_t ws_bytes, hipStream_t st);
// The bit matrix in the workspace of launch_idx_transpose if it holds all heads at once, else null: a caller that has filled it
// (launch_sort_rows) says `built`.
uint32_t *transpose_matrix(const dsv_problem &p, void *ws);
// out = the rows of idx in ascending order (same layout), and their bitmaps if bits is given; can_sort_rows: whether this L is covered.
bool can_sort_rows(const dsv_problem &p);
dsv_status launch_sort_rows(const dsv_problem &p, const HeadTable *tabs, int n_tabs, const int32_t *idx, int32_t *out,
                            uint32_t *bits, hipStream_t st);
// col[bh, 0 .. L] = exclusive prefix sums of cnt[bh, 0 .. L - 1] for the heads of one table.
dsv_status launch_col_scan(const int32_t *cnt, int64_t *col, int L, const HeadTable &tab, hipStream_t st);

}  // namespace dsv
