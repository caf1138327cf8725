// Tiles of 32 rows that the kernels over dense tiles share in LDS (dense.hip, dense_bwd.hip), and choices between the results of matrix products.
#pragma once

#include "stage2_core.h"
#include "pair_slots.h"

namespace dsv {

constexpr int kTile = 32;          // rows of a tile
constexpr int kChunkPitch = 1088;  // bytes from one kilobyte of a parked tile to the next: 16 banks on

typedef __attribute__((__vector_size__(16 * sizeof(__bf16)))) __bf16 bf16x16_t;

template <int D> struct TileLayout {
    static constexpr int PPR = D / 8;              // 16-byte pieces per row
    static constexpr int CHUNKS = kTile * PPR / 64;  // kilobytes, one load instruction of a wave each
    static constexpr int BYTES = CHUNKS * kChunkPitch;
    __device__ __forceinline__ static int chunk(int r) { return D == 128 ? r >> 2 : (r >> 2) & 3; }
    __device__ __forceinline__ static int slot(int r) { return D == 128 ? r & 3 : (r & 3) + 4 * (r >> 4); }
    __device__ __forceinline__ static int row(int chunk, int slot) { return D == 128 ? 4 * chunk + slot : 4 * chunk + (slot & 3) + 16 * (slot >> 2); }
    // piece p of row r lies at base(r) + 16 (p ^ r % 4)
    __device__ __forceinline__ static int base(int r) { return chunk(r) * kChunkPitch + slot(r) * (2 * D); }
};

// Tiles tile .. tile + COUNT - 1 of a [L, D] matrix into LDS, one after the other (rows past the end repeat the last one): this wave's share
// of the chunks.  Two vector instructions per load: a lane's place in the matrix is its place in the first tiles plus what all lanes
// add (the matrix has less than 2^32 bytes; wave is the same in all lanes, also for the compiler).
template <int D, int WAVES, int COUNT> struct TileLoads {
    typedef TileLayout<D> TL;
    static constexpr int N = COUNT * TL::CHUNKS / WAVES;
    static_assert(N * WAVES == COUNT * TL::CHUNKS, "every chunk has its wave");
    uint32_t at[N], last[N];
    int wave;
    __device__ __forceinline__ TileLoads(int L, int wave_, int lane) : wave(wave_)
    {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int c = wave * N + i, r = TL::row(c % TL::CHUNKS, lane / TL::PPR);
            const uint32_t piece = (uint32_t)((lane % TL::PPR) ^ (r & 3)) * 16u;
            at[i] = (uint32_t)(c / TL::CHUNKS * kTile + r) * (2 * D) + piece;
            last[i] = (uint32_t)(L - 1) * (2 * D) + piece;
        }
    }
    __device__ __forceinline__ void request(const unsigned char *__restrict__ mat, int tile, unsigned char *lds) const
    {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const unsigned char *src = mat + min(at[i] + (uint32_t)tile * (kTile * 2 * D), last[i]);
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                             (__attribute__((address_space(3))) void *)(lds + (wave * N + i) * kChunkPitch), 16, 0, 0);
        }
    }
};

// Plain expressions, because their operands are results of matrix products: the compiler puts the wait that such a read needs before
// an instruction of its own, and none before one written in inline assembly.  The empty statement only hides from it that a
// mask is a bit spread out, which it would turn into a compare and a select per use (dq at L = 32768, four heads, k = 2048: 4.65 ms, 4.77
// without).
template <int BIT> __device__ __forceinline__ uint32_t bit_mask(uint32_t w)  // all ones where the bit is set, else zero
{
    uint32_t m = (uint32_t)__builtin_amdgcn_sbfe((int)w, BIT, 1);
    asm("" : "+v"(m));
    return m;
}
__device__ __forceinline__ float pick(uint32_t mask, float a, float b)  // mask all ones: a, zero: b
{
    return __uint_as_float((mask & __float_as_uint(a)) | (~mask & __float_as_uint(b)));
}
__device__ __forceinline__ float keep(uint32_t mask, float a) { return __uint_as_float(mask & __float_as_uint(a)); }

}  // namespace dsv
