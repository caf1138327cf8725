// Slots of the sparse matrix product over a tile of selected pairs (dense_bwd.hip): plain integer arithmetic, the same on host and device.
#pragma once

#include <cstdint>

#if defined(__HIP__)
#include <hip/hip_runtime.h>
#define DSV_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define DSV_HOST_DEVICE inline
#endif

namespace dsv {

// The first two selected pairs of every group of four, from the mask word of a lane's row shifted so that accumulator 4 g + i has
// bit 4 i + 2 (g % 2) + 16 (g / 2).  All groups at once, a bit plane per i.  Slot 0 takes the first of 0, 1, 2 (2 if none), slot
// 1 the last of the others.  Pairs left over -- 1, 2 or both -- take the slots of a second round: 1 and 2, or 2 and 3.  In both
// rounds the numbers of a group's slots ascend whatever the mask, as the instruction's index operand wants them.
struct PairSlots {
    uint32_t b0, b1, n2, n3, v0, v1;  // slot 0: b0 ? 0 : b1 ? 1 : 2; slot 1: n3 ? (n2 ? 1 : 2) : 3; v0, v1: a selected pair
    uint32_t index;                   // the instruction's index operand: slot numbers, two bits each
    uint32_t r1, r2;                  // pairs number 1 and 2 that are left
    static constexpr uint32_t M = 0x00050005u;
    // slot 0 = lo0 + 2 hi0, slot 1 = lo1 + 2 hi1; the groups' bits moved together: bytes 0 and 2 of z
    DSV_HOST_DEVICE static uint32_t index_of(uint32_t lo0, uint32_t hi0, uint32_t lo1, uint32_t hi1)
    {
        const uint32_t x = (lo0 & M) | ((hi0 & M) << 1), y = (lo1 & M) | ((hi1 & M) << 1);
        const uint32_t z = (x & 0x00030003u) | ((x & 0x000C000Cu) << 2) | ((y & 0x00030003u) << 2) | ((y & 0x000C000Cu) << 4);
        return (z & 0xFFu) | ((z >> 8) & 0xFF00u);
    }
    DSV_HOST_DEVICE explicit PairSlots(uint32_t w)
    {
        b0 = w & M;
        b1 = (w >> 4) & M;
        const uint32_t b2 = (w >> 8) & M, b3 = (w >> 12) & M;
        const uint32_t a = b0 | b1;
        n3 = a & ~b3;
        n2 = b0 & ~b2;
        v0 = a | b2;
        v1 = (n3 & ((n2 & b1) | (~n2 & b2))) | (~n3 & b3);
        index = index_of(b1 & ~b0, ~a, ~n3 | n2, ~n3 | ~n2);
        r1 = b1 & b0 & (b2 | b3);
        r2 = b2 & a & b3;
    }
    DSV_HOST_DEVICE uint32_t index_left() const { return index_of(r1, ~r1, ~r1, ~0u); }
};

}  // namespace dsv
