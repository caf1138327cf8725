// Grids of more blocks than one dimension takes (host).
#pragma once

#include <algorithm>
#include <cstdint>

namespace dsv {

struct GridXY {
    uint32_t x, y;
};

// At least `blocks` blocks (up to 2^20 * 65535): a multiple of eight of them in x, so that consecutive blocks take the XCDs in turn in every
// row, and at most 2^20, since a dimension has less than 2^32 work items and a block up to 1024.
inline GridXY grid_of(int64_t blocks)
{
    const int64_t x = std::min<int64_t>((blocks + 7) / 8 * 8, 1 << 20);
    return GridXY{(uint32_t)x, (uint32_t)((blocks + x - 1) / x)};
}

}  // namespace dsv
