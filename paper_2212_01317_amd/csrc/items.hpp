// The order of a launch's work items over its workgroups.
#pragma once
#include <cstdint>

namespace mpr {

constexpr uint32_t kItemRow = 1u << 22;          // workgroups of a grid row: 2^31 threads of 512 (a launch dimension holds 2^32)
constexpr uint32_t kNoItem = 0xffffffffu;

// The item of workgroup x of grid row y, or kNoItem.  A row of `row` workgroups (a multiple of 8) takes the next `row` of the
// nwork items, the last row what is left.  XCD-aware: workgroup x runs on XCD x % 8, and an XCD takes an eighth of the row's
// items, consecutive ones (adjacent tiles).
constexpr uint32_t item_of(uint32_t x, uint32_t y, uint32_t row, uint32_t nwork)
{
    const uint32_t base = y * row, left = nwork - base, n = left < row ? left : row, eighth = (n + 7u) / 8u;
    const uint32_t k = x >> 3, i = (x & 7u) * eighth + k;
    return k < eighth && i < n ? base + i : kNoItem;
}

}  // namespace mpr
