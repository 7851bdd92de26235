// How batched matching divides train ranges: rules of sizes alone, the same on the host.
#pragma once

#include "internal.h"

namespace latch {

constexpr int kMinPartTiles = 80;
constexpr int kMaxParts = kBatchMaxParts;

// Cost class of a pair, 0 for the longest items: 255 - floor(8 log2(tiles + 1))
// with the fraction taken from the three bits after the leading one.
__host__ __device__ inline int cost_class(int64_t nt)
{
    nt = nt < 0 ? 0 : nt > kMaxSplitRows ? kMaxSplitRows : nt;              // invalid pairs: any class
    const uint32_t x = (uint32_t)((nt + kTileRows - 1) / kTileRows) + 1u;   // <= 2^16
    const int lz = __builtin_clz(x);
    const uint32_t frac = ((x << lz) >> 28) & 7u;
    const int c = 8 * (31 - lz) + (int)frac;
    return 255 - (c < 255 ? c : 255);
}

// Parts of a train range of `tiles` tiles with `left` tiles of work from its pair on
// and `resident` workgroups: about left / resident tiles each, within the limits, and
// no part empty.
__host__ __device__ inline int train_parts(int tiles, unsigned long long left, int resident)
{
    const unsigned long long share = left / (uint32_t)resident;
    const int chunk = share < (unsigned)kMinPartTiles ? kMinPartTiles : (int)(share < (1ull << 20) ? share : 1ull << 20);
    int parts = (tiles + chunk - 1) / chunk;
    parts = parts < kMaxParts ? parts : kMaxParts;
    if (parts <= 1) return 1;
    const int per_part = (tiles + parts - 1) / parts;
    return (tiles + per_part - 1) / per_part;
}

}  // namespace latch
