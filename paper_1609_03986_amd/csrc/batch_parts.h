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

// Whether dividing can shorten a batch of `groups` query groups with `work` train tiles
// in all, `longest` in its longest train range.  It cannot where every range is at most
// a least part.  Where all units start at once (no more of them than workgroups), the
// batch takes as long as its longest range, and dividing cannot beat the workgroups'
// share of the work; what parts cost beside their tiles (starts, query fragments, merging)
// comes to some 30 tiles.  With and without this rule, us: 63 pairs of 2754 rows (87 tiles,
// share 86) 122 and 154, 30 of 5000 (157, share 129) 170 and 193, 15 of 12,000 (375, share
// 352) 355 and 373; 30 of 3840 (120, share 70), divided, take 150 against 146 undivided.
constexpr int kWholeSlack = 32;

__host__ __device__ inline bool may_divide(int longest, unsigned long long groups, unsigned long long work,
                                           int resident)
{
    if (longest <= kMinPartTiles) return false;
    return groups > (unsigned)resident || (unsigned)longest > work / (unsigned)resident + kWholeSlack;
}

// Parts of a train range of `tiles` tiles with `left` tiles of work from its pair on
// and `resident` workgroups: as many as of left / resident tiles, or of the least part's,
// cover it, within the limit, the range then divided evenly (a part has at least half of
// those tiles) and no part empty.
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
