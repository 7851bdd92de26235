// Ranges of a grid-stride loop per XCD.  Included inside
// namespace latch { namespace { ... } } of each kernel file.
#pragma once

// The items (keypoints, tiles) one workgroup of a grid-stride loop takes.  The
// chip's 8 XCDs (workgroups go to them round-robin by index) take contiguous
// eighths of [0, n), so that one XCD's L2 holds the images (or, for items in
// raster order, the rows) its own workgroups read, rather than every XCD
// fetching everything; within its eighth an XCD's workgroups stride over the
// items.  Item m of the range is first + m * stride.
struct XcdRange {
    int64_t first, end, stride;
};

__device__ __forceinline__ XcdRange xcd_range(int64_t n)
{
    constexpr int kXcds = 8;
    const int g = gridDim.x, b = blockIdx.x;
    XcdRange r;
    if (g < kXcds) {
        r.first = b;
        r.end = n;
        r.stride = g;
        return r;
    }
    const int xcd = b % kXcds;
    const int64_t per = (n + kXcds - 1) / kXcds;
    r.first = (int64_t)xcd * per + b / kXcds;
    r.end = min(n, (int64_t)(xcd + 1) * per);
    r.stride = (g - xcd + kXcds - 1) / kXcds;     // workgroups on this XCD
    return r;
}
