// Reductions over lane rows that scatter their results.  Included inside
// namespace latch { namespace { ... } }.
//
// Every lane row (16 lanes) of a wavefront holds partial results of four blocks
// 0..3.  Exchanging blocks b and b + 2 between the wavefront's halves, then the
// kept pair between the rows of a half, leaves lane row b with all four partials
// of block b, merged step by step: three exchanges of each value instead of
// eight.
#pragma once

// x and y are two blocks' values on every lane.  Afterwards a lane of the first
// half (kHalves) or of an even row (otherwise) holds its own and its partner
// lane's value of block x, the others those of block y.
template <bool kHalves>
__device__ __forceinline__ void exchange(int &x, int &y)
{
    if constexpr (kHalves) {
        const auto v = __builtin_amdgcn_permlane32_swap(x, y, false, false);
        x = (int)v[0];
        y = (int)v[1];
    } else {
        const auto v = __builtin_amdgcn_permlane16_swap(x, y, false, false);
        x = (int)v[0];
        y = (int)v[1];
    }
}

template <bool kHalves>
__device__ __forceinline__ void exchange(float &x, float &y)
{
    int a = __float_as_int(x), b = __float_as_int(y);
    exchange<kHalves>(a, b);
    x = __int_as_float(a);
    y = __int_as_float(b);
}

__device__ __forceinline__ int larger(int a, int b) { return max(a, b); }
__device__ __forceinline__ int smaller(int a, int b) { return min(a, b); }
__device__ __forceinline__ float larger(float a, float b) { return fmaxf(a, b); }
__device__ __forceinline__ float smaller(float a, float b) { return fminf(a, b); }

// Two blocks' running top two, x1 >= x2 and y1 >= y2, merged into x1, x2.
template <bool kHalves, typename T>
__device__ __forceinline__ void exchange_top2(T &x1, T &x2, T &y1, T &y2)
{
    exchange<kHalves>(x1, y1);
    exchange<kHalves>(x2, y2);
    const T lo = smaller(x1, y1);
    x1 = larger(x1, y1);
    x2 = larger(lo, larger(x2, y2));
}

// Two blocks' sums, added into x.
template <bool kHalves>
__device__ __forceinline__ void exchange_sum(int &x, int &y)
{
    exchange<kHalves>(x, y);
    x += y;
}
