// Keypoint detection for gfx950: FAST-9 corners with suppression and an
// intensity-centroid orientation (the paper detects FAST keypoints and
// extracts LATCH at their orientation, Sec. 3.2; the score, suppression and
// orientation method are not stated there and are fixed as follows).
//
//   * Score: for the 16 pixels of the radius-3 circle and c the centre, the
//     largest over the 16 arcs of 9 consecutive circle pixels and over both
//     polarities of the smallest difference on the arc (q - c brighter,
//     c - q darker).  A corner for threshold t has score > t.
//   * Pixels at least kDetectBorder from every edge are tested; others score
//     0.  Suppression keeps p iff S(p) > 0 and S(p) > S(q) for its 8
//     neighbours.
//   * Output in raster order, appended after the keypoints already counted
//     in *n_kps.
//   * Orientation: moments m10 = sum dx I, m01 = sum dy I over the disc of
//     radius kOrientRadius, bin = rne(atan2(m01, m10) * 4096 / 2 pi) mod 4096
//     in double (integer moments keep the angle far enough from a bin
//     boundary that the bin does not depend on the last bits of atan2), and
//     the keypoint angle bin * 360 / 4096 degrees, exact in float.
//
// Two launches, or three for large images:
//   1. detect_tile_kernel: a 64 x 16 tile per workgroup.  The image tile with
//      a 4-pixel halo is staged in LDS; the pixels of the tile and a 1-pixel
//      halo that pass a test on four of the circle's pixels are listed and
//      scored, and each wavefront's ballot over one tile row is that row's
//      64-bit survivor mask; the mask and its popcount (one byte per row and
//      tile, rows of the count array padded to 16 bytes) go to the workspace,
//      with the tile's total or, in large images, without.
//   2. detect_scan_kernel, in large images: one workgroup sums each row's count
//      bytes (two rows per thread) and scans them into each row's first output
//      slot and the new total.
//   3. detect_emit_kernel: per tile, the image window of every disc staged in
//      LDS; the slot of each survivor from what precedes its row (the scan's
//      slots, or the totals and counts) and the mask, its orientation with one
//      disc row per lane (two keypoints per wavefront), then the keypoint
//      written once, complete.
//
// What bounds it (1920 x 1080, 55,000 keypoints at threshold 20): every
// workgroup of a launch is resident at once, so a launch takes its few
// microseconds of start and staging latency plus its vector work, 407
// instructions per wavefront in the tile kernel (5 of 10.6 us) and 690 in the emit
// kernel (9 of 13.2 us).  Scoring every pixel one per lane took 17 us, the scan
// 4 us and an emit kernel that ran a double atan2 in every wavefront 17 us: 37.7
// -> 25.0 us per call.  39% of that image's pixels pass the four-pixel test.
#include "internal.h"

namespace latch {
namespace {

constexpr int kTileW = 64, kTileH = 16;
constexpr int kHaloImg = 4;                            // circle radius 3 + suppression 1
constexpr int kImgW = kTileW + 2 * kHaloImg;           // 72
constexpr int kImgH = kTileH + 2 * kHaloImg;           // 24
constexpr int kScoreW = kTileW + 2, kScoreH = kTileH + 2;   // 66 x 18
constexpr int kThreads = 256;
constexpr int kScanThreads = 1024;
constexpr int kDiscRows = 2 * kOrientRadius + 1;       // 31

// Circle offsets, clockwise from the top (y downwards).
struct Offset {
    int x, y;
};
constexpr Offset kCircle[16] = {{0, -3}, {1, -3},  {2, -2},  {3, -1}, {3, 0},   {3, 1},
                                {2, 2},  {1, 3},   {0, 3},   {-1, 3}, {-2, 2},  {-3, 1},
                                {-3, 0}, {-3, -1}, {-2, -2}, {-1, -3}};

typedef unsigned short ushort2v __attribute__((ext_vector_type(2)));
typedef short short2v __attribute__((ext_vector_type(2)));

__device__ __forceinline__ ushort2v pk_min(ushort2v a, ushort2v b) { return __builtin_elementwise_min(a, b); }
__device__ __forceinline__ ushort2v pk_max(ushort2v a, ushort2v b) { return __builtin_elementwise_max(a, b); }

// FAST-9 scores of the two pixels at p and q (an LDS image tile of row stride
// kImgW), one per 16-bit half.  On the circle values themselves: the best arc
// of 9 for "brighter" has the largest minimum, that for "darker" the smallest
// maximum, and the centre is subtracted at the end.  The arcs from k and from
// k + 1 share the 8 pixels k + 1 .. k + 8, so the better of the two is
// min(min of those 8, max of pixels k and k + 9): 8 such pairs.
__device__ __forceinline__ short2v fast_scores(const uint8_t *p, const uint8_t *q)
{
    ushort2v d[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int off = kCircle[i].y * kImgW + kCircle[i].x;
        d[i] = ushort2v{p[off], q[off]};
    }
    ushort2v lo[8], hi[8];                                  // arcs of 2, then 4, from odd pixels
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        lo[i] = pk_min(d[2 * i + 1], d[(2 * i + 2) & 15]);
        hi[i] = pk_max(d[2 * i + 1], d[(2 * i + 2) & 15]);
    }
    ushort2v lo4[8], hi4[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        lo4[i] = pk_min(lo[i], lo[(i + 1) & 7]);
        hi4[i] = pk_max(hi[i], hi[(i + 1) & 7]);
    }
    ushort2v best_lo = ushort2v{0, 0}, best_hi = ushort2v{255, 255};
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const ushort2v a = d[2 * i], b = d[(2 * i + 9) & 15];
        best_lo = pk_max(best_lo, pk_min(pk_min(lo4[i], lo4[(i + 2) & 7]), pk_max(a, b)));
        best_hi = pk_min(best_hi, pk_max(pk_max(hi4[i], hi4[(i + 2) & 7]), pk_min(a, b)));
    }
    const short2v c = {(short)p[0], (short)q[0]};
    return __builtin_elementwise_max(__builtin_bit_cast(short2v, best_lo) - c,
                                     c - __builtin_bit_cast(short2v, best_hi));
}

// Copies rows ry0 .. ry0 + kRows - 1 and columns cx0 .. cx0 + kCols - 1 of
// the image into LDS (row stride kStride), coordinates clamped to the image
// (callers never use the clamped values).  kDword: 4-byte loads, for a
// 4-byte-aligned image whose pitch and width are multiples of 4 (cx0 and
// kCols are); otherwise byte loads.  Every load is issued before the first
// LDS write; lds must hold kStageRows<kDword, kRows, kCols> rows.
template <bool kDword, int kRows, int kCols>
struct Stage {
    static constexpr int kUnit = kDword ? 4 : 1;
    static constexpr int kPerRow = kCols / kUnit;
    static constexpr int kLoads = (kRows * kPerRow + kThreads - 1) / kThreads;
    static constexpr int kLdsRows = (kLoads * kThreads + kPerRow - 1) / kPerRow;
};

template <bool kDword, int kRows, int kCols, int kStride>
__device__ __forceinline__ void stage_window(const uint8_t *__restrict__ img, int height, int width,
                                             int pitch, int ry0, int cx0, uint8_t *lds)
{
    using S = Stage<kDword, kRows, kCols>;
    const int t = threadIdx.x;
    uint32_t v[S::kLoads];
#pragma unroll
    for (int k = 0; k < S::kLoads; ++k) {
        const int i = t + k * kThreads;
        const int yy = min(max(ry0 + i / S::kPerRow, 0), height - 1);
        const int xx = min(max(cx0 + S::kUnit * (i % S::kPerRow), 0), width - S::kUnit);
        const uint8_t *p = img + (size_t)yy * pitch + xx;
        if constexpr (kDword)
            v[k] = *reinterpret_cast<const uint32_t *>(p);
        else
            v[k] = *p;
    }
#pragma unroll
    for (int k = 0; k < S::kLoads; ++k) {
        const int i = t + k * kThreads;
        uint8_t *q = lds + (i / S::kPerRow) * kStride + S::kUnit * (i % S::kPerRow);
        if constexpr (kDword)
            *reinterpret_cast<uint32_t *>(q) = v[k];
        else
            *q = (uint8_t)v[k];
    }
}

template <int kRows, int kCols>
constexpr int stage_lds_rows()
{
    return Stage<true, kRows, kCols>::kLdsRows > Stage<false, kRows, kCols>::kLdsRows
               ? Stage<true, kRows, kCols>::kLdsRows
               : Stage<false, kRows, kCols>::kLdsRows;
}

template <bool kDword>
__global__ __launch_bounds__(kThreads) void detect_tile_kernel(
    const uint8_t *__restrict__ img, int height, int width, int pitch, int threshold, int tiles_x,
    uint64_t *__restrict__ masks, uint8_t *__restrict__ counts, int count_stride,
    uint16_t *__restrict__ tile_total, const int64_t *__restrict__ n_kps, int64_t *__restrict__ base)
{
    __shared__ __align__(16) uint8_t timg[stage_lds_rows<kImgH, kImgW>() * kImgW];
    // Scores of the tile and a 1-pixel halo, at the pixels' places in timg.
    __shared__ uint8_t tscore[kImgH * kImgW];
    __shared__ uint16_t list[kScoreH * kScoreW + 1];       // places of the pixels to score
    __shared__ int listed, kept;
    const int tx = (int)(blockIdx.x % (unsigned)tiles_x), ty = (int)(blockIdx.x / (unsigned)tiles_x);
    const int x0 = tx * kTileW, y0 = ty * kTileH;
    const int t = threadIdx.x;

    if (t == 0) listed = kept = 0;
    // The count on entry, for the emit kernel (one writer, before the count
    // is replaced).
    if (base && blockIdx.x == 0 && t == 0) *base = max(*n_kps, (int64_t)0);
    // Image tile with halo.  Clamped pixels only reach scores outside the
    // tested region, which are 0 regardless.
    stage_window<kDword, kImgH, kImgW, kImgW>(img, height, width, pitch, y0 - kHaloImg, x0 - kHaloImg,
                                              timg);
    __syncthreads();

    // An arc of 9 holds two neighbouring compass points of the circle, so a
    // corner has min(max(n, s), max(e, w)) - c or c - max(min(n, s), min(e, w))
    // above the threshold.  The pixels that pass are listed and scored two per
    // thread; the others score 0.
    const int lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    constexpr int kPasses = (kScoreH * kScoreW + kThreads - 1) / kThreads;
    uint64_t pass[kPasses];
    int at[kPasses], total = 0;
#pragma unroll
    for (int k = 0; k < kPasses; ++k) {
        const int i = t + k * kThreads;
        const int sy = i / kScoreW, sx = i % kScoreW;
        const int yy = y0 - 1 + sy, xx = x0 - 1 + sx;
        at[k] = (sy + kHaloImg - 1) * kImgW + sx + kHaloImg - 1;
        bool ok = false;
        if (i < kScoreH * kScoreW) {
            const uint8_t *p = timg + at[k];
            const int n = p[-3 * kImgW], e = p[3], s = p[3 * kImgW], w = p[-3], c = p[0];
            const int brighter = min(max(n, s), max(e, w)) - c, darker = c - max(min(n, s), min(e, w));
            ok = (max(brighter, darker) > threshold) & (yy >= kDetectBorder) &
                 (yy < height - kDetectBorder) & (xx >= kDetectBorder) & (xx < width - kDetectBorder);
            tscore[at[k]] = 0;
        }
        pass[k] = __ballot(ok);
        total += __popcll(pass[k]);
    }
    int first = 0;
    if (lane == 0) first = atomicAdd(&listed, total);
    first = __builtin_amdgcn_readfirstlane(first);
#pragma unroll
    for (int k = 0; k < kPasses; ++k) {
        const int rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(pass[k] >> 32),
                                                   __builtin_amdgcn_mbcnt_lo((uint32_t)pass[k], 0));
        if ((pass[k] >> lane) & 1) list[first + rank] = (uint16_t)at[k];
        first += __popcll(pass[k]);
    }
    __syncthreads();
    const int n = listed;
    for (int i = 2 * t; i < n; i += 2 * kThreads) {
        const int a = list[i], b = list[min(i + 1, n - 1)];
        const short2v s = fast_scores(timg + a, timg + b);
        tscore[a] = (uint8_t)(s[0] > threshold ? s[0] : 0);
        tscore[b] = (uint8_t)(s[1] > threshold ? s[1] : 0);
    }
    __syncthreads();

    // Suppression: wavefront w takes tile rows 4 w .. 4 w + 3; lane = column.
    // A pixel stays if its score exceeds the largest of its 8 neighbours
    // (and so 0).
    constexpr int kRows = kTileH / (kThreads / 64);
    const uint8_t *p = &tscore[(kRows * wave + kHaloImg) * kImgW + lane + kHaloImg];
    int mid[kRows + 2], side[kRows + 2], survivors = 0;
#pragma unroll
    for (int r = 0; r < kRows + 2; ++r) {
        const uint8_t *q = p + (r - 1) * kImgW;
        mid[r] = q[0];
        side[r] = max((int)q[-1], (int)q[1]);
    }
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        const int y = y0 + kRows * wave + r;
        const int above = max(mid[r], side[r]), below = max(mid[r + 2], side[r + 2]);
        const uint64_t m = __ballot(mid[r + 1] > max(max(above, below), side[r + 1]));
        if (lane == 0 && y < height) {
            masks[(size_t)tx * height + y] = m;
            counts[(size_t)y * count_stride + tx] = (uint8_t)__popcll(m);
            survivors += __popcll(m);
        }
    }
    if (tile_total) {
        if (lane == 0) atomicAdd(&kept, survivors);
        __syncthreads();
        if (t == 0) tile_total[blockIdx.x] = (uint16_t)kept;
    }
}

// Inclusive scan over the 1024 threads of the workgroup (wavefront shuffles,
// then the 16 wavefront totals).
__device__ __forceinline__ int64_t block_inclusive_scan(int64_t v, int64_t *wave_tot)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int64_t u = __shfl_up(v, o);
        if (lane >= o) v += u;
    }
    if (lane == 63) wave_tot[wave] = v;
    __syncthreads();
    int64_t before = 0;
    for (int i = 0; i < wave; ++i) before += wave_tot[i];
    __syncthreads();                                    // wave_tot is reused by the next call
    return v + before;
}

__global__ __launch_bounds__(kScanThreads) void detect_scan_kernel(
    const uint8_t *__restrict__ counts, int count_stride, int height, int tiles_x,
    int64_t *__restrict__ row_first, int64_t *__restrict__ base_out, int64_t *__restrict__ n_kps)
{
    __shared__ int64_t wave_tot[kScanThreads / 64];
    __shared__ int64_t base, chunk_total;
    if (threadIdx.x == 0) {
        const int64_t n0 = *n_kps;
        base = n0 > 0 ? n0 : 0;                          // a negative count is taken as 0
        *base_out = base;
    }
    __syncthreads();
    const int chunks = count_stride / 16;                 // 16 tile counts per chunk
    // Survivors of row r: its counts, one byte per tile, four 16-byte chunks
    // in flight; bytes past tiles_x (never written) are masked off.
    auto row_count = [&](const uint4 (&v)[4], int i) {
        int64_t c = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int valid = min(max(tiles_x - 16 * (i + k), 0), 16);
            const uint32_t w[4] = {v[k].x, v[k].y, v[k].z, v[k].w};
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const int nb = min(max(valid - 4 * d, 0), 4);
                const uint32_t keep = nb == 4 ? 0xffffffffu : (1u << (8 * nb)) - 1u;
                c += __builtin_amdgcn_sad_u8(w[d] & keep, 0u, 0u);
            }
        }
        return c;
    };
    int64_t carry = base;
    // Two rows per thread, so one pass covers 2048 rows.
    for (int r0 = 0; r0 < height; r0 += 2 * kScanThreads) {
        const int r = r0 + 2 * (int)threadIdx.x;
        int64_t c0 = 0, c1 = 0;
        if (r < height) {
            const uint4 *row0 = reinterpret_cast<const uint4 *>(counts + (size_t)r * count_stride);
            const uint4 *row1 =
                reinterpret_cast<const uint4 *>(counts + (size_t)min(r + 1, height - 1) * count_stride);
            for (int i = 0; i < chunks; i += 4) {
                uint4 v0[4], v1[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    v0[k] = row0[min(i + k, chunks - 1)];
                    v1[k] = row1[min(i + k, chunks - 1)];
                }
                c0 += row_count(v0, i);
                c1 += row_count(v1, i);
            }
            if (r + 1 >= height) c1 = 0;
        }
        const int64_t c = c0 + c1;
        const int64_t incl = block_inclusive_scan(c, wave_tot);
        if (r < height) row_first[r] = carry + incl - c;
        if (r + 1 < height) row_first[r + 1] = carry + incl - c1;
        if (threadIdx.x == kScanThreads - 1) chunk_total = incl;
        __syncthreads();
        carry += chunk_total;
        __syncthreads();
    }
    if (threadIdx.x == 0) *n_kps = carry;
}

// Image window of one tile for the orientation: rows y0 - 15 .. y0 + 30 and
// columns x0 - 16 .. x0 + 79 (every disc of a pixel of the tile), row stride
// kOriStride bytes (25 dwords: the lanes of a disc, one row each, fall in
// distinct banks).
constexpr int kOriRows = kTileH + 2 * kOrientRadius;          // 46
constexpr int kOriCols = kTileW + 32;                          // 96
constexpr int kOriStride = 100;

// Byte masks of disc row dy (lane = dy + 15): of the 32 bytes starting at
// dx = -15, bytes k = 15 - r .. 15 + r with r = floor(sqrt(15^2 - dy^2)).
__device__ __forceinline__ void disc_masks(int dy, uint32_t (&bm)[8])
{
    const int r2 = kOrientRadius * kOrientRadius - dy * dy;
    // floor(sqrt(r2)) for r2 in [0, 225]: sqrt(k^2 + 1/2) and sqrt(k^2 - 1/2)
    // lie 1/(4k) from k, far beyond the rounding of sqrtf.
    const int r = (int)__builtin_sqrtf((float)r2 + 0.5f);
    const uint32_t keep = (uint32_t)(((1ull << (kOrientRadius + r + 1)) - 1ull) &
                                     ~((1ull << (kOrientRadius - r)) - 1ull));
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const uint32_t nib = (keep >> (4 * i)) & 15u;
        bm[i] = ((nib * 0x00204081u) & 0x01010101u) * 0xffu;
    }
}

// Disc row dy of the keypoint at tile column j and tile row r_tile:
// S = sum I and W = sum k I with k = dx + 15, from 9 aligned dwords of the
// window.
__device__ __forceinline__ void disc_row(const uint8_t *win, int j, int r_tile, int dy,
                                         const uint32_t (&bm)[8], uint32_t &S, uint32_t &W)
{
    const int c = j + 1;                                   // window column of dx = -15
    const uint32_t *w =
        reinterpret_cast<const uint32_t *>(win + (r_tile + kOrientRadius + dy) * kOriStride) + (c >> 2);
    const uint32_t sh = (uint32_t)(c & 3);
    uint32_t d[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) d[i] = w[i];
    S = 0;
    W = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const uint32_t v = __builtin_amdgcn_alignbyte(d[i + 1], d[i], sh) & bm[i];
        S = __builtin_amdgcn_udot4(v, 0x01010101u, S, false);
        W = __builtin_amdgcn_udot4(v, (uint32_t)(4 * i) * 0x01010101u + 0x03020100u, W, false);
    }
}

// Sum over each row of 16 lanes (DPP: swap neighbours, swap pairs, mirror
// halves, mirror the row); every lane of the row gets the row's sum.
__device__ __forceinline__ int row16_sum(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false);   // quad_perm [1,0,3,2]
    v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false);   // quad_perm [2,3,0,1]
    v += __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, false);  // row_half_mirror
    v += __builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, false);  // row_mirror
    return v;
}

// Sum over each half-wavefront, on every lane of it.
__device__ __forceinline__ int half_sum(int v)
{
    v = row16_sum(v);
    const auto w = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return (int)w[0] + (int)w[1];
}

// Mask of the n lowest bytes of a dword (none for n <= 0, all for n >= 4).
__device__ __forceinline__ uint32_t low_bytes(int n)
{
    return n >= 4 ? 0xffffffffu : n <= 0 ? 0u : (1u << (8 * n)) - 1u;
}

// acc + the two 16-bit halves of v.
__device__ __forceinline__ uint32_t sum_u16(uint32_t v, uint32_t acc)
{
    return acc + (v & 0xffffu) + (v >> 16);
}

__device__ __forceinline__ int64_t readlane64(int64_t v, int lane)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), lane);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Angle bin of moments (m10, m01), in double as the definition states.
__device__ __forceinline__ int orientation_bin_f64(int m10, int m01)
{
    const double a = atan2((double)m01, (double)m10);
    return (int)((int64_t)rint(a * (4096.0 / (2.0 * 3.14159265358979323846))) & 4095);
}

// The same bin from a float atan2 (the moments are below 2^24, exact): its
// error of at most 6 ulp, 9.4e-4 bins at pi, and the roundings of the product,
// 2.4e-4 bins, only matter within 1/256 bin of a boundary, where the double
// decides (about one keypoint in 128).
__device__ __forceinline__ int orientation_bin(int m10, int m01)
{
    const float x = atan2f((float)m01, (float)m10) * (float)(4096.0 / (2.0 * 3.14159265358979323846));
    const float r = rintf(x);
    int bin = (int)r & 4095;
    if (fabsf(x - r) > 0.5f - 1.0f / 256.0f) bin = orientation_bin_f64(m10, m01);
    return bin;
}

// One workgroup per tile: the tile's image window goes to LDS, then wavefront
// w takes the survivors of tile rows 4 w .. 4 w + 3, listed in LDS (64 at most:
// no two survivors are neighbours).  Moments are summed two keypoints per pass
// (one per half-wavefront, a disc row per lane) and parked in LDS; then lane n
// computes the n-th keypoint's angle and writes it.
constexpr int kEmitRows = kTileH / (kThreads / 64);
constexpr int kEmitMost = kEmitRows / 2 * (kTileW / 2);

//
// kFused (at most kFusedTilesX tiles across and kFusedTiles in all): no scan
// kernel ran; the workgroup adds up the survivors of the bands of tiles above it
// from the per-tile totals (2 bytes each, read by every workgroup), then those of
// the rows above in its own band, and the last one writes the new count.
// 1920 x 1080 (2,040 tiles): 26.9 us with the scan, 25.0 without; 1277 x 719:
// 17.9 and 15.7.  The totals read grow with the square of the tile count, and at
// 3840 x 2160 (8,100 tiles) the two are equal (79.9, 80.7), so larger images
// take the scan.
constexpr int kFusedTilesX = 64, kFusedTiles = 1 << 12;

template <bool kDword, bool kFused>
__global__ __launch_bounds__(kThreads) void detect_emit_kernel(
    const uint8_t *__restrict__ img, int height, int width, int pitch, int tiles_x,
    const uint64_t *__restrict__ masks, const uint8_t *__restrict__ counts, int count_stride,
    const int64_t *__restrict__ row_first, const uint16_t *__restrict__ tile_total,
    const int64_t *__restrict__ base, int64_t *__restrict__ n_kps, float4 *__restrict__ kps,
    int64_t max_kps, int32_t *__restrict__ image_id, int32_t image_index)
{
    // Rows past kOriRows take the rounding of the load count (never read).
    __shared__ __align__(16) uint8_t win[stage_lds_rows<kOriRows, kOriCols>() * kOriStride];
    __shared__ uint8_t place[kThreads / 64][kEmitMost + 1];      // tile row - 4 w, column
    __shared__ int2 moments[kThreads / 64][kEmitMost + 1];
    __shared__ int row_total[kTileH], above_part[kThreads / 64];
    static_assert(kEmitRows * kTileW <= 256 && kEmitMost <= 64, "one byte per place, one lane per keypoint");
    const int tx = (int)(blockIdx.x % (unsigned)tiles_x), ty = (int)(blockIdx.x / (unsigned)tiles_x);
    const int x0 = tx * kTileW, y0 = ty * kTileH;
    const int t = threadIdx.x;
    const int lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int half = lane >> 5, hl = lane & 31;
    const int dy = hl - kOrientRadius;

    // Coordinates clamped to the image: discs of survivors never leave it.
    stage_window<kDword, kOriRows, kOriCols, kOriStride>(img, height, width, pitch, y0 - kOrientRadius,
                                                         x0 - 16, win);
    uint32_t bm[8];
    disc_masks(dy, bm);

    // Survivors of the wavefront's rows: masks (uniform), and in the 16 lanes
    // of row r those of the tiles to the left, four count bytes per lane.
    const int yw = y0 + kEmitRows * wave;
    uint64_t m[kEmitRows];
    int before[kEmitRows + 1];
    before[0] = 0;
#pragma unroll
    for (int r = 0; r < kEmitRows; ++r) {
        m[r] = yw + r < height ? masks[(size_t)tx * height + yw + r] : 0ull;
        before[r + 1] = before[r] + __popcll(m[r]);
    }
    const int n = __builtin_amdgcn_readfirstlane(before[kEmitRows]);
    const int rl = lane >> 4;
    const int yl = min(yw + rl, height - 1);
    int left = 0, row = 0;
    for (int c = 4 * (lane & 15); c < (kFused ? tiles_x : tx); c += 64) {
        const uint32_t v = *reinterpret_cast<const uint32_t *>(counts + (size_t)yl * count_stride + c);
        left = (int)__builtin_amdgcn_sad_u8(v & low_bytes(tx - c), 0u, (uint32_t)left);
        if (kFused) row = (int)__builtin_amdgcn_sad_u8(v & low_bytes(tiles_x - c), 0u, (uint32_t)row);
    }
    left = row16_sum(left);
    int64_t slot;                                            // of the row's first survivor in this tile
    if (kFused) {
        row = row16_sum(row);
        if ((lane & 15) == 0) row_total[kEmitRows * wave + rl] = yw + rl < height ? row : 0;
        uint32_t part = 0;
        const int tiles_above = ty * tiles_x;
        for (int i = 8 * t; i < tiles_above; i += 8 * kThreads) {
            const uint4 v = *reinterpret_cast<const uint4 *>(tile_total + i);
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const int nb = 2 * (tiles_above - i) - 4 * d;
                part = sum_u16(w[d] & low_bytes(nb), part);
            }
        }
        int sum = half_sum((int)part);
        sum = __builtin_amdgcn_readlane(sum, 0) + __builtin_amdgcn_readlane(sum, 32);
        if (lane == 0) above_part[wave] = sum;
    } else {
        slot = row_first[yl] + left;
    }

    uint8_t *at = place[wave];
    int2 *mom = moments[wave];
#pragma unroll
    for (int r = 0; r < kEmitRows; ++r) {
        const int rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(m[r] >> 32),
                                                   __builtin_amdgcn_mbcnt_lo((uint32_t)m[r], 0));
        if ((m[r] >> lane) & 1) at[before[r] + rank] = (uint8_t)(r * kTileW + lane);
    }
    __syncthreads();
    if (kFused) {
        int64_t all = *base;
#pragma unroll
        for (int i = 0; i < kThreads / 64; ++i) all += above_part[i];
        slot = all + left;
#pragma unroll
        for (int i = 0; i < kTileH; ++i) {
            const int v = row_total[i];
            all += v;
            slot += i < kEmitRows * wave + rl ? v : 0;
        }
        if (blockIdx.x == gridDim.x - 1 && t == 0) *n_kps = all;
    }
    // First slot of each row's survivors in this tile (uniform; read with
    // every lane active).
    int64_t first[kEmitRows];
#pragma unroll
    for (int r = 0; r < kEmitRows; ++r) first[r] = readlane64(slot, 16 * r);

    for (int k = 0; k < n; k += 2) {
        const int e = at[min(k + half, n - 1)];
        uint32_t S = 0, W = 0;
        if (hl < kDiscRows) disc_row(win, e % kTileW, kEmitRows * wave + e / kTileW, dy, bm, S, W);
        int2 v;
        v.x = half_sum((int)W - kOrientRadius * (int)S);
        v.y = half_sum(dy * (int)S);
        if (hl == 0 && k + half < n) mom[k + half] = v;
    }
    // The wavefront's own moments: its LDS accesses are in order.
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (lane < n) {
        const int e = at[lane];
        const int r = e / kTileW;
        const int2 v = mom[lane];
        int bf = 0;
        int64_t s = 0;
#pragma unroll
        for (int i = 0; i < kEmitRows; ++i)
            if (r == i) {
                bf = before[i];
                s = first[i];
            }
        s += lane - bf;
        if (s < max_kps) {
            kps[s] = make_float4((float)(x0 + e % kTileW), (float)(yw + r),
                                 (float)orientation_bin(v.x, v.y) * (360.0f / 4096.0f), 1.0f);
            if (image_id) image_id[s] = image_index;
        }
    }
}

}  // namespace

hipError_t launch_detect(const DetectArgs &a, hipStream_t stream)
{
    const int tiles_x = (a.width + kTileW - 1) / kTileW;
    const int64_t tiles = (int64_t)tiles_x * ((a.height + kTileH - 1) / kTileH);
    const bool dword = (reinterpret_cast<uintptr_t>(a.img) & 3) == 0 && (a.pitch & 3) == 0 &&
                       (a.width & 3) == 0;
    // The per-tile totals take the place of the rows' first slots (2 bytes per
    // tile, at most 64 tiles per band of 16 rows, against 8 bytes per row).
    const bool fused = tiles_x <= kFusedTilesX && tiles <= kFusedTiles;
    static_assert(2 * kFusedTilesX <= 8 * kTileH, "totals fit the rows' first slots");
    uint16_t *totals = fused ? reinterpret_cast<uint16_t *>(a.row_first) : nullptr;
    hipLaunchKernelGGL(dword ? detect_tile_kernel<true> : detect_tile_kernel<false>,
                       dim3((unsigned)tiles), dim3(kThreads), 0, stream, a.img, a.height, a.width,
                       a.pitch, a.threshold, tiles_x, a.masks, a.counts, a.count_stride, totals, a.n_kps,
                       fused ? a.base : nullptr);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (!fused) {
        hipLaunchKernelGGL(detect_scan_kernel, dim3(1), dim3(kScanThreads), 0, stream, a.counts,
                           a.count_stride, a.height, tiles_x, a.row_first, a.base, a.n_kps);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    const auto emit = fused ? (dword ? detect_emit_kernel<true, true> : detect_emit_kernel<false, true>)
                            : (dword ? detect_emit_kernel<true, false> : detect_emit_kernel<false, false>);
    hipLaunchKernelGGL(emit, dim3((unsigned)tiles), dim3(kThreads), 0, stream, a.img, a.height, a.width,
                       a.pitch, tiles_x, a.masks, a.counts, a.count_stride, a.row_first, totals, a.base,
                       a.n_kps, a.kps, a.max_kps, a.image_id, a.image_index);
    return hipGetLastError();
}

}  // namespace latch
