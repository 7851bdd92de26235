// Dense CLATCH and dense matching for gfx950 (Sec. 6 proposes CLATCH for
// dense pixel matching).
//
// Dense extraction: the descriptor of every pixel p of a region, upright and
// at scale 1 (the resampling rule then samples I(p + (u, v)) with clamping,
// so the window is the edge-padded image around p).  For a triplet with
// patch centres A, C1, C2 (window coordinates), Eq. 1 compares
//     S1 - S2 = sum over the 7 x 7 box of G(q),
//     G(q) = (I(q + c1) - I(q + c2)) (I(q + c1) + I(q + c2) - 2 I(q + a)),
// with a, c1, c2 the centres minus (24, 24): bit = [box7x7(G)(p) > 0].  So a
// workgroup that owns a tile of pixels evaluates G once per position and
// triplet and sums it over 7 rows and 7 columns, instead of 3 x 49 products per
// pixel and triplet.  |G| <= 130,050, a column's prefix sum over 38 rows and the
// box sum stay below 2^23, so int32 is exact, and the result is bit-identical
// to extracting at every pixel.
//
// A lane holds two neighbouring columns.  Their pixels are one dword of 16-bit
// lanes (two copies of the window in LDS, one shifted by a pixel, make that so
// for odd offsets too), so the two factors of -G take three packed instructions
// per two pixels, and v_mad_i32_i16 adds their product to each column's prefix
// sum; two prefix sums 7 rows apart differ by a 7-row sum.  The 7-column sums of
// two columns share the sums of column pairs: six adds with the neighbour's value
// through DPP and one without, for two outputs.  The sign of a sum is shifted
// into the output word by one v_alignbit.  In all 16 instructions per two pixels
// and triplet, plus 5 for the 6 rows of halo.
//
// What bounds it: vector issue, 88% of the time on the SIMDs of a 1920 x 1080
// frame.  One column per lane with byte pixels took 14 instructions per pixel
// (and 6 of 64 lanes of halo, now 6 of 128 columns): 618 -> 320 us there,
// 258 -> 51 us for 64 x 48, where a workgroup now computes 4 of the 16 words and
// the tile's 512 triplets spread over 4 workgroups.  The words of a pixel leave
// as 16 bytes through LDS: HBM writes fell from 629 MB to the 130 MB of the
// output.
//
// Dense matching: per query pixel, the two nearest train pixels by Hamming
// distance within +/- R rows and columns (R <= 8), ties to the lower raster
// index, ratio test as in hamming_knn.  A workgroup owns 16 x 16 queries, stages
// the packed train descriptors around them in LDS and forms the distances on
// the FP4 matrix cores.
#include <algorithm>
#include <type_traits>

#include "internal.h"

namespace latch {
namespace {

#include "codegen.h"
#include "fp4.h"
#include "lanes.h"
#include "packed16.h"
#include "xcd_range.h"

constexpr int kDThreads = 256;
constexpr int kDTileW = 122;                        // output columns: 2 l, 2 l + 1 of lanes 0..60
constexpr int kDTileH = 32;                         // output rows per workgroup
constexpr int kDWords = 4;                          // descriptor words per workgroup, one per wavefront
constexpr int kDRegionRows = kDTileH + 6;           // rows of G per tile
constexpr int kDTexRows = kDRegionRows + 41;        // image rows: 79
constexpr int kDTexQuads = 43;                      // image columns in fours: 172 (128 + 41 are read)
constexpr int kDRowBytes = 2 * 170;                 // a row of 16-bit pixels: 85 dwords
constexpr int kDCopyBytes = kDTexRows * kDRowBytes;
constexpr int kDUnits = kDTexRows * kDTexQuads;
constexpr int kDLoads = (kDUnits + kDThreads - 1) / kDThreads;
constexpr int kDGroup = 3;                          // texture rows read together
constexpr int kDOutRows = 16;                       // rows per pass of the output transpose
constexpr int kDLdsBytes = 2 * kDCopyBytes + 8;     // 3 workgroups per CU
static_assert(2 * kDCopyBytes <= 65536, "16-bit patch offsets");
static_assert(3 * kDLdsBytes <= kLdsPerCu, "three workgroups per CU");
static_assert(kDOutRows * 128 * 16 <= kDLdsBytes && kDTileH % kDOutRows == 0, "output transpose fits");

// Lane l receives lane l + 1's value (DPP wave_shl:1; lane 63 receives 0
// through bound_ctrl, so no old value has to be set up).
__device__ __forceinline__ int lane_next(int v)
{
    return __builtin_amdgcn_mov_dpp(v, 0x130, 0xF, 0xF, true);
}

// bits = bits << 1 | sign of h, in place.
__device__ __forceinline__ void shift_in_sign(uint32_t &bits, int h)
{
    asm("v_alignbit_b32 %0, %0, %1, 31" : "+v"(bits) : "v"(h));
}

// The image window of a tile, in LDS as 16-bit pixels in two copies: copy 0
// holds pixel (row, x) at element x of row `row`, copy 1 at element x - 1, so
// that the pixels x, x + 1 of any column x are one dword of copy x & 1.
// kInside: every column lies in the image and four pixels are one (unaligned)
// load; otherwise columns clamp to the image one by one (the rule's
// clamp-to-edge).  Rows clamp either way.
template <bool kInside>
__device__ __forceinline__ void stage_texture(const uint8_t *__restrict__ img, int height, int width,
                                              int pitch, int xs, int ys, uint8_t *__restrict__ tex)
{
    constexpr int kBatch = kInside ? 7 : 4;               // loads (of four pixels) in flight
    for (int k0 = 0; k0 < kDLoads; k0 += kBatch) {
        uint32_t v[kBatch];
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            const int i = min((int)threadIdx.x + (k0 + k) * kDThreads, kDUnits - 1);
            const int x = xs + 4 * (i % kDTexQuads);
            const uint8_t *row = img + (size_t)min(max(ys + i / kDTexQuads, 0), height - 1) * pitch;
            if constexpr (kInside) {
                __builtin_memcpy(&v[k], row + x, 4);
            } else {
                uint32_t w = 0;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    w |= (uint32_t)row[min(max(x + j, 0), width - 1)] << (8 * j);
                v[k] = w;
            }
        }
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            const int i = (int)threadIdx.x + (k0 + k) * kDThreads;
            if (i >= kDUnits) break;
            const int q = i % kDTexQuads;
            uint8_t *to = tex + i / kDTexQuads * kDRowBytes + 8 * q;
            const uint32_t p01 = __builtin_amdgcn_perm(0, v[k], 0x0c010c00), p12 = __builtin_amdgcn_perm(0, v[k], 0x0c020c01),
                           p23 = __builtin_amdgcn_perm(0, v[k], 0x0c030c02);
            // Columns 170 and 171 of the last quad would land in the next row.
            *reinterpret_cast<uint32_t *>(to) = p01;
            if (q < kDTexQuads - 1) *reinterpret_cast<uint32_t *>(to + 4) = p23;
            uint8_t *to1 = to + kDCopyBytes;
            if (q > 0) *reinterpret_cast<uint16_t *>(to1 - 2) = (uint16_t)p01;
            *reinterpret_cast<uint32_t *>(to1) = p12;
            if (q < kDTexQuads - 1) *reinterpret_cast<uint16_t *>(to1 + 4) = (uint16_t)(p23 >> 16);
        }
    }
}

// Block b covers words 4 y .. 4 y + 3 of tile t; the four blocks of a tile run
// on one XCD (workgroups go to the 8 XCDs round-robin by index), whose L2 then
// joins their quarters of each 64-byte descriptor.
__global__ __launch_bounds__(kDThreads) __attribute__((amdgpu_waves_per_eu(3, 3))) void
dense_extract_kernel(const uint8_t *__restrict__ img, int height, int width, int pitch, int x0, int y0,
                     int gw, int gh, int tiles_x, int tiles, const uint2 *__restrict__ toff,
                     uint32_t *__restrict__ desc)
{
    __shared__ __align__(16) uint8_t tex[kDLdsBytes];
    const int local = (int)(blockIdx.x >> 3);
    const int tile = (local / (kWords / kDWords)) * 8 + (int)(blockIdx.x & 7);
    const int part = local % (kWords / kDWords);
    if (tile >= tiles) return;
    const int X0 = x0 + tile % tiles_x * kDTileW, Y0 = y0 + tile / tiles_x * kDTileH;
    const int t = threadIdx.x;
    const int lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);

    // Image rows Y0 - 24 .. Y0 + 54 and columns X0 - 24 .. X0 + 147.
    const int xs = X0 - 24, ys = Y0 - 24;
    if (xs >= 0 && xs + 4 * kDTexQuads <= width)
        stage_texture<true>(img, height, width, pitch, xs, ys, tex);
    else
        stage_texture<false>(img, height, width, pitch, xs, ys, tex);
    __syncthreads();

    const int word = kDWords * part + wave;
    uint32_t bits[kDTileH][2];                      // of columns 2 l, 2 l + 1
#pragma unroll
    for (int o = 0; o < kDTileH; ++o) bits[o][0] = bits[o][1] = 0u;
    for (int b = 0; b < 32; ++b) {
        const uint2 off = toff[32 * word + b];      // uniform: scalar loads
        const uint8_t *pa = tex + 4 * lane + (off.x & 0xffffu);
        const uint8_t *p1 = tex + 4 * lane + (off.x >> 16);
        const uint8_t *p2 = tex + 4 * lane + off.y;
        int pre0[7], pre1[7];                       // prefix sums of -G down the two columns
        int s0 = 0, s1 = 0, v0[2], v1[2];
        // Rows are read in groups, one group ahead of their use; the groups are
        // kept apart (left alone, the compiler reads most rows first and
        // spills).
        short2v px[2][kDGroup][3];
        auto read_rows = [&](int rr) {
#pragma unroll
            for (int k = 0; k < kDGroup; ++k) {
                if (rr + k >= kDRegionRows) break;
                short2v *to = px[rr / kDGroup & 1][k];
                to[0] = *reinterpret_cast<const short2v *>(pa + (rr + k) * kDRowBytes);
                to[1] = *reinterpret_cast<const short2v *>(p1 + (rr + k) * kDRowBytes);
                to[2] = *reinterpret_cast<const short2v *>(p2 + (rr + k) * kDRowBytes);
            }
        };
        read_rows(0);
#pragma unroll
        for (int rr = 0; rr < kDRegionRows; ++rr) {
            if (rr % kDGroup == 0) {
                __builtin_amdgcn_sched_barrier(0);
                read_rows(rr + kDGroup);
            }
            const short2v *at = px[rr / kDGroup & 1][rr % kDGroup];
            const short2v a = at[0], c1 = at[1], c2 = at[2];
            const short2v d = c2 - c1;
            const short2v s = pk_mad_i16(a, kPkMinus2, c1 + c2);
            s0 = mad_i32_lo16(d, s, s0);
            s1 = mad_i32_hi16(d, s, s1);
            if (rr >= 6) {
                // Rows rr - 6 .. rr of the two columns.
                v0[rr & 1] = rr > 6 ? s0 - pre0[rr % 7] : s0;
                v1[rr & 1] = rr > 6 ? s1 - pre1[rr % 7] : s1;
            }
            if (rr > 6 && (rr & 1)) {
                // Seven columns from each, for two rows: with p = v0 + v1 and
                // lanes l, l + 1, ..: p + p + p + v0 and v1 + p + p + p, in
                // Horner form, the four chains in step (a DPP operand is not to
                // be one of the last two results).
                int h[2][2];
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    h[k][0] = v0[k];
                    h[k][1] = v0[k] + v1[k];
                }
                const int p[2] = {h[0][1], h[1][1]};
#pragma unroll
                for (int step = 0; step < 3; ++step)
#pragma unroll
                    for (int c = 0; c < 2; ++c)
#pragma unroll
                        for (int k = 0; k < 2; ++k)
                            h[k][c] = (c == 1 && step == 2 ? v1[k] : p[k]) + lane_next(h[k][c]);
                // Shift the sign (box sum of G > 0) in from the right: triplet b
                // ends at bit 31 - b.
#pragma unroll
                for (int k = 0; k < 2; ++k)
#pragma unroll
                    for (int c = 0; c < 2; ++c) shift_in_sign(bits[rr - 7 + k][c], h[k][c]);
            }
            pre0[rr % 7] = s0;
            pre1[rr % 7] = s1;
        }
    }

    // The four wavefronts' words of a pixel meet in LDS and leave as 16 bytes.
#pragma unroll
    for (int o0 = 0; o0 < kDTileH; o0 += kDOutRows) {
        __syncthreads();                            // texture or the previous rows are read
#pragma unroll
        for (int o = 0; o < kDOutRows; ++o)
#pragma unroll
            for (int c = 0; c < 2; ++c)
                reinterpret_cast<uint32_t *>(tex)[((2 * o + c) * 64 + lane) * kDWords + wave] =
                    __builtin_bitreverse32(bits[o0 + o][c]);
        __syncthreads();
        for (int i = t; i < kDOutRows * kDTileW; i += kDThreads) {
            const int o = i / kDTileW, c = i % kDTileW;
            const int px = X0 - x0 + c, py = Y0 - y0 + o0 + o;
            if (px < gw && py < gh)
                reinterpret_cast<uint4 *>(desc)[((size_t)py * gw + px) * (kWords / 4) + part] =
                    reinterpret_cast<const uint4 *>(tex)[(2 * o + (c & 1)) * 64 + (c >> 1)];
        }
    }
}

// ---------------------------------------------------------------------------
// Dense matching on the FP4 matrix cores (v_mfma_f32_16x16x128_f8f6f4).
//
// A wavefront owns 4 x 16 query pixels (4 columns, 16 rows) as four blocks of
// 4 x 4, and a workgroup of four wavefronts 16 x 16.  A block of 16 queries
// meets the S x S train pixels around it, S = 4 + 2 RP with RP the radius
// rounded up to even: S^2 is then a multiple of 16 and the train pixels of the
// stack's columns, S per row, form whole 16-row MFMA tiles of which block b
// uses the S rows from 4 b on.  Four train rows (a quad) are S / 4 tiles, and
// blocks one below the other share all but one of their S / 4 quads, so an
// expanded tile serves up to four blocks.  Of the S^2 distances a query gets,
// (2 R + 1)^2 are candidates (0.56 at radius 4, 0.72 at radius 8); the matrix
// instruction still makes them at several times the rate of XOR and popcount.
//
// Operands (fp4.h).  A: train pixels, lane l = 16 g + m holds words 4 g ..
// 4 g + 3 of tile row m (one ds_read_b128 of packed bits, expanded in
// registers), word 4 g + s in step s.  B: queries, lane l holds the same words
// of query n = l % 16, as +-1 / c.  The f32 sum is |a| - d, exact.  (No block
// scales: the instruction without them issues in half the time.)
//
// Keys.  Output lane 16 g + n, register r is train row 4 g + r of the tile
// against query n.  The accumulator starts at 512 + (a constant - p) / 1024 for
// position p of the quad, or at -2^15 where p lies outside the query's own
// (2 R + 1)^2 window, and the block's best two move up by the positions of a quad
// when the next one starts, so a key ends as 512 + |a| - d + (1023 - p) / 1024 for
// position p of the S x S region (larger is better: smaller distance, then
// lower raster index) or below zero: multiples of 1/1024 below 2^11, exact in f32,
// whose bit patterns order like the signed integers they are compared as.  Only a
// block's first and last quads hold rows outside a query's window, so three
// kinds of start values, kept in registers over the workgroup's tiles, do for
// all of them.  Train pixels outside the grid are masked after the product, in
// workgroup tiles at its border only.
//
// What bounds it: vector issue.  At 1920 x 1080 and radius 4 a wavefront takes
// about 900 vector instructions and 145 matrix instructions per 64 queries, and
// the SIMDs issue vector instructions 82% of the time; the 0.30 GB of
// descriptors, indices and distances take 48 us by themselves (radius 0).
// Measured (2-NN, accept flags) against XOR and popcount over the same staged
// region: radius 2 99 -> 70 us, radius 4 256 -> 98 us, radius 8 1069 -> 182 us.
// Not kept, no faster: the next tile's loads issued before this one's
// arithmetic, bit 3 of a train nibble used in place as the sign (one
// instruction less per word, with a per-query correction).

constexpr int kMTile = 16;                               // queries per side of a workgroup
constexpr int kWindowPosBits = 10;                          // positions are a key's fraction
constexpr float kWindowPos = 1.0f / (1 << kWindowPosBits);
constexpr float kWindowNone = -32768.0f;
constexpr float kWindowBias = 512.0f;                       // keys are positive

template <int RP>
struct WindowGeom {
    static_assert(RP % 2 == 0 && RP > 0 && RP <= kDenseMaxRadius, "even region margin");
    static constexpr int kS = 4 + 2 * RP;                // region side of a block
    static constexpr int kQuadTiles = kS / 4;            // MFMA tiles per four train rows
    static constexpr int kSide = kMTile + 2 * RP;        // staged train pixels per side
    static constexpr int kQuads = kSide / 4;
    static constexpr int kRowsPerWave = kSide / 4;       // staged by each wavefront
    static constexpr int kExtraCols = 2 * RP;            // past the first 16
    static constexpr int kExtraLoads = (kRowsPerWave * 2 * RP + 15) / 16;
    // LDS: 16-byte chunk c of pixel (row, col) at c kPlane + row kStride + col.
    // kStride - S is a multiple of 16, so 16 consecutive region positions fall
    // in distinct banks also across a row's end; the planes are 4 pixels (64
    // bytes) apart in banks, so staging writes of four chunks do not collide.
    static constexpr int kStride = kS + 16;
    static constexpr int kPlane = kSide * kStride + 4;
    // Positions count down from kFirst within a quad, and a block's keys move
    // up by kQuadPos when its next quad starts.
    static constexpr int kQuadPos = 16 * kQuadTiles;
    static constexpr int kFirst = (1 << kWindowPosBits) - 1 - kQuadPos * (kQuadTiles - 1);
    static_assert(kFirst >= kQuadPos, "positions below the distance");
    // Kinds of quads of a block: first, between, last.  Rows between are in
    // every query's window (RP - R <= 1), so those quads have the same masks.
    static constexpr int kKinds = kQuadTiles < 3 ? kQuadTiles : 3;
    static constexpr int kind_of(int dq) { return dq == 0 ? 0 : dq == kQuadTiles - 1 ? kKinds - 1 : 1; }
    static constexpr int kind_row(int c) { return c == 0 ? 0 : c == kKinds - 1 ? kS - 4 : 4; }
    static_assert(kPlane % 16 == 4, "planes spread over the banks");
    // Wavefronts per SIMD, and so workgroups of four per CU: what LDS and the
    // registers of start values allow.
    static constexpr int kWaves = RP >= 4 ? 2 : 3;
    static_assert(kWaves * kPlane * 64 <= kLdsPerCu, "workgroups per CU fit the LDS");
};

__device__ __forceinline__ int imed3(int a, int b, int c) { return max(min(a, b), min(max(a, b), c)); }

// Two keys into a running top two (k1 >= k2): med3, max3, max.  The max3 is
// written out (the compiler would reuse the median's inner maximum and take
// two instructions); it names the median so that it follows it, and with it
// the wait states that the compiler puts between a matrix instruction and the
// first use of its result.
__device__ __forceinline__ void insert_keys(int &k1, int &k2, int x, int y)
{
    const int m = imed3(k1, x, y);
    asm("v_max3_i32 %0, %0, %1, %2" : "+v"(k1) : "v"(x), "v"(y), "v"(m));
    k2 = max(k2, m);
}

template <int RP>
__global__ __launch_bounds__(kDThreads)
__attribute__((amdgpu_waves_per_eu(WindowGeom<RP>::kWaves, WindowGeom<RP>::kWaves))) void
dense_match_kernel(const uint32_t *__restrict__ query, const uint32_t *__restrict__ train, int gw,
                   int gh, int radius, int tiles_x, int64_t tiles, int k, float ratio,
                   int32_t *__restrict__ idx, int32_t *__restrict__ dist, uint8_t *__restrict__ accept)
{
    using G = WindowGeom<RP>;
    __shared__ uint4 region[4 * G::kPlane];
    const int t = threadIdx.x;
    const int lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int g = lane >> 4, n = lane & 15;
    const int qr = n >> 2, qc = n & 3;

    // Start values of tile j of a quad, for a block's first quad, its last one
    // and those between: positions 16 j + 4 g + r, all four in one region row
    // (S is a multiple of 4).
    v4f start[G::kKinds][G::kQuadTiles];
#pragma unroll
    for (int c = 0; c < G::kKinds; ++c)
#pragma unroll
        for (int j = 0; j < G::kQuadTiles; ++j) {
            const int p = 16 * j + 4 * g;
            const int row = G::kind_row(c) + p / G::kS, col = p % G::kS;
            const bool row_ok = abs(row - qr - RP) <= radius;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                start[c][j][r] = (row_ok & (abs(col + r - qc - RP) <= radius))
                                     ? kWindowBias + (float)(G::kFirst - p - r) * kWindowPos
                                     : kWindowNone;
        }
    // LDS position of tile row m = n of the quad's tiles.
    int frag_at[G::kQuadTiles];
#pragma unroll
    for (int j = 0; j < G::kQuadTiles; ++j) {
        const int p = 16 * j + n;
        frag_at[j] = g * G::kPlane + p / G::kS * G::kStride + p % G::kS + 4 * wave;
    }

    const int sc = lane & 3, scol = lane >> 2;           // staging: chunk, column
    const int stage_to = sc * G::kPlane + G::kRowsPerWave * wave * G::kStride;

    // A tile's loads.  Queries: words 4 g .. 4 g + 3 of query n of each block;
    // one outside the grid takes a pixel inside it and is not stored.  Train
    // pixels: rows kRowsPerWave wave .. of the region, columns 0 .. 15 with one
    // row per load (uniform row, lane = (column, chunk)), the columns past 15
    // with several.  Pixels outside the grid take one inside it (coordinates
    // clamped relative to the first staged row and column), and their distances
    // are masked.
    struct Loads {
        uint4 q[4], v[G::kRowsPerWave], vx[G::kExtraLoads];
    };
    auto fetch = [&](uint32_t x0, uint32_t y0, Loads &ld) {
        const uint32_t xq = min(4u * wave + qc, (uint32_t)gw - 1u - x0);
        const uint32_t yq = (uint32_t)gh - 1u - y0;
        const uint4 *at = reinterpret_cast<const uint4 *>(query) + ((size_t)y0 * gw + x0) * 4;
#pragma unroll
        for (int b = 0; b < 4; ++b)
            ld.q[b] = at[(uint64_t)min(4u * b + qr, yq) * (uint32_t)gw * 4 + 4 * xq + g];

        const int left = x0 < RP ? RP - (int)x0 : 0, above = y0 < RP ? RP - (int)y0 : 0;
        const uint32_t xb = x0 + left - RP, yb = y0 + above - RP;
        const int xlim = (int)min((uint32_t)gw - 1u - xb, (uint32_t)kMTile + 2 * RP);
        const int ylim = (int)min((uint32_t)gh - 1u - yb, (uint32_t)kMTile + 2 * RP);
        at = reinterpret_cast<const uint4 *>(train) + ((size_t)yb * gw + xb) * 4;
        const uint32_t xa = 4u * min(max(scol - left, 0), xlim) + sc;
#pragma unroll
        for (int i = 0; i < G::kRowsPerWave; ++i) {
            const int row = min(max(G::kRowsPerWave * wave + i - above, 0), ylim);
            ld.v[i] = (at + (size_t)row * gw * 4)[xa];
        }
#pragma unroll
        for (int i = 0; i < G::kExtraLoads; ++i) {
            const int e = scol + 16 * i;
            const int row = min(max(G::kRowsPerWave * wave + e / G::kExtraCols - above, 0), ylim);
            const int xe = min(max(16 + e % G::kExtraCols - left, 0), xlim);
            ld.vx[i] = at[(uint64_t)(uint32_t)row * (uint32_t)gw * 4 + (uint32_t)(4 * xe + sc)];
        }
    };

    // Tile coordinates, stepped without divisions.  (Pixel coordinates are in
    // 32-bit unsigned arithmetic: one below 0 or past 2^31 compares as outside
    // the grid.)
    const XcdRange range = xcd_range(tiles);
    uint32_t tx = (uint32_t)range.first % (uint32_t)tiles_x, ty = (uint32_t)range.first / (uint32_t)tiles_x;
    const uint32_t step_x = (uint32_t)range.stride % (uint32_t)tiles_x;
    const uint32_t step_y = (uint32_t)range.stride / (uint32_t)tiles_x;
    for (int64_t tile = range.first; tile < range.end; tile += range.stride) {
        const uint32_t x0 = tx * kMTile, y0 = ty * kMTile;
        tx += step_x;
        ty += step_y;
        if (tx >= (uint32_t)tiles_x) {
            tx -= (uint32_t)tiles_x;
            ++ty;
        }

        Loads ld;
        fetch(x0, y0, ld);
        __syncthreads();                       // the previous tile's reads are done
#pragma unroll
        for (int i = 0; i < G::kRowsPerWave; ++i) region[stage_to + i * G::kStride + scol] = ld.v[i];
#pragma unroll
        for (int i = 0; i < G::kExtraLoads; ++i) {
            const int e = scol + 16 * i;
            if (G::kRowsPerWave * 2 * RP % 16 == 0 || e < G::kRowsPerWave * 2 * RP)
                region[stage_to + e / G::kExtraCols * G::kStride + 16 + e % G::kExtraCols] = ld.vx[i];
        }

        uint4 bq[4][4];
        int na[4], k1[4], k2[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const uint32_t w[4] = {ld.q[b].x, ld.q[b].y, ld.q[b].z, ld.q[b].w};
            na[b] = 0;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                bq[b][s] = fp4_query(w[s]);
                na[b] += __popc(w[s]);
            }
            k1[b] = k2[b] = __float_as_int(kWindowNone);
        }
        __syncthreads();

        // Some staged pixel lies outside the grid (uniform).
        const bool border = x0 < RP || y0 < RP || x0 + kMTile + RP > (uint32_t)gw ||
                            y0 + kMTile + RP > (uint32_t)gh;
        // Wavefronts in the distances issue before those that stage: radius 4 103 -> 98 us,
        // radius 6 145 -> 137; the other way round 99 and 142.
        __builtin_amdgcn_s_setprio(2);
        auto distances = [&](auto at_border) {
            uint4 packed = region[frag_at[0]];
#pragma unroll
            for (int q = 0; q < G::kQuads; ++q) {
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    if (q > b && q < b + G::kQuadTiles) {
                        k1[b] = __float_as_int(__int_as_float(k1[b]) + G::kQuadPos * kWindowPos);
                        k2[b] = __float_as_int(__int_as_float(k2[b]) + G::kQuadPos * kWindowPos);
                    }
#pragma unroll
                for (int j = 0; j < G::kQuadTiles; ++j) {
                    // The next tile's packed rows are read one tile ahead; tiles
                    // are kept apart so that the reads do not all move up and
                    // spill.
                    __builtin_amdgcn_sched_barrier(0);
                    const uint32_t w[4] = {packed.x, packed.y, packed.z, packed.w};
                    if (j + 1 < G::kQuadTiles)
                        packed = region[frag_at[j + 1] + 4 * q * G::kStride];
                    else if (q + 1 < G::kQuads)
                        packed = region[frag_at[0] + 4 * (q + 1) * G::kStride];
                    v4f acc[4];
#pragma unroll
                    for (int s = 0; s < 4; ++s) {
                        const v8i a = fp4_operand(fp4_train(w[s]));
#pragma unroll
                        for (int b = 0; b < 4; ++b) {
                            if (q < b || q >= b + G::kQuadTiles) continue;
                            acc[b] = fp4_mfma(a, fp4_operand(bq[b][s]),
                                              s == 0 ? start[G::kind_of(q - b)][j] : acc[b]);
                        }
                    }
                    if constexpr (decltype(at_border)::value) {
                        const int o = 16 * j + 4 * opaque(g);
                        const uint32_t y = y0 + (uint32_t)(4 * q + o / G::kS - RP);
                        const uint32_t x = x0 + (uint32_t)(4 * wave + o % G::kS - RP);
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const bool real = (y < (uint32_t)gh) & (x + r < (uint32_t)gw);
#pragma unroll
                            for (int b = 0; b < 4; ++b)
                                if (q >= b && q < b + G::kQuadTiles) acc[b][r] = real ? acc[b][r] : kWindowNone;
                        }
                    }
#pragma unroll
                    for (int r = 0; r < 4; r += 2)
#pragma unroll
                        for (int b = 0; b < 4; ++b)
                            if (q >= b && q < b + G::kQuadTiles)
                                insert_keys(k1[b], k2[b], __float_as_int(acc[b][r]),
                                            __float_as_int(acc[b][r + 1]));
                    // A tile's keys are taken before the next tile's products (left
                    // alone, the compiler regroups the maxima and spills sums).
#pragma unroll
                    for (int b = 0; b < 4; ++b)
                        if (q >= b && q < b + G::kQuadTiles) {
                            k1[b] = opaque(k1[b]);
                            k2[b] = opaque(k2[b]);
                        }
                }
            }
        };
        if (border)
            distances(std::true_type{});
        else
            distances(std::false_type{});

        __builtin_amdgcn_s_setprio(0);
        // The four lane rows hold partial results of all four blocks: lane row
        // b ends with block b's.
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            exchange_top2<true>(k1[b], k2[b], k1[b + 2], k2[b + 2]);
            exchange_sum<true>(na[b], na[b + 2]);
        }
        exchange_top2<false>(k1[0], k2[0], k1[1], k2[1]);
        exchange_sum<false>(na[0], na[1]);

        const uint32_t qy = y0 + 4 * g + qr, qx = x0 + 4 * wave + qc;
        if (qy < (uint32_t)gh && qx < (uint32_t)gw) {
            auto decode = [&](int bits, int32_t &i_out, int32_t &d_out) {
                if (bits < 0) {
                    i_out = -1;
                    d_out = 513;
                    return;
                }
                const int key = (int)(__int_as_float(bits) * (1 << kWindowPosBits));
                const int p = 1023 - (key & 1023);              // of the S x S region
                i_out = ((int)qy + p / G::kS - qr - RP) * gw + (int)qx + p % G::kS - qc - RP;
                d_out = na[0] + 512 - (key >> kWindowPosBits);
            };
            int32_t i1, d1, i2, d2;
            decode(k1[0], i1, d1);
            decode(k2[0], i2, d2);
            const size_t q = (size_t)qy * gw + qx;
            if (k == 2) {
                reinterpret_cast<int2 *>(idx)[q] = make_int2(i1, i2);
                reinterpret_cast<int2 *>(dist)[q] = make_int2(d1, d2);
            } else {
                idx[q] = i1;
                dist[q] = d1;
            }
            // Two candidates in the window and the exact ratio test.
            if (accept) accept[q] = (uint8_t)(k2[0] >= 0 && (double)d1 < (double)ratio * (double)d2);
        }
    }
}

// ---------------------------------------------------------------------------
// Dense matching at radius 0 and 1: XOR and popcount, one query per lane.  At
// most 9 candidates per query do not pay for expanding train and query bits
// into matrix operands (1920 x 1080, 2-NN with accept flags: radius 0 48 us
// against 54 us, radius 1 64 us against 70 us, radius 2 99 us against 70 us).

constexpr int kPopcountRadius = 1;

__global__ __launch_bounds__(kDThreads) void window_popcount_kernel(
    const uint32_t *__restrict__ query, const uint32_t *__restrict__ train, int gw, int gh, int radius,
    int tiles_x, int k, float ratio, int32_t *__restrict__ idx, int32_t *__restrict__ dist,
    uint8_t *__restrict__ accept)
{
    // Train descriptors of the (16 + 2 radius)^2 region, 64 B each, stored
    // chunk-major: the 16-byte chunk c of position p is region[c plane + p].
    // The 16 lanes of a query row read chunk c of 16 consecutive positions,
    // 256 contiguous bytes, which LDS serves without bank conflicts.
    __shared__ uint4 region[4 * (kMTile + 2 * kPopcountRadius) * (kMTile + 2 * kPopcountRadius)];
    const int tx = (int)(blockIdx.x % (unsigned)tiles_x), ty = (int)(blockIdx.x / (unsigned)tiles_x);
    const int t = threadIdx.x;
    const int side = kMTile + 2 * radius;
    const int plane = side * side;
    const int rx0 = tx * kMTile - radius, ry0 = ty * kMTile - radius;
    for (int i = t; i < side * side * 4; i += kDThreads) {
        const int p = i >> 2, c = i & 3;
        const int gy = ry0 + p / side, gx = rx0 + p % side;
        uint4 val = make_uint4(0u, 0u, 0u, 0u);
        if (gy >= 0 && gy < gh && gx >= 0 && gx < gw)
            val = reinterpret_cast<const uint4 *>(train + ((size_t)gy * gw + gx) * kWords)[c];
        region[c * plane + p] = val;
    }
    const int qx = tx * kMTile + (t & 15), qy = ty * kMTile + (t >> 4);
    const bool real = qx < gw && qy < gh;
    uint32_t qd[kWords];
    {
        const uint4 *src = reinterpret_cast<const uint4 *>(query + ((size_t)(real ? qy : 0) * gw + (real ? qx : 0)) * kWords);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const uint4 w = src[c];
            qd[4 * c] = w.x;
            qd[4 * c + 1] = w.y;
            qd[4 * c + 2] = w.z;
            qd[4 * c + 3] = w.w;
        }
    }
    __syncthreads();

    // Keys d << 9 | window index: smaller is better; the window index grows
    // with the raster index of the candidate, so ties go to the lower one.
    uint32_t best1 = 0xffffffffu, best2 = 0xffffffffu;
    const int wside = 2 * radius + 1;
    for (int dy = -radius; dy <= radius; ++dy) {
        const bool row_ok = qy + dy >= 0 && qy + dy < gh;
        for (int dx = -radius; dx <= radius; ++dx) {
            const int p = ((t >> 4) + radius + dy) * side + (t & 15) + radius + dx;
            uint32_t d = 0;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const uint4 w = region[c * plane + p];
                d += __builtin_popcount(w.x ^ qd[4 * c]) + __builtin_popcount(w.y ^ qd[4 * c + 1]) +
                     __builtin_popcount(w.z ^ qd[4 * c + 2]) + __builtin_popcount(w.w ^ qd[4 * c + 3]);
            }
            const bool ok = row_ok && qx + dx >= 0 && qx + dx < gw;
            const uint32_t key = ok ? (d << 9) | (uint32_t)((dy + radius) * wside + dx + radius) : 0xffffffffu;
            const uint32_t lo = min(best1, key);
            best2 = min(best2, max(best1, key));
            best1 = lo;
        }
    }
    if (!real) return;
    const int ny = min(gh - 1, qy + radius) - max(0, qy - radius) + 1;
    const int nx = min(gw - 1, qx + radius) - max(0, qx - radius) + 1;
    const int n = ny * nx;
    auto decode = [&](uint32_t key, int32_t &i_out, int32_t &d_out) {
        if (key == 0xffffffffu) {
            i_out = -1;
            d_out = 513;
            return;
        }
        const int w = (int)(key & 511u);
        const int dy = w / wside - radius, dx = w % wside - radius;
        i_out = (qy + dy) * gw + qx + dx;
        d_out = (int)(key >> 9);
    };
    const size_t q = (size_t)qy * gw + qx;
    int32_t i1, d1, i2, d2;
    decode(best1, i1, d1);
    decode(best2, i2, d2);
    idx[k * q] = i1;
    dist[k * q] = d1;
    if (k == 2) {
        idx[k * q + 1] = i2;
        dist[k * q + 1] = d2;
    }
    if (accept) accept[q] = (uint8_t)(n >= 2 && (double)d1 < (double)ratio * (double)d2);
}

}  // namespace

uint32_t dense_patch_offset(int r, int c)
{
    const int x = c - 3;
    return (uint32_t)((x & 1) * kDCopyBytes + (r - 3) * kDRowBytes + 4 * (x >> 1));
}

hipError_t launch_dense_extract(const DenseArgs &a, hipStream_t stream)
{
    const int tiles_x = (int)(((int64_t)a.gw + kDTileW - 1) / kDTileW);
    const int64_t tiles = tiles_x * (((int64_t)a.gh + kDTileH - 1) / kDTileH);
    const int64_t blocks = (tiles + 7) / 8 * 8 * (kWords / kDWords);
    hipLaunchKernelGGL(dense_extract_kernel, dim3((unsigned)blocks), dim3(kDThreads), 0, stream, a.img,
                       a.height, a.width, a.pitch, a.x0, a.y0, a.gw, a.gh, tiles_x, (int)tiles, a.toff,
                       a.desc);
    return hipGetLastError();
}

namespace {

template <int RP>
void launch_window(const DenseMatchArgs &a, hipStream_t stream)
{
    const int tiles_x = (int)(((int64_t)a.gw + kMTile - 1) / kMTile);
    const int64_t tiles = tiles_x * (((int64_t)a.gh + kMTile - 1) / kMTile);
    const int64_t resident = (int64_t)a.num_cus * WindowGeom<RP>::kWaves;
    hipLaunchKernelGGL(dense_match_kernel<RP>, dim3((unsigned)std::min(tiles, resident)), dim3(kDThreads),
                       0, stream, a.query, a.train, a.gw, a.gh, a.radius, tiles_x, tiles, a.k, a.ratio,
                       a.idx, a.dist, a.accept);
}

}  // namespace

hipError_t launch_dense_match(const DenseMatchArgs &a, hipStream_t stream)
{
    if (a.radius < 0 || a.radius > kDenseMaxRadius) return hipErrorInvalidValue;
    if (a.radius <= kPopcountRadius) {
        const int tiles_x = (int)(((int64_t)a.gw + kMTile - 1) / kMTile);
        const int64_t tiles = tiles_x * (((int64_t)a.gh + kMTile - 1) / kMTile);
        hipLaunchKernelGGL(window_popcount_kernel, dim3((unsigned)tiles), dim3(kDThreads), 0, stream,
                           a.query, a.train, a.gw, a.gh, a.radius, tiles_x, a.k, a.ratio, a.idx, a.dist,
                           a.accept);
        return hipGetLastError();
    }
    switch ((a.radius + 1) / 2) {          // the smallest even margin that holds the radius
    case 1: launch_window<2>(a, stream); break;
    case 2: launch_window<4>(a, stream); break;
    case 3: launch_window<6>(a, stream); break;
    default: launch_window<8>(a, stream); break;
    }
    return hipGetLastError();
}

}  // namespace latch
