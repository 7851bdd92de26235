// Brute-force 2-NN Hamming matching for gfx950 (Sec. 4, "Descriptor matching
// on the GPU": exhaustive distances between all query/train pairs).
//
// Two interchangeable paths produce identical partial results:
//
//   MFMA.  With a, b in {0,1}^512, Hamming(a, b) = |a| + |b| - 2 a.b, and a.b
//   over all pairs is an int8 x int8 -> int32 matrix product with K = 512.
//   Packed train tiles (32 rows, 2 KB) are expanded to 0/1 bytes in the exact
//   fragment order of v_mfma_i32_32x32x32_i8 while being staged in LDS, so
//   HBM carries packed bits only and the MFMA operands come from contiguous,
//   conflict-free ds_read_b128.  Queries stay resident in VGPRs (64 queries,
//   128 VGPRs per wavefront).  The sum is exact in int32 (<= 512).
//
//   POPCOUNT.  Each lane owns one query (16 VGPRs); train rows are uniform
//   across the wavefront and arrive through scalar loads; 16 x (v_xor,
//   v_bcnt) per pair.
//
// Top-2 selection packs (distance, split-local index) into one 32-bit key so
// that a max3, a med3 and a max fold two keys into the two best per lane;
// ties resolve to the lowest index because the index is part of the key.  Each (query,
// train split) writes its best two as 64-bit (distance << 32 | index) values;
// a merge kernel reduces over splits and applies the ratio test.
#include <algorithm>
#include <type_traits>

#include "batch_parts.h"
#include "internal.h"
#include "part_keys.h"

namespace latch {
namespace {

#include "fp4.h"
#include "lanes.h"

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr uint32_t kLocalBits = 21;
constexpr uint32_t kLocalMask = (1u << kLocalBits) - 1;

__device__ __forceinline__ uint32_t umed3(uint32_t a, uint32_t b, uint32_t c)
{
    return max(min(a, b), min(max(a, b), c));
}

// Two keys x, y into a running top two (k1 >= k2, as a multiset): the new
// largest is max(k1, x, y); the new second is max(k2, med3(k1, x, y)), since
// if k1 stays largest the second is max(k2, x, y) = max(k2, med3), and if x
// (or y) is largest the second is max(k1, y) (or max(k1, x)), which is the
// median of k1, x, y and is >= k2.  Three operations per two keys, against
// two per key inserted one at a time.
__device__ __forceinline__ void insert_pair_u32(uint32_t &k1, uint32_t &k2, uint32_t x, uint32_t y)
{
    k2 = max(k2, umed3(k1, x, y));
    k1 = max(max(k1, x), y);
}


// Four bits -> four bytes of value 0/1 (bit e of nib -> byte e).  The four
// shifted copies of nib occupy disjoint bit ranges, so the product has no
// carries; nib < 16 and the constant < 2^24 make it a full-rate 24-bit multiply.
__device__ __forceinline__ uint32_t spread_nibble(uint32_t nib)
{
    return __umul24(nib, 0x00204081u) & 0x01010101u;
}

// 16 bits -> 16 bytes of value 0/1, byte m = bit m.
__device__ __forceinline__ v4i expand16(uint32_t x)
{
    v4i r;
    r[0] = (int)spread_nibble(x & 0xfu);
    r[1] = (int)spread_nibble((x >> 4) & 0xfu);
    r[2] = (int)spread_nibble((x >> 8) & 0xfu);
    r[3] = (int)spread_nibble((x >> 12) & 0xfu);
    return r;
}

// ---------------------------------------------------------------------------
// MFMA matcher.  Workgroup = 4 wavefronts x 64 queries; grid (query groups,
// train splits).
//
// Operands.  Train bits enter as bytes b_k in {0, 1} (operand A), query bits
// as signed bytes 2 a_k - 1 in {-1, +1} (operand B, resident in VGPRs), so the
// int8 MFMA sum over K = 512 is directly
//   s = sum_k (2 a_k - 1) b_k = 2 a.b - |b| = |a| - Hamming(a, b),
// exact in int32, and no train-side popcount is needed.
//
// Fragment order.  For a 32-row train tile, step s (0..15) and lane l
// (0..63), the A fragment is 16 bytes: bits 32 s + 16 (l / 32) + m, m = 0..15,
// of tile row l % 32.  Query fragments use the same bit -> (step, lane, byte)
// map, so the MFMA k-sum covers every bit exactly once whatever its internal k
// order.  Each tile is expanded from its packed 2 KB into this order while
// being staged in LDS (16 KB) and read back with contiguous, conflict-free
// ds_read_b128.
//
// Keys.  For train row j with split-local index jl,
//   key = ((s + 512) << 21) + (2^21 - 1 - jl),   s + 512 in [0, 1024],
// so for a fixed query the largest key is the smallest (distance, index).
// Split-local indices stay below 2^21 - 1, so a real key is never 0; rows
// past nt (only in the last tile) are forced to key 0 = "no neighbour".
//
// Accumulator layout of v_mfma_i32_32x32x32_i8 (output 32 x 32, 16 values
// per lane): lane l holds column l % 32 and rows 8 (r / 4) + 4 (l / 32) + r % 4
// for r = 0..15.  Train rows are the MFMA rows and queries the columns, so
// each lane keeps a running top-2 for one query; lanes l and l ^ 32 merge at
// the end.
// ---------------------------------------------------------------------------
constexpr int kMfmaThreads = kMfmaWaves * 64;
constexpr int kQueryBlocks = 2;                        // 32-query blocks per wavefront
constexpr int kQueriesPerWave = 32 * kQueryBlocks;
constexpr int kQueriesPerGroup = kMfmaWaves * kQueriesPerWave;
static_assert(kQueriesPerGroup == 256, "query groups of 256 in every matcher");
constexpr int kTileVec = kTileBytes / 16;              // 16-byte fragments per tile (1024)
static_assert(kMfmaThreads == 8 * kTileRows, "staging: 8 threads per tile row");

// 16 bits -> 16 signed bytes, +1 for a set bit and -1 for a clear one: byte
// b in {0, 1} becomes 0xff ^ 0xfe b, and 0xfe b = (b << 8) - (b << 1) stays
// inside its own byte, so the whole dword is ~((x << 8) - (x << 1)) mod 2^32.
__device__ __forceinline__ v4i expand16_pm1(uint32_t x)
{
    v4i r = expand16(x);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t b = (uint32_t)r[i];
        r[i] = (int)~((b << 8) - (b << 1));
    }
    return r;
}

// Staging role of a thread: tile row tid % 32, packed words 2 (tid / 32) and
// 2 (tid / 32) + 1, i.e. steps 2 (tid / 32) + {0, 1}, both halves.
__device__ __forceinline__ uint2 load_tile(const uint32_t *__restrict__ train, int nt, int tile,
                                           int tid)
{
    // Rows past nt load row nt - 1 (or row 0 of an empty set, which is never
    // staged) and are zeroed, without a branch.
    const int row = tile * kTileRows + (tid & 31);
    const int src = max(min(row, nt - 1), 0);
    const uint2 w = reinterpret_cast<const uint2 *>(train + (size_t)src * kWords)[tid >> 5];
    const uint32_t keep = row < nt ? 0xffffffffu : 0u;
    return make_uint2(w.x & keep, w.y & keep);
}

__device__ __forceinline__ void stage_tile(uint2 w, int tid, v4i *__restrict__ buf)
{
    const int r = tid & 31;
    const int c = tid >> 5;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const uint32_t word = e == 0 ? w.x : w.y;
#pragma unroll
        for (int h = 0; h < 2; ++h)
            buf[(2 * c + e) * 64 + 32 * h + r] = expand16((word >> (16 * h)) & 0xffffu);
    }
}

// Where a work item's results go: per-(split, query) partials for a later
// merge, or (one split only) the final idx / dist / accept rows directly.
struct ItemOut {
    uint64_t *partial;      // partial + (split * nq + q) * 2, or nullptr for direct
    int32_t *idx;           // direct: rows q of this item's query range
    int32_t *dist;
    uint8_t *accept;
    int k;
    float ratio;
};

// Final results of one query from its two best packed (distance << 32 | index).
__device__ __forceinline__ void store_final(uint64_t b1, uint64_t b2, int nt, const ItemOut &o,
                                            int q)
{
    const int d1 = b1 == kNoNeighbour ? 513 : (int)(b1 >> 32);
    const int d2 = b2 == kNoNeighbour ? 513 : (int)(b2 >> 32);
    const int j1 = b1 == kNoNeighbour ? -1 : (int)(uint32_t)b1;
    const int j2 = b2 == kNoNeighbour ? -1 : (int)(uint32_t)b2;
    o.idx[(size_t)q * o.k] = j1;
    o.dist[(size_t)q * o.k] = d1;
    if (o.k == 2) {
        o.idx[(size_t)q * o.k + 1] = j2;
        o.dist[(size_t)q * o.k + 1] = d2;
    }
    if (o.accept) o.accept[q] = (uint8_t)(nt >= 2 && (double)d1 < (double)o.ratio * (double)d2);
}

__device__ __forceinline__ void store_pair(uint64_t b1, uint64_t b2, int nq, int nt, int split,
                                           const ItemOut &o, int q)
{
    if (o.partial) {
        uint64_t *dst = o.partial + ((size_t)split * nq + q) * 2;
        dst[0] = b1;
        dst[1] = b2;
    } else {
        store_final(b1, b2, nt, o, q);
    }
}

// The 16 words of query row qn, zeros past nq, with every load issued
// before any is used: one memory round trip per row.  (Loads guarded word by
// word compile to a branch and a wait per word.)
__device__ __forceinline__ void load_query_row(const uint32_t *__restrict__ query, int nq, int qn,
                                               uint32_t (&w)[kWords])
{
    const bool real = qn < nq;
#pragma unroll
    for (int i = 0; i < kWords; ++i) w[i] = 0u;
    if (nq > 0) {
        const uint32_t *src = query + (size_t)(real ? qn : 0) * kWords;
#pragma unroll
        for (int i = 0; i < kWords; ++i) w[i] = src[i];
    }
#pragma unroll
    for (int i = 0; i < kWords; ++i) w[i] = real ? w[i] : 0u;
}

// One work item of the MFMA matcher: queries qgroup * 256 .. + 255 of
// `query` (nq rows) against train rows split * split_rows .. + split_rows - 1
// of `train` (nt rows).  All 256 threads of the workgroup take part; tbuf is
// the workgroup's 2 x 16 KB LDS staging buffer.
__device__ __forceinline__ void mfma_item(const uint32_t *__restrict__ query, int nq,
                                          const uint32_t *__restrict__ train, int nt, int qgroup,
                                          int split, int split_rows, const ItemOut &out,
                                          v4i (*tbuf)[kTileVec])
{
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int qbase = qgroup * kQueriesPerGroup + wave * kQueriesPerWave;

    const int ntiles_all = (nt + kTileRows - 1) / kTileRows;
    const int tiles_per_split = split_rows / kTileRows;
    const int t_begin = split * tiles_per_split;
    const int t_end = min(ntiles_all, t_begin + tiles_per_split);

    // The next tile's load is issued at the start of a tile and staged at
    // its end (the query fragments leave no registers for a deeper queue).
    uint2 ld0 = make_uint2(0, 0);
    if (t_begin < t_end) ld0 = load_tile(train, nt, t_begin, tid);

    // Resident query fragments and query popcounts.
    v4i bq[kQueryBlocks][16];
    int na[kQueryBlocks];
    uint32_t qw[kQueryBlocks][kWords];
#pragma unroll
    for (int qb = 0; qb < kQueryBlocks; ++qb) load_query_row(query, nq, qbase + 32 * qb + (lane & 31), qw[qb]);
#pragma unroll
    for (int qb = 0; qb < kQueryBlocks; ++qb) {
        int pc = 0;
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            const uint32_t w = qw[qb][s];
            pc += __popc(w);
            bq[qb][s] = expand16_pm1((w >> (16 * half)) & 0xffffu);
        }
        na[qb] = pc;
    }

    uint32_t k1[kQueryBlocks], k2[kQueryBlocks];
#pragma unroll
    for (int qb = 0; qb < kQueryBlocks; ++qb) k1[qb] = k2[qb] = 0u;

    __syncthreads();       // the staging buffer may still be read by a previous item
    if (t_begin < t_end) stage_tile(ld0, tid, tbuf[0]);
    __syncthreads();

    // One tile: MFMAs over LDS buffer `buf`, then the top-2 update.
    auto tile_step = [&](int tile, int buf) {
        v16i acc[kQueryBlocks];
#pragma unroll
        for (int qb = 0; qb < kQueryBlocks; ++qb) acc[qb] = (v16i){};
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            const v4i a = tbuf[buf][s * 64 + lane];
#pragma unroll
            for (int qb = 0; qb < kQueryBlocks; ++qb)
                acc[qb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, bq[qb][s], acc[qb], 0, 0, 0);
        }

        // Epilogue.  Register r = 4 g + e holds tile row m = 8 g + 4 half + e,
        // split-local index tile * 32 - split * split_rows + m.  Padding rows
        // (past nt, last tile only) have all-zero bytes, so s = 0 there and a
        // zero key base makes their key 0.
        const uint32_t kt = (512u << kLocalBits) + kLocalMask -
                            (uint32_t)(tile * kTileRows - split * split_rows) - 4u * half;
        const int valid_rows = nt - tile * kTileRows;        // < 32 only in the last tile
        uint32_t cb[16];
        if (valid_rows >= kTileRows) {
#pragma unroll
            for (int r = 0; r < 16; ++r) cb[r] = kt - (uint32_t)(8 * (r >> 2) + (r & 3));
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int m = 8 * (r >> 2) + 4 * half + (r & 3);
                cb[r] = m < valid_rows ? kt - (uint32_t)(8 * (r >> 2) + (r & 3)) : 0u;
            }
        }
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
#pragma unroll
            for (int qb = 0; qb < kQueryBlocks; ++qb)
                insert_pair_u32(k1[qb], k2[qb], ((uint32_t)acc[qb][r] << kLocalBits) + cb[r],
                                ((uint32_t)acc[qb][r + 1] << kLocalBits) + cb[r + 1]);
        }
    };

    // Straight-line body: the load past the split reads train rows of the
    // next split or none (rows past nt load nothing and give zeros), and
    // staging into the idle buffer is harmless.
    for (int tile = t_begin; tile < t_end; ++tile) {
        const int buf = (tile - t_begin) & 1;
        const uint2 ld = load_tile(train, nt, tile + 1, tid);
        tile_step(tile, buf);
        stage_tile(ld, tid, tbuf[buf ^ 1]);
        __syncthreads();
    }

    // Merge the two row halves, decode (d = |a| + 512 - (key >> 21)), store.
#pragma unroll
    for (int qb = 0; qb < kQueryBlocks; ++qb) {
        const uint32_t o1 = __shfl_xor(k1[qb], 32);
        const uint32_t o2 = __shfl_xor(k2[qb], 32);
        const uint32_t b1 = max(k1[qb], o1);
        const uint32_t b2 = max(min(k1[qb], o1), max(k2[qb], o2));
        const int qn = qbase + 32 * qb + (lane & 31);
        if (half == 0 && qn < nq) {
            uint64_t r[2];
            const uint32_t kk[2] = {b1, b2};
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                if (kk[e] == 0u) {
                    r[e] = kNoNeighbour;
                } else {
                    const uint32_t score = kk[e] >> kLocalBits;
                    const uint32_t d = (uint32_t)na[qb] + 512u - score;
                    const uint32_t j = (uint32_t)split * (uint32_t)split_rows +
                                       (kLocalMask - (kk[e] & kLocalMask));
                    r[e] = ((uint64_t)d << 32) | j;
                }
            }
            store_pair(r[0], r[1], nq, nt, split, out, qn);
        }
    }
}

// The two smallest of the pairs (a1 <= a2) and (c1 <= c2).
__device__ __forceinline__ void top2_pair(uint64_t &a1, uint64_t &a2, uint64_t c1, uint64_t c2)
{
    const uint64_t lo = min(a1, c1);
    a2 = min(max(a1, c1), min(a2, c2));
    a1 = lo;
}

// ---------------------------------------------------------------------------
// FP4 matcher (LATCH_PATH_MFMA_FP4).  Same staging as the int8 path, on the FP4
// matrix instruction v_mfma_f32_16x16x128_f8f6f4 (K = 128 per instruction, twice
// the int8 rate on gfx950).
//
// Operands.  FP4 (e2m1) holds 0 (0x0), +-0.5 (0x1 / 0x9), +-1 (0x2 / 0xa)
// and +-2 (0x4 / 0xc) exactly.  A train bit enters as 0 or c (c = 0.5, 1 or
// 2 by its place in the fragment, below), and the query bit it meets as
// +1 / c or -1 / c (set / clear), so each product is 0 or +-1 and the f32 sum
// over K = 512 is s = |a| - Hamming(a, b) as in the int8 path, exact.
//
// Keys.  In units of 2^-14: for tile row m the accumulator starts at
// c_m = 2^14 - 1 - m, so it ends at 2^14 s + c_m; the running top-2 of a lane is
// kept in the frame of the current tile and moved up by 32 when the next tile
// starts, so a key from split-local row jl = 32 t + m ends as
// 2^14 s + 2^14 - 1 - jl + 32 (T - 1) after T tiles (T <= 512): integers below
// 2^24 in magnitude, exact in f32.  For a fixed query the largest key is the
// smallest (distance, index).  Rows past nt (last tile only) take -2048 (before
// the scaling) instead, below every real key,
// which also marks "no neighbour".  Top-2 selection takes the keys two at a
// time: v_med3_f32, v_max3_f32 and v_max_f32 per two pairs.
//
// Fragment order.  Step s (0..3), lane l = 16 g + n: the 32 elements of row n
// (of a subtile of 16 train rows, of a block of 16 queries) at K = 128 s + 32 g
// + 0..31 are the bits of packed word 4 g + s of that row, bit 4 i + j in nibble
// i of dword j (16 bytes).  Train rows and queries use the same map, so the K
// sum covers every bit once, and a lane's four query words are one 16-byte load.
// In this order a train word becomes FP4 with four AND masks and one shift, no
// table: dword j keeps its bits where they are, as nibble bit 0, 1, 2 (values
// 0.5, 1, 2) for j = 0, 1, 2, and bit 3 (the sign) is moved down to bit 2 for
// j = 3, so c = 0.5, 1, 2, 2 by dword.
//
// Bound: the matrix cores, and through their power the clock.  On random bits
// this instruction alone sustains 9.15 PFLOP/s and the 32x32x64 one, which
// moves twice the accumulator registers per product, 7.55 PFLOP/s; the
// matcher reaches 6.7 to 7.1 PFLOP/s by machine at 8000 x 1,000,000, since four lane rows select from every block and
// the selection (12 VALU instructions per 8 MFMAs) shares the issue slots.
//
// Tile shape.  A wavefront holds 2 QB blocks of 16 queries (QB = 2 or 3, from
// the tuning table), so each train fragment read from LDS feeds 2 QB MFMAs and
// each staged tile serves 128 QB queries of the workgroup; QB = 4 spills.  A
// lane's 4 accumulators per block and subtile are rows of one query, whose
// top two live in all four lane rows until the end of the range.  Both subtiles'
// products come before their selection; a hand-written software pipeline that
// selected the previous subtile between MFMAs was slower (1370 us), and so was
// a frame of 64 rows, whose start values take the batched kernel's last
// registers.  Measured, 32x32x64 with block scales -> 16x16x128 with -> without:
// 8000 x 1,000,000 1359 -> 1231 -> 1176 us, 9973 x 10007 27.4 -> 24.3 -> 23.9 us;
// QB = 2 is about 5% slower where it pads as little.
// ---------------------------------------------------------------------------
constexpr int kFp4Steps = 4;                          // K = 512 = 4 x 128
constexpr int kFp4SubRows = 16;                       // train rows per MFMA
constexpr int kFp4Subs = kTileRows / kFp4SubRows;     // subtiles per staged tile
constexpr int kFp4TileVec = kFp4Subs * kFp4Steps * 64;    // 16-byte fragments per tile (512)
constexpr int kFp4MaxTiles = (int)kFp4MaxSplitRows / kTileRows;
constexpr float kFp4Row = 1.0f / (1 << 14);           // a row's step in a key
constexpr float kFp4None = -2048.0f;                  // below every key

// A wavefront's queries with QB (2 or 3): blocks of 16, and sets of four
// blocks whose results meet one lane row each.
template <int QB>
struct Fp4Shape {
    static constexpr int kBlocks = 2 * QB;
    static constexpr int kSets = (kBlocks + 3) / 4;
    static constexpr int kQueries = 16 * kBlocks;
};

// Two keys into a running top two (k1 >= k2), as insert_pair_u32 does for
// integer keys: v_med3_f32, v_max3_f32 and v_max_f32.  (This file is compiled
// without NaNs in mind: the IEEE-mode maxima would otherwise quiet every operand.
// Keys are never NaN, nor is the ratio of the test at the end, which the host checks.)
__device__ __forceinline__ void insert_pair(float &k1, float &k2, float x, float y)
{
    k2 = fmaxf(k2, __builtin_amdgcn_fmed3f(k1, x, y));
    k1 = fmaxf(fmaxf(k1, x), y);
}

// Staging role of a thread: tile row tid % 32, packed words 2 (tid / 32) and
// 2 (tid / 32) + 1.  Word w of row r is lane 16 (w / 4) + r % 16 of step w % 4 of
// subtile r / 16.
__device__ __forceinline__ void stage_tile_fp4(uint2 w, int tid, uint4 *__restrict__ buf)
{
    const int r = tid & 31, c = tid >> 5;
    uint4 *to = buf + ((r >> 4) * kFp4Steps + 2 * (c & 1)) * 64 + 16 * (c >> 1) + (r & 15);
    to[0] = fp4_train(w.x);
    to[64] = fp4_train(w.y);
}

// One (query group, train range) of the FP4 matcher.  Train tiles
// t_begin .. t_end - 1 (at most 2^14 rows); the best two
// (distance << 32 | index) of query n = lane % 16 of block 4 t + lane / 16 are
// merged into best[t].
template <int QB>
__device__ __forceinline__ void fp4_item(const uint32_t *__restrict__ query, int nq,
                                         const uint32_t *__restrict__ train, int nt, int qgroup,
                                         int t_begin, int t_end,
                                         uint64_t (&best)[Fp4Shape<QB>::kSets][2],
                                         uint4 (*tbuf)[kFp4TileVec])
{
    constexpr int kBlocks = Fp4Shape<QB>::kBlocks, kSets = Fp4Shape<QB>::kSets;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int g = lane >> 4, n = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int qbase = (qgroup * kMfmaWaves + wave) * Fp4Shape<QB>::kQueries;

    // Tile loads two tiles ahead of staging.
    uint2 ld0 = make_uint2(0, 0), ra = ld0, rb = ld0;
    if (t_begin < t_end) ld0 = load_tile(train, nt, t_begin, tid);
    if (t_begin + 1 < t_end) ra = load_tile(train, nt, t_begin + 1, tid);
    if (t_begin + 2 < t_end) rb = load_tile(train, nt, t_begin + 2, tid);

    // Resident query fragments: words 4 g .. 4 g + 3 of query n of each block
    // (of row 0 past nq: not stored), and their popcounts.
    uint4 bq[kBlocks][kFp4Steps];
    int na[4 * kSets] = {};
    {
        uint4 qw[kBlocks];
#pragma unroll
        for (int b = 0; b < kBlocks; ++b) {
            const int qn = qbase + 16 * b + n;
            qw[b] = make_uint4(0u, 0u, 0u, 0u);
            if (nq > 0)
                qw[b] = reinterpret_cast<const uint4 *>(query + (size_t)(qn < nq ? qn : 0) * kWords)[g];
        }
#pragma unroll
        for (int b = 0; b < kBlocks; ++b) {
            const uint32_t w[4] = {qw[b].x, qw[b].y, qw[b].z, qw[b].w};
#pragma unroll
            for (int s = 0; s < kFp4Steps; ++s) {
                bq[b][s] = fp4_query(w[s]);
                na[b] += __popc(w[s]);
            }
        }
    }

    float k1[4 * kSets], k2[4 * kSets];
#pragma unroll
    for (int b = 0; b < 4 * kSets; ++b) k1[b] = k2[b] = kFp4None;

    // Accumulator start values c_m; register r of subtile h holds tile row
    // m = 16 h + 4 g + r.
    v4f c0[kFp4Subs];
#pragma unroll
    for (int h = 0; h < kFp4Subs; ++h)
#pragma unroll
        for (int r = 0; r < 4; ++r) c0[h][r] = (float)((1 << 14) - 1 - (kFp4SubRows * h + 4 * g + r)) * kFp4Row;

    __syncthreads();       // the staging buffers may still be read for a previous range
    if (t_begin < t_end) stage_tile_fp4(ld0, tid, tbuf[0]);
    __syncthreads();

    // Rows past nt (in the last tile only) take a key below every real one.
    auto mask_tail = [&](int tile, int h, v4f (&acc)[kBlocks]) {
        const int valid_rows = nt - tile * kTileRows - kFp4SubRows * h;
        if (valid_rows < kFp4SubRows) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (4 * g + r >= valid_rows)
#pragma unroll
                    for (int b = 0; b < kBlocks; ++b) acc[b][r] = kFp4None;
        }
    };
    auto sub_mfma = [&](int buf, int h, v4f (&acc)[kBlocks]) {
#pragma unroll
        for (int s = 0; s < kFp4Steps; ++s) {
            const v8i a = fp4_operand(tbuf[buf][(h * kFp4Steps + s) * 64 + lane]);
#pragma unroll
            for (int b = 0; b < kBlocks; ++b)
                acc[b] = fp4_mfma(a, fp4_operand(bq[b][s]), s == 0 ? c0[h] : acc[b]);
        }
    };
    auto tile_step = [&](int tile, int buf) {
        v4f acc0[kBlocks], acc1[kBlocks];
        sub_mfma(buf, 0, acc0);
        sub_mfma(buf, 1, acc1);
#pragma unroll
        for (int b = 0; b < kBlocks; ++b) {
            k1[b] += kTileRows * kFp4Row;
            k2[b] += kTileRows * kFp4Row;
        }
        mask_tail(tile, 0, acc0);
        mask_tail(tile, 1, acc1);
#pragma unroll
        for (int b = 0; b < kBlocks; ++b) {
            insert_pair(k1[b], k2[b], acc0[b][0], acc0[b][1]);
            insert_pair(k1[b], k2[b], acc0[b][2], acc0[b][3]);
            insert_pair(k1[b], k2[b], acc1[b][0], acc1[b][1]);
            insert_pair(k1[b], k2[b], acc1[b][2], acc1[b][3]);
        }
    };
    for (int tile = t_begin; tile < t_end; tile += 2) {
        tile_step(tile, 0);
        stage_tile_fp4(ra, tid, tbuf[1]);
        ra = load_tile(train, nt, tile + 3, tid);
        __syncthreads();
        if (tile + 1 >= t_end) break;
        tile_step(tile + 1, 1);
        stage_tile_fp4(rb, tid, tbuf[0]);
        rb = load_tile(train, nt, tile + 4, tid);
        __syncthreads();
    }

    // Every lane row holds partial results of all blocks (its rows of every
    // tile, its words' popcounts): lane row g ends with those of block 4 t + g.
    // Then decode key = 2^14 (|a| - d) + 2^14 - 1 - jl + 32 (tiles - 1).
    const int shift = 32 * max(t_end - t_begin - 1, 0);
#pragma unroll
    for (int t = 0; t < kSets; ++t) {
#pragma unroll
        for (int b = 4 * t; b < 4 * t + 2; ++b) {
            exchange_top2<true>(k1[b], k2[b], k1[b + 2], k2[b + 2]);
            exchange_sum<true>(na[b], na[b + 2]);
        }
        exchange_top2<false>(k1[4 * t], k2[4 * t], k1[4 * t + 1], k2[4 * t + 1]);
        exchange_sum<false>(na[4 * t], na[4 * t + 1]);
        uint64_t r[2];
        const float kk[2] = {k1[4 * t], k2[4 * t]};
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            if (kk[e] < kFp4None / 2) {                  // a row past nt, or none
                r[e] = kNoNeighbour;
            } else {
                const int key = (int)(kk[e] * (1 << 14)) - shift;
                const uint32_t d = (uint32_t)(na[4 * t] - (key >> 14));
                const uint32_t j = (uint32_t)t_begin * (uint32_t)kTileRows +
                                   (uint32_t)((1 << 14) - 1 - (key & 0x3fff));
                r[e] = ((uint64_t)d << 32) | j;
            }
        }
        top2_pair(best[t][0], best[t][1], r[0], r[1]);
    }
}

template <int QB>
__device__ __forceinline__ void fp4_init_best(uint64_t (&best)[Fp4Shape<QB>::kSets][2])
{
#pragma unroll
    for (int t = 0; t < Fp4Shape<QB>::kSets; ++t) best[t][0] = best[t][1] = kNoNeighbour;
}

// Every lane stores its queries' results, one per set.
template <int QB>
__device__ __forceinline__ void fp4_store(const uint64_t (&best)[Fp4Shape<QB>::kSets][2], int nq, int nt,
                                          int qgroup, int split, const ItemOut &out)
{
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
#pragma unroll
    for (int t = 0; t < Fp4Shape<QB>::kSets; ++t) {
        const int b = 4 * t + (lane >> 4);
        const int qn = (qgroup * kMfmaWaves + wave) * Fp4Shape<QB>::kQueries + 16 * b + (lane & 15);
        if (b < Fp4Shape<QB>::kBlocks && qn < nq)
            store_pair(best[t][0], best[t][1], nq, nt, split, out, qn);
    }
}

// ---------------------------------------------------------------------------
// Popcount matcher.  One query per lane; grid (query blocks of 256, splits).
// key = (d << 21) | jl with d <= 512, jl < 2^21 - 1, so ~0u means "none".
// ---------------------------------------------------------------------------
__device__ __forceinline__ void popcount_item(const uint32_t *__restrict__ query, int nq,
                                              const uint32_t *__restrict__ train, int nt,
                                              int qgroup, int split, int split_rows,
                                              const ItemOut &out)
{
    const int qn = qgroup * 256 + threadIdx.x;
    const int j0 = split * split_rows;
    const int j1 = min(nt, j0 + split_rows);

    uint32_t q[kWords];
    load_query_row(query, nq, qn, q);

    uint32_t k1 = ~0u, k2 = ~0u;
#pragma unroll 4
    for (int j = j0; j < j1; ++j) {
        const uint32_t *t = train + (size_t)j * kWords;
        uint32_t d = 0;
#pragma unroll
        for (int w = 0; w < kWords; ++w) d = __popc(q[w] ^ t[w]) + d;
        const uint32_t key = (d << kLocalBits) | (uint32_t)(j - j0);
        k2 = umed3(k1, k2, key);
        k1 = min(k1, key);
    }

    if (qn < nq) {
        const uint32_t kk[2] = {k1, k2};
        uint64_t r[2];
#pragma unroll
        for (int e = 0; e < 2; ++e)
            r[e] = kk[e] == ~0u ? kNoNeighbour
                                : (((uint64_t)(kk[e] >> kLocalBits) << 32) |
                                   (uint32_t)(j0 + (int)(kk[e] & kLocalMask)));
        store_pair(r[0], r[1], nq, nt, split, out, qn);
    }
}

// ---------------------------------------------------------------------------
// Merge per-split partials (64-bit keys: distance << 32 | global index, so the
// integer order is the lexicographic one) and apply the ratio test exactly:
// a float32 ratio times an integer <= 512 is exact in double.
// ---------------------------------------------------------------------------
// Arguments of the split matchers.  nsplit == 1: results go straight to
// idx / dist / accept; otherwise per-(split, query) partials for the merge
// kernel.
struct SplitArgs {
    const uint32_t *query;
    const uint32_t *train;
    int nq, nt, split_rows, nsplit;
    uint64_t *partial;
    int k;
    float ratio;
    int32_t *idx, *dist;
    uint8_t *accept;
};

__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t v, int m)
{
    const uint32_t lo = __shfl_xor((uint32_t)v, m), hi = __shfl_xor((uint32_t)(v >> 32), m);
    return ((uint64_t)hi << 32) | lo;
}

// Sixteen lanes per query: lane g of a query reads splits g, g + 16, ... (four
// loads in flight), then four shuffle rounds combine the top-2 pairs.  Bound by the
// latency of those loads: 500 x 1,000,000 with 256 splits took 109.6 us in all with
// 4 lanes, 101.9 with 8, 99.5 with 16 and 98.9 with 32; 2000 x 2000 7.4 us with 16
// and 8.2 with 4.
constexpr int kMergeLanes = 16;
constexpr int kMergeQueries = 256 / kMergeLanes;         // per workgroup and pass
// A launch holds fewer than 2^32 work items, which 16 lanes per query pass at 2^28
// queries: from 2^20 on the workgroups take several passes (2^16 workgroups are 32
// times what the GPU holds at once).
constexpr int64_t kMergeMaxBlocks = 1 << 16;

__global__ __launch_bounds__(256) void knn_merge_kernel(const uint64_t *__restrict__ partial, int nq,
                                                        int nsplit, int nt, int k, float ratio,
                                                        int32_t *__restrict__ idx,
                                                        int32_t *__restrict__ dist,
                                                        uint8_t *__restrict__ accept)
{
    const int g = threadIdx.x & (kMergeLanes - 1);
    // (nq < 2^31 and a pass takes at most kMergeMaxBlocks kMergeQueries queries: 32 bits.)
    for (uint32_t q0 = blockIdx.x * kMergeQueries; q0 < (uint32_t)nq; q0 += gridDim.x * kMergeQueries) {
        const uint32_t q = q0 + threadIdx.x / kMergeLanes;
        const bool real = q < (uint32_t)nq;
        uint64_t b1 = kNoNeighbour, b2 = kNoNeighbour;
        for (int s0 = g; s0 < nsplit; s0 += 4 * kMergeLanes) {
            ulonglong2 v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int sp = s0 + kMergeLanes * i;
                v[i] = real && sp < nsplit
                           ? reinterpret_cast<const ulonglong2 *>(partial)[(size_t)sp * nq + q]
                           : make_ulonglong2(kNoNeighbour, kNoNeighbour);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) top2_pair(b1, b2, v[i].x, v[i].y);
        }
        // (Every lane takes part: the loop's bounds are the workgroup's.)
#pragma unroll
        for (int m = 1; m < kMergeLanes; m <<= 1)
            top2_pair(b1, b2, shfl_xor_u64(b1, m), shfl_xor_u64(b2, m));
        if (real && g == 0)
            store_final(b1, b2, nt, ItemOut{nullptr, idx, dist, accept, k, ratio}, (int)q);
    }
}

__global__ __launch_bounds__(kMfmaThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void
knn_mfma_kernel(SplitArgs a)
{
    __shared__ v4i tbuf[2][kTileVec];
    const ItemOut direct{nullptr, a.idx, a.dist, a.accept, a.k, a.ratio};
    const ItemOut part{a.partial, nullptr, nullptr, nullptr, 2, 0.f};
    mfma_item(a.query, a.nq, a.train, a.nt, blockIdx.x, blockIdx.y, a.split_rows,
              a.nsplit == 1 ? direct : part, tbuf);
}

template <int QB>
__global__ __launch_bounds__(kMfmaThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void
knn_fp4_kernel(SplitArgs a)
{
    __shared__ uint4 tbuf[2][kFp4TileVec];
    const ItemOut direct{nullptr, a.idx, a.dist, a.accept, a.k, a.ratio};
    const ItemOut part{a.partial, nullptr, nullptr, nullptr, 2, 0.f};
    uint64_t best[Fp4Shape<QB>::kSets][2];
    fp4_init_best<QB>(best);
    const int tiles = (a.nt + kTileRows - 1) / kTileRows, per_split = a.split_rows / kTileRows;
    const int t_begin = blockIdx.y * per_split;
    fp4_item<QB>(a.query, a.nq, a.train, a.nt, blockIdx.x, t_begin, min(tiles, t_begin + per_split), best,
                 tbuf);
    fp4_store<QB>(best, a.nq, a.nt, blockIdx.x, blockIdx.y, a.nsplit == 1 ? direct : part);
}

__global__ __launch_bounds__(256) void knn_popcount_kernel(SplitArgs a)
{
    const ItemOut direct{nullptr, a.idx, a.dist, a.accept, a.k, a.ratio};
    const ItemOut part{a.partial, nullptr, nullptr, nullptr, 2, 0.f};
    popcount_item(a.query, a.nq, a.train, a.nt, blockIdx.x, blockIdx.y, a.split_rows,
                  a.nsplit == 1 ? direct : part);
}

// ---------------------------------------------------------------------------
// Batched matching: many (query range, train range, output range) pairs in
// one persistent launch.  Work unit = (pair, query group, part of the pair's
// train range); where a pair has one part, as most do, a unit's results are final
// and go straight to the outputs.  A one-block setup kernel validates the pairs,
// lays their units out and resets the atomic work counter (so the sequence is
// replayable from a HIP graph without memset nodes); a fill kernel writes the
// unit -> pair map; persistent workgroups then claim units through the counter.
//
// Units are laid out longest first (an undivided unit's time grows with its
// pair's train rows): pairs go to 256 cost classes, 8 per doubling of the train
// tile count, and the classes are laid out in decreasing order, so that the
// last units claimed are the shortest and the workgroups finish together.
// The order within a class follows the atomics and does not matter: every
// query group writes its own outputs.
//
// Parts (FP4 matcher).  A unit should not outlast what is left for everyone: with
// R train tiles of work from a pair's first item on and S resident workgroups, its
// train range is divided into as many parts as hold about R / S tiles each, counted
// with at least kMinPartTiles (shorter ones cost more in query fragments and merging than
// they even out: 48, 64, 96 and 128 were tried), and at most kMaxParts (batch_parts.h,
// which also has the batches that are not divided at all).  Long pairs among short ones
// and the last rounds of a batch of equal pairs are divided, the rest is not.  Parts of a
// query group meet in a slot (part_keys.h), the one that arrives last writes the outputs,
// and none waits for another.  Bound without parts: the longest unit and the last round.
// Measured, undivided -> divided, us: 47 pairs of log-normal sizes around 5000 (sigma 1)
// 627 -> 315, 29 around 2000 256 -> 97, one pair of 20,000 x 20,000 476 -> 115, 15 such
// pairs 1097 -> 908, 63 3794 -> 3602.  Parts of R / 2 S, 3 R / 4 S and 3 R / 2 S were up to
// 10% slower.
// ---------------------------------------------------------------------------
__device__ __forceinline__ bool pair_ok(const PairEntry &e, int64_t query_rows, int64_t train_rows,
                                        int64_t out_rows)
{
    return e.nq >= 0 && e.nt >= 0 && e.nq <= kMaxRows && e.nt <= kMaxSplitRows &&
           e.query_first >= 0 && e.query_first + e.nq <= query_rows &&
           (e.nt == 0 || (e.train_first >= 0 && e.train_first + e.nt <= train_rows)) &&
           e.out_first >= 0 && e.out_first + e.nq <= out_rows;
}

// Inclusive scan of 256 values in LDS: within the wavefronts, then over their totals.
__device__ __forceinline__ void scan256(unsigned long long *v, unsigned long long *totals, int tid)
{
    __syncthreads();
    const int lane = tid & 63;
    unsigned long long x = v[tid];
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const unsigned long long y = __shfl_up(x, off);
        if (lane >= off) x += y;
    }
    if (lane == 63) totals[tid >> 6] = x;
    __syncthreads();
    for (int w = 0; w < tid >> 6; ++w) x += totals[w];
    v[tid] = x;
    __syncthreads();
}

// First slot of this lane's `groups` query groups if it `wants` them and they are to
// be had, else -1.  A wavefront's lanes take theirs in turn and the wavefront all of them at
// once, so a pair that does not fit takes none from those after it.  (With one atomic
// add per pair, undone for no one, a refused pair's slots were lost to the rest.)
__device__ __forceinline__ int take_slots(int *used, bool wants, int groups, int slots)
{
    const uint64_t wanting = __ballot(wants);
    if (wanting == 0) return -1;
    const int lane = threadIdx.x & 63, first = __builtin_ctzll(wanting);
    int seen = 0;
    for (;;) {                        // (another round only if another wavefront took slots)
        int slot = -1, at = seen;
        for (uint64_t m = wanting; m != 0; m &= m - 1) {
            const int l = __builtin_ctzll(m);
            const int g = __builtin_amdgcn_readlane(groups, l);
            if (at + g > slots) continue;
            if (lane == l) slot = at;
            at += g;
        }
        int old = 0;
        if (lane == first) old = atomicCAS(used, seen, at);
        old = __builtin_amdgcn_readlane(old, first);
        if (old == seen) return slot;
        seen = old;
    }
}

// resident: workgroups that run at once; slots: query groups that may be divided (0: no
// pair is).  Bound by latency, so a thread keeps its first pair in registers between the
// steps, and a batch that divides no pair has neither a scan of work nor a second count.
__global__ __launch_bounds__(256) void knn_batch_setup_kernel(
    const PairEntry *__restrict__ pairs, int n_pairs, int64_t query_rows, int64_t train_rows,
    int64_t out_rows, int64_t item_capacity, int group, int resident, int slots,
    PairInfo *__restrict__ info, BatchState *__restrict__ st, uint32_t *__restrict__ flags)
{
    __shared__ unsigned long long classes[256], works[256], totals[4];
    __shared__ int slots_s, longest_s[4];
    const int tid = threadIdx.x;
    classes[tid] = 0;
    works[tid] = 0;
    if (tid == 0) slots_s = 0;
    __syncthreads();
    // Items (pair, query group) and their train tiles per class.  Until a pair's units
    // are placed, unit_first is its rank in its class, and until its parts are known,
    // `parts` its train tiles.
    PairInfo mine = {};
    int mine_class = 0;
    bool bad = false;
    int longest = 0;
    for (int p = tid; p < n_pairs; p += 256) {
        const PairEntry e = pairs[p];
        const bool ok = pair_ok(e, query_rows, train_rows, out_rows);
        bad |= !ok;
        const unsigned long long groups = ok ? (unsigned long long)((e.nq + group - 1) / group) : 0ull;
        const int tiles = ok ? (int)((e.nt + kTileRows - 1) / kTileRows) : 0;
        const int c = cost_class(e.nt);
        const PairInfo pi{(int32_t)atomicAdd(&classes[c], groups), (int32_t)groups, (uint32_t)tiles, 0u};
        if (slots > 0 && groups > 0) {
            atomicAdd(&works[c], groups * (unsigned long long)tiles);
            longest = max(longest, tiles);
        }
        if (p == tid) {
            mine = pi;
            mine_class = c;
        } else {
            info[p] = pi;
        }
    }
    auto each_pair = [&](auto f) {
        if (tid < n_pairs) f(mine, mine_class);
        for (int p = tid + 256; p < n_pairs; p += 256) {
            PairInfo pi = info[p];
            f(pi, cost_class(pairs[p].nt));
            info[p] = pi;
        }
    };
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) longest = max(longest, __shfl_xor(longest, off));
    if ((tid & 63) == 0) longest_s[tid >> 6] = longest;
    scan256(classes, totals, tid);
    longest = max(max(longest_s[0], longest_s[1]), max(longest_s[2], longest_s[3]));
    // The map holds item_capacity items, enough for every batch whose pairs'
    // output ranges do not overlap; a batch that needs more is not run.
    const bool overflow = (int64_t)classes[255] > item_capacity;
    if (bad || (overflow && tid == 0)) atomicOr(flags, kFlagBadPair);
    bool divides = !overflow && longest > kMinPartTiles, divided = false;
    unsigned long long all_work = 0;
    if (divides) {
        scan256(works, totals, tid);
        all_work = works[255];
        divides = may_divide(longest, classes[255], all_work, resident);
    }
    if (divides) {
        // Parts and slots.
        each_pair([&](PairInfo &pi, int c) {
            int parts = 1;
            if (pi.groups > 0 && pi.groups <= slots) {
                // Work from this pair on: its class's remaining items and later classes.
                const unsigned long long in_class = classes[c] - (c > 0 ? classes[c - 1] : 0ull);
                const unsigned long long left =
                    all_work - works[c] + (in_class - (uint32_t)pi.unit_first) * pi.parts;
                parts = train_parts((int)pi.parts, left, resident);
            }
            const int slot = take_slots(&slots_s, parts > 1, pi.groups, slots);
            pi.parts = slot < 0 ? 1u : (uint32_t)parts;
            pi.slot = slot < 0 ? 0u : (uint32_t)slot;
            divided |= slot >= 0;
        });
    }
    // With parts, units per class and each pair's rank among them.
    if (__syncthreads_or(divided)) {
        classes[tid] = 0;
        __syncthreads();
        each_pair([&](PairInfo &pi, int c) {
            pi.unit_first = (int32_t)atomicAdd(&classes[c], (unsigned long long)pi.groups * pi.parts);
        });
        scan256(classes, totals, tid);
    }
    each_pair([&](PairInfo &pi, int c) {
        pi.unit_first += (int32_t)(c > 0 ? classes[c - 1] : 0ull);
        if (overflow) pi.groups = 0;
        if (!divides) {
            pi.parts = 1u;
            pi.slot = 0u;
        }
    });
    if (tid < n_pairs) info[tid] = mine;
    if (tid == 255) {
        st->units = overflow ? 0 : (int64_t)classes[255];
        st->next_unit = 0;
    }
}

// The unit -> pair map, and the slots of divided pairs: no neighbours, no part done.
__global__ __launch_bounds__(256) void knn_batch_fill_kernel(const PairInfo *__restrict__ info,
                                                             int n_pairs,
                                                             int32_t *__restrict__ unit_pair,
                                                             BatchSlots slots)
{
    const int first = 256 * blockIdx.y + threadIdx.x, step = 256 * gridDim.y;
    for (int p = blockIdx.x; p < n_pairs; p += gridDim.x) {
        const PairInfo pi = info[p];
        const int units = pi.groups * (int)pi.parts;
        for (int i = first; i < units; i += step) unit_pair[pi.unit_first + i] = p;
        if (pi.parts == 1) continue;
        PartKeys *keys = slots.keys + (size_t)pi.slot * kBatchSlotQueries;
        for (int i = first; i < pi.groups * kBatchSlotQueries; i += step) keys[i].clear();
        for (int i = first; i < pi.groups; i += step) slots.done[pi.slot + i].clear();
    }
}

// Claims the next work unit for the whole workgroup; -1 when none is left.
__device__ __forceinline__ int64_t claim_unit(BatchState *__restrict__ st, int *slot)
{
    if (threadIdx.x == 0) {
        const uint32_t it = atomicAdd(&st->next_unit, 1u);
        *slot = (int64_t)it < st->units ? (int)it : -1;
    }
    __syncthreads();
    const int it = *slot;
    __syncthreads();
    return it;
}

// A part's best two of each query into the query group's slot; the part that
// arrives last writes the group's outputs.
template <int QB>
__device__ __forceinline__ void fp4_merge_part(const uint64_t (&best)[Fp4Shape<QB>::kSets][2], int nq,
                                               int nt, int qgroup, uint32_t parts, PartKeys *slot,
                                               PartCount *done, int *last_s, const ItemOut &out)
{
    static_assert(kMfmaWaves * Fp4Shape<QB>::kQueries <= kBatchSlotQueries, "a group fits its slot");
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    auto each_query = [&](auto f) {
#pragma unroll
        for (int t = 0; t < Fp4Shape<QB>::kSets; ++t) {
            const int b = 4 * t + (lane >> 4);
            const int at = wave * Fp4Shape<QB>::kQueries + 16 * b + (lane & 15);
            const int qn = qgroup * kMfmaWaves * Fp4Shape<QB>::kQueries + at;
            if (b < Fp4Shape<QB>::kBlocks && qn < nq) f(t, PartKeys::of(slot, at), qn);
        }
    };
    each_query([&](int t, PartKeys *to, int) { to->merge(best[t][0], best[t][1]); });
    wait_device_accesses();
    __syncthreads();
    if (threadIdx.x == 0) *last_s = done->add_one() == parts - 1;
    __syncthreads();
    if (!*last_s) return;
    each_query([&](int, PartKeys *from, int qn) { store_final(from->first(), from->second(), nt, out, qn); });
}

enum class BatchKind { kPopcount, kMfmaI8, kMfmaFp4 };

// Arguments of the persistent matchers.
struct BatchLoopArgs {
    const uint32_t *query, *train;
    const PairEntry *pairs;
    int n_pairs;
    const PairInfo *info;
    const int32_t *unit_pair;
    BatchState *st;
    BatchSlots slots;
    int k;
    float ratio;
    int32_t *idx, *dist;
    uint8_t *accept;
};

template <BatchKind kKind, int QB>
__device__ __forceinline__ void batch_loop(const BatchLoopArgs &a, void *tbuf, int *slot_s)
{
    for (;;) {
        const int unit = claim_unit(a.st, slot_s);
        if (unit < 0) break;
        const int p = a.unit_pair[unit];
        if (p < 0 || p >= a.n_pairs) continue;   // cannot happen for a map written by the fill kernel
        const PairEntry e = a.pairs[p];
        const int local = unit - a.info[p].unit_first;
        const int nt = (int)e.nt;
        const ItemOut out{nullptr, a.idx + e.out_first * a.k, a.dist + e.out_first * a.k,
                          a.accept ? a.accept + e.out_first : nullptr, a.k, a.ratio};
        const uint32_t *q = a.query + (size_t)e.query_first * kWords;
        const uint32_t *t = a.train + (size_t)(nt ? e.train_first : 0) * kWords;
        if constexpr (kKind == BatchKind::kMfmaFp4) {
            // The part in ranges of at most 2^14 rows (the keys' index field),
            // merged in registers.
            const int groups = a.info[p].groups, parts = (int)a.info[p].parts;
            const int part = parts > 1 ? local / groups : 0, qgroup = local - part * groups;
            const int tiles = (nt + kTileRows - 1) / kTileRows, per_part = (tiles + parts - 1) / parts;
            const int t_end = min(tiles, (part + 1) * per_part);
            uint64_t best[Fp4Shape<QB>::kSets][2];
            fp4_init_best<QB>(best);
            int from = part * per_part;
            do {
                fp4_item<QB>(q, (int)e.nq, t, nt, qgroup, from, min(t_end, from + kFp4MaxTiles), best,
                             reinterpret_cast<uint4 (*)[kFp4TileVec]>(tbuf));
                from += kFp4MaxTiles;
            } while (from < t_end);
            if (parts == 1) {
                fp4_store<QB>(best, (int)e.nq, nt, qgroup, 0, out);
            } else {
                const uint32_t slot = a.info[p].slot + (uint32_t)qgroup;
                fp4_merge_part<QB>(best, (int)e.nq, nt, qgroup, (uint32_t)parts,
                                   a.slots.keys + (size_t)slot * kBatchSlotQueries,
                                   a.slots.done + slot, slot_s + 1, out);
            }
        } else {
            const int split_rows = max(kTileRows, (nt + kTileRows - 1) / kTileRows * kTileRows);
            if constexpr (kKind == BatchKind::kMfmaI8)
                mfma_item(q, (int)e.nq, t, nt, local, 0, split_rows, out,
                          reinterpret_cast<v4i (*)[kTileVec]>(tbuf));
            else
                popcount_item(q, (int)e.nq, t, nt, local, 0, split_rows, out);
        }
    }
}

// (Kernel parameters of their own, not fields of a struct, tell the compiler that the rows
// and tables which these two read alias nothing that the loop writes: a train row, uniform
// over a wavefront, then comes through scalar loads in the popcount matcher.  Struct ->
// parameters: popcount 9 pairs of 1855 rows 536 -> 436 us, 64 of 1846 818 -> 680; int8 the
// former 102 -> 96.  The FP4 matcher, whose registers are full, is as fast either way.)
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void knn_batch_mfma_kernel(
    const uint32_t *__restrict__ query, const uint32_t *__restrict__ train,
    const PairEntry *__restrict__ pairs, int n_pairs, const PairInfo *__restrict__ info,
    const int32_t *__restrict__ unit_pair, BatchState *__restrict__ st, int k, float ratio,
    int32_t *__restrict__ idx, int32_t *__restrict__ dist, uint8_t *__restrict__ accept)
{
    const BatchLoopArgs a{query, train, pairs, n_pairs, info, unit_pair, st, BatchSlots{}, k, ratio, idx, dist, accept};
    __shared__ v4i tbuf[2][kTileVec];
    __shared__ int slot[1];
    batch_loop<BatchKind::kMfmaI8, kQueryBlocks>(a, tbuf, slot);
}

template <int QB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void
knn_batch_fp4_kernel(BatchLoopArgs a)
{
    __shared__ uint4 tbuf[2][kFp4TileVec];
    __shared__ int slot[2];
    batch_loop<BatchKind::kMfmaFp4, QB>(a, tbuf, slot);
}

__global__ __launch_bounds__(256) void knn_batch_popcount_kernel(
    const uint32_t *__restrict__ query, const uint32_t *__restrict__ train,
    const PairEntry *__restrict__ pairs, int n_pairs, const PairInfo *__restrict__ info,
    const int32_t *__restrict__ unit_pair, BatchState *__restrict__ st, int k, float ratio,
    int32_t *__restrict__ idx, int32_t *__restrict__ dist, uint8_t *__restrict__ accept)
{
    const BatchLoopArgs a{query, train, pairs, n_pairs, info, unit_pair, st, BatchSlots{}, k, ratio, idx, dist, accept};
    __shared__ int slot[1];
    batch_loop<BatchKind::kPopcount, 1>(a, nullptr, slot);
}

}  // namespace

int queries_per_group(SplitKernel which, int fp4_query_blocks)
{
    return which == SplitKernel::kMfmaFp4 ? kMfmaWaves * 32 * fp4_query_blocks : 256;
}

hipError_t launch_knn_split(const KnnSplitArgs &a, SplitKernel which, hipStream_t stream)
{
    const SplitArgs k{a.query, a.train, (int)a.plan.nq, (int)a.plan.nt, (int)a.plan.split_rows,
                      a.plan.nsplit, a.partial, a.k, a.ratio, a.idx, a.dist, a.accept};
    const int64_t group = queries_per_group(which, a.plan.query_blocks);
    const int64_t qgroups = (a.plan.nq + group - 1) / group;
    const dim3 grid((unsigned)qgroups, (unsigned)a.plan.nsplit);
    if (which == SplitKernel::kMfmaI8)
        hipLaunchKernelGGL(knn_mfma_kernel, grid, dim3(kMfmaThreads), 0, stream, k);
    else if (which == SplitKernel::kMfmaFp4 && a.plan.query_blocks == 3)
        hipLaunchKernelGGL(knn_fp4_kernel<3>, grid, dim3(kMfmaThreads), 0, stream, k);
    else if (which == SplitKernel::kMfmaFp4)
        hipLaunchKernelGGL(knn_fp4_kernel<2>, grid, dim3(kMfmaThreads), 0, stream, k);
    else
        hipLaunchKernelGGL(knn_popcount_kernel, grid, dim3(256), 0, stream, k);
    return hipGetLastError();
}

int64_t merge_blocks(int64_t nq)
{
    return std::min((nq + kMergeQueries - 1) / kMergeQueries, kMergeMaxBlocks);
}

hipError_t launch_knn_merge(const KnnSplitArgs &a, hipStream_t stream)
{
    hipLaunchKernelGGL(knn_merge_kernel, dim3((unsigned)merge_blocks(a.plan.nq)), dim3(256), 0, stream, a.partial,
                       (int)a.plan.nq, a.plan.nsplit, (int)a.plan.nt, a.k, a.ratio, a.idx, a.dist,
                       a.accept);
    return hipGetLastError();
}

// Workgroups of a batch: the tuned number per CU, and no more than there can be units (parts
// only where a train range can exceed a least part).  A
// workgroup that finds no unit still takes its turn at the counter, some 40 ns, which was
// most of a small batch's time: 4 pairs of 200 rows 34.0 -> 15.8 us on the FP4 path (31.3
// with a setup that divided nothing), 36.3 -> 18.2 on int8, 161 -> 30 on popcount; 63 of 20
// rows 31.1 -> 13.4 (28.6).
int64_t batch_blocks(const BatchArgs &a)
{
    const int64_t resident = (int64_t)a.num_cus * (a.kind == SplitKernel::kPopcount ? 8 : a.shape.batch_groups_per_cu);
    const bool divides = a.kind == SplitKernel::kMfmaFp4 && a.train_rows > kMinPartTiles * kTileRows;
    const int64_t parts = divides ? std::min<int64_t>(a.slots.count, a.item_capacity) * (kBatchMaxParts - 1) : 0;
    return std::min(resident, a.item_capacity + parts);
}

hipError_t launch_knn_batch(const BatchArgs &a, hipStream_t stream)
{
    const bool fp4 = a.kind == SplitKernel::kMfmaFp4;
    // Two workgroups of the FP4 matcher fit a CU.
    hipLaunchKernelGGL(knn_batch_setup_kernel, dim3(1), dim3(256), 0, stream, a.pairs, a.n_pairs,
                       a.query_rows, a.train_rows, a.out_rows, a.item_capacity,
                       queries_per_group(a.kind, a.shape.fp4_query_blocks), 2 * a.num_cus, fp4 ? a.slots.count : 0,
                       a.info, a.state, a.flags);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int fill_blocks = a.n_pairs < 4096 ? a.n_pairs : 4096;
    const int fill_slices = std::max(1, std::min(16, 512 / a.n_pairs));
    hipLaunchKernelGGL(knn_batch_fill_kernel, dim3(fill_blocks, fill_slices), dim3(256), 0, stream, a.info,
                       a.n_pairs, a.unit_pair, a.slots);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const dim3 blocks((unsigned)batch_blocks(a));
    if (fp4) {
        const BatchLoopArgs k{a.query, a.train, a.pairs, a.n_pairs, a.info, a.unit_pair, a.state, a.slots,
                              a.k, a.ratio, a.idx, a.dist, a.accept};
        hipLaunchKernelGGL(a.shape.fp4_query_blocks == 3 ? knn_batch_fp4_kernel<3> : knn_batch_fp4_kernel<2>,
                           blocks, dim3(256), 0, stream, k);
    } else {
        hipLaunchKernelGGL(a.kind == SplitKernel::kMfmaI8 ? knn_batch_mfma_kernel : knn_batch_popcount_kernel,
                           blocks, dim3(256), 0, stream, a.query, a.train, a.pairs, a.n_pairs, a.info,
                           a.unit_pair, a.state, a.k, a.ratio, a.idx, a.dist, a.accept);
    }
    return hipGetLastError();
}

}  // namespace latch
