// LATCH descriptor extraction for gfx950.
//
// A workgroup of four wavefronts computes one descriptor at a time
// (grid-stride over keypoints):
//   1. resampling rule steps 1-3 on the keypoint (uniform across the group);
//   2. gather of the 48 x 48 upright window (steps 4-5), one byte load per
//      window position.  Rounding half away from zero is odd, so positions
//      (u, v) and (-u, -v) sample at offsets (ox, oy) and (-ox, -oy), and the
//      unrounded offsets of (u + 1, v) are those of (u, v) plus a per-keypoint
//      constant: a thread takes 2 chains (3 in two of the wavefronts) (u, v),
//      (u + 1, v), (-u, -v), (-u - 1, -v) with two roundings per coordinate
//      each (over [-24, 24]^2; the extra row and column are gathered and not
//      read).  The chains are taken in an order that keeps each load's samples
//      on nearby image bytes: for the keypoint's angle class (32 bins), sorted
//      by the band of image rows their first member samples at the class's
//      middle angle, then by column (a host-built table).  The loads are
//      issued one keypoint ahead so that their latency overlaps the previous
//      descriptor's arithmetic;
//   3. the samples are written to a plain window in LDS, and a copy pass
//      builds eight byte-shifted copies of it in which every 7-byte patch
//      row is one 8-byte-aligned quadword with a zero last byte;
//   4. Eq. 1 (Sec. 3.1) for 512 triplets: each wavefront takes 2 rounds of 64
//      lanes, one triplet per lane per round, in exact integer arithmetic;
//   5. triplets sit in (wavefront, round, lane) slots chosen on the host so
//      that the 32-lane halves of a ds_read_b64 hit few bank conflicts; each
//      bit goes to its triplet's place in LDS as a byte, and after the next
//      descriptor's first barrier 8 lanes at a time pack and store the words.
// A wavefront's priority rises with the phases of a descriptor, triplets highest,
// gather lowest: windows that are ready are finished first, and the gathers, whose
// samples are wanted a descriptor later, fill what issue slots are left.  50,000 keypoints
// of 1920 x 1080: 122 -> 116 us, 111 -> 100 upright; the gather above all else 120 and
// 110, the triplets alone above the rest 117 and 104.
//
// Patch distances.  With A, C the 7 x 7 patches of the anchor and one
// companion, ||A - C||^2 = sum A^2 + sum C^2 - 2 sum A C.  sum A^2 is shared by
// both sides of Eq. 1, so bit = [sum C1^2 - 2 sum A C1 > sum C2^2 - 2 sum A C2].
// Each patch row is a quadword of 7 u8 and a zero byte, and each sum is a
// chain of v_dot4_u32_u8.  All sums are < 49 * 255^2 < 2^22, so the int32
// result equals the exact integer one.
//
// The paper's CUDA kernel (Sec. 3.2) spreads one descriptor over 32 warps of
// a 1024-thread block with float32 patches in shared memory; here four 64-lane
// wavefronts share a 20.4 KB byte window (eight per CU, eight wavefronts per
// SIMD) and synchronise twice per descriptor.
//
// What bounds it: no one unit.  Per keypoint the vector ALUs issue about 940
// instructions, the LDS is busy some 950 cycles (patch reads 82 of 96 possible
// bank cycles per row and group, copies, window) and the texture units 1,070 at
// scale 1 to 1,290 over scales 1 to 3.6 (a byte load costs about 12 cycles plus
// 1.2 per 16-byte chunk of each 16 lanes), of 1,250 to 1,400 in all.  50,000
// keypoints of a 1920 x 1080 image: with two wavefronts per window (four per
// SIMD), 1,060 instructions and 95 bank cycles 135 us at mixed scales and 127 us
// upright; now 116 and 100 us.  16 images of 3000 x 2000 with 20,000 keypoints
// each: 894 -> 795 us.  The registers just fit: 64 per
// wavefront, and a spill of 20 bytes took back all of the gain (its accesses go
// through the texture units).
#include <algorithm>

#include "internal.h"

namespace latch {
namespace {

constexpr int kThreads = kExtractWaves * 64;              // 256: four wavefronts per window
constexpr int kRoundsPerWave = 8 / kExtractWaves;         // 2
constexpr int kWaveTriplets = 64 * kRoundsPerWave;

// Gather slots per thread: chains 256 m + tid of the gather order, four
// samples each; the last slot in wavefronts 0 and 1 only.
constexpr int kGatherTailWaves = 2;
constexpr int kRawCentre = kRawBase + kHalf * kRawStride + kHalf;
static_assert(2 * kThreads + 64 * kGatherTailWaves == kGatherClassEntries, "chains per class");
static_assert(kRawStride >= kWin + 1, "raw rows hold u = -24 .. 24");

// Copy pass: units (row y, quadword q), 240 per window, unit e = 5 y + q.
constexpr int kCopyUnits = kWin * kCopyQwords;
static_assert(kCopyUnits <= kThreads, "at most one copy unit per thread");
static_assert(kWinLdsBytes * 8 <= kLdsPerCu, "eight windows per CU");

#include "keypoint.h"

// The image offsets of one chain of keypoint k: its members (u, v), (u + 1, v),
// (-u, -v), (-u - 1, -v) go to at[0 .. 3], and raw is the raw-window byte of
// (u, v) less that of the centre (the mirrors' sit at minus it).  The chain's
// entry is half `h` of t.
//
// Rule steps 4-5.  The unrounded offsets of (u, v) are sq (C u - S v) and
// sq (S u + C v), formed from 24-bit products (|C u - S v| < 2^20 and sq <= 2^10,
// so every product is exact and full rate; kSmall: sq < 2^9, where sq C and sq S
// are 24-bit factors themselves and save a product per coordinate); those of
// (u + 1, v) add sq C and sq S (|sq C| <= 2^24, a scalar product), and rounding
// half away from zero is odd, so the mirrors sample at the negated offsets.  Two
// roundings per coordinate serve the chain's four samples.
// kTies: an offset may lie halfway between two integers (three instructions per
// rounding instead of one).  kInterior: every sample lies inside the image, so
// no coordinate is clamped.
struct Chain {
    int raw;
    uint32_t a, b, c, d;
};

template <bool kInterior, bool kTies, bool kSmall>
__device__ __forceinline__ Chain chain_offsets(const Keypoint &k, uint32_t t, int h, int half)
{
    Chain r;
    const int xm = k.width - 1, ym = k.height - 1;
    const int sqc = k.sq * k.c, sqs = k.sq * k.s;
    const int u = __builtin_amdgcn_sbfe((int)t, 16 * h, 8);
    const int v = __builtin_amdgcn_sbfe((int)t, 16 * h + 8, 8);
    r.raw = mad_i24(v, kRawStride, u);
    int mx, my;                                    // offsets + 2^21
    if constexpr (kSmall) {
        mx = mad_i24_s(sqc, u, mad_i24_s(-sqs, v, half));
        my = mad_i24_s(sqs, u, mad_i24_s(sqc, v, half));
    } else {
        mx = mad_i24_s(k.sq, mad_i24_s(k.c, u, mul_i24_s(-k.s, v)), half);
        my = mad_i24_s(k.sq, mad_i24_s(k.s, u, mul_i24_s(k.c, v)), half);
    }
    const int ox0 = round_half<kTies>(mx), oy0 = round_half<kTies>(my);
    const int ox1 = round_half<kTies>(mx + sqc), oy1 = round_half<kTies>(my + sqs);
    if constexpr (kInterior) {
        // Every sample is inside the image, so |offset| * pitch < 2^31 and the
        // 24-bit multiply-adds are exact.
        const int d0 = mad_i24_s(k.pitch, oy0, ox0);
        const int d1 = mad_i24_s(k.pitch, oy1, ox1);
        r.a = (uint32_t)(k.centre + d0);
        r.b = (uint32_t)(k.centre + d1);
        r.c = (uint32_t)(k.centre - d0);
        r.d = (uint32_t)(k.centre - d1);
    } else {
        r.a = (uint32_t)mad_i24(clamp_med3(k.cy + oy0, 0, ym), k.pitch, clamp_med3(k.cx + ox0, 0, xm));
        r.b = (uint32_t)mad_i24(clamp_med3(k.cy + oy1, 0, ym), k.pitch, clamp_med3(k.cx + ox1, 0, xm));
        r.c = (uint32_t)mad_i24(clamp_med3(k.cy - oy0, 0, ym), k.pitch, clamp_med3(k.cx - ox0, 0, xm));
        r.d = (uint32_t)mad_i24(clamp_med3(k.cy - oy1, 0, ym), k.pitch, clamp_med3(k.cx - ox1, 0, xm));
    }
    return r;
}

// The offsets of one or two chains of an entry pair, by the keypoint's case
// (uniform branches).
template <bool kTwo>
__device__ __forceinline__ void chains_offsets(const Keypoint &k, uint32_t t, Chain &x, Chain &y)
{
    const int half = opaque(kRoundHalf);
    if (!k.interior) {
        x = chain_offsets<false, true, false>(k, t, 0, half);
        if (kTwo) y = chain_offsets<false, true, false>(k, t, 1, half);
    } else if (k.ties) {
        x = chain_offsets<true, true, false>(k, t, 0, half);
        if (kTwo) y = chain_offsets<true, true, false>(k, t, 1, half);
    } else if (k.sq < 512) {
        x = chain_offsets<true, false, true>(k, t, 0, half);
        if (kTwo) y = chain_offsets<true, false, true>(k, t, 1, half);
    } else {
        x = chain_offsets<true, false, false>(k, t, 0, half);
        if (kTwo) y = chain_offsets<true, false, false>(k, t, 1, half);
    }
}

// A chain's samples and the place of the first in the raw window.
struct Samples {
    int raw;
    uint32_t a, b, c, d;
};

__device__ __forceinline__ void load_chain(GlobalByte *img, const Chain &c, Samples &s)
{
    s.raw = c.raw;
    s.a = img[c.a];
    s.b = img[c.b];
    s.c = img[c.c];
    s.d = img[c.d];
}

// Loads this thread's entries of the keypoint's angle class (a 4-byte and, in
// the wavefronts with a third chain, a 2-byte load) and issues its gather.
__device__ __forceinline__ void issue_gather(const Keypoint &k, const uint16_t *__restrict__ order,
                                             int tid, bool tail, Samples &s0, Samples &s1, Samples &s2)
{
    // (A uniform base and 32-bit offsets: no address registers over the loop.)
    const GlobalWord *cls = uniform_words((uint32_t *)(order + (size_t)k.cls * kGatherClassEntries));
    const uint32_t t0 = cls[(uint32_t)opaque(tid)];
    const uint32_t t1 = tail ? ((const GlobalHalf *)cls)[(uint32_t)opaque(tid + 2 * kThreads)] : 0u;
    GlobalByte *img = (GlobalByte *)k.img;
    Chain x, y;
    chains_offsets<true>(k, t0, x, y);
    load_chain(img, x, s0);
    load_chain(img, y, s1);
    if (tail) {
        chains_offsets<false>(k, t1, x, y);
        load_chain(img, x, s2);
    }
}

// The gathered samples into the raw window.  Chains overlap at the end of a
// row and the padding slots repeat the centre's chain: such bytes are written
// more than once, always with the same sample.
__device__ __forceinline__ void write_chain(uint8_t *lds, const Samples &s)
{
    uint8_t *p = lds + kRawCentre + s.raw, *q = lds + kRawCentre - s.raw;
    p[0] = (uint8_t)s.a;
    p[1] = (uint8_t)s.b;
    q[0] = (uint8_t)s.c;
    q[-1] = (uint8_t)s.d;
}

// Copy unit e = 5 y + q: from raw bytes (y, 8 q .. 8 q + 15) build the
// quadword q of row y of every copy (and of the edge copies when q = 4).
__device__ __forceinline__ void copy_unit(uint8_t *lds, int e)
{
    const int y = e / kCopyQwords, q = e - kCopyQwords * y;
    const uint32_t *src = reinterpret_cast<const uint32_t *>(lds + kRawBase + y * kRawStride + 8 * q);
    const uint32_t d0 = src[0], d1 = src[1], d2 = src[2], d3 = src[3];
    constexpr uint32_t m = 0x00ffffffu;
    uint32_t lo[kCopies], hi[kCopies];
    lo[0] = d0;
    lo[1] = __builtin_amdgcn_alignbyte(d1, d0, 1);
    lo[2] = __builtin_amdgcn_alignbyte(d1, d0, 2);
    lo[3] = __builtin_amdgcn_alignbyte(d1, d0, 3);
    lo[4] = d1;
    lo[5] = __builtin_amdgcn_alignbyte(d2, d1, 1);
    lo[6] = __builtin_amdgcn_alignbyte(d2, d1, 2);
    lo[7] = __builtin_amdgcn_alignbyte(d2, d1, 3);
#pragma unroll
    for (int s = 0; s < 4; ++s) hi[s] = lo[s + 4] & m;
    hi[4] = d2 & m;
    hi[5] = __builtin_amdgcn_alignbyte(d3, d2, 1) & m;
    hi[6] = __builtin_amdgcn_alignbyte(d3, d2, 2) & m;
    hi[7] = __builtin_amdgcn_alignbyte(d3, d2, 3) & m;
#pragma unroll
    for (int s = 0; s < kCopies; ++s)
        *reinterpret_cast<uint2 *>(lds + s * kCopyBytes + 8 * e) = make_uint2(lo[s], hi[s]);
    if (q == kCopyQwords - 1) {
        // Columns 40..46 and 41..47.
        *reinterpret_cast<uint2 *>(lds + kEdgeBase + 8 * e) = make_uint2(d2, d3 & m);
        *reinterpret_cast<uint2 *>(lds + kEdgeBase + 8 + 8 * e) =
            make_uint2(__builtin_amdgcn_alignbyte(d3, d2, 1), d3 >> 8);
    }
}

// One row of the three patches of a triplet: anchor, companion 1, companion 2.
// Rows are read one row before their use (eight wavefronts per SIMD hide the
// rest of the latency; two rows ahead are no faster, three spill registers).
constexpr int kPatchRows = 2 * kPatchR + 1;
constexpr int kRowsAhead = 1;

struct PatchRow {
    uint64_t a, c, e;
};

// Sums of Eq. 1 on one triplet, via ||A - Ck||^2 - sum A^2 = sum Ck^2 - 2 sum A Ck.
// The zero last byte of every row quadword keeps them to the 7 x 7 patch.
struct TripletSums {
    uint32_t ac1 = 0, ac2 = 0, q1 = 0, q2 = 0;

    __device__ __forceinline__ void add(const PatchRow &r)
    {
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            const uint32_t a = (uint32_t)(r.a >> (32 * d)), c = (uint32_t)(r.c >> (32 * d)),
                           e = (uint32_t)(r.e >> (32 * d));
            ac1 = dot4(a, c, ac1);
            ac2 = dot4(a, e, ac2);
            q1 = dot4(c, c, q1);
            q2 = dot4(e, e, q2);
        }
    }

    // [||A - C1||^2 > ||A - C2||^2]: the sign of the difference the other way round.
    __device__ __forceinline__ uint32_t bit() const { return (((ac1 - ac2) << 1) + (q2 - q1)) >> 31; }
};

template <bool kTable>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(8, 8))) void extract_kernel(
    ImageSource src, const float4 *__restrict__ kps, int64_t begin, int64_t n_host,
    const int64_t *__restrict__ n_dev,
    const int2 *__restrict__ rot, const uint2 *__restrict__ trip_off,
    const uint32_t *__restrict__ bit_of, const uint16_t *__restrict__ gather_order,
    uint32_t *__restrict__ desc, uint32_t *__restrict__ flags)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds[kWinLdsBytes];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // Wavefront w evaluates the triplets in slots 128 w + 64 r + lane, r = 0, 1,
    // where the bank-aware assignment put them; `places` names their output
    // bits (constant over keypoints).
    // Offsets: anchor | companion 1 << 16 per round, and the companion-2
    // offsets of both rounds packed in off_2 (all < 2^16).
    uint32_t off_a1[kRoundsPerWave], off_2 = 0;
#pragma unroll
    for (int r = 0; r < kRoundsPerWave; ++r) {
        const uint2 o = trip_off[kWaveTriplets * wave + 64 * r + lane];
        off_a1[r] = o.x;
        off_2 |= o.y << (16 * r);
    }
    uint8_t *out_bits = lds + kBitBase;
    const bool tail = wave < kGatherTailWaves;

    // The end of the positions: a host value, or (batches) a device value capped by it.
    int64_t n_all = n_host;
    if (n_dev) n_all = min(n_all, *n_dev);
    const XcdRange range = xcd_range(n_all - begin);
    const int64_t n = begin + range.end;
    int64_t p = begin + range.first;
    if (p >= n) return;
    const uint32_t places = bit_of[64 * wave + lane];
    const int64_t stride = range.stride;
    Samples s0, s1, s2;                       // s2 in the wavefronts with a third chain
    KeypointBatch batch = prepare_batch<kTable, kHalf>(kps, n, p, stride, lane, rot, src);
    bool bad_image = false;
    Keypoint cur = batch_get<kTable>(batch, 0, src, &bad_image);
    if (cur.ok) issue_gather(cur, gather_order, tid, tail, s0, s1, s2);

    int64_t pending = -1;                     // row whose bits are complete in LDS
    for (int i = 0; p < n; ++i, p += stride) {
        const bool compute = cur.ok;
        // Descriptor row of this position's keypoint (the position itself
        // unless a batch order permutes the keypoints).
        const int64_t q = kTable && src.order ? (int64_t)cur.key : p;
        if (!compute) {
            if (tid < kWords) uniform_words(desc + q * kWords)[(uint32_t)tid] = 0u;
            if (tid == 0) atomicOr(flags, bad_image ? kFlagBadImage : kFlagBadKeypoint);
        } else {
            __builtin_amdgcn_s_setprio(0);
            // The raw window was last read by the previous descriptor's copy
            // pass, which ended before that descriptor's second barrier.
            write_chain(lds, s0);
            write_chain(lds, s1);
            if (tail) write_chain(lds, s2);
            __syncthreads();   // raw window complete; the previous triplets are done
            __builtin_amdgcn_s_setprio(1);
            if (pending >= 0) pack_words(lds + kBitBase, wave, lane, desc + pending * kWords);
            if (tid < kCopyUnits) copy_unit(lds, tid);
            __syncthreads();   // copies complete
        }

        __builtin_amdgcn_s_setprio(0);
        // Start the next keypoint's gather; it completes during the arithmetic below.
        const int j = (i + 1) & 63;
        if (j == 0) batch = prepare_batch<kTable, kHalf>(kps, n, p + stride, stride, lane, rot, src);
        cur = batch_get<kTable>(batch, j, src, &bad_image);
        if (cur.ok) issue_gather(cur, gather_order, tid, tail, s0, s1, s2);
        if (!compute) continue;
        __builtin_amdgcn_s_setprio(2);

        // Eq. 1 for this wavefront's 128 triplets, each bit as a byte in the
        // place of its triplet.
        constexpr int kAllRows = kRoundsPerWave * kPatchRows;
        PatchRow rows[kRowsAhead + 1];
        auto read = [&](int n) {
            const int r = n / kPatchRows, at = n % kPatchRows * kCopyRowBytes;
            PatchRow &to = rows[n % (kRowsAhead + 1)];
            to.a = read_quad(lds + (off_a1[r] & 0xffffu) + at);
            to.c = read_quad(lds + (off_a1[r] >> 16) + at);
            to.e = read_quad(lds + ((off_2 >> (16 * r)) & 0xffffu) + at);
        };
#pragma unroll
        for (int n = 0; n < kRowsAhead; ++n) read(n);
        TripletSums sums;
#pragma unroll
        for (int n = 0; n < kAllRows; ++n) {
            __builtin_amdgcn_sched_barrier(0);
            if (n + kRowsAhead < kAllRows) read(n + kRowsAhead);
            sums.add(rows[n % (kRowsAhead + 1)]);
            if (n % kPatchRows == kPatchRows - 1) {
                out_bits[(places >> (16 * (n / kPatchRows))) & 0xffffu] = (uint8_t)sums.bit();
                sums = TripletSums();
            }
        }
        pending = q;
    }
    __syncthreads();                          // the last triplets are done
    if (pending >= 0) pack_words(lds + kBitBase, wave, lane, desc + pending * kWords);
}

}  // namespace

// An ordered batch of many keypoints runs in equal launches of at least this many.
// Within a launch the workgroups of an XCD drift apart, and with them the bands of
// rows that its L2 has to hold: L2 misses per keypoint were 27 lines over 320,000
// keypoints of 3000 x 2000 images and 74 over 1,280,000; each launch starts them
// together again.  1,280,000: 3465 -> 3250 us in three, 3205 in five, 3223 in ten;
// 1,910,000 of uneven images 5890 -> 5450 in four, 5495 in eight.  At the lower end, in
// two instead of one: 800,000 of 3000 x 2000 images 2120 -> 2030 us, 1,014,000 of uneven
// ones 2720 -> 2600, 800,000 of 1280 x 720 1931 and 1930, 832,000 of 640 x 480 2000 and
// 1993; 580,000 of 1280 x 720, which drift costs little, would take 0.6% longer.
constexpr int64_t kSegment = 400000;
// With a count on the device, launches are cut by the capacity, and those past the count
// find nothing to do, about 3 us each.  Four instead of one at a capacity of 2,000,000:
// 21.9 -> 31.1 us for a count of 1000, 146 -> 151 for 50,000, 1675 -> 1657 for 667,000,
// 5650 -> 5020 for all.
constexpr int64_t kMostCounted = 4;

hipError_t launch_extract(const ExtractArgs &a, hipStream_t stream)
{
    if (a.n <= 0) return hipSuccess;
    const int64_t resident = (int64_t)a.num_cus * (kLdsPerCu / kWinLdsBytes);
    int64_t launches = a.order ? std::max<int64_t>(1, a.n / kSegment) : 1;
    if (a.n_dev) launches = std::min(launches, kMostCounted);
    const int64_t segment = (a.n + launches - 1) / launches;
    ImageSource src{a.img, a.height, a.width, a.pitch, a.table, a.image_id, a.n_images, a.order};
    for (int64_t begin = 0; begin < a.n; begin += segment) {
        const int64_t end = std::min(a.n, begin + segment);
        const unsigned blocks = (unsigned)std::min(end - begin, resident);
        hipLaunchKernelGGL(a.table ? extract_kernel<true> : extract_kernel<false>, dim3(blocks), dim3(kThreads), 0,
                           stream, src, a.kps, begin, end, a.n_dev, a.rot, a.trip_off, a.bit_of, a.gather,
                           a.desc, a.flags);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace latch
