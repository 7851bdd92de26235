// LATCH extraction with the paper's CLATCH geometry and per-pixel patch
// weights (Sec. 3.2: 64 x 64 windows, 8 x 8 patches, an integer weight per
// patch pixel; zero weights on one row and one column give the 7 x 7 patch).
//
// For each triplet, S_j = sum w[a][b] (A[a][b] - P_j[a][b])^2 over the patch
// pixels and bit = [S_1 > S_2].  Per pixel,
//     w (A - P_1)^2 - w (A - P_2)^2 = w d (P_1 + P_2) - 2 w d A,  d = P_1 - P_2,
// so bit = [sum w d (P_1 + P_2) > 2 sum w d A].  Weights lie in [0, 128] and d in
// [-255, 255], so d, w d and P_1 + P_2 fit signed 16-bit lanes: per patch row of 8
// pixels (4 pairs) the kernel forms d, w d and P_1 + P_2 with packed 16-bit
// subtract, multiply and add, and accumulates both sums with v_dot2_i32_i16.
// |sum w d (P_1 + P_2)| <= 64 * 128 * 255 * 510 < 2^31, and so is twice the other:
// exact.  7 x 7 patches run as 8 x 8 ones whose last row and column weigh 0.
//
// A workgroup of eight wavefronts (W = 48: four) computes one descriptor at a
// time (grid-stride over keypoints):
//   1. resampling rule steps 1-3 on the keypoint (uniform);
//   2. the W x W window gathered with the rule, issued one keypoint ahead and
//      along image rows (Positions below), written to a plain byte window in
//      LDS, from which a copy pass makes four copies of 16-bit pixels shifted by
//      0..3 columns, so that the 8 pixels of any patch row start on a quadword
//      of one copy (two ds_read_b64);
//   3. one triplet per thread (W = 48: two), in (wavefront, lane) slots the host
//      chose over all triplets so that the 32-lane halves of a ds_read_b64 hit
//      few bank conflicts; each bit goes to its triplet's place in LDS as a byte,
//      and after the next descriptor's first barrier 8 lanes at a time pack and
//      store the words.
//
// What bounds it: LDS (patch rows) and vector issue, about two thirds busy each,
// between two barriers per descriptor.  20,000 keypoints of a
// 1920 x 1080 image, W = 64: in raster order with four wavefronts, 16 at a time per
// CU, 142 us (the texture units 67% busy: a row of the window crosses up to 64 image
// rows); along image rows 137, reads one patch row ahead 134, eight wavefronts and
// free slots 122, a copy pass (64 byte writes and 64 of quadwords per descriptor
// and wavefronts in place of 256 conflicting 16-bit ones) 110, priorities by phase 100.
// 50,000 keypoints of 3840 x 2160: 387 -> 246 us; upright 125 -> 94; W = 48 104 -> 96.
#include "internal.h"

namespace latch {
namespace {

#include "keypoint.h"
#include "packed16.h"

constexpr int kPatchRows = 8;
constexpr int kRowsAhead = 1;

template <int kW>
struct WGeom {
    static constexpr int kThreads = kW == 64 ? 512 : 256;
    static constexpr int kWaves = kThreads / 64;
    static constexpr int kRounds = kTriplets / kThreads;         // triplets per thread
    static constexpr int kHalfW = kW / 2;
    static constexpr int kRowBytes = 2 * (kW + 4);               // 16-bit pixels; 4 spare spread the banks
    static constexpr int kCopyBytes = (kW + 1) * kRowBytes;      // 7 x 7 patches reach a row past W
    static constexpr int kRawStride = kW + 4;                    // the window as gathered, bytes
    static constexpr int kRawBase = 4 * kCopyBytes;
    static constexpr int kBitBase = kRawBase + kW * kRawStride + 16;   // the descriptor's bits, a byte each
    static constexpr int kLds = kBitBase + kTriplets;
    static constexpr int kRowQuads = kW / 4;                     // patch rows start at multiples of 4 below
    static constexpr int kUnits = kW * kRowQuads;                // W - 4 and read two quads
    static constexpr int kSamples = kW * kW / kThreads;         // per thread
    static_assert(kW * kW % kThreads == 0, "whole samples per thread");
};

// Rule steps 4-5 for a sample with unrounded offsets m - 2^21 (kTies: they may lie
// halfway between two integers; kInterior: the sample lies inside the image).
template <bool kInterior, bool kTies>
__device__ __forceinline__ uint32_t sample_at(const Keypoint &k, GlobalByte *img, int mx, int my)
{
    const int ox = round_half<kTies>(mx), oy = round_half<kTies>(my);
    if constexpr (kInterior) return img[(uint32_t)(k.centre + mad_i24_s(k.pitch, oy, ox))];
    const int x = clamp_med3(k.cx + ox, 0, k.width - 1);
    const int y = clamp_med3(k.cy + oy, 0, k.height - 1);
    return img[(uint32_t)mad_i24(y, k.pitch, x)];
}

// Which window positions a thread samples.  W = 64: lane a of wavefront w takes
// position a of one axis and b = (w + 8 m + k) mod 64, m = 0..7, of the other,
// where k is the lane's shear: along an axis the samples move away from an image
// row by the tangent of its angle, and k undoes it to the nearest position, so the
// 64 lanes of a load sample one or a few image rows (any k covers the window
// once).  The lanes run along the axis nearer to the image rows.  Other W: q = tid
// + 256 m in raster order.
struct Positions {
    bool rows;      // lanes along u, m along v
    int b;          // (w + k) mod 64
};

template <int kW>
__device__ __forceinline__ Positions positions(const Keypoint &k, int tid)
{
    Positions t = {true, 0};
    if constexpr (kW == 64) {
        t.rows = abs(k.c) >= abs(k.s);
        // S u + C v stays constant where v falls by S / C per u (u by C / S per v).
        const float slope = t.rows ? -(float)k.s * __builtin_amdgcn_rcpf((float)k.c)
                                   : -(float)k.c * __builtin_amdgcn_rcpf((float)k.s);
        t.b = ((tid >> 6) + (int)rintf((float)((tid & 63) - 32) * slope)) & 63;
    }
    return t;
}

template <int kW, bool kInterior, bool kTies>
__device__ __forceinline__ void load_samples(const Keypoint &k, const Positions &t, int tid,
                                             uint32_t (&g)[WGeom<kW>::kSamples])
{
    using G = WGeom<kW>;
    GlobalByte *img = (GlobalByte *)k.img;
    // |C u - S v| < 2^20 and sq <= 2^10, so the 24-bit products are exact.
    if constexpr (kW == 64) {
        // Offsets of (a, b): sq (ca a + cb b), sq (da a + db b), a step of kWaves in b
        // away from each other, less 64 past the wrap (|64 sq cb| <= 2^30).
        const int ca = t.rows ? k.c : -k.s, cb = t.rows ? -k.s : k.c;
        const int da = t.rows ? k.s : k.c, db = t.rows ? k.c : k.s;
        const int a = (tid & 63) - G::kHalfW, b = t.b - G::kHalfW;
        const int half = opaque(kRoundHalf);
        const int mx = mad_i24_s(k.sq, mad_i24_s(ca, a, mul_i24_s(cb, b)), half);
        const int my = mad_i24_s(k.sq, mad_i24_s(da, a, mul_i24_s(db, b)), half);
        const int sx = G::kWaves * k.sq * cb, sy = G::kWaves * k.sq * db;
        const int wx = mx - G::kSamples * sx, wy = my - G::kSamples * sy;
#pragma unroll
        for (int m = 0; m < G::kSamples; ++m) {
            const bool wrapped = t.b >= 64 - G::kWaves * m;
            g[m] = sample_at<kInterior, kTies>(k, img, (wrapped ? wx : mx) + m * sx,
                                               (wrapped ? wy : my) + m * sy);
        }
    } else {
#pragma unroll
        for (int m = 0; m < G::kSamples; ++m) {
            const int q = tid + G::kThreads * m;
            const int u = q % kW - G::kHalfW, v = q / kW - G::kHalfW;
            g[m] = sample_at<kInterior, kTies>(
                k, img, mad_i24_s(k.sq, mad_i24_s(k.c, u, mul_i24_s(-k.s, v)), opaque(kRoundHalf)),
                mad_i24_s(k.sq, mad_i24_s(k.s, u, mul_i24_s(k.c, v)), opaque(kRoundHalf)));
        }
    }
}

template <int kW>
__device__ __forceinline__ void issue_samples(const Keypoint &k, const Positions &t, int tid,
                                              uint32_t (&g)[WGeom<kW>::kSamples])
{
    if (!k.interior)
        load_samples<kW, false, true>(k, t, tid, g);
    else if (k.ties)
        load_samples<kW, true, true>(k, t, tid, g);
    else
        load_samples<kW, true, false>(k, t, tid, g);
}

// This thread's samples into the raw window.
template <int kW>
__device__ __forceinline__ void write_window(uint8_t *lds, const Positions &t, int tid,
                                             const uint32_t (&g)[WGeom<kW>::kSamples])
{
    using G = WGeom<kW>;
    const int step_a = t.rows ? 1 : G::kRawStride, step_b = t.rows ? G::kRawStride : 1;
    const int at = step_a * (tid & 63) + step_b * t.b, wrapped_at = at - 64 * step_b;
    uint8_t *raw = lds + G::kRawBase;
#pragma unroll
    for (int m = 0; m < G::kSamples; ++m) {
        const int q = tid + G::kThreads * m;
        const int to = kW == 64 ? (t.b >= 64 - G::kWaves * m ? wrapped_at : at) + G::kWaves * m * step_b
                                : q / kW * G::kRawStride + q % kW;
        raw[to] = (uint8_t)g[m];
    }
}

// Copy pass: quadword q of row i of copy s holds pixels 4 q + s .. 4 q + s + 3.
// (Pixels past column W - 1, and the row past W - 1, meet zero weights only.)
template <int kW>
__device__ __forceinline__ void copy_window(uint8_t *lds, int tid)
{
    using G = WGeom<kW>;
#pragma unroll
    for (int e0 = 0; e0 < G::kUnits; e0 += G::kThreads) {
        const int e = e0 + tid;
        if (G::kUnits % G::kThreads != 0 && e >= G::kUnits) break;
        const int i = e / G::kRowQuads, q = e % G::kRowQuads;
        const uint32_t *src = reinterpret_cast<const uint32_t *>(lds + G::kRawBase + i * G::kRawStride + 4 * q);
        const uint32_t d0 = src[0], d1 = src[1];
        uint8_t *to = lds + i * G::kRowBytes + 8 * q;
        // Bytes k, k + 1 of d1:d0 as 16-bit halves.
        const uint32_t p[6] = {__builtin_amdgcn_perm(d1, d0, 0x0c010c00), __builtin_amdgcn_perm(d1, d0, 0x0c020c01),
                               __builtin_amdgcn_perm(d1, d0, 0x0c030c02), __builtin_amdgcn_perm(d1, d0, 0x0c040c03),
                               __builtin_amdgcn_perm(d1, d0, 0x0c050c04), __builtin_amdgcn_perm(d1, d0, 0x0c060c05)};
#pragma unroll
        for (int s = 0; s < 4; ++s)
            *reinterpret_cast<uint2 *>(to + s * G::kCopyBytes) = make_uint2(p[s], p[s + 2]);
    }
}

// One row of the three patches, two quadwords each: anchor, companion 1, companion 2.
struct PatchRow {
    uint64_t a[2], c[2], e[2];
};

// One patch row (4 pixel pairs) of sum w d (P_1 + P_2) and sum w d A.
__device__ __forceinline__ void weighted_row(const uint32_t *wrow, const PatchRow &r, int &sum_p, int &sum_a)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const auto pair = [&](const uint64_t (&q)[2]) {
            return __builtin_bit_cast(short2v, (uint32_t)(q[i / 2] >> (32 * (i % 2))));
        };
        const short2v wv = __builtin_bit_cast(short2v, wrow[i]);
        const short2v A = pair(r.a), P1 = pair(r.c), P2 = pair(r.e);
        const short2v wd = wv * (P1 - P2);
        sum_p = __builtin_amdgcn_sdot2(wd, P1 + P2, sum_p, false);
        sum_a = __builtin_amdgcn_sdot2(wd, A, sum_a, false);
    }
}

template <bool kTable, int kW>
__global__ __launch_bounds__(WGeom<kW>::kThreads) __attribute__((amdgpu_waves_per_eu(kW == 64 ? 8 : 5))) void
extract_weighted_kernel(
    ImageSource src, const float4 *__restrict__ kps, int64_t n_host, const int64_t *__restrict__ n_dev,
    const int2 *__restrict__ rot, const uint2 *__restrict__ trip_off,
    const uint32_t *__restrict__ bit_of, WeightRows w, uint32_t *__restrict__ desc,
    uint32_t *__restrict__ flags)
{
    using G = WGeom<kW>;
    __shared__ __attribute__((aligned(16))) uint8_t lds[G::kLds];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // This lane's slots (round r: 64 (kRounds wave + r) + lane) and the places of
    // their bits.
    uint2 off[G::kRounds];
    uint32_t places = 0;
#pragma unroll
    for (int r = 0; r < G::kRounds; ++r) {
        const int slot = 64 * (G::kRounds * wave + r) + lane;
        off[r] = trip_off[slot];
        places |= bit_of[slot] << (16 * r);
    }

    int64_t n_all = n_host;
    if (n_dev) n_all = min(n_all, *n_dev);
    const XcdRange range = xcd_range(n_all);
    const int64_t n = range.end;
    int64_t p = range.first;
    if (p >= n) return;
    const int64_t stride = range.stride;
    uint32_t g[G::kSamples];
    KeypointBatch batch = prepare_batch<kTable, G::kHalfW>(kps, n, p, stride, lane, rot, src);
    bool bad_image = false;
    Keypoint cur = batch_get<kTable>(batch, 0, src, &bad_image);
    Positions at = positions<kW>(cur, tid);
    if (cur.ok) issue_samples<kW>(cur, at, tid, g);

    // A wavefront's priority by phase, as in the default kernel: 110 -> 100 us, 104 -> 94
    // upright.  (W = 48, five wavefronts per SIMD, is 3% slower with it.)
    constexpr bool kPriorities = kW == 64;
    int64_t pending = -1;      // row whose bits are complete in LDS
    for (int i = 0; p < n; ++i, p += stride) {
        const bool compute = cur.ok;
        if (!compute) {
            if (tid < kWords) uniform_words(desc + p * kWords)[(uint32_t)tid] = 0u;
            if (tid == 0) atomicOr(flags, bad_image ? kFlagBadImage : kFlagBadKeypoint);
        } else {
            if (kPriorities) __builtin_amdgcn_s_setprio(0);
            // The raw window was last read by the previous descriptor's copy
            // pass, which ended before that descriptor's second barrier.
            write_window<kW>(lds, at, tid, g);
            __syncthreads();   // raw window complete; the previous triplets are done
            if (kPriorities) __builtin_amdgcn_s_setprio(1);
            if (pending >= 0 && wave < kTriplets / 128)
                pack_words(lds + G::kBitBase, wave, lane, desc + pending * kWords);
            copy_window<kW>(lds, tid);
            __syncthreads();   // copies complete
        }

        if (kPriorities) __builtin_amdgcn_s_setprio(0);
        // Next keypoint's gather, in flight during the arithmetic below.
        const int j = (i + 1) & 63;
        if (j == 0) batch = prepare_batch<kTable, G::kHalfW>(kps, n, p + stride, stride, lane, rot, src);
        cur = batch_get<kTable>(batch, j, src, &bad_image);
        at = positions<kW>(cur, tid);
        if (cur.ok) issue_samples<kW>(cur, at, tid, g);
        if (!compute) continue;
        if (kPriorities) __builtin_amdgcn_s_setprio(2);

        constexpr int kAllRows = G::kRounds * kPatchRows;
        PatchRow rows[kRowsAhead + 1];
        auto read = [&](int n) {
            const uint2 t = off[n / kPatchRows];
            const int row = n % kPatchRows * G::kRowBytes;
            PatchRow &to = rows[n % (kRowsAhead + 1)];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                to.a[h] = read_quad(lds + (t.x & 0xffffu) + row + 8 * h);
                to.c[h] = read_quad(lds + (t.x >> 16) + row + 8 * h);
                to.e[h] = read_quad(lds + t.y + row + 8 * h);
            }
        };
#pragma unroll
        for (int n = 0; n < kRowsAhead; ++n) read(n);
        int sum_p = 0, sum_a = 0;
        int wfirst = 0;                // unknown to the compiler: the weights are read here, not kept
        asm volatile("" : "+s"(wfirst));
#pragma unroll
        for (int n = 0; n < kAllRows; ++n) {
            __builtin_amdgcn_sched_barrier(0);
            if (n + kRowsAhead < kAllRows) read(n + kRowsAhead);
            weighted_row(w.pair + wfirst + 4 * (n % kPatchRows), rows[n % (kRowsAhead + 1)], sum_p, sum_a);
            if (n % kPatchRows == kPatchRows - 1) {
                lds[G::kBitBase + ((places >> (16 * (n / kPatchRows))) & 0xffffu)] = (uint8_t)(sum_p > 2 * sum_a);
                sum_p = sum_a = 0;
            }
        }
        pending = p;
    }
    __syncthreads();       // the last bits are written
    if (pending >= 0 && wave < kTriplets / 128)
        pack_words(lds + G::kBitBase, wave, lane, desc + pending * kWords);
}

template <int kW>
hipError_t launch_weighted_w(const ExtractArgs &a, hipStream_t stream)
{
    int64_t blocks = a.n;
    // As many workgroups as the LDS holds.  For W = 48 that is six per CU where five
    // wavefronts per SIMD let five run at once; with five, 2,000 keypoints take 15.0 ->
    // 14.0 us, 20,000 92.6 -> 92.2 and 50,000 223.2 -> 224.1.
    const int64_t resident = (int64_t)a.num_cus * (kLdsPerCu / WGeom<kW>::kLds);
    if (blocks > resident) blocks = resident;
    ImageSource src{a.img, a.height, a.width, a.pitch, a.table, a.image_id, a.n_images, nullptr};
    if (a.table)
        hipLaunchKernelGGL((extract_weighted_kernel<true, kW>), dim3((unsigned)blocks), dim3(WGeom<kW>::kThreads),
                           0, stream, src, a.kps, a.n, a.n_dev, a.rot, a.wtrip_off, a.wbit_of, a.weights,
                           a.desc, a.flags);
    else
        hipLaunchKernelGGL((extract_weighted_kernel<false, kW>), dim3((unsigned)blocks),
                           dim3(WGeom<kW>::kThreads), 0, stream, src, a.kps, a.n, a.n_dev, a.rot, a.wtrip_off,
                           a.wbit_of, a.weights, a.desc, a.flags);
    return hipGetLastError();
}

}  // namespace

uint32_t weighted_patch_offset(int window, int top, int left)
{
    const int s = left & 3, e = left - s;
    if (window == 64)
        return (uint32_t)(s * WGeom<64>::kCopyBytes + top * WGeom<64>::kRowBytes + 2 * e);
    return (uint32_t)(s * WGeom<48>::kCopyBytes + top * WGeom<48>::kRowBytes + 2 * e);
}

hipError_t launch_extract_weighted(const ExtractArgs &a, hipStream_t stream)
{
    if (a.n <= 0) return hipSuccess;
    return a.window == 64 ? launch_weighted_w<64>(a, stream) : launch_weighted_w<48>(a, stream);
}

}  // namespace latch
