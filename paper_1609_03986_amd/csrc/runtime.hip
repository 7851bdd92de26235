// C ABI of the LATCH library: handle, argument checks, tables, workspace and
// launches.  Every call only enqueues on the caller's stream (see latch.h).
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <string>
#include <algorithm>
#include <array>
#include <map>
#include <mutex>
#include <vector>

#include "../../include/latch.h"
#include "internal.h"
#include "part_keys.h"

using namespace latch;

struct latch_ctx {
    int device = 0;
    int num_cus = 0;
    int2 *rot_dev = nullptr;           // [4096] {cos_q14 | sin_q14 << 16, tie masks}
    uint2 *trip_off_dev = nullptr;     // [512] by slot: LDS byte offsets of the three patches
    uint32_t *bit_of_dev = nullptr;    // [256] output bits of the slots per (wavefront, lane)
    uint16_t *gather_dev = nullptr;    // [kGatherClasses][kGatherClassEntries] window gather order
    uint32_t *flags_dev = nullptr;     // sticky error word
    // Weighted geometry (latch_create_geometry); window 0 runs the default kernel.
    int window = 0;
    uint2 *wtrip_dev = nullptr;        // [512] by slot: weighted-kernel patch offsets
    uint32_t *wbit_of_dev = nullptr;   // [512] by slot: output bits of the weighted kernel
    uint2 *dense_off_dev = nullptr;    // [512] in triplet order: dense-kernel texture offsets
    WeightRows weights = {};
    uint8_t *ws = nullptr;             // grow-only workspace
    size_t ws_bytes = 0;
    uint8_t *parts = nullptr;          // handle_parts(): what dividing train ranges needs
    uint8_t *scratch = nullptr;        // this device's copy of the static scratch array
    latch_tuning tuning;               // LATCH_PATH_AUTO table and split targets
    std::string last_error;
    // Event timing (latch_timing_enable).
    bool timing = false;
    struct Timed {
        const char *name;
        hipEvent_t start, stop;
    };
    std::vector<Timed> timed;
    std::vector<hipEvent_t> event_pool;
};

namespace {

int fail(latch_handle h, int code, const char *fmt, ...) __attribute__((format(printf, 3, 4)));

int fail(latch_handle h, int code, const char *fmt, ...)
{
    if (h) {
        char buf[512];
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(buf, sizeof buf, fmt, ap);
        va_end(ap);
        h->last_error = buf;
    }
    return code;
}

int hip_fail(latch_handle h, hipError_t e, const char *what)
{
    return fail(h, e == hipErrorOutOfMemory ? LATCH_ENOMEM : LATCH_EDEVICE, "%s: %s", what,
                hipGetErrorString(e));
}

// Rule step 2: the first octant from libm, the rest from the exact
// symmetries cos(90 - a) = sin(a) and (C, S)(a + 90) = (-S, C)(a).
void rotation_table(int16_t *c, int16_t *s)
{
    const double step = M_PI / 2048.0;
    for (int a = 0; a <= 512; ++a) {
        c[a] = (int16_t)std::lrint(16384.0 * std::cos(step * a));
        s[a] = (int16_t)std::lrint(16384.0 * std::sin(step * a));
    }
    for (int a = 513; a < 1024; ++a) {
        c[a] = s[1024 - a];
        s[a] = c[1024 - a];
    }
    for (int a = 1024; a < kBins; ++a) {
        c[a] = (int16_t)(-s[a - 1024]);
        s[a] = c[a - 1024];
    }
}

// Per angle bin, the numbers k of trailing zero bits of sq (bits 0..10) for
// which some position (u, v) with |u|, |v| <= 24 (low half of the word) or 32
// (high half) has an unrounded offset halfway between two integers: sq (C u - S v)
// is an odd multiple of 2^21 iff C u - S v has exactly 21 - k trailing zeros.
// The second coordinate S u + C v takes the same values over the square, and so
// do the bins that quarter turns and the swap of C and S relate.
std::vector<uint32_t> tie_masks(const int16_t *c, const int16_t *s)
{
    std::vector<uint32_t> mask(kBins);
    for (int a = 0; a <= 512; ++a) {
        uint32_t m = 0;
        for (int v = 0; v <= 32; ++v)
            for (int u = -32; u <= 32; ++u) {
                const int x = c[a] * u - s[a] * v;
                if (x == 0) continue;
                const int k = 21 - __builtin_ctz((unsigned)x);
                if (k > 10) continue;                      // (|x| < 2^21, so k >= 1)
                m |= 1u << (16 + k);
                if (v <= kHalf && u >= -kHalf && u <= kHalf) m |= 1u << k;
            }
        for (int q = 0; q < kBins; q += 1024) {
            mask[(a + q) % kBins] = m;
            mask[(1024 - a + q) % kBins] = m;
        }
    }
    return mask;
}

// Gather order of the extraction kernel.  Rounding half away from zero is
// odd, so positions (u, v) and (-u, -v) sample at offsets (ox, oy) and
// (-ox, -oy), and the unrounded offsets of (u + 1, v) are those of (u, v)
// plus s C and s S: the kernel takes positions in chains (u, v), (u + 1, v),
// (-u, -v), (-u - 1, -v), with two rounded offset pairs per chain.  Over
// [-24, 24]^2 (the window and one more row and column, which nothing reads)
// the first members run over rows v = 1..24 with u = -24, -22, .., 22 and 23
// (the last chain overlaps the one before it at (23, v)), and over row 0
// with u = 0, 2, .., 22 and 23: 613 chains, whose mirrors cover the other
// half.  For angle class c (bins 32 c .. 32 c + 31), with (C, S) the cosine
// and sine of the class's middle angle, position (u, v) samples image row
// offset about s (S u + C v) and column offset s (C u - S v) at scale s.
// Chains are sorted by the band floor(4 (S u + C v)) of their first member
// (a quarter row at unit scale), then by its column offset (ties by
// position), so that the lanes of a load sample nearby image bytes and the
// mirrored members form the mirrored band.  Sorted chain k goes to thread
// k % 256, slot k / 256 (0, 1, and 2 for the first 128 threads); the 27 slots
// left over repeat the centre's chain (0, 0), (1, 0).  Entry:
// u & 0xff | (v & 0xff) << 8, laid out as internal.h says.
std::vector<uint16_t> gather_order()
{
    constexpr int kThreads = 2 * 64;
    std::vector<uint16_t> table((size_t)kGatherClasses * kGatherClassEntries, 0);
    std::vector<std::pair<int, int>> units;                      // first members
    for (int v = 0; v <= kHalf; ++v) {
        for (int u = v > 0 ? -kHalf : 0; u < kHalf - 1; u += 2) units.emplace_back(u, v);
        units.emplace_back(kHalf - 1, v);                        // (23, v), (24, v)
    }
    const int n = (int)units.size();                             // 24 * 25 + 13 = 613
    std::vector<int> idx(n);
    std::vector<double> row(n), col(n);
    for (int c = 0; c < kGatherClasses; ++c) {
        const double a = 2.0 * M_PI * (32.0 * c + 16.0) / kBins;
        const double cs = std::cos(a), sn = std::sin(a);
        for (int p = 0; p < n; ++p) {
            const int u = units[p].first, v = units[p].second;
            idx[p] = p;
            row[p] = std::floor(4.0 * (sn * u + cs * v));
            col[p] = cs * u - sn * v;
        }
        std::sort(idx.begin(), idx.end(), [&](int x, int y) {
            if (row[x] != row[y]) return row[x] < row[y];
            if (col[x] != col[y]) return col[x] < col[y];
            return x < y;
        });
        for (int k = 0; k < kThreads * kGatherChains; ++k) {
            const int p = k < n ? idx[k] : 0;                    // units[0]: the centre's chain
            const int u = units[p].first, v = units[p].second;
            const int t = k % 256, m = k / 256;
            const int at = m < 2 ? 2 * t + m : 512 + t;
            table[(size_t)c * kGatherClassEntries + at] = (uint16_t)((u & 0xff) | ((v & 0xff) << 8));
        }
    }
    static_assert(24 * 25 + 13 <= kThreads * kGatherChains, "chains per thread");
    static_assert(kGatherChains == kGatherHeadChains + 1, "one chain after the head");
    return table;
}

// LDS byte offset of the top-left byte of the 7 x 7 patch centred on (r, c):
// the quadword of the copy that holds its first row (see internal.h).
uint32_t patch_offset(int r, int c)
{
    const int x = c - kPatchR, y = r - kPatchR;
    if (x < 8 * kCopyQwords)
        return (uint32_t)((x & 7) * kCopyBytes + y * kCopyRowBytes + 8 * (x >> 3));
    return (uint32_t)(kEdgeBase + 8 * (x - 8 * kCopyQwords) + y * kCopyRowBytes + 8 * (kCopyQwords - 1));
}

// Slot assignment of the extraction kernels: n triplets in slots of 64-lane
// rounds, slot 64 r + l being lane l of round r.  On gfx950 (measured with a
// probe over random and structured address patterns):
//  * a ds_read_b64 is served 32 lanes at a time over 64 dword banks, so its
//    32-lane halves read without conflicts when their quadword addresses
//    differ mod 32;
//  * a ds_read2_b64 is served 16 lanes and one address at a time over 32
//    banks, so its 16-lane quarters read without conflicts when their
//    quadword addresses differ mod 16.
// `group` (lanes served together) and `cols` (quadword banks) name the
// model of the kernel's row reads.  Every patch row read of a lane is its
// patch offset plus a uniform row offset, so the bank of all rows follows
// from the patch offset, and a read costs as many cycles as the largest number
// of a group's lanes on one bank.  A deterministic annealing search over swaps
// puts triplets into lane groups so that these maxima, per group and per patch
// (anchor, companion 1, companion 2), sum to as little as it gets.  The table
// itself sets a floor: a bank that holds more patches than there are groups
// doubles up in some group.  So what helps is to gather the doubled lanes in few
// groups: beside the maxima the objective counts the square root of a group's
// lanes that share a bank with another.  (Sums for the default table: 82 with
// all 512 triplets free, 88 within halves of 256, 103 within quarters of 128;
// 96 is two cycles everywhere, and the sum of squared counts as the second
// objective gives 95 within halves.)
// slot[i] is the slot of triplet i; results never depend on it, only speed
// does.
void search_slots(const uint2 *toff, int n, int group, int cols, uint16_t *slot)
{
    constexpr int kItersPerTriplet = 8000, kMaxGroup = 64;
    constexpr float kMaximum = 100.0f, kShared = 20.0f, kTemperature = 10.0f;
    // One group's lanes by the bank of one patch.
    struct Banks {
        int count[32], banks_with[kMaxGroup + 1], shared, most;
    };
    const int groups = n / group;
    std::vector<std::array<int, 3>> col(n);
    for (int i = 0; i < n; ++i) {
        const uint32_t off[3] = {toff[i].x & 0xffffu, toff[i].x >> 16, toff[i].y};
        for (int k = 0; k < 3; ++k) col[i][k] = (int)((off[k] >> 3) & (uint32_t)(cols - 1));
    }
    std::vector<std::array<Banks, 3>> state(groups);
    auto add = [&](Banks &b, int c) {
        const int v = b.count[c]++;
        --b.banks_with[v];
        ++b.banks_with[v + 1];
        b.shared += v >= 1;
        if (v + 1 > b.most) b.most = v + 1;
    };
    auto remove = [&](Banks &b, int c) {
        const int v = b.count[c]--;
        --b.banks_with[v];
        ++b.banks_with[v - 1];
        b.shared -= v >= 2;
        while (b.banks_with[b.most] == 0) --b.most;
    };
    std::vector<int> group_of(n);
    for (auto &g : state)
        for (Banks &b : g) {
            std::memset(&b, 0, sizeof b);
            b.banks_with[0] = cols;
        }
    for (int i = 0; i < n; ++i) {
        group_of[i] = i / group;
        for (int k = 0; k < 3; ++k) add(state[group_of[i]][k], col[i][k]);
    }
    float root[kMaxGroup + 1];
    for (int v = 0; v <= kMaxGroup; ++v) root[v] = kShared * std::sqrt((float)v);
    auto cost = [&](int g) {
        float c = 0.0f;
        for (const Banks &b : state[g]) c += kMaximum * (float)b.most + root[b.shared];
        return c;
    };
    uint32_t rs = 0x9e3779b9u;
    auto rnd = [&]() {
        rs ^= rs << 13;
        rs ^= rs >> 17;
        rs ^= rs << 5;
        return rs;
    };
    auto swap_members = [&](int i, int j, int g, int h) {
        for (int k = 0; k < 3; ++k) {
            const int a = col[i][k], b = col[j][k];
            if (a == b) continue;
            remove(state[g][k], a);
            add(state[g][k], b);
            remove(state[h][k], b);
            add(state[h][k], a);
        }
        group_of[i] = h;
        group_of[j] = g;
    };
    const int iters = kItersPerTriplet * n;
    for (int it = 0; it < iters; ++it) {
        const int i = (int)(rnd() % (uint32_t)n), j = (int)(rnd() % (uint32_t)n);
        const int g = group_of[i], h = group_of[j];
        if (g == h) continue;
        const float before = cost(g) + cost(h);
        swap_members(i, j, g, h);
        // Worse moves pass with a probability that shrinks to zero over the
        // search.
        const float d = cost(g) + cost(h) - before;
        const float temp = kTemperature * (1.0f - (float)it / (float)iters);
        if (d > 0.0f && !(d < 12.0f * temp && (float)(rnd() & 0xffffu) < 65536.0f * std::exp(-d / temp)))
            swap_members(j, i, g, h);
    }
    // Group g = (64 / group) r + h is lanes group h .. group (h + 1) - 1 of
    // round r.
    const int per_round = 64 / group;
    std::vector<int> fill(groups, 0);
    for (int i = 0; i < n; ++i) {
        const int g = group_of[i];
        slot[i] = (uint16_t)(64 * (g / per_round) + group * (g % per_round) + fill[g]++);
    }
}

// search_slots takes a few hundred milliseconds; its result depends only on
// the offsets, so it is kept per process for each offset table.
void assign_slots(const uint2 *toff, int n, int group, int cols, uint16_t *slot)
{
    static std::mutex mu;
    static std::map<std::vector<uint32_t>, std::vector<uint16_t>> cache;
    std::vector<uint32_t> key;
    key.reserve(2 * n + 3);
    key.push_back((uint32_t)n);
    key.push_back((uint32_t)group);
    key.push_back((uint32_t)cols);
    for (int i = 0; i < n; ++i) {
        key.push_back(toff[i].x);
        key.push_back(toff[i].y);
    }
    {
        std::lock_guard<std::mutex> lock(mu);
        auto it = cache.find(key);
        if (it != cache.end()) {
            std::copy(it->second.begin(), it->second.end(), slot);
            return;
        }
    }
    search_slots(toff, n, group, cols, slot);
    std::lock_guard<std::mutex> lock(mu);
    cache.emplace(std::move(key), std::vector<uint16_t>(slot, slot + n));
}

// The same for `waves` sets of per_wave (at most 256) triplets, each in the
// slots of its own wavefront (the host-code tests check the search in this form).
void assign_slots(const uint2 *toff, int waves, int per_wave, int group, int cols, uint8_t *slot_of)
{
    std::vector<uint16_t> slot(per_wave);
    for (int w = 0; w < waves; ++w) {
        assign_slots(toff + per_wave * w, per_wave, group, cols, slot.data());
        for (int i = 0; i < per_wave; ++i) slot_of[per_wave * w + i] = (uint8_t)slot[i];
    }
}

// Work calls never allocate or wait: a call whose need exceeds the handle's
// workspace fails before it enqueues anything (latch_reserve sizes it).
int check_workspace(latch_handle h, size_t need, const char *call)
{
    if (need <= h->ws_bytes) return LATCH_OK;
    return fail(h, LATCH_EWORKSPACE,
                "%s needs %zu workspace bytes and the handle holds %zu: call latch_reserve first",
                call, need, h->ws_bytes);
}

// Table uploads of handle creation: host arrays copied (or, with a null
// source, zero-filled) on a private stream, waiting for that stream only.
struct Upload {
    void *dst;
    const void *src;
    size_t bytes;
};

hipError_t upload(const Upload *u, int n)
{
    hipStream_t s = nullptr;
    hipError_t e = hipStreamCreateWithFlags(&s, hipStreamNonBlocking);
    for (int i = 0; i < n && e == hipSuccess; ++i)
        e = u[i].src ? hipMemcpyAsync(u[i].dst, u[i].src, u[i].bytes, hipMemcpyHostToDevice, s)
                     : hipMemsetAsync(u[i].dst, 0, u[i].bytes, s);
    if (s) {
        const hipError_t e2 = hipStreamSynchronize(s);
        if (e == hipSuccess) e = e2;
        (void)hipStreamDestroy(s);
    }
    return e;
}

hipEvent_t pool_event(latch_handle h)
{
    if (!h->event_pool.empty()) {
        hipEvent_t e = h->event_pool.back();
        h->event_pool.pop_back();
        return e;
    }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
}

// Runs one launch, bracketed by events when timing is on.
template <typename F>
hipError_t timed_launch(latch_handle h, const char *name, hipStream_t stream, F &&launch)
{
    if (!h->timing) return launch();
    latch_ctx::Timed t{name, pool_event(h), pool_event(h)};
    if (!t.start || !t.stop) return hipErrorOutOfMemory;
    hipError_t e = hipEventRecord(t.start, stream);
    if (e != hipSuccess) return e;
    e = launch();
    if (e != hipSuccess) return e;
    e = hipEventRecord(t.stop, stream);
    if (e != hipSuccess) return e;
    h->timed.push_back(t);
    return hipSuccess;
}

void release_timed(latch_handle h)
{
    for (auto &t : h->timed) {
        h->event_pool.push_back(t.start);
        h->event_pool.push_back(t.stop);
    }
    h->timed.clear();
}

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Bucket of a row count in the tuning's path table.
int size_bucket(int64_t n)
{
    int b = 0;
    while (b < 7 && (n >> (2 * (b + 1))) > 0) ++b;
    return b;
}

void default_tuning(latch_tuning *t)
{
    std::memset(t, 0, sizeof *t);
    std::memset(t->path, LATCH_PATH_MFMA_FP4, sizeof t->path);
    t->batch_path = LATCH_PATH_MFMA_FP4;
    t->fp4_query_blocks = 3;
    t->mfma_groups_per_cu = 2;
    t->popcount_groups_per_cu = 8;
    t->batch_groups_per_cu = 2;
}

KnnShape knn_shape(const latch_tuning &t)
{
    KnnShape s;
    s.fp4_query_blocks = t.fp4_query_blocks;
    s.batch_groups_per_cu = t.batch_groups_per_cu;
    return s;
}

SplitKernel split_kernel(int path)
{
    return path == LATCH_PATH_MFMA       ? SplitKernel::kMfmaI8
           : path == LATCH_PATH_MFMA_FP4 ? SplitKernel::kMfmaFp4
                                         : SplitKernel::kPopcount;
}

// Split plan of a single-pair call for query groups of `group`.  The base
// choice fills the GPU's workgroup slots once (slots / query groups splits),
// raised to what the split-local index needs and capped at 2 tiles per split (up
// to 8 tiles, one split: the second launch takes longer than the tiles).  With caps
// of 8 and 4 tiles a call of 2000 x 2000 took 10.0 and 8.0 us instead of 7.4,
// 1000 x 1000 10.2 and 8.0 instead of 6.8.  Work items (query group, split) then
// run in rounds of `slots`, each costing about its
// split's tiles; when the base count leaves the last round partly empty (the
// index raised it, or the query groups alone exceed the slots), a larger
// count can spread the same tiles over fuller rounds.  Over counts up to 4x
// the base (at most 512 more), within `partial_cap` bytes of partials, the
// smallest count whose rounds x tiles per split is within 2% of the least is
// taken (more splits also mean more merge work and partials), unless the
// base itself is.
struct SplitCount {
    int64_t tiles_per_split, rounds;
    int nsplit;
};

SplitCount count_splits(int64_t nq, int64_t tiles, int64_t group, int64_t slots, int64_t max_rows,
                        size_t partial_cap)
{
    const int64_t qgroups = (nq + group - 1) / group;
    int64_t nsplit = qgroups >= slots ? 1 : slots / qgroups;
    const int64_t max_by_size = tiles <= 8 ? 1 : (tiles + 1) / 2;
    if (nsplit > max_by_size) nsplit = max_by_size;
    const int64_t max_by_cap = (int64_t)(partial_cap / ((size_t)nq * 2 * sizeof(uint64_t)));
    if (nsplit > max_by_cap) nsplit = max_by_cap;
    if (nsplit < 1) nsplit = 1;
    const int64_t max_tiles = max_rows / kTileRows;
    const int64_t min_by_index = (tiles + max_tiles - 1) / max_tiles;
    if (nsplit < min_by_index) nsplit = min_by_index;
    if (nsplit > kMaxSplits) nsplit = kMaxSplits;
    auto tiles_per = [&](int64_t n) { return (tiles + n - 1) / n; };
    auto rounds = [&](int64_t n) {
        const int64_t tps = tiles_per(n), used = (tiles + tps - 1) / tps;
        return (qgroups * used + slots - 1) / slots;
    };
    auto cost = [&](int64_t n) { return rounds(n) * tiles_per(n); };
    const int64_t n_hi = std::min({(int64_t)kMaxSplits, std::max(nsplit, max_by_size), 4 * nsplit + 8,
                                   nsplit + 512});
    const int64_t top = std::min(n_hi, std::max(nsplit, max_by_cap));
    // The cost depends on the tiles per split alone: only the smallest count of each is
    // tried (a few dozen instead of hundreds of counts, each some divisions long).
    auto each_count = [&](auto stop) {
        for (int64_t n = nsplit; tiles_per(n) > 1;) {
            const int64_t fewer = tiles_per(n) - 1;
            n = (tiles + fewer - 1) / fewer;
            if (n > top || stop(n)) break;
        }
    };
    const int64_t base_cost = cost(nsplit);
    int64_t least = base_cost;
    each_count([&](int64_t n) {
        least = std::min(least, cost(n));
        return false;
    });
    if (base_cost * 50 > least * 51) {
        int64_t chosen = nsplit;
        each_count([&](int64_t n) {
            if (cost(n) * 50 > least * 51) return false;
            chosen = n;
            return true;
        });
        nsplit = chosen;
    }
    const int64_t tps = tiles_per(nsplit);
    return {tps, rounds(nsplit), (int)((tiles + tps - 1) / tps)};
}

// The plan: splits, and for the FP4 path the 32-query blocks per wavefront, 2 or (if
// the tuning has 3) 3.  A tile costs a workgroup of 2 blocks 0.78 of one of 3
// (more per query: its staging and fragment reads serve fewer), and a work item
// starts and ends in the time of 5 and 6.5 such tiles: fewer blocks win where the
// splits are short or where 3 pad the queries more.  With 3 and 2 blocks: 1000 x 1000
// 7.5 and 6.8 us, 4000 x 3000 11.0 and 9.7, 500 x 1,000,000 126 and 99, 1200 x 200,000
// 56.0 and 53.6, 9973 x 10007 24.6 and 25.6, 3000 x 10,000 13.1 and 13.1.
KnnPlan plan_knn(int64_t nq, int64_t nt, int path, int num_cus, const latch_tuning &tune,
                 size_t partial_cap)
{
    KnnPlan p;
    p.nq = nq;
    p.nt = nt;
    p.query_blocks = tune.fp4_query_blocks;
    p.nsplit = 1;
    p.split_rows = kTileRows;
    const int64_t tiles = (nt + kTileRows - 1) / kTileRows;
    if (tiles == 0) return p;
    const SplitKernel which = split_kernel(path);
    const bool fp4 = which == SplitKernel::kMfmaFp4;
    const int64_t slots = (int64_t)num_cus * (path == LATCH_PATH_POPCOUNT ? tune.popcount_groups_per_cu
                                                                        : tune.mfma_groups_per_cu);
    const int64_t max_rows = fp4 ? kFp4MaxSplitRows : kMaxSplitRows;
    auto splits = [&](int blocks) {
        return count_splits(nq, tiles, queries_per_group(which, blocks), slots, max_rows, partial_cap);
    };
    SplitCount c = splits(p.query_blocks);
    if (fp4 && p.query_blocks == 3) {
        const SplitCount two = splits(2);
        if (two.rounds * (78 * two.tiles_per_split + 500) < c.rounds * (100 * c.tiles_per_split + 650)) {
            c = two;
            p.query_blocks = 2;
        }
    }
    p.split_rows = c.tiles_per_split * kTileRows;
    p.nsplit = c.nsplit;
    return p;
}

// The split kernel a single-pair call runs: LATCH_PATH_AUTO resolved by the
// tuning table, and the FP4 path, whose keys hold a 14-bit split-local
// index, replaced by the int8 one (identical results) when the train rows
// would need more than the 65,535 splits a grid dimension allows.
int resolve_path(latch_handle h, int path, int64_t nq, int64_t nt)
{
    if (path == LATCH_PATH_AUTO) path = h->tuning.path[size_bucket(nq)][size_bucket(nt)];
    if (path == LATCH_PATH_MFMA_FP4 && nt > kMaxSplits * kFp4MaxSplitRows) path = LATCH_PATH_MFMA;
    return path;
}

// Partial top-2 keys of a split plan: 16 bytes per (split, query).
size_t knn_workspace_bytes(const KnnPlan &p)
{
    return p.nsplit > 1 ? align_up((size_t)p.nsplit * p.nq * 2 * sizeof(uint64_t), 256) : 0;
}

// Detection: survivor masks (one u64 per row and 64-column tile), the first
// output slot of every row, the per-(row, tile) survivor counts (rows padded
// to 16 bytes) and the count on entry.
struct DetectLayout {
    size_t mask_bytes, first_bytes, count_bytes, total;
    int count_stride;
};

DetectLayout detect_layout(int height, int width)
{
    DetectLayout l;
    l.mask_bytes = align_up((size_t)height * ((width + 63) / 64) * sizeof(uint64_t), 256);
    l.first_bytes = align_up((size_t)height * sizeof(int64_t), 256);
    l.count_stride = (int)align_up((size_t)(width + 63) / 64, 16);
    l.count_bytes = align_up((size_t)height * l.count_stride, 256);
    l.total = l.mask_bytes + l.first_bytes + l.count_bytes + sizeof(int64_t);
    return l;
}

// Workspace of a batched matching: the pairs' state, the header and the unit map of
// undivided pairs.
struct BatchLayout {
    int64_t item_capacity;
    size_t info_bytes, total;
};

BatchLayout batch_layout(int n_pairs, int64_t out_rows)
{
    BatchLayout l;
    l.item_capacity = out_rows / 256 + n_pairs + 1;
    l.info_bytes = align_up((size_t)n_pairs * sizeof(PairInfo), 256);
    l.total = l.info_bytes + 256 + align_up((size_t)l.item_capacity * sizeof(int32_t), 256);
    return l;
}

size_t batch_workspace_bytes(int n_pairs, int64_t out_rows) { return batch_layout(n_pairs, out_rows).total; }

// What dividing train ranges needs beyond the workspace: the slots' keys and counts,
// and a unit map with room for their parts.  A handle holds it for its calls from its
// creation on and a plan its own, so that no call depends on how large a workspace
// earlier ones left.
struct PartMemory {
    int64_t slots, units;
    size_t key_bytes, done_bytes, total;
};

PartMemory part_memory(int64_t slots, int64_t units)
{
    PartMemory m;
    m.slots = slots;
    m.units = units;
    m.key_bytes = (size_t)slots * kBatchSlotQueries * sizeof(PartKeys);
    m.done_bytes = align_up((size_t)slots * sizeof(PartCount), 256);
    m.total = m.key_bytes + m.done_bytes + (size_t)units * sizeof(int32_t);
    return m;
}

// A handle's: 2^20 units, so batches of which out_rows / 256 + n_pairs is below 1,017,000.
// (Larger ones, of a thousand rounds of units, are not divided; a plan's memory fits its
// batch.)
PartMemory handle_parts() { return part_memory(kBatchMaxSlots, 1 << 20); }

PartMemory plan_parts(int n_pairs, int64_t out_rows)
{
    const int64_t items = batch_layout(n_pairs, out_rows).item_capacity;
    const int64_t slots = std::min(items, kBatchMaxSlots);
    return part_memory(slots, items + slots * (kBatchMaxParts - 1));
}

// Arguments of the batched matcher with its workspace (batch_workspace_bytes bytes) at
// `ws` and the memory of parts `m` at `parts` (nullptr: no train range is divided).
BatchArgs batch_args(latch_handle h, uint8_t *ws, uint8_t *parts, const PartMemory &m,
                     const uint32_t *query_dev, int64_t query_rows, const uint32_t *train_dev,
                     int64_t train_rows, const latch_pair *pairs_dev, int n_pairs, int k, float ratio,
                     int32_t *idx_dev, int32_t *dist_dev, uint8_t *accept_dev, int64_t out_rows,
                     int path)
{
    const BatchLayout l = batch_layout(n_pairs, out_rows);
    BatchArgs a;
    a.query = query_dev;
    a.train = train_dev;
    a.query_rows = query_rows;
    a.train_rows = train_rows;
    a.out_rows = out_rows;
    a.pairs = reinterpret_cast<const PairEntry *>(pairs_dev);
    a.n_pairs = n_pairs;
    a.item_capacity = l.item_capacity;
    a.info = reinterpret_cast<PairInfo *>(ws);
    a.state = reinterpret_cast<BatchState *>(ws + l.info_bytes);
    a.unit_pair = reinterpret_cast<int32_t *>(ws + l.info_bytes + 256);
    a.slots = BatchSlots{nullptr, nullptr, 0};
    if (parts && l.item_capacity + m.slots * (kBatchMaxParts - 1) <= m.units) {
        a.slots = BatchSlots{reinterpret_cast<PartKeys *>(parts),
                             reinterpret_cast<PartCount *>(parts + m.key_bytes), (int)m.slots};
        a.unit_pair = reinterpret_cast<int32_t *>(parts + m.key_bytes + m.done_bytes);
    }
    a.k = k;
    a.ratio = ratio;
    a.idx = idx_dev;
    a.dist = dist_dev;
    a.accept = accept_dev;
    a.flags = h->flags_dev;
    a.num_cus = h->num_cus;
    a.kind = split_kernel(path);
    a.shape = knn_shape(h->tuning);
    return a;
}

ExtractArgs batch_extract_args(latch_handle h, const latch_image *images_dev, int n_images,
                               const int32_t *image_id_dev, const latch_keypoint *kps_dev,
                               int64_t max_kps, const int64_t *n_kps_dev, uint32_t *desc_dev)
{
    ExtractArgs a;
    a.img = nullptr;
    a.height = a.width = a.pitch = 0;
    a.table = reinterpret_cast<const ImageEntry *>(images_dev);
    a.image_id = image_id_dev;
    a.n_images = n_images;
    a.kps = reinterpret_cast<const float4 *>(kps_dev);
    a.n = max_kps;
    a.n_dev = n_kps_dev;
    a.rot = h->rot_dev;
    a.trip_off = h->trip_off_dev;
    a.bit_of = h->bit_of_dev;
    a.gather = h->gather_dev;
    a.desc = desc_dev;
    a.flags = h->flags_dev;
    a.num_cus = h->num_cus;
    a.window = h->window;
    a.wtrip_off = h->wtrip_dev;
    a.wbit_of = h->wbit_of_dev;
    a.weights = h->weights;
    return a;
}

// The handle's extraction kernel: the weighted one for a geometry handle.
hipError_t run_extract(const ExtractArgs &a, hipStream_t stream)
{
    return a.window ? launch_extract_weighted(a, stream) : launch_extract(a, stream);
}

// Workspace of a batched extraction's spatial order (0: extracted as given).
constexpr int kOrderMaxImages = 1 << 16;

size_t extract_batch_workspace(latch_handle h, int n_images, int64_t max_kps)
{
    if (h->window || max_kps < kOrderMinKeypoints || n_images < 1 || n_images > kOrderMaxImages)
        return 0;
    return order_layout(n_images, max_kps).total;
}

// A batched extraction: the order's kernels (when the batch has one, in
// workspace `ws`), then the extraction kernel.  A plan's capture records no
// timing events (timed = false).
hipError_t run_extract_batch(latch_handle h, ExtractArgs a, uint8_t *ws, hipStream_t stream,
                             bool timed)
{
    auto launch = [&](const char *name, auto &&f) {
        return timed ? timed_launch(h, name, stream, f) : f();
    };
    if (extract_batch_workspace(h, a.n_images, a.n) > 0) {
        const hipError_t e = launch("extract_order", [&] { return launch_order(a, ws, stream); });
        if (e != hipSuccess) return e;
        a.order = reinterpret_cast<const int32_t *>(ws + order_layout(a.n_images, a.n).order);
    }
    return launch("extract", [&] { return run_extract(a, stream); });
}

// Scratch of hamming_knn_noalloc: a static device array, one copy per GPU
// the library runs on, held until the process ends.  Host code never names
// it directly (on the host `scratch` is only a stand-in symbol): it uses the
// device address hipGetSymbolAddress gives, looked up once per device.
static __device__ __align__(256) uint8_t scratch[LATCH_NOALLOC_SCRATCH_BYTES];

std::mutex scratch_mutex;
std::map<int, uint8_t *> scratch_by_device;

// Address of `device`'s copy of the scratch array; `device` must be current.
hipError_t scratch_address(int device, uint8_t **out)
{
    std::lock_guard<std::mutex> lock(scratch_mutex);
    auto it = scratch_by_device.find(device);
    if (it == scratch_by_device.end()) {
        void *ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!ptr) return hipErrorInvalidSymbol;
        it = scratch_by_device.emplace(device, static_cast<uint8_t *>(ptr)).first;
    }
    *out = it->second;
    return hipSuccess;
}

// A handle with the rotation table and the error word (no triplet data).
int create_base(latch_ctx **out)
{
    latch_ctx *h = new latch_ctx();
    default_tuning(&h->tuning);
    hipError_t e = hipGetDevice(&h->device);
    if (e == hipSuccess)
        e = hipDeviceGetAttribute(&h->num_cus, hipDeviceAttributeMultiprocessorCount, h->device);
    if (e == hipSuccess && h->num_cus >= 1) e = scratch_address(h->device, &h->scratch);
    if (e != hipSuccess || h->num_cus < 1) {
        delete h;
        return LATCH_EDEVICE;
    }
    int16_t c[kBins], s[kBins];
    rotation_table(c, s);
    const std::vector<uint32_t> ties = tie_masks(c, s);
    int2 rot[kBins];
    for (int a = 0; a < kBins; ++a)
        rot[a] = make_int2((int)((uint16_t)c[a] | (uint32_t)(uint16_t)s[a] << 16), (int)ties[a]);
    if ((e = hipMalloc((void **)&h->rot_dev, sizeof rot)) == hipSuccess &&
        (e = hipMalloc((void **)&h->parts, handle_parts().total)) == hipSuccess &&
        (e = hipMalloc((void **)&h->flags_dev, sizeof(uint32_t))) == hipSuccess) {
        const Upload u[2] = {{h->rot_dev, rot, sizeof rot}, {h->flags_dev, nullptr, sizeof(uint32_t)}};
        e = upload(u, 2);
    }
    if (e != hipSuccess) {
        const int rc = e == hipErrorOutOfMemory ? LATCH_ENOMEM : LATCH_EDEVICE;
        latch_destroy(h);
        return rc;
    }
    *out = h;
    return LATCH_OK;
}

// hamming_knn and hamming_knn_noalloc: the same checks and launches; the
// split partials go to the handle's workspace or to the static scratch.
int knn_call(latch_handle h, const uint32_t *query_dev, int64_t nq, const uint32_t *train_dev,
             int64_t nt, int k, float ratio, int32_t *idx_dev, int32_t *dist_dev,
             uint8_t *accept_dev, int path, hipStream_t stream, bool noalloc)
{
    if (!h) return LATCH_EINVAL;
    h->last_error.clear();
    if (nq < 0 || nq > LATCH_MAX_ROWS || nt < 0 || nt > LATCH_MAX_ROWS)
        return fail(h, LATCH_EINVAL, "sizes nq = %lld, nt = %lld out of [0, 2^31)", (long long)nq,
                    (long long)nt);
    if (k != 1 && k != 2) return fail(h, LATCH_ERANGE, "k = %d (must be 1 or 2)", k);
    if (!(ratio > 0.0f && ratio <= 1.0f))
        return fail(h, LATCH_ERANGE, "ratio = %g (must be in (0, 1])", (double)ratio);
    if (path < LATCH_PATH_AUTO || path > LATCH_PATH_MFMA_FP4)
        return fail(h, LATCH_EINVAL, "unknown path %d", path);
    if (nq == 0) return LATCH_OK;
    if (!query_dev || !idx_dev || !dist_dev || (nt > 0 && !train_dev))
        return fail(h, LATCH_EINVAL, "null buffer");
    path = resolve_path(h, path, nq, nt);

    KnnSplitArgs a;
    a.query = query_dev;
    a.train = train_dev;
    a.plan = plan_knn(nq, nt, path, h->num_cus, h->tuning,
                      noalloc ? (size_t)LATCH_NOALLOC_SCRATCH_BYTES : SIZE_MAX);
    a.partial = nullptr;
    a.k = k;
    a.ratio = ratio;
    a.idx = idx_dev;
    a.dist = dist_dev;
    a.accept = accept_dev;
    if (a.plan.nsplit > 1) {
        const size_t need = knn_workspace_bytes(a.plan);
        if (noalloc) {
            // Every (split, query) partial is written by the split kernel
            // before the merge reads it, so nothing needs clearing.
            if (need > LATCH_NOALLOC_SCRATCH_BYTES)
                return fail(h, LATCH_ERANGE,
                            "hamming_knn_noalloc needs %zu scratch bytes (%d train splits x %lld "
                            "queries) and its static scratch holds %zu",
                            need, a.plan.nsplit, (long long)nq, (size_t)LATCH_NOALLOC_SCRATCH_BYTES);
            a.partial = reinterpret_cast<uint64_t *>(h->scratch);
        } else {
            const int rc = check_workspace(h, need, "hamming_knn");
            if (rc != LATCH_OK) return rc;
            a.partial = reinterpret_cast<uint64_t *>(h->ws);
        }
    }
    const SplitKernel which = split_kernel(path);
    const char *name = which == SplitKernel::kMfmaI8    ? "knn_mfma"
                       : which == SplitKernel::kMfmaFp4 ? "knn_fp4"
                                                        : "knn_popcount";
    // The allocation-free call records no timing events (creating one may allocate).
    auto launch = [&](const char *what, auto &&f) {
        return noalloc ? f() : timed_launch(h, what, stream, f);
    };
    hipError_t e = launch(name, [&] { return launch_knn_split(a, which, stream); });
    if (e != hipSuccess) return hip_fail(h, e, name);
    if (a.plan.nsplit > 1) {
        e = launch("knn_merge", [&] { return launch_knn_merge(a, stream); });
        if (e != hipSuccess) return hip_fail(h, e, "merge launch");
    }
    return LATCH_OK;
}

}  // namespace

struct latch_plan_ctx {
    latch_handle h = nullptr;
    uint8_t *ws = nullptr;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
};

extern "C" {

const char *latch_version(void) { return "latch-gfx950 0.2"; }

int latch_rotation_table(int16_t *cos_q14, int16_t *sin_q14)
{
    if (!cos_q14 || !sin_q14) return LATCH_EINVAL;
    rotation_table(cos_q14, sin_q14);
    return LATCH_OK;
}

int latch_create(latch_handle *out, const uint8_t *triplets_host)
{
    if (!out || !triplets_host) return LATCH_EINVAL;
    *out = nullptr;
    for (int i = 0; i < kTriplets * 6; ++i)
        if (triplets_host[i] < kPatchR || triplets_host[i] > kWin - 1 - kPatchR) return LATCH_ERANGE;

    latch_ctx *h = nullptr;
    int rc = create_base(&h);
    if (rc != LATCH_OK) return rc;
    uint2 toff[kTriplets];
    for (int t = 0; t < kTriplets; ++t) {
        const uint8_t *tr = triplets_host + 6 * t;
        toff[t].x = patch_offset(tr[0], tr[1]) | (patch_offset(tr[2], tr[3]) << 16);
        toff[t].y = patch_offset(tr[4], tr[5]);
    }
    // Triplets by slot, and per (wavefront w, lane l) the output bits of its
    // slots 128 w + l and 128 w + 64 + l.
    uint16_t slot_of[kTriplets];
    assign_slots(toff, kTriplets, 32, 32, slot_of);   // row reads: ds_read_b64
    uint2 toff_slot[kTriplets];
    uint32_t bit_of[kExtractWaves * 64] = {};
    for (int t = 0; t < kTriplets; ++t) {
        const int s = slot_of[t], w = s >> 7, r = (s >> 6) & 1, l = s & 63;
        toff_slot[s] = toff[t];
        bit_of[64 * w + l] |= (uint32_t)t << (16 * r);
    }
    uint2 doff[kTriplets];
    for (int t = 0; t < kTriplets; ++t) {
        const uint8_t *tr = triplets_host + 6 * t;
        doff[t] = make_uint2(dense_patch_offset(tr[0], tr[1]) | (dense_patch_offset(tr[2], tr[3]) << 16),
                             dense_patch_offset(tr[4], tr[5]));
    }
    const std::vector<uint16_t> order = gather_order();
    const size_t order_bytes = order.size() * sizeof(uint16_t);
    hipError_t e;
    if ((e = hipMalloc((void **)&h->trip_off_dev, sizeof toff_slot)) == hipSuccess &&
        (e = hipMalloc((void **)&h->bit_of_dev, sizeof bit_of)) == hipSuccess &&
        (e = hipMalloc((void **)&h->dense_off_dev, sizeof doff)) == hipSuccess &&
        (e = hipMalloc((void **)&h->gather_dev, order_bytes)) == hipSuccess) {
        const Upload u[4] = {{h->dense_off_dev, doff, sizeof doff},
                             {h->trip_off_dev, toff_slot, sizeof toff_slot},
                             {h->bit_of_dev, bit_of, sizeof bit_of},
                             {h->gather_dev, order.data(), order_bytes}};
        e = upload(u, 4);
    }
    if (e != hipSuccess) {
        rc = e == hipErrorOutOfMemory ? LATCH_ENOMEM : LATCH_EDEVICE;
        latch_destroy(h);
        return rc;
    }
    *out = h;
    return LATCH_OK;
}

int latch_create_geometry(latch_handle *out, const uint8_t *triplets_host, int window, int patch,
                          const uint8_t *weights_host)
{
    if (!out || !triplets_host) return LATCH_EINVAL;
    *out = nullptr;
    if ((window != 48 && window != 64) || (patch != 7 && patch != 8)) return LATCH_ERANGE;
    uint8_t w[64];
    bool unit = true;
    for (int i = 0; i < patch * patch; ++i) {
        w[i] = weights_host ? weights_host[i] : 1;
        if (w[i] > 128) return LATCH_ERANGE;
        unit = unit && w[i] == 1;
    }
    for (int i = 0; i < kTriplets * 6; ++i) {
        const int first = triplets_host[i] - patch / 2;
        if (first < 0 || first + patch > window) return LATCH_ERANGE;
    }
    if (window == kWin && patch == 2 * kPatchR + 1 && unit) return latch_create(out, triplets_host);

    latch_ctx *h = nullptr;
    int rc = create_base(&h);
    if (rc != LATCH_OK) return rc;
    h->window = window;
    // 7 x 7 patches run as 8 x 8 ones whose last row and column weigh 0.
    for (int r = 0; r < 8; ++r)
        for (int i = 0; i < 4; ++i) {
            const int c0 = 2 * i, c1 = 2 * i + 1;
            const uint32_t lo = (r < patch && c0 < patch) ? w[r * patch + c0] : 0u;
            const uint32_t hi = (r < patch && c1 < patch) ? w[r * patch + c1] : 0u;
            h->weights.pair[4 * r + i] = lo | (hi << 16);
        }
    uint2 toff[kTriplets];
    for (int t = 0; t < kTriplets; ++t) {
        const uint8_t *tr = triplets_host + 6 * t;
        uint32_t o[3];
        for (int k = 0; k < 3; ++k)
            o[k] = weighted_patch_offset(window, tr[2 * k] - patch / 2, tr[2 * k + 1] - patch / 2);
        toff[t] = make_uint2(o[0] | (o[1] << 16), o[2]);
    }
    // Bank-aware slots over all triplets (row reads: ds_read_b64).
    uint16_t slot_of[kTriplets];
    assign_slots(toff, kTriplets, 32, 32, slot_of);
    uint2 toff_slot[kTriplets];
    uint32_t bit_of[kTriplets];
    for (int t = 0; t < kTriplets; ++t) {
        toff_slot[slot_of[t]] = toff[t];
        bit_of[slot_of[t]] = (uint32_t)t;
    }
    hipError_t e;
    if ((e = hipMalloc((void **)&h->wtrip_dev, sizeof toff_slot)) == hipSuccess &&
        (e = hipMalloc((void **)&h->wbit_of_dev, sizeof bit_of)) == hipSuccess) {
        const Upload u[2] = {{h->wtrip_dev, toff_slot, sizeof toff_slot},
                             {h->wbit_of_dev, bit_of, sizeof bit_of}};
        e = upload(u, 2);
    }
    if (e != hipSuccess) {
        rc = e == hipErrorOutOfMemory ? LATCH_ENOMEM : LATCH_EDEVICE;
        latch_destroy(h);
        return rc;
    }
    *out = h;
    return LATCH_OK;
}

void latch_destroy(latch_handle h)
{
    if (!h) return;
    (void)hipDeviceSynchronize();
    if (h->rot_dev) (void)hipFree(h->rot_dev);
    if (h->trip_off_dev) (void)hipFree(h->trip_off_dev);
    if (h->bit_of_dev) (void)hipFree(h->bit_of_dev);
    if (h->gather_dev) (void)hipFree(h->gather_dev);
    if (h->flags_dev) (void)hipFree(h->flags_dev);
    if (h->wtrip_dev) (void)hipFree(h->wtrip_dev);
    if (h->wbit_of_dev) (void)hipFree(h->wbit_of_dev);
    if (h->dense_off_dev) (void)hipFree(h->dense_off_dev);
    if (h->ws) (void)hipFree(h->ws);
    if (h->parts) (void)hipFree(h->parts);
    release_timed(h);
    for (hipEvent_t e : h->event_pool) (void)hipEventDestroy(e);
    delete h;
}

const char *latch_last_error(latch_handle h) { return h ? h->last_error.c_str() : "null handle"; }

int latch_extract(latch_handle h, const uint8_t *img_dev, int height, int width, int pitch,
                  const latch_keypoint *kps_dev, int64_t n_kps, uint32_t *desc_dev,
                  hipStream_t stream)
{
    if (!h) return LATCH_EINVAL;
    h->last_error.clear();
    if (n_kps < 0 || n_kps > LATCH_MAX_ROWS)
        return fail(h, LATCH_EINVAL, "n_kps = %lld out of [0, 2^31)", (long long)n_kps);
    if (height < 1 || width < 1 || pitch < width)
        return fail(h, LATCH_EINVAL, "bad image shape %d x %d, pitch %d", height, width, pitch);
    if ((int64_t)height * pitch > (int64_t)INT32_MAX || height >= (1 << 23) || pitch >= (1 << 23))
        return fail(h, LATCH_EINVAL, "image of %d rows x %d pitch: need rows, pitch < 2^23 and "
                    "rows * pitch < 2^31", height, pitch);
    if (n_kps == 0) return LATCH_OK;
    if (!img_dev || !kps_dev || !desc_dev) return fail(h, LATCH_EINVAL, "null buffer");
    ExtractArgs a;
    a.img = img_dev;
    a.height = height;
    a.width = width;
    a.pitch = pitch;
    a.table = nullptr;
    a.image_id = nullptr;
    a.n_images = 0;
    a.kps = reinterpret_cast<const float4 *>(kps_dev);
    a.n = n_kps;
    a.n_dev = nullptr;
    a.rot = h->rot_dev;
    a.trip_off = h->trip_off_dev;
    a.bit_of = h->bit_of_dev;
    a.gather = h->gather_dev;
    a.desc = desc_dev;
    a.flags = h->flags_dev;
    a.num_cus = h->num_cus;
    a.window = h->window;
    a.wtrip_off = h->wtrip_dev;
    a.wbit_of = h->wbit_of_dev;
    a.weights = h->weights;
    hipError_t e = timed_launch(h, "extract", stream, [&] { return run_extract(a, stream); });
    return e == hipSuccess ? LATCH_OK : hip_fail(h, e, "extract launch");
}

int latch_extract_batch(latch_handle h, const latch_image *images_dev, int n_images,
                        const int32_t *image_id_dev, const latch_keypoint *kps_dev, int64_t max_kps,
                        const int64_t *n_kps_dev, uint32_t *desc_dev, hipStream_t stream)
{
    if (!h) return LATCH_EINVAL;
    h->last_error.clear();
    if (max_kps < 0 || max_kps > LATCH_MAX_ROWS)
        return fail(h, LATCH_EINVAL, "max_kps = %lld out of [0, 2^31)", (long long)max_kps);
    if (n_images < 0) return fail(h, LATCH_EINVAL, "n_images = %d < 0", n_images);
    if (max_kps == 0) return LATCH_OK;
    if (!images_dev || !image_id_dev || !kps_dev || !desc_dev || n_images == 0)
        return fail(h, LATCH_EINVAL, "null buffer or empty image table");
    const int rc = check_workspace(h, extract_batch_workspace(h, n_images, max_kps),
                                   "latch_extract_batch");
    if (rc != LATCH_OK) return rc;
    const ExtractArgs a = batch_extract_args(h, images_dev, n_images, image_id_dev, kps_dev,
                                             max_kps, n_kps_dev, desc_dev);
    const hipError_t e = run_extract_batch(h, a, h->ws, stream, true);
    return e == hipSuccess ? LATCH_OK : hip_fail(h, e, "batched extract launch");
}

int latch_extract_dense(latch_handle h, const uint8_t *img_dev, int height, int width, int pitch,
                        int x0, int y0, int gw, int gh, uint32_t *desc_dev, hipStream_t stream)
{
    if (!h) return LATCH_EINVAL;
    h->last_error.clear();
    if (!h->dense_off_dev)
        return fail(h, LATCH_EINVAL, "dense extraction needs a handle of the default geometry");
    if (height < 1 || width < 1 || pitch < width || height >= (1 << 23) || pitch >= (1 << 23) ||
        (int64_t)height * pitch > (int64_t)INT32_MAX)
        return fail(h, LATCH_EINVAL, "image %d x %d, pitch %d outside the limits", height, width, pitch);
    if (gw < 0 || gh < 0 || (int64_t)gw * gh > LATCH_MAX_ROWS || x0 < -(1 << 24) || y0 < -(1 << 24) ||
        (int64_t)x0 + gw > (1 << 24) || (int64_t)y0 + gh > (1 << 24))
        return fail(h, LATCH_ERANGE, "region (%d, %d) + %d x %d outside the limits", x0, y0, gw, gh);
    if (gw == 0 || gh == 0) return LATCH_OK;
    if (!img_dev || !desc_dev) return fail(h, LATCH_EINVAL, "null buffer");
    DenseArgs a;
    a.img = img_dev;
    a.height = height;
    a.width = width;
    a.pitch = pitch;
    a.x0 = x0;
    a.y0 = y0;
    a.gw = gw;
    a.gh = gh;
    a.toff = h->dense_off_dev;
    a.desc = desc_dev;
    const hipError_t e =
        timed_launch(h, "dense_extract", stream, [&] { return launch_dense_extract(a, stream); });
    return e == hipSuccess ? LATCH_OK : hip_fail(h, e, "dense extract launch");
}

int hamming_knn_window(latch_handle h, const uint32_t *query_dev, const uint32_t *train_dev, int gw,
                       int gh, int radius, int k, float ratio, int32_t *idx_dev, int32_t *dist_dev,
                       uint8_t *accept_dev, hipStream_t stream)
{
    if (!h) return LATCH_EINVAL;
    h->last_error.clear();
    if (gw < 0 || gh < 0 || (int64_t)gw * gh > LATCH_MAX_ROWS)
        return fail(h, LATCH_EINVAL, "grid %d x %d", gw, gh);
    if (radius < 0 || radius > kDenseMaxRadius)
        return fail(h, LATCH_ERANGE, "radius %d (must be in [0, %d])", radius, kDenseMaxRadius);
    if (k != 1 && k != 2) return fail(h, LATCH_ERANGE, "k = %d (must be 1 or 2)", k);
    if (!(ratio > 0.0f && ratio <= 1.0f))
        return fail(h, LATCH_ERANGE, "ratio = %g (must be in (0, 1])", (double)ratio);
    if (gw == 0 || gh == 0) return LATCH_OK;
    if (!query_dev || !train_dev || !idx_dev || !dist_dev) return fail(h, LATCH_EINVAL, "null buffer");
    DenseMatchArgs a;
    a.query = query_dev;
    a.train = train_dev;
    a.gw = gw;
    a.gh = gh;
    a.radius = radius;
    a.k = k;
    a.ratio = ratio;
    a.idx = idx_dev;
    a.dist = dist_dev;
    a.accept = accept_dev;
    a.num_cus = h->num_cus;
    const hipError_t e =
        timed_launch(h, "knn_window", stream, [&] { return launch_dense_match(a, stream); });
    return e == hipSuccess ? LATCH_OK : hip_fail(h, e, "dense match launch");
}

int latch_detect(latch_handle h, const uint8_t *img_dev, int height, int width, int pitch,
                 int threshold, latch_keypoint *kps_dev, int64_t max_kps, int64_t *n_kps_dev,
                 int32_t *image_id_dev, int32_t image_index, hipStream_t stream)
{
    if (!h) return LATCH_EINVAL;
    h->last_error.clear();
    if (!img_dev || !n_kps_dev || (max_kps > 0 && !kps_dev))
        return fail(h, LATCH_EINVAL, "null buffer");
    if (height < 1 || width < 1 || pitch < width || height >= (1 << 23) || pitch >= (1 << 23) ||
        (int64_t)height * pitch > (int64_t)0x7fffffff)
        return fail(h, LATCH_EINVAL, "image %d x %d, pitch %d outside the limits", height, width,
                    pitch);
    if (threshold < 0 || threshold > 255)
        return fail(h, LATCH_ERANGE, "threshold %d (must be in [0, 255])", threshold);
    if (max_kps < 0 || max_kps > LATCH_MAX_ROWS)
        return fail(h, LATCH_EINVAL, "max_kps = %lld", (long long)max_kps);
    const DetectLayout l = detect_layout(height, width);
    const int rc = check_workspace(h, l.total, "latch_detect");
    if (rc != LATCH_OK) return rc;
    DetectArgs a;
    a.img = img_dev;
    a.height = height;
    a.width = width;
    a.pitch = pitch;
    a.threshold = threshold;
    a.masks = reinterpret_cast<uint64_t *>(h->ws);
    a.row_first = reinterpret_cast<int64_t *>(h->ws + l.mask_bytes);
    a.counts = h->ws + l.mask_bytes + l.first_bytes;
    a.count_stride = l.count_stride;
    a.base = reinterpret_cast<int64_t *>(h->ws + l.mask_bytes + l.first_bytes + l.count_bytes);
    a.kps = reinterpret_cast<float4 *>(kps_dev);
    a.max_kps = max_kps;
    a.n_kps = n_kps_dev;
    a.image_id = image_id_dev;
    a.image_index = image_index;
    const hipError_t e = timed_launch(h, "detect", stream, [&] { return launch_detect(a, stream); });
    return e == hipSuccess ? LATCH_OK : hip_fail(h, e, "detect launch");
}

int hamming_knn(latch_handle h, const uint32_t *query_dev, int64_t nq, const uint32_t *train_dev,
                int64_t nt, int k, float ratio, int32_t *idx_dev, int32_t *dist_dev,
                uint8_t *accept_dev, int path, hipStream_t stream)
{
    return knn_call(h, query_dev, nq, train_dev, nt, k, ratio, idx_dev, dist_dev, accept_dev, path,
                    stream, false);
}

int hamming_knn_noalloc(latch_handle h, const uint32_t *query_dev, int64_t nq,
                        const uint32_t *train_dev, int64_t nt, int k, float ratio,
                        int32_t *idx_dev, int32_t *dist_dev, uint8_t *accept_dev, int path,
                        hipStream_t stream)
{
    return knn_call(h, query_dev, nq, train_dev, nt, k, ratio, idx_dev, dist_dev, accept_dev, path,
                    stream, true);
}

int hamming_knn_workspace_size(latch_handle h, int64_t nq, int64_t nt, int path, size_t *bytes)
{
    if (!h || !bytes) return LATCH_EINVAL;
    if (nq < 0 || nq > LATCH_MAX_ROWS || nt < 0 || nt > LATCH_MAX_ROWS)
        return fail(h, LATCH_EINVAL, "sizes nq = %lld, nt = %lld out of [0, 2^31)", (long long)nq,
                    (long long)nt);
    if (path < LATCH_PATH_AUTO || path > LATCH_PATH_MFMA_FP4)
        return fail(h, LATCH_EINVAL, "unknown path %d", path);
    path = resolve_path(h, path, nq, nt);
    *bytes = nq == 0 ? 0 : knn_workspace_bytes(plan_knn(nq, nt, path, h->num_cus, h->tuning, SIZE_MAX));
    return LATCH_OK;
}

int hamming_knn_batch_workspace_size(latch_handle h, int n_pairs, int64_t out_rows, size_t *bytes)
{
    if (!h || !bytes) return LATCH_EINVAL;
    if (n_pairs < 0 || out_rows < 0 || out_rows > LATCH_MAX_ROWS)
        return fail(h, LATCH_EINVAL, "negative or too large batch size");
    *bytes = n_pairs == 0 ? 0 : batch_workspace_bytes(n_pairs, out_rows);
    return LATCH_OK;
}

int latch_detect_workspace_size(latch_handle h, int height, int width, size_t *bytes)
{
    if (!h || !bytes) return LATCH_EINVAL;
    if (height < 1 || width < 1 || height >= (1 << 23))
        return fail(h, LATCH_EINVAL, "image %d x %d outside the limits", height, width);
    *bytes = detect_layout(height, width).total;
    return LATCH_OK;
}

int latch_extract_batch_workspace_size(latch_handle h, int n_images, int64_t max_kps,
                                       size_t *bytes)
{
    if (!h || !bytes) return LATCH_EINVAL;
    if (n_images < 0 || max_kps < 0 || max_kps > LATCH_MAX_ROWS)
        return fail(h, LATCH_EINVAL, "n_images = %d, max_kps = %lld out of range", n_images,
                    (long long)max_kps);
    *bytes = extract_batch_workspace(h, n_images, max_kps);
    return LATCH_OK;
}

int latch_reserve(latch_handle h, size_t bytes, size_t *held_out)
{
    if (!h) return LATCH_EINVAL;
    h->last_error.clear();
    if (bytes > h->ws_bytes) {
        const size_t want = align_up(bytes, 256);
        if (h->ws) {
            // Work enqueued on any stream may still use the old buffer.
            hipError_t e = hipDeviceSynchronize();
            if (e != hipSuccess) return hip_fail(h, e, "hipDeviceSynchronize");
            (void)hipFree(h->ws);
            h->ws = nullptr;
            h->ws_bytes = 0;
        }
        const hipError_t e = hipMalloc((void **)&h->ws, want);
        if (e != hipSuccess) {
            h->ws = nullptr;
            if (held_out) *held_out = 0;
            return hip_fail(h, e, "hipMalloc(workspace)");
        }
        h->ws_bytes = want;
    }
    if (held_out) *held_out = h->ws_bytes;
    return LATCH_OK;
}

int latch_get_tuning(latch_handle h, latch_tuning *out)
{
    if (!h || !out) return LATCH_EINVAL;
    *out = h->tuning;
    return LATCH_OK;
}

int latch_set_tuning(latch_handle h, const latch_tuning *t)
{
    if (!h || !t) return LATCH_EINVAL;
    auto ok_path = [](int p) {
        return p == LATCH_PATH_MFMA || p == LATCH_PATH_POPCOUNT || p == LATCH_PATH_MFMA_FP4;
    };
    for (int i = 0; i < 8; ++i)
        for (int j = 0; j < 8; ++j)
            if (!ok_path(t->path[i][j])) return fail(h, LATCH_ERANGE, "tuning path[%d][%d]", i, j);
    if (!ok_path(t->batch_path)) return fail(h, LATCH_ERANGE, "tuning batch_path");
    if (t->mfma_groups_per_cu < 1 || t->popcount_groups_per_cu < 1)
        return fail(h, LATCH_ERANGE, "tuning workgroup targets must be >= 1");
    if (t->fp4_query_blocks != 2 && t->fp4_query_blocks != 3)
        return fail(h, LATCH_ERANGE, "tuning fp4_query_blocks = %d (must be 2 or 3)",
                    t->fp4_query_blocks);
    if (t->batch_groups_per_cu < 1 || t->batch_groups_per_cu > 8)
        return fail(h, LATCH_ERANGE, "tuning batch_groups_per_cu = %d (must be in [1, 8])",
                    t->batch_groups_per_cu);
    h->tuning = *t;
    return LATCH_OK;
}

int latch_timing_enable(latch_handle h, int enable)
{
    if (!h) return LATCH_EINVAL;
    if (enable) {
        // Earlier records must be complete before their events are reused.
        for (auto &t : h->timed) (void)hipEventSynchronize(t.stop);
        release_timed(h);
    }
    h->timing = enable != 0;
    return LATCH_OK;
}

int latch_timing_read(latch_handle h, const char *kernel, int *launches, double *total_ms)
{
    if (!h || !kernel || !launches || !total_ms) return LATCH_EINVAL;
    int n = 0;
    double ms = 0.0;
    for (auto &t : h->timed) {
        if (std::strcmp(t.name, kernel) != 0) continue;
        hipError_t e = hipEventSynchronize(t.stop);
        float v = 0.0f;
        if (e == hipSuccess) e = hipEventElapsedTime(&v, t.start, t.stop);
        if (e != hipSuccess) return hip_fail(h, e, "reading timing events");
        ++n;
        ms += v;
    }
    *launches = n;
    *total_ms = ms;
    return LATCH_OK;
}

int hamming_knn_batch(latch_handle h, const uint32_t *query_dev, int64_t query_rows,
                      const uint32_t *train_dev, int64_t train_rows, const latch_pair *pairs_dev,
                      int n_pairs, int k, float ratio, int32_t *idx_dev, int32_t *dist_dev,
                      uint8_t *accept_dev, int64_t out_rows, int path, hipStream_t stream)
{
    if (!h) return LATCH_EINVAL;
    h->last_error.clear();
    if (n_pairs < 0 || query_rows < 0 || train_rows < 0 || out_rows < 0 ||
        query_rows > LATCH_MAX_ROWS || train_rows > LATCH_MAX_ROWS || out_rows > LATCH_MAX_ROWS)
        return fail(h, LATCH_EINVAL, "negative or too large batch size");
    if (k != 1 && k != 2) return fail(h, LATCH_ERANGE, "k = %d (must be 1 or 2)", k);
    if (!(ratio > 0.0f && ratio <= 1.0f))
        return fail(h, LATCH_ERANGE, "ratio = %g (must be in (0, 1])", (double)ratio);
    if (path < LATCH_PATH_AUTO || path > LATCH_PATH_MFMA_FP4)
        return fail(h, LATCH_EINVAL, "unknown path %d", path);
    if (n_pairs == 0) return LATCH_OK;
    if (!pairs_dev || !idx_dev || !dist_dev || (query_rows > 0 && !query_dev) ||
        (train_rows > 0 && !train_dev))
        return fail(h, LATCH_EINVAL, "null buffer");
    if (path == LATCH_PATH_AUTO) path = h->tuning.batch_path;

    const int rc = check_workspace(h, batch_workspace_bytes(n_pairs, out_rows), "hamming_knn_batch");
    if (rc != LATCH_OK) return rc;
    const BatchArgs a = batch_args(h, h->ws, h->parts, handle_parts(), query_dev, query_rows, train_dev, train_rows,
                                   pairs_dev, n_pairs, k, ratio, idx_dev, dist_dev, accept_dev,
                                   out_rows, path);
    const char *name = a.kind == SplitKernel::kPopcount  ? "knn_batch_popcount"
                       : a.kind == SplitKernel::kMfmaFp4 ? "knn_batch_fp4"
                                                         : "knn_batch_mfma";
    hipError_t e = timed_launch(h, name, stream,
                                [&] { return launch_knn_batch(a, stream); });
    return e == hipSuccess ? LATCH_OK : hip_fail(h, e, "batched knn launch");
}

int latch_plan_create(latch_handle h, const latch_plan_desc *d, latch_plan *out)
{
    if (!h || !d || !out) return LATCH_EINVAL;
    *out = nullptr;
    h->last_error.clear();
    if (d->max_kps < 0 || d->max_kps > LATCH_MAX_ROWS || d->n_images < 1 || d->n_pairs < 0 ||
        d->out_rows < 0 || d->out_rows > LATCH_MAX_ROWS)
        return fail(h, LATCH_EINVAL, "bad plan sizes");
    if (d->k != 1 && d->k != 2) return fail(h, LATCH_ERANGE, "k = %d (must be 1 or 2)", d->k);
    if (!(d->ratio > 0.0f && d->ratio <= 1.0f))
        return fail(h, LATCH_ERANGE, "ratio = %g (must be in (0, 1])", (double)d->ratio);
    if (d->path < LATCH_PATH_AUTO || d->path > LATCH_PATH_MFMA_FP4)
        return fail(h, LATCH_EINVAL, "unknown path %d", d->path);
    if (!d->images || !d->image_id || !d->kps || !d->desc ||
        (d->n_pairs > 0 && (!d->pairs || !d->idx || !d->dist)))
        return fail(h, LATCH_EINVAL, "null buffer");

    latch_plan_ctx *p = new latch_plan_ctx();
    p->h = h;
    // Plan workspace: the matcher's state, on the FP4 path what its parts need, then
    // the extraction's order.
    const int path = d->path == LATCH_PATH_AUTO ? h->tuning.batch_path : d->path;
    const size_t state_bytes = batch_workspace_bytes(d->n_pairs, d->out_rows);
    const PartMemory parts = plan_parts(d->n_pairs, d->out_rows);
    const bool divides = split_kernel(path) == SplitKernel::kMfmaFp4;
    const size_t knn_bytes = state_bytes + (divides ? align_up(parts.total, 256) : 0);
    const size_t order_bytes = extract_batch_workspace(h, d->n_images, d->max_kps);
    hipError_t e = hipMalloc((void **)&p->ws, knn_bytes + order_bytes);
    if (e != hipSuccess) {
        delete p;
        return hip_fail(h, e, "hipMalloc(plan workspace)");
    }
    const ExtractArgs ea = batch_extract_args(h, d->images, d->n_images, d->image_id, d->kps,
                                              d->max_kps, d->n_kps, d->desc);
    const BatchArgs ba = batch_args(h, p->ws, divides ? p->ws + state_bytes : nullptr, parts, d->desc,
                                    d->max_kps, d->desc, d->max_kps, d->pairs, d->n_pairs, d->k, d->ratio, d->idx,
                                    d->dist, d->accept, d->out_rows, path);
    hipStream_t s = nullptr;
    e = hipStreamCreateWithFlags(&s, hipStreamNonBlocking);
    if (e == hipSuccess) e = hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal);
    if (e == hipSuccess && d->max_kps > 0) e = run_extract_batch(h, ea, p->ws + knn_bytes, s, false);
    if (e == hipSuccess && d->n_pairs > 0) e = launch_knn_batch(ba, s);
    hipGraph_t graph = nullptr;
    if (s) {
        const hipError_t e2 = hipStreamEndCapture(s, &graph);
        if (e == hipSuccess) e = e2;
    }
    if (e == hipSuccess) e = hipGraphInstantiate(&p->exec, graph, nullptr, nullptr, 0);
    p->graph = graph;
    if (s) (void)hipStreamDestroy(s);
    if (e != hipSuccess) {
        latch_plan_destroy(p);
        return hip_fail(h, e, "plan capture");
    }
    *out = p;
    return LATCH_OK;
}

int latch_plan_run(latch_plan p, hipStream_t stream)
{
    if (!p) return LATCH_EINVAL;
    const hipError_t e = hipGraphLaunch(p->exec, stream);
    return e == hipSuccess ? LATCH_OK : hip_fail(p->h, e, "graph launch");
}

void latch_plan_destroy(latch_plan p)
{
    if (!p) return;
    (void)hipDeviceSynchronize();
    if (p->exec) (void)hipGraphExecDestroy(p->exec);
    if (p->graph) (void)hipGraphDestroy(p->graph);
    if (p->ws) (void)hipFree(p->ws);
    delete p;
}

int latch_check_errors(latch_handle h, hipStream_t stream, uint32_t *flags_out, int clear)
{
    if (!h || !flags_out) return LATCH_EINVAL;
    uint32_t v = 0;
    hipError_t e = hipMemcpyAsync(&v, h->flags_dev, sizeof v, hipMemcpyDeviceToHost, stream);
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
    if (e != hipSuccess) return hip_fail(h, e, "reading error word");
    *flags_out = v;
    if (clear) {
        e = hipMemsetAsync(h->flags_dev, 0, sizeof v, stream);
        if (e == hipSuccess) e = hipStreamSynchronize(stream);
        if (e != hipSuccess) return hip_fail(h, e, "clearing error word");
    }
    return LATCH_OK;
}

}  // extern "C"
