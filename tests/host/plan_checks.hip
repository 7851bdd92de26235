// Host rules of the library, checked without a GPU: this file includes the
// runtime's source, so that its internal host functions are reachable, and links
// with the built library for the rest.  It launches no kernel.  Prints the name of
// each group of checks; exits non-zero on a failed one.
#include "../../paper_1609_03986_amd/csrc/runtime.hip"
#include "../../paper_1609_03986_amd/csrc/batch_parts.h"

#include <cstdio>

namespace {

int failures = 0;

void check(bool ok, const char *what, long long a = 0, long long b = 0, long long c = 0)
{
    if (ok) return;
    std::fprintf(stderr, "check failed: %s (%lld, %lld, %lld)\n", what, a, b, c);
    ++failures;
}

// The merge of a split call: a launch holds fewer than 2^32 work items, for every
// query count that the C ABI takes.
void merge_launch()
{
    for (int64_t nq : {1LL, 15LL, 16LL, 17LL, 1LL << 20, (1LL << 20) + 1, (1LL << 28) - 1, 1LL << 28,
                       300000000LL, 1LL << 30, LATCH_MAX_ROWS}) {
        const int64_t blocks = merge_blocks(nq);
        check(blocks >= 1 && blocks * 256 < (1LL << 32), "merge work items", nq, blocks);
        check(nq > 1000000 || blocks * 16 >= nq, "one pass for ordinary query counts", nq, blocks);
    }
    std::puts("merge launch");
}

// Batched matching: the workspace holds what undivided pairs need; the memory of parts
// holds its three arrays one after the other, and serves a call whose unit map it holds.
void batch_memory()
{
    latch_ctx h;
    default_tuning(&h.tuning);
    h.num_cus = 256;
    uint8_t *ws = reinterpret_cast<uint8_t *>(1 << 20), *mem = reinterpret_cast<uint8_t *>(1 << 30);
    auto up = [](size_t v) { return (v + 255) / 256 * 256; };
    for (int n_pairs : {1, 3, 63, 100000, 300000})
        for (int64_t rows : {1LL, 1280000LL, 183000000LL, 262000000LL, LATCH_MAX_ROWS}) {
            const int64_t items = rows / 256 + n_pairs + 1;
            check(batch_workspace_bytes(n_pairs, rows) == up(16 * (size_t)n_pairs) + 256 + up(4 * (size_t)items),
                  "batch workspace", n_pairs, rows);
            for (const PartMemory &m : {handle_parts(), plan_parts(n_pairs, rows)}) {
                BatchArgs a = batch_args(&h, ws, mem, m, nullptr, 0, nullptr, LATCH_MAX_ROWS, nullptr, n_pairs, 2,
                                         0.8f, nullptr, nullptr, nullptr, rows, LATCH_PATH_MFMA_FP4);
                const bool fits = items + m.slots * (kBatchMaxParts - 1) <= m.units;
                check(a.item_capacity == items && a.slots.count == (fits ? m.slots : 0), "slots", n_pairs, rows);
                const int64_t units = items + std::min<int64_t>(a.slots.count, items) * (kBatchMaxParts - 1);
                check(batch_blocks(a) == std::min<int64_t>(units, 2 * h.num_cus), "workgroups of a batch", n_pairs, rows);
                a.train_rows = kMinPartTiles * kTileRows;         // no range to divide
                check(batch_blocks(a) == std::min<int64_t>(items, 2 * h.num_cus), "undivided batch", n_pairs, rows);
                const uint8_t *map = reinterpret_cast<const uint8_t *>(a.unit_pair);
                if (!fits) {
                    check(map >= ws && map + 4 * items <= ws + batch_workspace_bytes(n_pairs, rows),
                          "map in the workspace", n_pairs, rows);
                    continue;
                }
                const int64_t done = reinterpret_cast<uint8_t *>(a.slots.done) - mem;
                check(reinterpret_cast<uint8_t *>(a.slots.keys) == mem && done >= m.slots * kBatchSlotQueries * 16 &&
                          done % 256 == 0 && (map - mem) % 256 == 0 && map - mem >= done + 4 * m.slots &&
                          map - mem + 4 * (items + m.slots * (kBatchMaxParts - 1)) <= (int64_t)m.total,
                      "memory of parts", n_pairs, rows);
            }
            const PartMemory own = plan_parts(n_pairs, rows);
            check(own.units >= items + own.slots * (kBatchMaxParts - 1), "a plan's parts fit its batch", rows);
            check((rows / 256 + n_pairs < 1017000) ==
                      (items + kBatchMaxSlots * (kBatchMaxParts - 1) <= handle_parts().units),
                  "a handle's parts fit ordinary batches", n_pairs, rows);
        }
    check(batch_args(&h, ws, nullptr, handle_parts(), nullptr, 0, nullptr, 0, nullptr, 1, 2, 0.8f, nullptr, nullptr,
                     nullptr, 1, LATCH_PATH_MFMA).slots.count == 0, "no memory, no slots");
    std::puts("batch memory");
}

// Parts of a train range: none empty, the limits kept.
void part_rule()
{
    for (int tiles : {0, 1, 79, 80, 81, 159, 160, 161, 1279, 1280, 1281, 10000, 65535})
        for (unsigned long long left : {0ull, 1ull, 512ull * 80, 512ull * 81, 512ull * 5000, 1ull << 40}) {
            const int parts = train_parts(tiles, left, 512);
            check(parts >= 1 && parts <= kBatchMaxParts, "part count", tiles, (long long)left, parts);
            const int per_part = (tiles + parts - 1) / parts;
            check(parts == 1 || ((parts - 1) * per_part < tiles && tiles >= kMinPartTiles), "no empty part", tiles,
                  (long long)left, parts);
        }
    // No division where every range is at most a least part, or where all units start at
    // once and the longest range hardly exceeds the workgroups' share.
    check(!may_divide(80, 5, 400, 512) && may_divide(81, 5, 405, 512), "least part");
    check(!may_divide(87, 504, 504 * 87, 512) && !may_divide(157, 420, 420 * 157, 512), "one full round");
    check(may_divide(157, 210, 210 * 157, 512) && may_divide(700, 504, 504 * 100, 512), "idle or uneven");
    check(may_divide(87, 513, 513 * 87, 512), "more than a round");
    // The pairs of the GPU test of more divided query groups than slots (31 pairs of 78
    // groups of 384 queries, train tiles from 16,384 down by a quarter octave): every
    // pair is divided, and together they want more slots than there are.
    const int pairs = 31, groups = 78, resident = 512;
    unsigned long long work[256] = {}, in_class[256] = {};
    int tiles[pairs];
    for (int i = 0; i < pairs; ++i) {
        tiles[i] = (int)std::lround(16384.0 * std::exp2(-i / 4.0));
        const int c = cost_class(32LL * tiles[i]);
        work[c] += (unsigned long long)groups * tiles[i];
        in_class[c] += groups;
    }
    unsigned long long all_work = 0;
    for (unsigned long long w : work) all_work += w;
    check(may_divide(tiles[0], (unsigned long long)groups * pairs, all_work, resident), "that batch divides");
    int wanted = 0;
    for (int i = 0; i < pairs; ++i) {
        const int c = cost_class(32LL * tiles[i]);
        check(in_class[c] == (unsigned long long)groups, "one pair a class", i, c);
        unsigned long long left = in_class[c] * tiles[i];
        for (int later = c + 1; later < 256; ++later) left += work[later];
        check(train_parts(tiles[i], left, resident) > 1, "divided pair", i, tiles[i]);
        wanted += groups;
    }
    check(wanted > kBatchMaxSlots, "more divided groups than slots", wanted);
    std::puts("part rule");
}

// Split plans within a cap on the partials' bytes, as the allocation-free call makes
// them: the plan covers the train rows, and its partials fit wherever those of the
// fewest splits that the index allows do.
void capped_plans()
{
    latch_ctx probe;
    default_tuning(&probe.tuning);
    const size_t cap = LATCH_NOALLOC_SCRATCH_BYTES;
    for (int per_cu : {1, 2, 8, 64})
        for (int qb : {2, 3})
            for (int path : {LATCH_PATH_MFMA, LATCH_PATH_POPCOUNT, LATCH_PATH_MFMA_FP4})
                for (int64_t nq : {1LL, 385LL, 2000LL, 16000LL, 40000LL, 150000LL, 700000LL, 1100000LL, LATCH_MAX_ROWS})
                    for (int64_t nt : {1LL, 257LL, 2000LL, 16384LL, 16385LL, 100000LL, 1000000LL, LATCH_MAX_ROWS}) {
                        latch_tuning t = probe.tuning;
                        t.fp4_query_blocks = (int8_t)qb;
                        t.mfma_groups_per_cu = t.popcount_groups_per_cu = per_cu;
                        const int run = resolve_path(&probe, path, nq, nt);
                        const KnnPlan p = plan_knn(nq, nt, run, 256, t, cap);
                        const int64_t most = run == LATCH_PATH_MFMA_FP4 ? kFp4MaxSplitRows : kMaxSplitRows;
                        const int64_t fewest = (nt + most - 1) / most;
                        check(p.split_rows % kTileRows == 0 && p.split_rows <= most && p.nsplit >= fewest &&
                                  (int64_t)p.nsplit * p.split_rows >= nt && (p.nsplit - 1) * p.split_rows < nt,
                              "capped plan covers the rows", nq, nt, p.nsplit);
                        const size_t need = knn_workspace_bytes(p);
                        if (fewest == 1 || (size_t)fewest * nq * 16 <= cap)
                            check(need <= cap || p.nsplit == 1, "capped partials", nq, nt, p.nsplit);
                        else
                            check(need > cap, "more than the cap", nq, nt, p.nsplit);
                    }
    // The plan depends on the query count through the numbers of query groups of 256
    // and 384 alone, so the need is largest at multiples of 128 queries.
    for (int64_t nt : {3000LL, 20000LL, 1000000LL})
        for (int64_t g = 1; g <= 400; g += g < 40 ? 1 : 13) {
            const KnnPlan a = plan_knn(128 * g - 127, nt, LATCH_PATH_MFMA_FP4, 256, probe.tuning, SIZE_MAX);
            const KnnPlan b = plan_knn(128 * g, nt, LATCH_PATH_MFMA_FP4, 256, probe.tuning, SIZE_MAX);
            check(a.nsplit == b.nsplit && a.split_rows == b.split_rows && a.query_blocks == b.query_blocks,
                  "plan within a group count", nt, g);
        }
    std::puts("capped plans");
}

// Slots of the 512 triplets as both kinds of handle place them.
void slots_of_handles()
{
    uint32_t rng = 12345;
    auto next = [&](int n) {
        rng = rng * 1664525u + 1013904223u;
        return (int)((rng >> 8) % (uint32_t)n);
    };
    for (int kind : {0, 64, 48}) {
        uint2 toff[kTriplets];
        for (uint2 &t : toff) {
            uint32_t o[3];
            for (uint32_t &x : o)
                x = kind == 0 ? patch_offset(3 + next(42), 3 + next(42))
                              : weighted_patch_offset(kind, next(kind - 7), next(kind - 7));
            t = make_uint2(o[0] | (o[1] << 16), o[2]);
            check(o[0] < 65536 && o[1] < 65536 && o[2] < 65536, "patch offsets", kind);
        }
        uint16_t slot[kTriplets], again[kTriplets];
        assign_slots(toff, kTriplets, 32, 32, slot);
        assign_slots(toff, kTriplets, 32, 32, again);
        int used[kTriplets] = {};
        for (int t = 0; t < kTriplets; ++t) {
            check(slot[t] < kTriplets && slot[t] == again[t], "slot", kind, t, slot[t]);
            if (slot[t] < kTriplets) ++used[slot[t]];
        }
        for (int i = 0; i < kTriplets; ++i) check(used[i] == 1, "slots are a permutation", kind, i);
    }
    std::puts("slots of handles");
}

// The tie masks of every angle bin, against each position's unrounded offset.
void ties()
{
    std::vector<int16_t> c(kBins), s(kBins);
    rotation_table(c.data(), s.data());
    const std::vector<uint32_t> mask = tie_masks(c.data(), s.data());
    for (int a = 0; a < kBins; ++a) {
        uint32_t want = 0;
        for (int v = -32; v <= 32; ++v)
            for (int u = -32; u <= 32; ++u) {
                const bool inner = std::abs(u) <= kHalf && std::abs(v) <= kHalf;
                const int xy[2] = {c[a] * u - s[a] * v, s[a] * u + c[a] * v};
                for (int x : xy)
                    for (int k = 0; k <= 10 && x != 0; ++k)        // sq = 2^k, or an odd multiple
                        if (((int64_t)x << k) % (1 << 21) == 0 && (((int64_t)x << k) >> 21) % 2 != 0)
                            want |= (1u << (16 + k)) | (inner ? 1u << k : 0u);
            }
        check(mask[a] == want, "tie mask", a, mask[a], want);
    }
    std::puts("tie masks");
}

}  // namespace

int main()
{
    capped_plans();
    slots_of_handles();
    ties();
    part_rule();
    merge_launch();
    batch_memory();
    return failures ? 1 : 0;
}
