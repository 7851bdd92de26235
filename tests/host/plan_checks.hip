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
    uint8_t *ws = reinterpret_cast<uint8_t *>(1 << 20), *mem = reinterpret_cast<uint8_t *>(1 << 30);
    auto up = [](size_t v) { return (v + 255) / 256 * 256; };
    for (int n_pairs : {1, 3, 63, 100000, 300000})
        for (int64_t rows : {1LL, 1280000LL, 58000000LL, 60000000LL, LATCH_MAX_ROWS}) {
            const int64_t items = rows / 256 + n_pairs + 1;
            check(batch_workspace_bytes(n_pairs, rows) == up(16 * (size_t)n_pairs) + 256 + up(4 * (size_t)items),
                  "batch workspace", n_pairs, rows);
            for (const PartMemory &m : {handle_parts(), plan_parts(n_pairs, rows)}) {
                const BatchArgs a = batch_args(&h, ws, mem, m, nullptr, 0, nullptr, 0, nullptr, n_pairs, 2, 0.8f,
                                               nullptr, nullptr, nullptr, rows, LATCH_PATH_MFMA_FP4);
                const bool fits = items + m.slots * (kBatchMaxParts - 1) <= m.units;
                check(a.item_capacity == items && a.slots.count == (fits ? m.slots : 0), "slots", n_pairs, rows);
                const uint8_t *map = reinterpret_cast<const uint8_t *>(a.unit_pair);
                if (!fits) {
                    check(map >= ws && map + 4 * items <= ws + batch_workspace_bytes(n_pairs, rows),
                          "map in the workspace", n_pairs, rows);
                    continue;
                }
                const int64_t done = reinterpret_cast<uint8_t *>(a.slots.done) - mem;
                check(reinterpret_cast<uint8_t *>(a.slots.best) == mem && done >= m.slots * kBatchSlotQueries * 16 &&
                          done % 256 == 0 && (map - mem) % 256 == 0 && map - mem >= done + 4 * m.slots &&
                          map - mem + 4 * (items + m.slots * (kBatchMaxParts - 1)) <= (int64_t)m.total,
                      "memory of parts", n_pairs, rows);
            }
            const PartMemory own = plan_parts(n_pairs, rows);
            check(own.units >= items + own.slots * (kBatchMaxParts - 1), "a plan's parts fit its batch", rows);
            check(rows > 58000000 || n_pairs > 3 ||
                      items + kBatchMaxSlots * (kBatchMaxParts - 1) <= handle_parts().units,
                  "a handle's parts fit ordinary batches", rows);
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

}  // namespace

int main()
{
    part_rule();
    merge_launch();
    batch_memory();
    return failures ? 1 : 0;
}
