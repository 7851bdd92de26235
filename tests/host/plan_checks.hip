// Host rules of the library, checked without a GPU: this file includes the
// runtime's source, so that its internal host functions are reachable, and links
// with the built library for the rest.  It launches no kernel.  Prints the name of
// each group of checks; exits non-zero on a failed one.
#include "../../paper_1609_03986_amd/csrc/runtime.hip"

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

}  // namespace

int main()
{
    merge_launch();
    return failures ? 1 : 0;
}
