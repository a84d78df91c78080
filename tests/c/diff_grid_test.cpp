// Grids of the diff kernel (csrc/diff_grid.h) over unit counts from none to the
// largest page space (2^32 pages of 4 units' size and more), groups and limits.
#include "diff_grid.h"

#include <cstdio>
#include <initializer_list>

using namespace crum;

static int bad = 0;

static void expect(uint64_t got, uint64_t want, const char* what)
{
    if (got != want) {
        std::printf("%s: %llu, not %llu\n", what, (unsigned long long)got,
                    (unsigned long long)want);
        ++bad;
    }
}

int main()
{
    expect(diff_grid(0, 1, kDiffBlocksMax), 0, "no units");
    expect(diff_grid(1, 1, kDiffBlocksMax), 1, "one unit");
    expect(diff_grid(4, 1, kDiffBlocksMax), 1, "four waves");
    expect(diff_grid(5, 1, kDiffBlocksMax), 2, "five waves");
    expect(diff_grid(8, 2, kDiffBlocksMax), 1, "four waves of two units");
    expect(diff_grid(9, 2, kDiffBlocksMax), 2, "a wave of one unit left");
    expect(diff_grid(16, 4, kDiffBlocksMax), 1, "four waves of four units");
    expect(diff_grid(1 << 20, 1, 7), 7, "a limit");
    expect(diff_grid(3, 1, 7), 1, "a limit above the need");
    // the default of 8 workgroups on each of 256 compute units was a limit, and stays
    // one for a caller or a cache that sets it
    expect(diff_grid(131072, 1, kDiffBlocksMax), 32768, "no limit by default");
    expect(diff_grid(131072, 1, 2048), 2048, "2048 is a limit");
    // the launch's own limit: 256 GiB of 4 KiB units, one a wave, and far above
    for (uint64_t units : {1ull << 26, (1ull << 26) + 1, 1ull << 32, ~0ull})
        for (uint32_t group : {1u, 2u, 4u})
            for (uint32_t blocks : {1u, 2048u, kDiffBlocksMax, ~0u}) {
                const uint64_t n = diff_grid(units, group, blocks);
                if (n == 0 || n * 256 >= 1ull << 32 || n > blocks) {
                    std::printf("%llu units, %u a wave, limit %u: %llu workgroups\n",
                                (unsigned long long)units, group, blocks, (unsigned long long)n);
                    ++bad;
                }
            }
    if (!bad)
        std::printf("diff grid: ok\n");
    return bad != 0;
}
