// Host unit check of the split of the maps into runs, against every other split.  Built
// and run by tests/test_map_runs.py.
#include "map_runs.h"

#include <cstdio>
#include <vector>

using namespace dsdp;

static int failures = 0;
#define CHECK(c)                                                                         \
    do {                                                                                 \
        if (!(c)) {                                                                      \
            std::fprintf(stderr, "map runs check failed: %s (line %d)\n", #c, __LINE__); \
            failures++;                                                                  \
        }                                                                                \
    } while (0)

// the least possible cost of the most costly of at most `want` runs
static int least(uint32_t first, int T, int from, int want)
{
    int best = run_cost(first, from, T);
    if (want > 1)
        for (int cut = from + 1; cut < T; cut++)
            if (first >> cut & 1u) {
                const int head = run_cost(first, from, cut), rest = least(first, T, cut, want - 1);
                best = std::min(best, std::max(head, rest));
            }
    return best;
}

int main()
{
    int part[18];
    // one radius of one map, one of one, one of two: 22, 22 and 26
    CHECK(split_maps(0x7u, 4, 3, part) == 3 && part[1] == 1 && part[2] == 2 && part[3] == 4);
    CHECK(split_maps(0x7u, 4, 1, part) == 1 && part[1] == 4);
    CHECK(split_maps(0x1u, 9, 4, part) == 1 && part[1] == 9);   // one radius: never cut
    // rows of cells over every spacing that a box may have (the edge is a float where it is
    // used), and that no position of a tile touches more
    int most = 0;
    for (double h = 0.05; h <= 4.0; h += 0.001) {
        const double edge = (double)(float)cell_edge(h);
        most = std::max(most, cell_rows(h, edge));
        for (double at = 0.0; at < 1.0; at += 0.05) {
            const auto touched = [&](int nodes) {
                const double lo = at * edge, hi = lo + (nodes - 1) * h + 16.0;
                return (int)(hi / edge) - (int)(lo / edge) + 1;
            };
            CHECK(touched(kTileY) * touched(kTileZ) <= cell_rows(h, edge));
        }
    }
    CHECK(most == 70 && most <= kMaxRows && cell_rows(4.0, 2.0) > kMaxRows);
    // the runs wanted: what fills the device, one to six, three from 13 maps on
    CHECK(runs_wanted(1, 3072, 4) == 6 && runs_wanted(512, 3072, 17) == 6 && runs_wanted(513, 3072, 17) == 5);
    CHECK(runs_wanted(1024, 3072, 9) == 3 && runs_wanted(1025, 3072, 9) == 2 && runs_wanted(1537, 3072, 9) == 1);
    CHECK(runs_wanted(1L << 20, 3072, 12) == 1 && runs_wanted(1L << 20, 3072, 13) == 3);
    // every arrangement of up to eight radii with one to three maps, every number of runs
    for (uint32_t code = 0; code < 6561; code++)
        for (int radii = 1; radii <= kMaxRadii; radii++) {
            uint32_t first = 0u, c = code;
            int T = 0;
            for (int r = 0; r < radii; r++, c /= 3) {
                first |= 1u << T;
                T += 1 + (int)(c % 3);
            }
            if (T > 17 || (radii < kMaxRadii && c != 0)) continue;
            for (int want = 1; want <= kMaxRadii; want++) {
                const int n = split_maps(first, T, want, part);
                int worst = 0;
                bool ends = n >= 1 && n <= want && n <= radii && part[0] == 0 && part[n] == T;
                for (int r = 0; r < n && ends; r++) {
                    ends = part[r + 1] > part[r] && (part[r] == 0 || (first >> part[r] & 1u));
                    worst = std::max(worst, run_cost(first, part[r], part[r + 1]));
                }
                CHECK(ends && worst == least(first, T, 0, want));
                CHECK(n == 1 || least(first, T, 0, n - 1) > worst);   // the fewest runs
            }
        }
    if (failures) return 1;
    std::printf("the runs are as specified\n");
    return 0;
}
