// Host unit check of the range allocator used from both ends, against a brute-force
// model of the pool (one flag per unit), on seeded random sequences.  Built and run by
// tests/test_range_alloc_ends.py with AddressSanitizer and UBSan.
#include "range_alloc.h"

#include <cstdio>
#include <random>
#include <vector>

using dsdp::host::RangeAlloc;

int main()
{
    for (int seed = 0; seed < 100; seed++) {
        std::mt19937 rng(seed);
        const long total = 1 + (long)(rng() % 2048);
        RangeAlloc a;
        a.init((size_t)total);
        std::vector<char> taken((size_t)total, 0);
        struct Block { size_t off, n; };
        std::vector<Block> live;
        auto model = [&](long need, bool high) {   // offset, or -1
            for (long k = 0; k + need <= total; k++) {
                const long at = high ? total - need - k : k;
                bool free = true;
                for (long u = at; u < at + need && free; u++) free = !taken[(size_t)u];
                if (free) return at;
            }
            return -1L;
        };
        for (int step = 0; step < 1000; step++) {
            if (live.empty() || rng() % 3 != 0) {
                const size_t n = rng() % 97;   // 0 is rounded up to one unit
                const long need = n ? (long)n : 1;
                const bool high = rng() % 2;
                const long expect = model(need, high);
                size_t off = 0;
                const bool ok = high ? a.alloc_high(n, off) : a.alloc(n, off);
                if (ok != (expect >= 0) || (ok && (long)off != expect)) {
                    std::fprintf(stderr, "differs from the model (seed %d, step %d)\n", seed, step);
                    return 1;
                }
                if (!ok) continue;
                for (long u = 0; u < need; u++) taken[off + (size_t)u] = 1;
                live.push_back({off, n});
            } else {
                const size_t k = rng() % live.size();
                const Block b = live[k];
                live[k] = live.back();
                live.pop_back();
                a.release(b.off, b.n);
                for (size_t u = b.off; u < b.off + (b.n ? b.n : 1); u++) taken[u] = 0;
            }
            size_t used = 0;
            for (char t : taken) used += (size_t)t;
            if (used != a.used) {
                std::fprintf(stderr, "used count (seed %d, step %d)\n", seed, step);
                return 1;
            }
        }
        for (const Block &b : live) a.release(b.off, b.n);
        if (a.used != 0 || a.free_.size() != 1 || a.free_.begin()->second != (size_t)total) {
            std::fprintf(stderr, "not whole again (seed %d)\n", seed);
            return 1;
        }
    }
    std::printf("both ends match the model\n");
    return 0;
}
