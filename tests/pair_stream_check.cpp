// Host unit check of the pair stream's construction against a plain one that goes,
// for every chunk, through every lane's whole list, and of the time it takes.
// Built and run by tests/test_pair_stream.py.
#include "pair_stream.h"

#include <chrono>
#include <cstdio>
#include <random>

using namespace dsdp;
using namespace dsdp::host;

static int failures = 0;
#define CHECK(c)                                                                            \
    do {                                                                                    \
        if (!(c)) {                                                                         \
            std::fprintf(stderr, "pair stream check failed: %s (line %d)\n", #c, __LINE__); \
            failures++;                                                                     \
        }                                                                                   \
    } while (0)

struct Plain {
    std::vector<uint32_t> words;
    std::vector<uint8_t> list;
    uint32_t chunk_words[2] = {0, 0}, plain = 0;
};
static Plain plain_chunks(const std::vector<uint32_t> &pairs, const std::vector<std::vector<uint16_t>> &lanes)
{
    Plain s;
    const int np = (int)pairs.size();
    for (int c = 0; c * 127 < np; c++) {
        std::vector<int> order, classes;
        for (int p = c * 127; p < std::min(np, c * 127 + 127); p++) ((pairs[p] >> 16) ? classes : order).push_back(p);
        const int n = (int)(order.size() + classes.size()), slots = n > 63 ? 2 : 1;
        s.plain |= (uint32_t)(classes.empty() ? slots : (int)order.size() / 64) << (2 * c);
        order.insert(order.end(), classes.begin(), classes.end());
        for (int k = 0; k < 64 * slots; k++) s.words.push_back(k < n ? pairs[order[k]] : 0x80000000u);
        std::vector<std::vector<uint8_t>> out(64);
        size_t longest = 0;
        for (int l = 0; l < 64; l++) {
            for (uint16_t e : lanes[l])
                for (int k = 0; k < n; k++)
                    if (order[k] == (e & 0x7fff)) out[l].push_back((uint8_t)(k + ((e & 0x8000) ? 128 : 0)));
            longest = std::max(longest, out[l].size());
        }
        const size_t words = (longest + 3) / 4;
        s.chunk_words[c / 8] |= (uint32_t)words << (4 * (c % 8));
        for (size_t m = 0; m < words; m++)
            for (int l = 0; l < 64; l++)
                for (size_t b = 4 * m; b < 4 * m + 4; b++)
                    s.list.push_back(b < out[l].size() ? out[l][b] : (uint8_t)(64 * slots - 1));
    }
    return s;
}

// every pair (i, j) with j - i > gap of n atoms, by distance, as the library orders them
static void shape(int n, int gap, int every, std::mt19937 &rng, std::vector<uint32_t> &pairs,
                  std::vector<std::vector<uint16_t>> &lanes)
{
    pairs.clear();
    lanes.assign(64, {});
    std::vector<std::vector<uint16_t>> atom(n);
    for (int d = gap + 1; d < n; d++)
        for (int i = 0; i + d < n; i++) {
            if (rng() % 100 >= (unsigned)every) continue;
            const uint32_t flags = rng() % 3 == 0 ? 1 + rng() % 2 : 0;
            atom[i].push_back((uint16_t)pairs.size());
            atom[i + d].push_back((uint16_t)(pairs.size() | 0x8000));
            pairs.push_back((uint32_t)i | ((uint32_t)(i + d) << 8) | (flags << 16));
        }
    const int per = n <= 32 ? 2 : 1;
    for (int l = 0; l < 64; l++) {
        const int a = per == 2 ? (l & 31) : l;
        if (a >= n) continue;
        for (size_t e = per == 2 ? l >> 5 : 0; e < atom[a].size(); e += per) lanes[l].push_back(atom[a][e]);
    }
}

int main()
{
    std::mt19937 rng(7);
    std::vector<uint32_t> pairs;
    std::vector<std::vector<uint16_t>> lanes;
    for (int n : {1, 2, 5, 13, 16, 17, 20, 31, 32, 33, 47, 60, 63, 64})
        for (int gap : {0, 3, 8})
            for (int every : {15, 60, 100}) {
                shape(n, gap, every, rng, pairs, lanes);
                const StreamChunks a = stream_chunks(pairs, lanes);
                const Plain b = plain_chunks(pairs, lanes);
                CHECK(a.n_chunks == (int)(pairs.size() + 126) / 127);
                CHECK(a.words == b.words && a.list == b.list && a.plain == b.plain);
                CHECK(a.chunk_words[0] == b.chunk_words[0] && a.chunk_words[1] == b.chunk_words[1]);
                CHECK(a.list_words * 256 == (int)a.list.size());
            }
    // more than fifteen list words in a chunk: refused (one atom in every pair of two chunks)
    pairs.assign(130, 0u);
    lanes.assign(64, {});
    for (int p = 0; p < 130; p++) lanes[0].push_back((uint16_t)p);
    CHECK(stream_chunks(pairs, lanes).n_chunks == -1);
#ifdef TIMED
    // one pass over the lists: 60 atoms, against collecting every chunk's entries from
    // whole lists
    shape(60, 3, 95, rng, pairs, lanes);
    auto seconds = [&](auto f) {
        double best = 1e30;
        for (int k = 0; k < 9; k++) {
            const auto t = std::chrono::steady_clock::now();
            for (int r = 0; r < 40; r++) f();
            best = std::min(best, std::chrono::duration<double>(std::chrono::steady_clock::now() - t).count() / 40);
        }
        return best;
    };
    size_t seen = 0;
    const double build = seconds([&] { seen += stream_chunks(pairs, lanes).list.size(); });
    const double whole = seconds([&] {
        for (int c = 0; c * 127 < (int)pairs.size(); c++) {
            std::vector<std::vector<uint8_t>> out(64);
            for (int l = 0; l < 64; l++)
                for (uint16_t e : lanes[l])
                    if ((e & 0x7fff) >= c * 127 && (e & 0x7fff) < c * 127 + 127) out[l].push_back((uint8_t)(e % 127));
            for (const auto &v : out) seen += v.size();
        }
    });
    std::printf("%.1f us, from whole lists %.1f us (%zu)\n", build * 1e6, whole * 1e6, seen);
    CHECK(2.0 * build < whole);
#endif
    if (failures) return 1;
    std::printf("the stream is as specified\n");
    return 0;
}
