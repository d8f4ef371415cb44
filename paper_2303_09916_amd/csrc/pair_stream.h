// Host construction of the pair stream, a layout of the intra-ligand term: plain C++,
// no device code, so it can be unit-tested on the host.  Private to the library.
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <vector>

namespace dsdp {

constexpr int kStreamPairs = 127;   // pairs per chunk

namespace host {

// The pair stream's sections, in the order the pairs of a chunk are stored: those
// without a class first (each part in list order).  Made in one pass over the pairs
// and one over the lanes' lists: a scoring call prepares its ligand every time (1000
// poses of 60 atoms: 81 us a call, 151 with every chunk collected from whole lists; 47
// atoms: 59 and 89).
struct StreamChunks {
    std::vector<uint32_t> words;   // stored pair words, whole slots
    std::vector<uint8_t> list;     // per chunk: [word][lane] of four entries each
    uint32_t chunk_words[2] = {0, 0}, plain = 0;
    int n_chunks = 0, list_words = 0;   // n_chunks < 0: the ligand does not fit the format
};
inline StreamChunks stream_chunks(const std::vector<uint32_t> &pairs, const std::vector<std::vector<uint16_t>> &lane_list)
{
    StreamChunks sc;
    const int np = (int)pairs.size();
    sc.n_chunks = (np + kStreamPairs - 1) / kStreamPairs;
    std::vector<uint8_t> at((size_t)np);   // a pair's index in its chunk
    size_t done[64] = {0};                 // entries of each lane's list in the chunks so far
    for (int c = 0; c < sc.n_chunks; c++) {
        const int p0 = c * kStreamPairs, p1 = std::min(np, p0 + kStreamPairs), n = p1 - p0;
        const int slots = n > 63 ? 2 : 1, zero = 64 * slots - 1;
        const size_t w0 = sc.words.size();
        sc.words.resize(w0 + (size_t)64 * slots, 0x80000000u);   // no pair
        int k = 0;
        for (int pass = 0; pass < 2; pass++) {
            for (int p = p0; p < p1; p++)
                if (((pairs[(size_t)p] >> 16) != 0) == (pass == 1)) {
                    at[(size_t)p] = (uint8_t)k;
                    sc.words[w0 + (size_t)k++] = pairs[(size_t)p];
                }
            // slots of class-free pairs only (a short last slot without a class pair counts)
            if (pass == 0) sc.plain |= (uint32_t)(k == n ? slots : k / 64) << (2 * c);
        }
        // a lane's list is in the order of the pairs: its entries of the chunk are one run
        size_t end[64], longest = 0;
        for (int l = 0; l < 64; l++) {
            const std::vector<uint16_t> &list = lane_list[(size_t)l];
            end[l] = done[l];
            while (end[l] < list.size() && (list[end[l]] & 0x7fff) < p1) end[l]++;
            longest = std::max(longest, end[l] - done[l]);
        }
        const int words = (int)((longest + 3) / 4);
        if (words > 15) {
            sc.n_chunks = -1;   // does not fit the format: the caller takes another layout
            return sc;
        }
        const size_t l0 = sc.list.size();
        sc.list.resize(l0 + (size_t)256 * words, (uint8_t)zero);
        for (int l = 0; l < 64; l++)
            for (size_t m = 0; done[l] < end[l]; m++, done[l]++) {
                const uint16_t e = lane_list[(size_t)l][done[l]];
                sc.list[l0 + (m / 4 * 64 + (size_t)l) * 4 + m % 4] =
                    (uint8_t)(at[(size_t)(e & 0x7fff)] | ((e & 0x8000) ? 128 : 0));
            }
        sc.chunk_words[c / 8] |= (uint32_t)words << (4 * (c % 8));
        sc.list_words += words;
    }
    return sc;
}

}  // namespace host
}  // namespace dsdp
