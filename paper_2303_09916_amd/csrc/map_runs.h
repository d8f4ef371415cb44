// Host rules of the map build (receptor cells, and how the maps of a small box are split
// into runs): plain C++, no device code, so they can be unit-tested on the host.
// Private to the library.
#pragma once

#include <algorithm>
#include <cstdint>

namespace dsdp {

constexpr int kMaxRadii = 8;   // distinct XS radii
constexpr int kTileX = 8, kTileY = 8, kTileZ = 4;   // nodes of a workgroup's tile
constexpr int kMaxRows = 128;                       // rows of cells that a tile can gather

// Edge of the receptor cells for node spacing h and the 8 A cutoff.
inline double cell_edge(double h) { return std::max(4.0, (8.0 * h + 16.0) / 9.0); }

// Rows of cells (along x) that a tile and the cutoff around it can touch, at most: a span of
// s cell edges touches floor(s) + 2 with its ends anywhere.  10 in y by 7 in z at spacing 2.5
// to 4, 6 by 6 below 0.57.
inline int cell_rows(double h, double edge)
{
    return ((int)(((kTileY - 1) * h + 16.0) / edge) + 2) * ((int)(((kTileZ - 1) * h + 16.0) / edge) + 2);
}

// Issue cost per atom of maps [a, b): about 18 instructions a radius, 4 a map.  Bit k of
// `first`: map k is the first of its radius.
inline int run_cost(uint32_t first, int a, int b)
{
    int cost = 0;
    for (int k = a; k < b; k++) cost += 4 + ((first >> k & 1u) ? 18 : 0);
    return cost;
}

// Runs wanted of T maps where one run is `waves` waves and `fill` waves fill the device.
//  - At least three from 13 maps on, where a lane would hold so many sums that few waves
//    share a SIMD (17 types, 75^3 nodes: 204 us, one run 246).
//  - Else what fills the device, since a wave's time is its own chain of atoms, but no more:
//    each run repeats the part that does not depend on the map (about 25 of 100 to 150
//    instructions an atom).  43^3 nodes, 4 types: two runs 37 us, three 39, one 46; 17^3, 9
//    types: four runs 31, one 51.
//  - At most six (27^3 nodes, 17 types: six runs 44 us, eight 47).
inline int runs_wanted(long waves, long fill, int T)
{
    return (int)std::max(T > 12 ? 3L : 1L, std::min(6L, fill / std::max(1L, waves)));
}

// Cuts T maps, ordered by radius, into at most `want` runs that end on a change of
// radius, so that the most costly run is as cheap as can be, with the fewest runs that
// do that: run r is maps part[r] to part[r + 1] - 1.  Returns the number of runs.
inline int split_maps(uint32_t first, int T, int want, int *part)
{
    int starts[kMaxRadii + 1], radii = 0;
    for (int k = 0; k < T; k++)
        if (k == 0 || (first >> k & 1u)) starts[radii++] = k;
    starts[radii] = T;
    int best_cost = 0, best_runs = 0;
    uint32_t best = 0u;
    for (uint32_t cuts = 0; cuts < (1u << (radii - 1)); cuts++) {   // bit r: a cut before radius r + 1
        int runs = 1, from = 0, worst = 0;
        for (int r = 1; r <= radii; r++)
            if (r == radii || (cuts >> (r - 1) & 1u)) {
                worst = std::max(worst, run_cost(first, starts[from], starts[r]));
                from = r;
                if (r < radii) runs++;
            }
        if (runs > want && cuts != 0) continue;
        if (best_runs == 0 || worst < best_cost || (worst == best_cost && runs < best_runs)) {
            best_cost = worst;
            best_runs = runs;
            best = cuts;
        }
    }
    int n = 0;
    part[0] = 0;
    for (int r = 1; r <= radii; r++)
        if (r == radii || (best >> (r - 1) & 1u)) part[++n] = starts[r];
    return n;
}

}  // namespace dsdp
