// Rules for the layout of a ligand's intra-ligand term and the waves of its chains:
// plain C++, no device code, so they can be unit-tested on the host.  Every choice
// gives the same bits, so the rules only move speed.  Private to the library.
#pragma once

#include "../../include/dsdp.h"
#include "pair_stream.h"

#include <algorithm>
#include <cstddef>

namespace dsdp {

// Layouts of the intra-ligand term.  Pair lists: lane l evaluates pairs
// l + 64 k once and stores each pair's force in LDS; every atom then gathers the
// forces of its pairs.  Atom lists: a lane owns an atom (or half of its partners
// when there are at most 32 atoms) and evaluates each of the atom's pairs from
// its own side, so every pair is evaluated twice but nothing per pair is kept
// in LDS.  Pair stream: the pair lists' arithmetic in chunks of kStreamPairs pairs,
// whose forces fit 2 KB, so that a compute unit holds more chains; chains of one wave
// share the ligand among up to kStreamChains of a workgroup.
constexpr int kFormPairs = 0;
constexpr int kFormAtoms = 1;
constexpr int kFormStream = 2;
constexpr int kStreamChains = 4;    // chains per workgroup

namespace host {

// Where a prepared ligand will run: the caller's layout request
// (DSDP_INTRA_*) and waves per chain (0: by the chain count), the chains of the
// launch and whether the launch mixes ligands.
struct IntraCtx {
    int form = DSDP_INTRA_AUTO;
    int waves = 0;
    long chains = 1;
    bool mixed = false;
    bool bb = false;   // Barzilai-Borwein: a chain's waves share each evaluation's pairs
    bool score = false;   // poses scored once each, a wave per pose whatever `waves` says
    int layout = -1;   // kForm*: this layout, whatever the rule
};
// Waves per compute unit that the search's launches aim at: pair and atom lists,
// pair stream (what their registers let a unit hold).
constexpr long kListWaves = 8, kStreamWaves = 12;

// Compute units and the LDS a workgroup may use.
struct Device {
    long cus;
    size_t max_lds;
};

// Waves per chain by the chain count: what fills `per_cu` waves of every compute unit.
inline int waves_for(long chains, long per_cu, long cus)
{
    return (int)std::max(1L, std::min(4L, per_cu * cus / std::max(1L, chains)));
}

// Chains with pair lists that the device holds at once, of `waves` waves and `lds`
// bytes each.
inline long resident_lists(size_t lds, int waves, const Device &dev)
{
    return std::min<long>((long)(dev.max_lds / lds), kListWaves / waves) * dev.cus;
}

// Waves per pose of a BFGS refinement whose waves are left to the library (0: by the
// rule of the searches).  Poses take 2 to some 100 evaluations and the launch ends on the
// slowest, which two waves shorten; one wave from where the extra waves cost more (2500 poses:
// 33 atoms 0.90 ms, one wave 1.10, 60 atoms 1.34 and 2.11; 4000 poses: 0.80 and 0.86, 1.86
// and 1.97; 6000 poses: 1.04 and 1.09, 2.57 and 2.55, 54 atoms 2.14 and 2.02).
inline int refine_waves(long poses, long cus)
{
    return poses > kStreamWaves / 2 * cus && poses <= 16 * cus ? 2 : 0;
}

// Layout of the intra-ligand term for a launch context; lists_lds(waves): the LDS of a
// workgroup of the ligand with pair lists.
//  - Pair lists have every pair in one go, the stream has chunks one after the other and
//    needs half the registers and a fraction of the LDS: lists while all workgroups are
//    resident, the stream when they would run in rounds.  Several waves per chain (BFGS, 47
//    atoms): 384 chains, 20 steps 3.5 and 4.0 ms; 1024 chains 6.5 and 4.8 at three waves.
//    One wave (Barzilai-Borwein, 10 steps): 47 atoms, 1024 chains 6.7 and 8.2 ms, 1300
//    chains (in rounds) 13.2 and 9.4; 33 atoms, 2048 chains 5.5 and 6.0, 2500 chains 9.2
//    and 7.5.
//  - One wave and hardly more than a chunk of pairs: the stream, which is one go too (12
//    atoms, 30 pairs, 384 to 2048 chains, 10 steps: 2.8 to 3.2 ms, lists 3.0 to 3.6; 60 steps of
//    1536 chains: 141 pairs 24.0 and 25.0, 154 pairs 25.0 both, 219 pairs 27.8 and 25.9).
//  - Barzilai-Borwein chains of several waves share each evaluation's pairs: lists.
//  - Scoring prepares the ligand in every call and is bound by that up to some 20 poses a
//    unit: pair lists while resident, then atom lists, the smaller sections (5000 poses a
//    call: 33 atoms 35.5 us, lists 39.8, stream 41.8; 60 atoms 82, 144 and 85), and
//    the stream where the kernel is what counts (20000 poses: 33 atoms 60 us, lists 64, atoms
//    76; 60 atoms 125, 471 and 126).
//  - Launches that mix ligands take atom lists, whose launches need not be split by pair
//    count, up to four chains a unit (1024), and the stream beyond, where lists would get one
//    wave per chain.  The stream's own waves are then those of kStreamWaves (pick_waves): two
//    up to six chains a unit (1536), one beyond.  Eight ligands of 14 to 60 atoms, 100 steps:
//    768 chains, atom lists 37.7 ms at two waves, stream 39.4; 1152 to 1536 chains, stream
//    45.5 at two waves and 73 at one, atom lists 46.2 and 75; 1600 chains, stream 73.7 at one
//    wave, atom lists 75.8.
template <typename ListsLds>
int choose_layout(const IntraCtx &ctx, int n_pairs, const Device &dev, ListsLds lists_lds)
{
    if (ctx.layout >= 0) return ctx.layout;
    if (ctx.form == DSDP_INTRA_ATOMS) return kFormAtoms;
    if (ctx.score) {
        if (ctx.chains > 20 * dev.cus) return kFormStream;
        if (ctx.chains <= resident_lists(lists_lds(1), 1, dev)) return kFormPairs;
        return ctx.form == DSDP_INTRA_AUTO ? kFormAtoms : kFormStream;
    }
    const bool by_mix = ctx.form == DSDP_INTRA_AUTO && ctx.mixed;
    const int waves = ctx.waves > 0 ? ctx.waves
                                    : waves_for(ctx.chains, ctx.bb || by_mix ? kListWaves : kStreamWaves, dev.cus);
    if (by_mix) return waves == 1 ? kFormStream : kFormAtoms;
    if (waves == 1 && n_pairs <= kStreamPairs * 5 / 4) return kFormStream;
    if (waves > 1 && ctx.bb) return kFormPairs;
    return ctx.chains <= resident_lists(lists_lds(waves), waves, dev) ? kFormPairs : kFormStream;
}

}  // namespace host
}  // namespace dsdp
