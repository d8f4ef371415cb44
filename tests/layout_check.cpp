// Host unit check of the layout rules on a device of 256 compute units with 160 KB of
// LDS each.  Built and run by tests/test_layout.py.
#include "layout.h"

#include <cstdio>

using namespace dsdp;
using namespace dsdp::host;

static int failures = 0;
#define CHECK(c)                                                                       \
    do {                                                                               \
        if (!(c)) {                                                                    \
            std::fprintf(stderr, "layout check failed: %s (line %d)\n", #c, __LINE__); \
            failures++;                                                                \
        }                                                                              \
    } while (0)

static const Device kDev{256, 160 << 10};

static IntraCtx ctx(int form, int waves, long chains, bool mixed = false, bool bb = false)
{
    IntraCtx c;
    c.form = form;
    c.waves = waves;
    c.chains = chains;
    c.mixed = mixed;
    c.bb = bb;
    return c;
}

int main()
{
    const int AUTO = DSDP_INTRA_AUTO, PAIRS = DSDP_INTRA_PAIRS, ATOMS = DSDP_INTRA_ATOMS;
    // a ligand whose pair lists leave four one-wave and two four-wave workgroups on a unit
    auto lds = [](int waves) { return (size_t)25000 + 13000 * (size_t)waves; };
    auto pick = [&](const IntraCtx &c, int n_pairs = 868) { return choose_layout(c, n_pairs, kDev, lds); };

    CHECK(waves_for(1, 8, 256) == 4 && waves_for(683, 8, 256) == 2 && waves_for(1025, 8, 256) == 1);
    CHECK(waves_for(1024, 12, 256) == 3 && waves_for(1536, 12, 256) == 2 && waves_for(1537, 12, 256) == 1);
    CHECK(resident_lists(lds(1), 1, kDev) == 1024 && resident_lists(lds(4), 4, kDev) == 512);
    CHECK(resident_lists(4000, 1, kDev) == 2048 && resident_lists(4000, 3, kDev) == 512);

    // one wave per chain: lists while all workgroups are resident, then the stream
    for (bool bb : {false, true})
        for (int form : {AUTO, PAIRS}) {
            CHECK(pick(ctx(form, 1, 9, false, bb)) == kFormPairs);
            CHECK(pick(ctx(form, 1, 1024, false, bb)) == kFormPairs);
            CHECK(pick(ctx(form, 1, 1025, false, bb)) == kFormStream);
            CHECK(pick(ctx(form, 1, 1 << 20, false, bb)) == kFormStream);
        }
    // a chunk and a quarter of pairs: the stream at once
    CHECK(pick(ctx(AUTO, 1, 9), 158) == kFormStream && pick(ctx(AUTO, 1, 9), 159) == kFormPairs);
    // several waves: the same rule for BFGS; lists for Barzilai-Borwein
    CHECK(pick(ctx(AUTO, 0, 512)) == kFormPairs && pick(ctx(AUTO, 0, 513)) == kFormStream);
    CHECK(pick(ctx(PAIRS, 4, 512)) == kFormPairs && pick(ctx(PAIRS, 4, 4096)) == kFormStream);
    CHECK(pick(ctx(AUTO, 4, 4096, false, true)) == kFormPairs && pick(ctx(PAIRS, 2, 4096, false, true)) == kFormPairs);
    // Barzilai-Borwein never has the stream at several waves (no such kernel)
    for (int form : {AUTO, PAIRS, ATOMS})
        for (int waves = 2; waves <= 4; waves++)
            for (long chains : {1L, 512L, 1025L, 100000L})
                for (bool mixed : {false, true}) CHECK(pick(ctx(form, waves, chains, mixed, true)) != kFormStream);
    // several ligands: atom lists until a wave per chain fills the device
    CHECK(pick(ctx(AUTO, 0, 1024, true)) == kFormAtoms && pick(ctx(AUTO, 0, 1025, true)) == kFormStream);
    CHECK(pick(ctx(AUTO, 1, 9, true)) == kFormStream && pick(ctx(AUTO, 2, 9000, true)) == kFormAtoms);
    // scoring: lists while resident, then atom lists (unless pairs are asked for), then the
    // stream; the waves asked for play no part
    for (int waves = 0; waves <= 4; waves++) {
        auto score = [&](int form, long poses) {
            IntraCtx c = ctx(form, waves, poses);
            c.score = true;
            return pick(c);
        };
        CHECK(score(AUTO, 1) == kFormPairs && score(AUTO, 1024) == kFormPairs && score(PAIRS, 1024) == kFormPairs);
        CHECK(score(AUTO, 1025) == kFormAtoms && score(AUTO, 5120) == kFormAtoms && score(PAIRS, 5120) == kFormStream);
        CHECK(score(AUTO, 5121) == kFormStream && score(PAIRS, 5121) == kFormStream && score(ATOMS, 1 << 20) == kFormAtoms);
    }
    // refinements: two waves where a search's chains would take one, up to 16 poses a unit
    CHECK(refine_waves(1536, 256) == 0 && refine_waves(1537, 256) == 2 && refine_waves(4096, 256) == 2 &&
          refine_waves(4097, 256) == 0 && refine_waves(0, 256) == 0);
    // what is asked for
    CHECK(pick(ctx(ATOMS, 1, 9)) == kFormAtoms && pick(ctx(ATOMS, 0, 9000, true)) == kFormAtoms);
    for (int f : {kFormPairs, kFormAtoms, kFormStream}) {
        IntraCtx c = ctx(ATOMS, 1, 4096, true, true);
        c.layout = f;
        CHECK(pick(c) == f);
    }
    if (failures) return 1;
    std::printf("the rules are as specified\n");
    return 0;
}
