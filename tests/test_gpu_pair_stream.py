"""GPU: the layouts of the intra-ligand term and the waves per chain move speed only.
Docks, refinements and scores are equal bit for bit between the pair stream (one
chain or pose per wave, one to four to a workgroup, or several waves), the pair
lists and the atom lists, at pair counts around the stream's chunks of 127 pairs and
chain counts that leave a workgroup partly filled."""
import numpy as np
import pytest

import paper_2303_09916_amd as D
from synth import make_ligand, make_receptor, make_box, PALETTE_T9
from helpers import box32

pytestmark = pytest.mark.gpu

PAIRS, ATOMS = 1, 2


@pytest.fixture(scope="module")
def grid():
    import gpu_common as gc
    rec = make_receptor(300, radius=12.0, seed=4)
    return gc.GpuGrid(rec.xyz, rec.types, box32(make_box(rec.pocket, 14.0, spacing=0.5)), PALETTE_T9)


def params(form, waves, **over):
    return D.dsdp_params_default(intra_form=form, waves_per_chain=waves, tune=0, **over)


def chain_bits(grid, lig, n_chains, steps, p):
    import gpu_common as gc
    poses, xyz, chains, st = gc.gpu_dock(grid, lig, n_chains, steps, 11, 5, p)
    rec = np.array([list(c.pos) + list(c.quat) + list(c.tors) + [c.e_total, c.e_inter, c.e_intra, c.e_wall]
                    for c in chains], np.float32)
    return rec, np.array([p_.chain for p_ in poses]), xyz, st.pose_evals, st.accepted


def same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a, b))


# atoms, torsions: no pairs; a handful; around one chunk; around two; several; the largest
SHAPES = [(5, 0), (8, 2), (19, 4), (20, 5), (26, 6), (33, 8), (47, 9), (64, 31)]


@pytest.mark.parametrize("atoms,tors", SHAPES)
def test_layouts_give_the_same_bits(grid, atoms, tors):
    lig = make_ligand(atoms, tors, seed=atoms, palette=PALETTE_T9)
    for over in ({}, {"optimizer": D.DSDP_OPT_BB, "bb_iters": 12}):
        ref = chain_bits(grid, lig, 9, 3, params(ATOMS, 1, **over))
        for form, waves in ((PAIRS, 1), (PAIRS, 2), (PAIRS, 4), (ATOMS, 3)):
            assert same(chain_bits(grid, lig, 9, 3, params(form, waves, **over)), ref), (over, form, waves)


@pytest.mark.parametrize("n_chains", [1027, 2051, 4099])
def test_chains_that_share_a_workgroup(grid, n_chains):
    """1027: several waves, in rounds; 2051 and 4099: two and four chains a workgroup,
    the last one partly filled."""
    lig = make_ligand(30, 6, seed=3, palette=PALETTE_T9)
    ref = chain_bits(grid, lig, n_chains, 1, params(ATOMS, 1))
    for waves in (1, 2, 3):
        assert same(chain_bits(grid, lig, n_chains, 1, params(PAIRS, waves)), ref), waves
    assert same(chain_bits(grid, lig, n_chains, 1, params(0, 0)), ref)


@pytest.mark.parametrize("n_chains", [513, 1024, 1537, 2049, 3072])
@pytest.mark.parametrize("atoms,tors", [(20, 5), (47, 9), (60, 12)])
def test_automatic_choices_around_their_limits(grid, n_chains, atoms, tors):
    """The tuner's pick and the fixed rule, on both sides of the chain counts at which
    candidates are left out."""
    lig = make_ligand(atoms, tors, seed=atoms, palette=PALETTE_T9)
    ref = chain_bits(grid, lig, n_chains, 1, params(ATOMS, 1))
    assert same(chain_bits(grid, lig, n_chains, 1, params(0, 0)), ref)
    assert same(chain_bits(grid, lig, n_chains, 1, D.dsdp_params_default(tune=1)), ref)


@pytest.mark.parametrize("n", [1, 1030, 4101])
def test_refine_and_score(grid, n):
    import gpu_common as gc
    lig = make_ligand(41, 7, seed=8, palette=PALETTE_T9)
    L = D.Ligand.from_synth(lig)
    rng = np.random.default_rng(n)
    poses = np.zeros((n, L.nx), np.float32)
    poses[:, :3] = rng.uniform(np.asarray(grid.origin), np.asarray(grid.origin) + (np.asarray(grid.n) - 1) * 0.5, (n, 3))
    q = rng.normal(size=(n, 4))
    poses[:, 3:7] = q * rng.uniform(0.2, 3.0, (n, 1))      # quaternions of any length
    poses[:, 7:] = rng.uniform(-np.pi, np.pi, (n, L.n_tors))
    poses[0, 3:7] = (1e-21, 0.0, 2e-21, 0.0)               # whose squared length is denormal
    ref = gc.gpu_local_opt(grid, lig, poses, params(ATOMS, 1))
    assert np.isfinite(ref[1]).all()
    for form, waves in ((PAIRS, 1), (PAIRS, 2), (PAIRS, 4), (0, 0)):
        assert same(gc.gpu_local_opt(grid, lig, poses, params(form, waves)), ref), (form, waves)
    ref = gc.gpu_eval(grid, lig, poses, params(ATOMS, 1))
    for form, waves in ((PAIRS, 1), (PAIRS, 2), (0, 0)):
        assert same(gc.gpu_eval(grid, lig, poses, params(form, waves)), ref), (form, waves)


def test_batch_of_mixed_sizes(grid):
    """A batch that shares launches between ligands of every size equals its docks alone,
    with chains that do not divide into workgroups."""
    import gpu_common as gc
    torch = grid.torch
    ligs = [make_ligand(a, t, seed=a, palette=PALETTE_T9) for a, t in SHAPES]
    Ls = [D.Ligand.from_synth(l) for l in ligs]
    n_chains = 519
    ws = gc.dev_bytes(torch, D.dsdp_dock_batch_workspace_bytes(Ls, n_chains))
    seeds = list(range(100, 100 + len(Ls)))
    for p in (params(PAIRS, 1), params(0, 0), None):
        res, _ = D.dsdp_dock_batch(grid.handle, Ls, n_chains, 2, seeds, 3, ws, p)
        for lig, L, seed, got in zip(ligs, Ls, seeds, res):
            w1 = gc.dev_bytes(torch, D.dsdp_dock_workspace_bytes(L, n_chains))
            want, _, _, _ = D.dsdp_dock(grid.handle, L, n_chains, 2, seed, 3, w1, params(ATOMS, 1))
            assert [(x.chain, x.e_total, list(x.pos)) for x in got] == [(x.chain, x.e_total, list(x.pos)) for x in want]


def test_members_that_need_most_lds_differ(grid):
    """A launch's LDS covers every member at its shape: of a ligand with many pairs and few
    torsions (large lists) and one with few atoms and many torsions (large chain state) the
    first needs more for one chain and the second for four; also through the scheduler."""
    import gpu_common as gc
    torch = grid.torch
    ligs = [make_ligand(46, 3, seed=5, palette=PALETTE_T9), make_ligand(36, 20, seed=6, palette=PALETTE_T9)]
    ligs += [make_ligand(60, 12, seed=7, palette=PALETTE_T9), make_ligand(44, 28, seed=9, palette=PALETTE_T9)]
    Ls = [D.Ligand.from_synth(l) for l in ligs]
    n_chains, steps = 1100, 2
    want = []
    for k, L in enumerate(Ls):
        w1 = gc.dev_bytes(torch, D.dsdp_dock_workspace_bytes(L, n_chains))
        want.append(D.dsdp_dock(grid.handle, L, n_chains, steps, 40 + k, 3, w1, params(ATOMS, 1))[0])

    def key(poses):
        return [(x.chain, x.e_total, list(x.pos), list(x.tors)) for x in poses]

    for lo, hi in ((0, 2), (2, 4), (0, 4)):
        ws = gc.dev_bytes(torch, D.dsdp_dock_batch_workspace_bytes(Ls[lo:hi], n_chains))
        for p in (params(PAIRS, 1), params(PAIRS, 2), params(ATOMS, 2), None):
            res, _ = D.dsdp_dock_batch(grid.handle, Ls[lo:hi], n_chains, steps, list(range(40 + lo, 40 + hi)), 3, ws, p)
            assert [key(r) for r in res] == [key(w) for w in want[lo:hi]], (lo, hi)
    rec = make_receptor(300, radius=12.0, seed=4)
    box = box32(make_box(rec.pocket, 14.0, spacing=0.5))
    pool = gc.dev_bytes(torch, D.dsdp_sched_fixed_bytes(8192) + (64 << 20))
    h = D.dsdp_sched_create(pool, 8192, 1)
    try:
        rid = D.dsdp_sched_add_receptor(h, rec.xyz, rec.types, box, list(PALETTE_T9))
        t = [D.dsdp_sched_submit(h, rid, L, n_chains, steps, 40 + k, 3) for k, L in enumerate(Ls)]
        for _ in range(8):
            D.dsdp_sched_tick(h)
        for k, ticket in enumerate(t):
            assert key(D.dsdp_sched_poll(h, ticket, 3)[1]) == key(want[k]), k
    finally:
        D.dsdp_sched_destroy(h)


def test_scoring_from_the_contiguous_copy():
    """Enough poses on large enough maps are scored from a copy of the maps with contiguous
    cells; the results are those of the same poses scored in small sets, which are not.
    Odd node counts, poses at and beyond every face."""
    import gpu_common as gc
    rec = make_receptor(300, radius=12.0, seed=4)
    g = gc.GpuGrid(rec.xyz, rec.types, box32(make_box(rec.pocket, (12.4, 13.3, 11.6), spacing=0.15)), PALETTE_T9)
    torch = g.torch
    nodes = int(np.prod(g.n)) * len(PALETTE_T9)
    assert nodes * 16 >= 32 << 20 and min(g.n) % 2 + max(g.n) % 2 >= 1
    lig = make_ligand(30, 5, seed=2, palette=PALETTE_T9)
    L = D.Ligand.from_synth(lig)
    n = 4 * nodes // L.n_atoms + 777
    gen = torch.Generator(device="cuda").manual_seed(5)
    P = torch.rand((n, L.nx), generator=gen, device="cuda")
    lo = torch.tensor(np.asarray(g.origin, np.float32), device="cuda")
    ext = torch.tensor([(a - 1) * 0.15 for a in g.n], device="cuda", dtype=torch.float32)
    P[:, :3] = lo - 2.0 + P[:, :3] * (ext + 4.0)
    P[:, 3:] = P[:, 3:] * 2 - 1
    P[:, 7:] *= np.pi
    E = torch.empty((n, 4), device="cuda")
    G = torch.empty((n, L.D), device="cuda")
    ws = gc.dev_bytes(torch, D.dsdp_dock_workspace_bytes(L, n))
    D.dsdp_eval_poses(g.handle, L, P, n, E, G, None, ws)
    small = n // 9
    for k in list(range(0, n - small, small))[:9]:
        e, gr = torch.empty((small, 4), device="cuda"), torch.empty((small, L.D), device="cuda")
        D.dsdp_eval_poses(g.handle, L, P[k:k + small].contiguous(), small, e, gr, None, ws)
        assert torch.equal(e, E[k:k + small]) and torch.equal(gr, G[k:k + small])


@pytest.mark.parametrize("atoms,tors", SHAPES)
def test_calls_in_a_row_with_ligands_of_every_size(grid, atoms, tors):
    """A ligand reaches the device as kernel arguments or as a copy, by its size: two
    ligands scored one after the other on one workspace, without a wait between, do not
    disturb each other, in either layout."""
    torch = grid.torch
    Ls = [D.Ligand.from_synth(make_ligand(a, t, seed=a, palette=PALETTE_T9)) for a, t in ((atoms, tors), (33, 8))]
    n = 40
    ws = torch.empty(max(D.dsdp_dock_workspace_bytes(L, n) for L in Ls), dtype=torch.uint8, device="cuda")
    lo = torch.tensor(np.asarray(grid.origin, np.float32), device="cuda")
    P = [torch.rand((n, L.nx), device="cuda") for L in Ls]
    for p in P:
        p[:, :3] = p[:, :3] * 13.0 + lo

    def score(k, form):
        e = torch.empty((n, 4), device="cuda")
        g = torch.empty((n, Ls[k].D), device="cuda")
        D.dsdp_eval_poses(grid.handle, Ls[k], P[k], n, e, g, None, ws, params(form, 0))
        return e, g

    alone = []
    for k in (0, 1):
        alone.append(score(k, ATOMS))
        torch.cuda.synchronize()
    got = [score(k, f) for _ in range(3) for k in (0, 1) for f in (PAIRS, ATOMS)]
    torch.cuda.synchronize()
    for i, (e, g) in enumerate(got):
        k = (i // 2) % 2
        assert torch.equal(e, alone[k][0]) and torch.equal(g, alone[k][1])
