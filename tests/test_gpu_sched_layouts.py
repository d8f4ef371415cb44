"""GPU: the scheduler's two layouts of a ligand.  A request holds atom lists; from four
chains a compute unit on, the running requests search by the pair stream where the pool
has room for it."""
import numpy as np
import pytest

import paper_2303_09916_amd as D
from synth import make_ligand, make_receptor, make_box, make_site_points, PALETTE_T9
from helpers import box32

pytestmark = pytest.mark.gpu

TYPES = list(PALETTE_T9)


def receptor(seed=4):
    rec = make_receptor(300, radius=12.0, seed=seed)
    return rec, box32(make_box(rec.pocket, 14.0, spacing=0.5))


def ligand(atoms, tors):
    return D.Ligand.from_synth(make_ligand(atoms, tors, seed=atoms, palette=PALETTE_T9))


class Sched:
    """A scheduler on a pool of its fixed part and `room` bytes."""

    def __init__(self, room, slots=4096, spt=1, params=None, recs=1):
        import gpu_common as gc
        self.pool = gc.dev_bytes(gc.torch_cuda(), D.dsdp_sched_fixed_bytes(slots) + room)
        self.h = D.dsdp_sched_create(self.pool, slots, spt, params)
        self.recs = [receptor(4 + k) for k in range(recs)]
        self.ids = [D.dsdp_sched_add_receptor(self.h, r.xyz, r.types, b, TYPES) for r, b in self.recs]

    def submit(self, L, chains, steps, seed, rec=0, top_k=3):
        return D.dsdp_sched_submit(self.h, self.ids[rec], L, chains, steps, seed, top_k)

    def tick(self, n=1):
        for _ in range(n):
            D.dsdp_sched_tick(self.h)

    def info(self):
        return D.dsdp_sched_get_info(self.h)

    def poses(self, ticket, top_k=3):
        state, poses, _, _ = D.dsdp_sched_poll(self.h, ticket, top_k)
        assert state == D.DSDP_REQ_DONE
        return [bytes(p) for p in poses]

    def finish(self, limit=400):
        for _ in range(limit):
            i = self.info()
            if i.queued == 0 and i.running == 0:
                return
            self.tick()
        raise AssertionError("scheduler made no progress")

    def __enter__(self):
        return self

    def __exit__(self, *exc):
        D.dsdp_sched_destroy(self.h)


def test_first_request_of_a_receptor_gets_the_stream():
    """Requests that bring their receptor's maps into the pool hold the same layouts there
    as requests that find them."""
    L = ligand(47, 9)
    free = []
    for warm in (True, False):
        with Sched(64 << 20) as s:
            if warm:
                s.submit(L, 8, 1, 1)
                s.tick()
                assert s.info().completed == 1
            for k in range(2):
                s.submit(L, 700, 3, 5 + k)
            s.tick()
            assert s.info().running == 2
            free.append(s.info().pool_free)
            s.finish()
    assert free[0] == free[1]


def ligand_bytes(L):
    """Pool bytes of a request's ligand as atom lists."""
    with Sched(64 << 20, slots=64, params=D.dsdp_params_default(intra_form=D.DSDP_INTRA_ATOMS)) as s:
        s.submit(L, 4, 1, 1)
        s.tick()
        free = s.info().pool_free
        s.submit(L, 4, 2, 1)
        s.tick()
        return free - s.info().pool_free


def maps_bytes(k):
    rec, box = receptor(4 + k)
    return (-(-D.dsdp_grids_bytes(box, len(TYPES)) // 256) * 256,
            -(-D.dsdp_build_grids_workspace_bytes(rec.n, box) // 256) * 256)


def alone(L, chains, steps, seed, rec=0, top_k=3, params=None, site=None):
    import gpu_common as gc
    r, box = receptor(4 + rec)
    g = gc.GpuGrid(r.xyz, r.types, box, TYPES)
    if site is not None:
        D.dsdp_grids_set_site(g.handle, *site)
    ws = gc.dev_bytes(g.torch, D.dsdp_dock_workspace_bytes(L, chains))
    return [bytes(p) for p in D.dsdp_dock(g.handle, L, chains, steps, seed, top_k, ws, params)[0]]


@pytest.mark.parametrize("waves", [0, 1])
def test_pool_sized_for_atom_lists_admits_as_many(waves):
    """A pool with room for the maps and the atom lists of 30 requests runs 30 at once,
    above the chain count from which they would search by the pair stream."""
    L = ligand(47, 9)
    maps, build = maps_bytes(0)
    one = ligand_bytes(L)
    assert build <= 30 * one
    with Sched(maps + 30 * one, params=D.dsdp_params_default(waves_per_chain=waves)) as s:
        s.submit(L, 4, 1, 1)     # brings the maps in
        s.tick()
        assert s.info().completed == 1
        t = [s.submit(L, 40, 3, 50 + k) for k in range(31)]
        s.tick()
        assert s.info().running == 30 and s.info().queued == 1
        s.finish()
        for k in (0, 29, 30):
            assert s.poses(t[k]) == alone(L, 40, 3, 50 + k)


def test_streams_make_way_for_maps():
    """Pair streams that lie in the pool do not keep another receptor's maps, or another
    request's ligand, out of it."""
    L = ligand(47, 9)
    (m0, b0), (m1, b1) = maps_bytes(0), maps_bytes(1)
    one = ligand_bytes(L)
    with Sched(m0 + m1 + b1 + 3 * one + 256, recs=2) as s:
        t = [s.submit(L, 700, 6, 60 + k) for k in range(2)]
        s.tick()
        s.tick()
        assert s.info().running == 2
        t.append(s.submit(L, 24, 4, 62, rec=1))
        s.tick()
        assert s.info().running == 3 and s.info().resident_receptors == 2 and s.info().evictions == 0
        s.finish()
        assert s.info().free_slots == 4096
        want = [alone(L, 700, 6, 60), alone(L, 700, 6, 61), alone(L, 24, 4, 62, rec=1)]
        assert [s.poses(x) for x in t] == want


@pytest.mark.parametrize("tight", [False, True])
@pytest.mark.parametrize("sites", [False, True])
@pytest.mark.parametrize("optimizer", [D.DSDP_OPT_BFGS, D.DSDP_OPT_BB])
def test_layout_changes_between_ticks(optimizer, sites, tight):
    """A small request ticks alone (atom lists), beside one that lifts the running chains
    over the limit (pair stream, where the pool holds it) and is cancelled, alone again,
    and beside a second such request; it and the second equal docking alone."""
    params = D.dsdp_params_default(optimizer=optimizer, bb_iters=12)
    small, large, other = ligand(33, 8), ligand(47, 9), ligand(26, 6)
    rec, _ = receptor(4)
    site = (make_site_points(rec, n=70, radius=5.0, clearance=2.5), 6.0) if sites else None
    maps, build = maps_bytes(0)
    room = maps + build + 2048 + ligand_bytes(small) + max(ligand_bytes(large), ligand_bytes(other)) if tight else 64 << 20
    with Sched(room, spt=2, params=params) as s:
        if sites:
            D.dsdp_sched_set_site(s.h, s.ids[0], *site)
        a = s.submit(small, 30, 13, 7)
        s.tick()
        b = s.submit(large, 1200, 40, 8)
        s.tick(2)
        assert s.info().running == 2
        D.dsdp_sched_cancel(s.h, b)
        s.tick()
        assert s.info().running == 1
        c = s.submit(other, 1100, 5, 9)
        s.finish()
        assert D.dsdp_sched_poll(s.h, b, 3)[0] == D.DSDP_REQ_CANCELLED
        assert s.poses(a) == alone(small, 30, 13, 7, params=params, site=site)
        assert s.poses(c) == alone(other, 1100, 5, 9, params=params, site=site)
        assert s.info().free_slots == 4096
