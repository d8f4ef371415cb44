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
