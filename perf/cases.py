"""Workloads of the docking library, through its public entry points.

A case is one call (or one short program) that a user of the library runs: building a
receptor's maps, scoring poses, refining poses, docking one ligand, docking a library of
ligands, serving a stream of requests, and extracting a binding site from a score volume.
Sizes follow the repository's own workloads (a 43^3, an 81^3 and a 107^3 node box, ligands
of 10-60 heavy atoms with 0-15 rotatable bonds, 32-384 chains); ``draw`` gives others of the
same ranges.

Inputs are synthetic and made from the seed alone: a receptor is a jittered lattice of heavy
atoms (0.025 per cubic Angstrom, at least 2.8 A apart) in a ball with a cleared pocket near
its surface, a ligand is a random tree of 1.5 A bonds cut into rigid fragments.
"""
import math

import numpy as np
import torch

import paper_2303_09916_amd as D

# XS codes: C_H 0, C_P 1, N_P 2, N_D 3, N_A 4, N_DA 5, O_A 8, O_DA 9, S_P 10
T4 = (0, 1, 4, 8)
T8 = (0, 1, 2, 3, 4, 8, 9, 10)
T9 = T8 + (5,)
T17 = tuple(range(17))
PALETTES = {4: T4, 8: T8, 9: T9, 17: T17}


# ------------------------------------------------------------------ cases
def listed():
    return [
        # the maps of a small receptor: a quick re-docking's fixed cost
        {"name": "maps_small", "kind": "maps", "rec": 300, "bx": 16.0, "by": 16.0, "bz": 16.0, "h": 0.375, "types": 4},
        # the maps of a usual request: the paper's 30 A search cube
        {"name": "maps_cube", "kind": "maps", "rec": 4000, "bx": 30.0, "by": 30.0, "bz": 30.0, "h": 0.375, "types": 8},
        # the maps of a large complex
        {"name": "maps_large", "kind": "maps", "rec": 12000, "bx": 40.0, "by": 40.0, "bz": 40.0, "h": 0.375, "types": 9},
        # re-scoring a handful of output poses, coordinates wanted
        {"name": "score_few", "kind": "score", "rec": 300, "box": 16.0, "types": 4, "atoms": 20, "tors": 4, "poses": 96,
         "xyz": True},
        # scoring a large pool of poses
        {"name": "score_pool", "kind": "score", "rec": 4000, "box": 30.0, "types": 8, "atoms": 32, "tors": 7,
         "poses": 1 << 20, "xyz": False},
        # refining given poses of a larger ligand (more than 32 atoms: another lane layout)
        {"name": "refine", "kind": "refine", "rec": 4000, "box": 30.0, "types": 9, "atoms": 47, "tors": 9, "poses": 1000,
         "opt": "bfgs", "site": False},
        # the smallest dock: few chains, one small ligand
        {"name": "dock_small", "kind": "dock", "rec": 300, "box": 16.0, "types": 4, "atoms": 20, "tors": 4, "chains": 32,
         "steps": 200, "opt": "bfgs", "site": False},
        # the usual dock: the paper's many-copies search of one drug-like ligand
        {"name": "dock_usual", "kind": "dock", "rec": 4000, "box": 30.0, "types": 8, "atoms": 32, "tors": 7, "chains": 384,
         "steps": 2000, "opt": "bfgs", "site": False},
        # the paper's own optimiser and one of its copies x steps settings, in a predicted site's search space
        {"name": "dock_bb_site", "kind": "dock", "rec": 4000, "box": 30.0, "types": 9, "atoms": 26, "tors": 6, "chains": 384,
         "steps": 40, "opt": "bb", "site": True},
        # a slice of a virtual-screening library against one receptor
        {"name": "library", "kind": "library", "rec": 4000, "box": 30.0, "types": 9, "ligands": 128, "chains": 128,
         "steps": 200, "opt": "bfgs"},
        # a burst of requests on a serving pool that keeps its receptors' maps
        {"name": "serving", "kind": "serving", "receptors": 4, "types": 9, "requests": 96, "chains": 128, "steps": 100,
         "tick": 25, "slots": 8192},
        # the binding site of a 36^3 score volume: its top 200 voxels, clustered
        {"name": "site", "kind": "site", "n": 36, "top": 200},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["maps", "maps", "score", "score", "refine", "dock", "dock", "dock", "library", "serving", "site"])
    if kind == "maps":
        h = rng.choice([0.375, 0.375, 0.3, 0.5])
        b = [round(rng.uniform(12.0, 40.0 if h >= 0.375 else 30.0), 2) for _ in range(3)]
        return {"kind": kind, "rec": _log(rng, 200, 12000), "bx": b[0], "by": b[1], "bz": b[2], "h": h,
                "types": rng.choice([4, 8, 9, 17])}
    na = rng.randint(6, 60)
    nt = min(rng.randint(0, 15), max(0, na // 3))
    box = round(rng.uniform(16.0, 30.0), 2)
    rec, types = _log(rng, 300, 8000), rng.choice([8, 9])
    opt = rng.choice(["bfgs", "bfgs", "bb"])
    if kind == "score":
        return {"kind": kind, "rec": rec, "box": box, "types": types, "atoms": na, "tors": nt, "poses": _log(rng, 1, 1 << 20),
                "xyz": rng.random() < 0.5}
    if kind == "refine":
        return {"kind": kind, "rec": rec, "box": box, "types": types, "atoms": na, "tors": nt, "poses": _log(rng, 1, 8192),
                "opt": opt, "site": rng.random() < 0.3}
    if kind == "dock":
        chains = _log(rng, 16, 2048)
        steps = _log(rng, 10, max(11, min(400, 120000 // chains)))
        return {"kind": kind, "rec": rec, "box": box, "types": types, "atoms": na, "tors": nt, "chains": chains,
                "steps": max(5, steps // 4) if opt == "bb" else steps, "opt": opt, "site": rng.random() < 0.3}
    if kind == "library":
        n, chains = _log(rng, 3, 160), _log(rng, 16, 128)
        return {"kind": kind, "rec": rec, "box": box, "types": 9, "ligands": n, "chains": chains, "steps": _log(rng, 10, 150),
                "opt": "bfgs"}
    if kind == "serving":
        return {"kind": kind, "receptors": rng.randint(1, 6), "types": 9, "requests": _log(rng, 4, 96),
                "chains": _log(rng, 16, 128), "steps": _log(rng, 10, 100), "tick": rng.choice([10, 25, 50]), "slots": 8192}
    return {"kind": "site", "n": rng.randint(16, 64), "top": _log(rng, 20, 1000)}


# ------------------------------------------------------------------ inputs
def _receptor(n, rng):
    """Coordinates, XS types and the pocket point of a synthetic receptor."""
    a = 0.025 ** (-1.0 / 3.0)
    R = (3.0 * n / (4.0 * math.pi * 0.025)) ** (1.0 / 3.0)
    m = int(math.ceil((1.4 * R + 8.0) / a))
    g = np.arange(-m, m + 1) * a
    P = np.stack(np.meshgrid(g, g, g, indexing="ij"), axis=-1).reshape(-1, 3) + rng.uniform(-0.5, 0.5, 3) * a
    P = P + rng.uniform(-0.5, 0.5, P.shape) * (a - 2.8)
    u = rng.normal(size=3)
    pocket = u / np.linalg.norm(u) * (R - 4.0)
    P = P[np.sum((P - pocket) ** 2, axis=1) >= 36.0]
    P = P[np.argsort(np.sum(P * P, axis=1), kind="stable")[:n]]
    P = P[rng.permutation(n)]
    q = np.linalg.qr(rng.normal(size=(3, 3)))[0]
    p = np.array([0.45 * .65, .55 * .65, .7 * .17, .15 * .17, .1 * .17, .05 * .17, .75 * .17, .25 * .17, .01])
    types = rng.choice([1, 0, 3, 2, 4, 5, 8, 9, 10], size=n, p=p / p.sum()).astype(np.int32)
    return (P @ q.T).astype(np.float32), types, pocket @ q.T


def _grow(n, rng):
    pos, elem, nb = [np.zeros(3)], ["C"], [[]]
    cap = {"C": 4, "N": 3, "O": 2, "S": 2}
    fails = 0
    while len(pos) < n:
        host = int(rng.integers(len(pos)))
        if len(nb[host]) >= cap[elem[host]]:
            fails += 1
            if fails > 2000:
                return None
            continue
        d = rng.normal(size=(16, 3))
        d /= np.linalg.norm(d, axis=1, keepdims=True)
        ok = np.ones(16, bool)
        for j in nb[host]:
            ok &= d @ ((pos[j] - pos[host]) / 1.5) <= -0.17
        X = pos[host] + 1.5 * d
        far = [k for k in range(len(pos)) if k != host and k not in nb[host]]
        if far:
            ok &= (np.sum((X[:, None] - np.array([pos[k] for k in far])[None]) ** 2, -1) >= 6.25).all(1)
        if not ok.any():
            fails += 1
            if fails > 2000:
                return None
            continue
        k = len(pos)
        pos.append(X[int(np.argmax(ok))])
        elem.append(str(rng.choice(["C", "N", "O", "S"], p=[.70, .12, .15, .03])))
        nb.append([host])
        nb[host].append(k)
    return np.array(pos), elem, nb


def _ligand(n, n_tors, palette, rng):
    """A random ligand tree as the arguments of D.Ligand: fragment-contiguous, parents first."""
    while (g := _grow(n, rng)) is None or sum(len(g[2][a]) > 1 and len(g[2][b]) > 1 for a in range(n) for b in g[2][a]) < 2 * min(n_tors, n // 3):
        pass
    pos, elem, nb = g
    opts = {"N": [(3, .7), (2, .15), (4, .1), (5, .05)], "O": [(8, .75), (9, .25)], "S": [(10, 1.)]}
    types = np.zeros(n, np.int32)
    for i in range(n):
        o = [(t, w) for t, w in opts.get(elem[i], []) if t in palette]
        if o:
            w = np.array([x[1] for x in o])
            types[i] = o[int(rng.choice(len(o), p=w / w.sum()))][0]
        else:
            types[i] = 1 if any(elem[j] in "NO" for j in nb[i]) else 0
    bonds = [(i, j) for i in range(n) for j in nb[i] if i < j]
    can = [b for b in bonds if len(nb[b[0]]) > 1 and len(nb[b[1]]) > 1]
    rot = {can[int(k)] for k in rng.permutation(len(can))[:n_tors]}
    frag = [-1] * n
    nf = 0
    for s in range(n):
        if frag[s] < 0:
            todo, frag[s] = [s], nf
            while todo:
                u = todo.pop()
                for v in nb[u]:
                    if frag[v] < 0 and (min(u, v), max(u, v)) not in rot:
                        frag[v] = nf
                        todo.append(v)
            nf += 1
    adj = [[] for _ in range(nf)]
    for u, v in sorted(rot):
        adj[frag[u]].append((frag[v], u, v))
        adj[frag[v]].append((frag[u], v, u))

    def walk(r):
        order, par, dep = [r], {r: (-1, -1, -1)}, {r: 0}
        for f in order:
            for g_, a, b in adj[f]:
                if g_ not in par:
                    par[g_], dep[g_] = (f, a, b), dep[f] + 1
                    order.append(g_)
        return order, par, max(dep.values())

    order, par, _ = walk(min(range(nf), key=lambda f: (walk(f)[2], f)))
    perm = [i for f in order for i in range(n) if frag[i] == f]
    at = {old: k for k, old in enumerate(perm)}
    start = np.concatenate([[0], np.cumsum([frag.count(f) for f in order])]).astype(np.int32)
    num = {f: k for k, f in enumerate(order)}
    parent = np.array([num[par[f][0]] if par[f][0] >= 0 else -1 for f in order], np.int32)
    axis = np.array([[at[par[f][1]], at[par[f][2]]] if par[f][0] >= 0 else [-1, -1] for f in order], np.int32)
    bl = np.array(sorted((min(at[i], at[j]), max(at[i], at[j])) for i, j in bonds), np.int32).reshape(-1, 2)
    return pos[perm].astype(np.float32), types[perm], start, parent, axis, bl


def _rng(seed, what):
    return np.random.default_rng([int(seed), what])


def _box(centre, size, h=0.375):
    return {"centre": np.asarray(centre, np.float32), "size": np.broadcast_to(np.asarray(size, np.float32), (3,)).copy(),
            "spacing": float(np.float32(h))}


def _bytes(n):
    return torch.empty(max(int(n), 256), dtype=torch.uint8, device="cuda")


class _Maps:
    """Maps on the GPU and the library's handle of them."""

    def __init__(self, rec, types, box, palette):
        self.maps = _bytes(D.dsdp_grids_bytes(box, len(palette)))
        ws = _bytes(D.dsdp_build_grids_workspace_bytes(len(types), box))
        self.handle = D.dsdp_build_grids(rec, types, box, palette, self.maps, ws)
        torch.cuda.synchronize()

    def __del__(self):
        D.dsdp_grids_release(self.handle)


class _Sched:
    """A serving pool with its receptors registered."""

    def __init__(self, case, seed):
        n = case["receptors"]
        rng = _rng(seed, 1)
        sizes = [(int(rng.integers(2000, 8001)), float(rng.uniform(22.0, 30.0))) for _ in range(n)]
        recs = [(_receptor(a, _rng(seed, 20 + i)), b) for i, (a, b) in enumerate(sizes)]
        palette = list(PALETTES[case["types"]])
        need = D.dsdp_sched_fixed_bytes(case["slots"]) + (32 << 20)
        for (xyz, types, pocket), size in recs:
            b = _box(pocket, size)
            need += D.dsdp_grids_bytes(b, len(palette)) + D.dsdp_build_grids_workspace_bytes(len(types), b) + 65536
        self.pool = _bytes(need)
        self.handle = D.dsdp_sched_create(self.pool, case["slots"], case["tick"])
        self.ids = [D.dsdp_sched_add_receptor(self.handle, xyz, types, _box(pocket, size), palette)
                    for (xyz, types, pocket), size in recs]

    def __del__(self):
        D.dsdp_sched_destroy(self.handle)


def _shapes(n, rng):
    out = []
    for _ in range(n):
        na = int(rng.integers(10, 61))
        out.append((na, int(rng.integers(0, 16))))
    return out


def _poses(lig_tors, n, origin, extent, seed):
    """n poses: root uniform in the box, uniform orientation and torsions."""
    g = torch.Generator(device="cuda").manual_seed(int(seed) * 7 + 3)
    P = torch.rand((n, 7 + lig_tors), generator=g, device="cuda")
    P[:, :3] = P[:, :3] * torch.tensor(extent, device="cuda") + torch.tensor(origin, device="cuda")
    q = torch.randn((n, 4), generator=g, device="cuda")
    P[:, 3:7] = q / q.norm(dim=1, keepdim=True)
    P[:, 7:] = (P[:, 7:] * 2 - 1) * math.pi
    return P


def _site_points(rec, pocket, rng, n=200):
    out = np.zeros((0, 3))
    while len(out) < n:
        c = rng.uniform(-9, 9, (400, 3))
        c = c[np.sum(c * c, 1) <= 81] + pocket
        far = np.min(np.sum((c[:, None] - rec[None].astype(np.float64)) ** 2, -1), 1) >= 9
        out = np.concatenate([out, c[far]])
    return out[:n].astype(np.float32)


def _single(case, seed):
    """Receptor, box and ligand of a one-ligand case."""
    xyz, types, pocket = _receptor(case["rec"], _rng(seed, 1))
    palette = PALETTES[case["types"]]
    return xyz, types, pocket, _box(pocket, case["box"]), palette, _ligand(case["atoms"], case["tors"], palette, _rng(seed, 2))


def prepare(case, seed):
    kind = case["kind"]
    if kind == "maps":
        xyz, types, pocket = _receptor(case["rec"], _rng(seed, 1))
        box = _box(pocket, (case["bx"], case["by"], case["bz"]), case["h"])
        palette = list(PALETTES[case["types"]])
        n, _ = D.dsdp_grid_dims(box)
        maps = torch.empty((len(palette), n[2], n[1], n[0], 4), dtype=torch.float32, device="cuda")
        ws = _bytes(D.dsdp_build_grids_workspace_bytes(len(types), box))
        return {"kind": kind, "xyz": xyz, "types": types, "box": box, "palette": palette, "maps": maps, "ws": ws}
    if kind == "site":
        vol, origin = _volume(case, seed)
        return {"kind": kind, "vol": torch.from_numpy(vol).cuda(), "dims": (case["n"],) * 3, "origin": origin,
                "top": case["top"], "ws": _bytes(D.dsdp_site_points_workspace_bytes(case["top"]))}
    if kind == "serving":
        s = _Sched(case, seed)
        rng = _rng(seed, 2)
        reqs = []
        for k, (na, nt) in enumerate(_shapes(case["requests"], rng)):
            lig = D.Ligand(*_ligand(na, nt, PALETTES[case["types"]], _rng(seed, 1000 + k)))
            reqs.append((s.ids[int(rng.integers(len(s.ids)))], lig, int(rng.integers(1 << 40))))
        return {"kind": kind, "sched": s, "reqs": reqs, "chains": case["chains"], "steps": case["steps"]}
    if kind == "library":
        xyz, types, pocket = _receptor(case["rec"], _rng(seed, 1))
        palette = PALETTES[case["types"]]
        rng = _rng(seed, 2)
        ligs = [D.Ligand(*_ligand(na, nt, palette, _rng(seed, 1000 + k)))
                for k, (na, nt) in enumerate(_shapes(case["ligands"], rng))]
        return {"kind": kind, "maps": _Maps(xyz, types, _box(pocket, case["box"]), list(palette)), "ligs": ligs,
                "seeds": [int(rng.integers(1 << 40)) for _ in ligs], "chains": case["chains"], "steps": case["steps"],
                "ws": _bytes(D.dsdp_dock_batch_workspace_bytes(ligs, case["chains"]))}
    xyz, types, pocket, box, palette, lg = _single(case, seed)
    maps = _Maps(xyz, types, box, list(palette))
    lig = D.Ligand(*lg)
    if case.get("site"):
        D.dsdp_grids_set_site(maps.handle, _site_points(xyz, pocket, _rng(seed, 4)), 7.0)
    params = D.dsdp_params_default(optimizer=D.DSDP_OPT_BB if case.get("opt") == "bb" else D.DSDP_OPT_BFGS)
    st = {"kind": kind, "maps": maps, "lig": lig, "params": params}
    if kind == "dock":
        return st | {"chains": case["chains"], "steps": case["steps"], "seed": int(_rng(seed, 3).integers(1 << 40)),
                     "ws": _bytes(D.dsdp_dock_workspace_bytes(lig, case["chains"]))}
    n, origin = D.dsdp_grid_dims(box)
    np_ = case["poses"]
    extent = [(a - 1) * box["spacing"] for a in n]
    st |= {"poses": _poses(lig.n_tors, np_, origin.tolist(), extent, seed), "n": np_,
           "energy": torch.empty((np_, 4), device="cuda"), "ws": _bytes(D.dsdp_dock_workspace_bytes(lig, np_))}
    if kind == "score":
        return st | {"grad": torch.empty((np_, lig.D), device="cuda"),
                     "xyz": torch.empty((np_, lig.n_atoms, 3), device="cuda") if case["xyz"] else None}
    return st | {"out": torch.empty_like(st["poses"]), "evals": torch.empty((np_,), dtype=torch.int32, device="cuda")}


# ------------------------------------------------------------------ one pass
def _pose_table(poses, k):
    """Ranked poses as arrays of k rows (zero, chain -1, past the last pose): pose vectors, energies and scores, chains."""
    x, e, c = np.zeros((k, 38), np.float32), np.zeros((k, 5), np.float32), np.full(k, -1, np.int64)
    for i, p in enumerate(poses):
        x[i, :3], x[i, 3:7], x[i, 7:] = p.pos, p.quat, p.tors
        e[i], c[i] = (p.e_total, p.e_inter, p.e_intra, p.e_wall, p.score), p.chain
    return x, e, c


def run(s):
    kind = s["kind"]
    if kind == "maps":
        h = D.dsdp_build_grids(s["xyz"], s["types"], s["box"], s["palette"], s["maps"], s["ws"])
        D.dsdp_grids_release(h)
        return s["maps"]
    if kind == "score":
        D.dsdp_eval_poses(s["maps"].handle, s["lig"], s["poses"], s["n"], s["energy"], s["grad"], s["xyz"], s["ws"],
                          s["params"])
        return {"energy": s["energy"], "grad": s["grad"]} | ({"xyz": s["xyz"]} if s["xyz"] is not None else {})
    if kind == "refine":
        D.dsdp_local_opt(s["maps"].handle, s["lig"], s["poses"], s["n"], s["out"], s["energy"], s["evals"], s["ws"],
                         s["params"])
        return {"poses": s["out"], "energy": s["energy"], "evals": s["evals"]}
    if kind == "dock":
        poses, xyz, _, stats = D.dsdp_dock(s["maps"].handle, s["lig"], s["chains"], s["steps"], s["seed"], 9, s["ws"],
                                           s["params"])
        x, e, c = _pose_table(poses, 9)
        full = np.zeros((9,) + xyz.shape[1:], np.float32)
        full[:len(xyz)] = xyz
        return {"pose": x, "energy": e, "chain": c, "xyz": full, "evals": stats.pose_evals, "accepted": stats.accepted}
    if kind == "library":
        res, stats = D.dsdp_dock_batch(s["maps"].handle, s["ligs"], s["chains"], s["steps"], s["seeds"], 9, s["ws"])
        t = [_pose_table(p, 9) for p in res]
        return {"pose": np.concatenate([a for a, _, _ in t]), "energy": np.concatenate([b for _, b, _ in t]),
                "chain": np.concatenate([c for _, _, c in t]), "evals": stats.pose_evals, "accepted": stats.accepted}
    if kind == "serving":
        h = s["sched"].handle
        order = {D.dsdp_sched_submit(h, r, lig, s["chains"], s["steps"], seed, 9): k
                 for k, (r, lig, seed) in enumerate(s["reqs"])}
        got = [None] * len(s["reqs"])
        while order:
            D.dsdp_sched_tick(h)
            for t in D.dsdp_sched_drain(h):
                _, poses, _, stats = D.dsdp_sched_poll(h, t, 9)
                D.dsdp_sched_release(h, t)
                got[order.pop(t)] = _pose_table(poses, 9) + (stats.pose_evals,)
        return {"pose": np.concatenate([g[0] for g in got]), "energy": np.concatenate([g[1] for g in got]),
                "chain": np.concatenate([g[2] for g in got]), "evals": np.array([g[3] for g in got], np.int64)}
    points, labels, centre = D.dsdp_site_points(s["vol"], s["dims"], s["origin"], 2.0, s["top"], s["ws"])
    return {"points": points, "labels": labels, "centre": centre}


# ------------------------------------------------------------------ the work of a pass
def _inside(n_atoms, extent):
    """Share of a box (edges `extent`, centred 4 A below the surface of the receptor's ball) that the ball covers, about."""
    R = (3.0 * n_atoms / (4.0 * math.pi * 0.025)) ** (1.0 / 3.0)
    g = [np.linspace(-0.5, 0.5, 17) * e for e in extent]
    X, Y, Z = np.meshgrid(*g, indexing="ij")
    return float(np.mean(X * X + Y * Y + (Z + R - 4.0) ** 2 <= R * R))


def _radii(types):
    r = (1.9, 1.9, 1.8, 1.8, 1.8, 1.8, 1.7, 1.7, 1.7, 1.7, 2.0, 2.1, 1.5, 1.8, 2.0, 2.2, 1.2)
    return len({r[t] for t in PALETTES[types]})


def work(case):
    """Bytes each input and output is worth once, and the operations of the terms the pass sums: about 25 for a pair
    term of one radius, 65 for an atom's trilinear energy, 66 more where its gradient is needed."""
    kind = case["kind"]
    if kind == "maps":
        ext = (case["bx"], case["by"], case["bz"])
        nodes = math.prod(int(e / case["h"]) + 1 for e in ext)
        pairs = nodes * 0.025 * 4.0 / 3.0 * math.pi * 512.0 * _inside(case["rec"], ext)
        return {"bytes": nodes * 16.0 * case["types"] + 16.0 * case["rec"], "flops": pairs * (10.0 + 25.0 * _radii(case["types"]))}
    if kind == "site":
        return {"bytes": 4.0 * case["n"] ** 3 + 16.0 * case["top"], "flops": float(case["n"] ** 3)}
    na = case.get("atoms", 35)
    pairs = 0.8 * na * (na - 1) / 2 if case.get("tors", 7) else 0.0
    ev = 131.0 * na + 63.0 * pairs
    if kind == "score":
        nt = case["tors"]
        maps = (int(case["box"] / 0.375) + 1) ** 3 * 16.0 * case["types"]
        return {"bytes": case["poses"] * 4.0 * (7 + nt + 4 + 6 + nt + (3 * na if case["xyz"] else 0))
                + min(maps, case["poses"] * na * 128.0), "flops": ev * case["poses"]}
    # evaluations of one local optimisation: about 36 with the line search, 101 with the fixed number of steps
    per = 101.0 if case.get("opt") == "bb" else 36.0
    n = case["poses"] if kind == "refine" else case["chains"] * case["steps"] * case.get("ligands", case.get("requests", 1))
    out = case["poses"] * 4.0 * (2 * (7 + case["tors"]) + 5) if kind == "refine" else 64.0 * case["chains"]
    return {"bytes": out, "flops": n * per * (65.0 * na + 45.0 * pairs)}


# ------------------------------------------------------------------ the same in 64 bits
_R = (1.9, 1.9, 1.8, 1.8, 1.8, 1.8, 1.7, 1.7, 1.7, 1.7, 2.0, 2.1, 1.5, 1.8, 2.0, 2.2, 1.2)
_HYD = (0, 12, 13, 14, 15)
_DON = (3, 5, 7, 9, 16)
_ACC = (4, 5, 8, 9)


def _class(a, b):
    """Hydrophobic and hydrogen-bond weight of an XS type pair."""
    hb = (a in _DON and b in _ACC) or (b in _DON and a in _ACC)
    return (-0.0351 if a in _HYD and b in _HYD else 0.0), (-0.587 if hb else 0.0)


def _pair(d, wh, wb):
    """Pair energy on the surface distance and its derivative."""
    b = d - 3.0
    g1, g2 = torch.exp(-4.0 * d * d), torch.exp(-0.25 * b * b)
    dn = torch.clamp(d, max=0.0)
    e = -0.0356 * g1 - 0.00516 * g2 + 0.840 * dn * dn
    de = 0.0356 * 8.0 * d * g1 + 0.00516 * 0.5 * b * g2 + 1.68 * dn
    e = e + wh * torch.clamp(1.5 - d, 0.0, 1.0) + wb * torch.clamp(d / -0.7, 0.0, 1.0)
    return e, de - wh * ((d > 0.5) & (d <= 1.5)) - wb / 0.7 * ((d > -0.7) & (d <= 0.0))


def _geometry(box):
    n = [int(math.floor(float(s) / box["spacing"])) + 1 for s in box["size"]]
    return n, [float(c) - 0.5 * (m - 1) * box["spacing"] for c, m in zip(box["centre"], n)]


def _maps64(xyz, types, box, palette):
    """[T, nz, ny, nx, 4] energy and gradient maps: direct sums over the receptor's atoms within 8 A of each node."""
    dev = "cuda"
    n, o = _geometry(box)
    h = box["spacing"]
    ax = [o[a] + h * torch.arange(n[a], dtype=torch.float64, device=dev) for a in range(3)]
    A = torch.from_numpy(xyz.astype(np.float64)).to(dev)
    near = torch.ones(len(A), dtype=torch.bool, device=dev)
    for a in range(2):
        near &= (A[:, a] > ax[a][0] - 8.0) & (A[:, a] < ax[a][-1] + 8.0)
    tp = [[(_R[t] + _R[r],) + _class(t, r) for r in range(17)] for t in palette]
    tp = torch.tensor(tp, dtype=torch.float64, device=dev)
    rt = torch.from_numpy(types.astype(np.int64)).to(dev)
    M = torch.zeros((len(palette), n[2], n[1], n[0], 4), dtype=torch.float64, device=dev)
    for k in range(n[2]):
        sel = near & ((A[:, 2] - ax[2][k]).abs() < 8.0)
        B, ty = A[sel], rt[sel]
        if not len(B):
            continue
        for j0 in range(0, n[1], 32):
            y = ax[1][j0:j0 + 32]
            dx = ax[0][None, :, None] - B[None, None, :, 0]
            dy = y[:, None, None] - B[None, None, :, 1]
            dz = ax[2][k] - B[None, None, :, 2]
            r = (dx * dx + dy * dy + dz * dz).sqrt()
            into = (r < 8.0).to(torch.float64)
            inv = into / r
            for t in range(len(palette)):
                p = tp[t][ty]
                e, de = _pair(r - p[:, 0], p[:, 1], p[:, 2])
                g = de * inv
                M[t, k, j0:j0 + 32] = torch.stack([(e * into).sum(-1), (g * dx).sum(-1), (g * dy).sum(-1), (g * dz).sum(-1)], -1)
    return M


def _cross(a, b):
    return torch.stack([a[..., 1] * b[..., 2] - a[..., 2] * b[..., 1], a[..., 2] * b[..., 0] - a[..., 0] * b[..., 2],
                        a[..., 0] * b[..., 1] - a[..., 1] * b[..., 0]], -1)


def _rotate(q, v):
    """Rotation of v by the unit quaternion q (w, x, y, z)."""
    r = q[..., 1:].expand(v.shape)
    t = 2.0 * _cross(r, v)
    return v + q[..., :1] * t + _cross(r, t)


def _qmul(a, b):
    w = a[..., :1] * b[..., :1] - (a[..., 1:] * b[..., 1:]).sum(-1, keepdim=True)
    return torch.cat([w, a[..., :1] * b[..., 1:] + b[..., :1] * a[..., 1:] + _cross(a[..., 1:], b[..., 1:])], -1)


def _score64(lg, maps, box, palette, P):
    """Energies [n, 4], gradients and coordinates of poses P."""
    xyz, types, start, parent, axis, bonds = lg
    dev, f8 = P.device, torch.float64
    ref = torch.from_numpy(xyz.astype(np.float64)).to(dev)
    na, nf = len(types), len(parent)
    org = [ref[start[0]:start[1]].mean(0)] + [ref[int(axis[k, 1])] for k in range(1, nf)]
    P = P.to(f8)
    q = [P[:, 3:7] / P[:, 3:7].norm(dim=1, keepdim=True)]
    o, u, X, frag = [P[:, :3]], [None], torch.zeros((len(P), na, 3), dtype=f8, device=dev), np.zeros(na, int)
    for k in range(nf):
        if k:
            p = int(parent[k])
            w = ref[int(axis[k, 1])] - ref[int(axis[k, 0])]
            w = w / w.norm()
            half = 0.5 * P[:, 6 + k:7 + k]
            u.append(_rotate(q[p], w.expand(len(P), 3)))
            o.append(o[p] + _rotate(q[p], (org[k] - org[p]).expand(len(P), 3)))
            q.append(_qmul(q[p], torch.cat([torch.cos(half), torch.sin(half) * w], -1)))
        a, b = int(start[k]), int(start[k + 1])
        frag[a:b] = k
        X[:, a:b] = o[k][:, None] + _rotate(q[k][:, None], (ref[a:b] - org[k]).expand(len(P), b - a, 3))
    n, og = _geometry(box)
    h = box["spacing"]
    F, wall, base, fr = torch.zeros_like(X), 0.0, [], []
    out_of = []
    for a in range(3):
        lo, hi = og[a], og[a] + (n[a] - 1) * h
        below, above = X[..., a] < lo, X[..., a] > hi
        wall = wall + 10.0 * (torch.where(below, lo - X[..., a], torch.zeros_like(X[..., a])) + torch.where(above, X[..., a] - hi, torch.zeros_like(X[..., a])))
        out_of.append((below | above, 10.0 * (above.to(f8) - below.to(f8))))
        c = (X[..., a].clamp(lo, hi) - lo) / h
        i = c.floor().clamp(0, n[a] - 2)
        base.append(i.long())
        fr.append(c - i)
    mi = torch.tensor([palette.index(int(t)) for t in types], device=dev)
    val = 0.0
    for cz in (0, 1):
        for cy in (0, 1):
            for cx in (0, 1):
                w = (fr[0] if cx else 1 - fr[0]) * (fr[1] if cy else 1 - fr[1]) * (fr[2] if cz else 1 - fr[2])
                val = val + w[..., None] * maps[mi, base[2] + cz, base[1] + cy, base[0] + cx]
    e_inter = (val[..., 0] + wall).sum(1)
    for a in range(3):
        F[..., a] = torch.where(out_of[a][0], torch.zeros_like(F[..., a]), val[..., 1 + a]) + out_of[a][1]
    dist = np.full((na, na), 9, int)
    for i, j in bonds:
        dist[i, j] = dist[j, i] = 1
    for s in (2, 3):
        reach = (dist <= s - 1).astype(int) @ (dist == 1).astype(int) > 0
        dist[reach & (dist > s)] = s
    pr = [(i, j) for i in range(na) for j in range(i + 1, na) if frag[i] != frag[j] and dist[i, j] > 3]
    e_intra = torch.zeros(len(P), dtype=f8, device=dev)
    if pr:
        I, J = (torch.tensor([p[c] for p in pr], device=dev) for c in (0, 1))
        R = torch.tensor([_R[types[i]] + _R[types[j]] for i, j in pr], dtype=f8, device=dev)
        W = torch.tensor([_class(int(types[i]), int(types[j])) for i, j in pr], dtype=f8, device=dev)
        d = X[:, I] - X[:, J]
        r = d.norm(dim=-1)
        e, de = _pair(r - R, W[:, 0], W[:, 1])
        into = (r < 8.0).to(f8)
        e_intra = (e * into).sum(1)
        f = (de * into / r)[..., None] * d
        F.index_add_(1, I, f)
        F.index_add_(1, J, -f)
    G = torch.zeros((len(P), 6 + nf - 1), dtype=f8, device=dev)
    G[:, :3], G[:, 3:6] = F.sum(1), _cross(X - P[:, None, :3], F).sum(1)
    for k in range(1, nf):
        below = [m for m in range(nf) if _under(m, k, parent)]
        s = torch.tensor([a for a in range(na) if frag[a] in below], device=dev)
        G[:, 5 + k] = (u[k] * _cross(X[:, s] - o[k][:, None], F[:, s]).sum(1)).sum(-1)
    return torch.stack([e_inter + e_intra, e_inter, e_intra, wall.sum(1)], -1), G, X


def _under(m, k, parent):
    while m > k:
        m = int(parent[m])
    return m == k


def _volume(case, seed):
    """A predictor's score volume: a peak on the site, a weaker decoy and noise."""
    rng = _rng(seed, 5)
    n = case["n"]
    g = np.arange(n) * 2.0
    z, y, x = np.meshgrid(g, g, g, indexing="ij")
    a, b = rng.uniform(0.25, 0.75, 3) * 2.0 * n, rng.uniform(0.1, 0.9, 3) * 2.0 * n
    d = [(x - c[0]) ** 2 + (y - c[1]) ** 2 + (z - c[2]) ** 2 for c in (a, b)]
    v = np.exp(-d[0] / 12.5) + 0.6 * np.exp(-d[1] / 12.5) + 0.05 * rng.random((n, n, n))
    return np.clip(v, 0, 1).astype(np.float32), rng.uniform(-40, 0, 3).astype(np.float32)


def exact(case, seed):
    """What run() computes, in 64 bits. Searches and refinements amplify the last bit of every
    evaluation over their steps, so no value of theirs is fixed by the inputs to a few digits."""
    if case["kind"] == "maps":
        xyz, types, pocket = _receptor(case["rec"], _rng(seed, 1))
        return _maps64(xyz, types, _box(pocket, (case["bx"], case["by"], case["bz"]), case["h"]), PALETTES[case["types"]])
    if case["kind"] == "score":
        xyz, types, _, box, palette, lg = _single(case, seed)
        M = _maps64(xyz, types, box, palette)
        n, o = _geometry(box)
        P = _poses(len(lg[3]) - 1, case["poses"], [float(np.float32(v)) for v in o], [(a - 1) * box["spacing"] for a in n], seed)
        got = [_score64(lg, M, box, list(palette), P[i:i + 16384]) for i in range(0, len(P), 16384)]
        E, G = (torch.cat([g[c] for g in got]) for c in (0, 1))
        return {"energy": E, "grad": G} | ({"xyz": torch.cat([g[2] for g in got])} if case["xyz"] else {})
    if case["kind"] == "site":
        vol, origin = _volume(case, seed)
        i = np.argsort(-vol.reshape(-1), kind="stable")[:case["top"]]
        n = case["n"]
        pts = origin.astype(np.float64) + 2.0 * np.stack([i % n, i // n % n, i // (n * n)], -1)
        return {"points": pts, "labels": None, "centre": pts[0]}
    return None
