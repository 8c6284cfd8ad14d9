"""Timed cases of the docking library: what a virtual-screening program has it do.

A program loads a docking site, docks ligands into it (one at a time while a
chemist looks on, in batches, streamed from host memory, into several sites of
one target), refines and rescores the kept poses, optimises poses through
autograd and ranks the library.  Every case goes through the public binding
(``paper_2303_06150_amd.lg`` and ``autograd``).  Sizes are those of the
repository's own workloads (tiny, mixed, screen, several sites, the
refinement configuration) cut to a share of the library, and the ragged sizes
of its parity tests.

Inputs are made on the GPU from the seed: a pocket of Gaussians inside a shell
of -5, rounded to multiples of 2^-10; ligands grown atom by atom as trees
whose atoms keep apart (1.5 A bonds, tetrahedral angles, preorder numbering,
rotatable bonds between inner atoms, listed parents first).
"""
import math

import numpy as np
import torch

from paper_2303_06150_amd import autograd, lg

CENTER = (10.0, -4.0, 6.5)
CLASH2 = 2.2 * 2.2
HALF_WIDTH = 2.0          # translation scans cover +-2 A

# docking sites: nodes per axis, spacing, Gaussians, shell atoms
GRIDS = {
    "tiny": (32, 0.5, 40, 300),
    "site": (96, 0.375, 200, 2000),
    "wide": (128, 0.375, 200, 2000),
}
# ligand libraries: least and most atoms, median (0: uniform), most bonds
LIBRARIES = {
    "tiny": (20, 40, 0, 6),
    "mixed": (12, 120, 38, 24),
    "screen": (12, 160, 38, 32),
    "ragged": (3, 256, 0, 32),
}


def listed():
    return [
        # one ligand at full effort while somebody waits for the poses
        dict(name="dock_one", kind="dock", grid="site", library="mixed", n=1, restarts=256, angles=256, shifts=256,
             sweeps=3, top=10, tuned=False),
        # a quick pass over a handful of small ligands (the tiny workload)
        dict(name="dock_tiny", kind="dock", grid="tiny", library="tiny", n=64, restarts=32, angles=64, shifts=64,
             sweeps=2, top=32, tuned=False),
        # fragments to peptide-sized ligands with sample counts that fill no wavefront
        dict(name="dock_ragged", kind="dock", grid="site", library="ragged", n=333, restarts=75, angles=130, shifts=100,
             sweeps=2, top=7, tuned=False),
        # the benchmark's mixed library, a fifth of it, in the benchmark's tuning
        dict(name="dock_mixed", kind="dock", grid="site", library="mixed", n=20000, restarts=256, angles=256,
             shifts=256, sweeps=3, top=10, tuned=True),
        # a batch of the large screen: wide site, ligands to 160 atoms, default tuning
        dict(name="dock_screen", kind="dock", grid="wide", library="screen", n=4000, restarts=256, angles=256,
             shifts=256, sweeps=3, top=8, tuned=False),
        # a small set into eight sites of one target
        dict(name="dock_sites", kind="sites", grid="site", library="mixed", n=300, sites=8, restarts=256, angles=256,
             shifts=256, sweeps=3, top=10),
        # a library in host memory, streamed in chunks
        dict(name="dock_stream", kind="stream", grid="site", library="mixed", n=6000, chunk=2000, restarts=256,
             angles=256, shifts=256, sweeps=3, top=10),
        # the kept poses of a few leads, refined
        dict(name="refine_leads", kind="refine", grid="site", library="mixed", n=100, poses=10, steps=50),
        # the refinement configuration (64 poses per ligand), a fifth of it
        dict(name="refine_mixed", kind="refine", grid="site", library="mixed", n=4000, poses=64, steps=50),
        # rescoring of many poses with force and torque, best thousand kept
        dict(name="score_poses", kind="score", grid="site", library="mixed", n=200000, top=1000),
        # one step of a pose optimiser written with torch: forward and backward
        dict(name="moves_autograd", kind="moves", grid="site", library="mixed", n=2000),
        # the ranking of a large screen: eight refined poses per ligand
        dict(name="rank_screen", kind="rank", n=1000000, poses=8, top=1000),
    ]


def draw(rng):
    def spread(lo, hi):
        return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))

    kind = rng.choice(["dock", "dock", "dock", "sites", "stream", "refine", "refine", "score", "moves", "rank"])
    if kind == "rank":
        n = spread(1000, 1000000)
        return dict(kind=kind, n=n, poses=rng.randint(1, 10), top=spread(10, min(n, 4000)))
    library = rng.choice(["tiny", "mixed", "mixed", "screen", "ragged"])
    case = dict(kind=kind, grid="tiny" if library == "tiny" else "wide" if library == "screen" else "site",
                library=library)
    if kind in ("dock", "sites", "stream"):
        case.update(restarts=rng.choice([32, 75, 100, 128, 256, 256]), angles=rng.choice([64, 100, 130, 200, 256, 256]),
                    shifts=rng.choice([64, 100, 130, 256, 256]), sweeps=rng.randint(1, 3), top=rng.randint(1, 12))
        most = 500 if library == "ragged" else 8000
        if kind == "dock":
            case.update(n=spread(1, most), tuned=rng.random() < 0.5)
        elif kind == "sites":
            sites = rng.randint(2, 10)
            case.update(n=spread(8, most // 2 // sites), sites=sites)
        else:
            n = spread(100, most // 2)
            case.update(n=n, chunk=max(40, n // rng.randint(1, 6)))
    elif kind == "refine":
        case.update(n=spread(20, 300 if library == "ragged" else 3000), poses=rng.choice([1, 3, 8, 10, 16, 64]),
                    steps=rng.randint(10, 50))
    elif kind == "score":
        n = spread(500, 8000 if library == "ragged" else 150000)
        case.update(n=n, top=spread(10, min(n, 3000)))
    else:
        case.update(n=spread(50, 1000 if library == "ragged" else 8000))
    return case


# ------------------------------------------------------------------ inputs
def generator(device, *words):
    seed = 0
    for w in words:
        seed = (seed * 1000003 + int(w) + 1) % (1 << 62)
    g = torch.Generator(device=device)
    g.manual_seed(seed)
    return g


def make_site(grid, seed, device):
    """Grid values [n, n, n] (x fastest) and the position of node (0, 0, 0)."""
    n, h, n_gauss, n_shell = GRIDS[grid]
    g = generator(device, seed, 11)
    origin = torch.tensor(CENTER, dtype=torch.float32, device=device) - 0.5 * h * (n - 1)

    def ball(count, lo, hi):
        d = torch.randn(count, 3, generator=g, device=device)
        d = d / d.norm(dim=1, keepdim=True)
        u = torch.rand(count, 1, generator=g, device=device)
        return d, lo + (hi - lo) * (u if lo else u.pow(1 / 3))

    d, r = ball(n_gauss, 0.0, 6.0)
    at = d * r
    amp = 0.2 + 0.8 * torch.rand(n_gauss, generator=g, device=device)
    d, r = ball(2 * n_shell, 6.0, 8.0)
    shell = (d * r)[d[:, 2] < math.cos(math.pi / 4)][:n_shell]     # the pocket opens upwards
    axis = (torch.arange(n, device=device, dtype=torch.float32) - 0.5 * (n - 1)) * h
    values = torch.zeros(n, n, n, device=device)
    for p, a in zip(at.tolist(), amp.tolist()):
        e = [torch.exp(-(axis - c).square() / (2 * 1.5 * 1.5)) for c in p]
        values += a * e[2][:, None, None] * e[1][None, :, None] * e[0][None, None, :]
    wall = torch.zeros(n, n, n, dtype=torch.bool, device=device)
    reach = int(2.0 / h) + 2
    off = torch.arange(-reach, reach + 1, device=device)
    for chunk in shell.split(256):
        near = (chunk / h + 0.5 * (n - 1)).round().long()
        ix, iy, iz = (near[:, a, None] + off[None] for a in range(3))
        dx, dy, dz = ((i.float() - 0.5 * (n - 1)) * h - chunk[:, a, None] for a, i in enumerate((ix, iy, iz)))
        d2 = dx.square()[:, None, None, :] + dy.square()[:, None, :, None] + dz.square()[:, :, None, None]
        inside = [(i >= 0) & (i < n) for i in (ix, iy, iz)]
        hit = ((d2 <= 4.0) & inside[0][:, None, None, :] & inside[1][:, None, :, None] & inside[2][:, :, None, None])
        flat = (iz[:, :, None, None] * n + iy[:, None, :, None]) * n + ix[:, None, None, :]
        wall.view(-1)[flat[hit]] = True
    values -= 5.0 * wall
    return (torch.round(values * 1024) / 1024).clamp(-63, 63), origin


def make_ligands(library, n, seed, device):
    """A library of `n` ligands: sizes, offsets and packed arrays (dict of tensors)."""
    lo, hi, median, most_bonds = LIBRARIES[library]
    r = np.random.RandomState(17)               # sizes are the library's, whatever the seed
    sizes = (np.clip(np.round(median * np.exp(0.4 * r.randn(n))), lo, hi) if median else r.randint(lo, hi + 1, n))
    sizes = sizes.astype(np.int64)
    wanted = np.clip(np.round(0.18 * sizes + 2 * r.randn(n)), 0, np.minimum(most_bonds, sizes - 1)).astype(np.int64)
    g = generator(device, seed, 23)
    N = int(sizes.max())
    rows = torch.arange(n, device=device)
    size = torch.from_numpy(sizes).to(device)
    pos = torch.zeros(n, N, 3, device=device)
    parent = torch.zeros(n, N, dtype=torch.long, device=device)
    children = torch.zeros(n, N, dtype=torch.long, device=device)

    def unit(v):
        return v / v.norm(dim=-1, keepdim=True).clamp_min(1e-6)

    bend = math.radians(180.0 - 109.47)
    for i in range(1, N):
        # three attachment points on the path from the last atom to the root, 16 directions each
        tried = []
        for climb in (0.3, 0.5, 0.8):
            p = torch.full((n,), i - 1, device=device)
            for _ in range(12):
                full = children[rows, p] >= 2
                up = (torch.rand(n, generator=g, device=device) < climb) | full
                p = torch.where(up & (p > 0), parent[rows, p], p)
            tried.append(torch.where(children[rows, p] >= 2, i - 1, p))
        p = torch.stack(tried, 1)                                      # [n, 3]
        at = pos[rows[:, None], p]
        q = parent[rows[:, None], p]
        back = torch.where((p > 0)[..., None], at - pos[rows[:, None], q],
                           torch.randn(n, 3, 3, generator=g, device=device))
        back = unit(back)
        side = unit(torch.linalg.cross(back, torch.randn(n, 3, 3, generator=g, device=device)))
        third = torch.linalg.cross(back, side)
        phi = 2 * math.pi * torch.rand(n, 3, 16, 1, generator=g, device=device)
        way = (math.cos(bend) * back[:, :, None] +
               math.sin(bend) * (torch.cos(phi) * side[:, :, None] + torch.sin(phi) * third[:, :, None]))
        new = (at[:, :, None] + 1.5 * way).reshape(n, 48, 3)
        room = torch.full((n, 48), 1e9, device=device)
        for j in range(0, i, 32):
            other = pos[:, j:min(i, j + 32)]
            d2 = sum((new[:, :, None, a] - other[:, None, :, a]).square() for a in range(3))
            own = p.repeat_interleave(16, 1)[:, :, None] == torch.arange(j, min(i, j + 32), device=device)
            room = torch.minimum(room, torch.where(own, 1e9, d2).amin(2))
        pick = (room.clamp(max=7.5) + torch.rand(n, 48, generator=g, device=device)).argmax(1)
        here = p[rows, pick // 16]
        live = i < size
        pos[:, i] = torch.where(live[:, None], new[rows, pick], pos[:, i])
        parent[:, i] = torch.where(live, here, 0)
        children[rows, here] += live.long()
    # preorder numbering: the subtree of an atom is a run of atoms
    idx = torch.arange(N, device=device)
    there = idx[None] < size[:, None]
    weight = there.long()
    for i in range(N - 1, 0, -1):
        weight[rows, parent[:, i]] += torch.where(there[:, i], weight[:, i], 0)
    end = idx[None] + weight
    inner = there & (idx[None] > 0) & (children > 0)
    up = torch.gather(children, 1, parent) + (parent > 0)
    inner &= up >= 2
    # inner bonds first; a ligand short of them takes bonds to end atoms
    last = torch.where(inner, 0.0, torch.where(there & (idx[None] > 0), 1.0, 2.0))
    rank = (torch.rand(n, N, generator=g, device=device) + last).argsort(1).argsort(1)
    chosen = rank < torch.from_numpy(wanted).to(device)[:, None]
    bonds = chosen.sum(1)
    order = chosen.long().cumsum(1) - 1                                  # bond number of its moving atom
    mask = torch.zeros(n, N, dtype=torch.long, device=device)
    for i in range(1, N):
        bit = torch.where(chosen[:, i], torch.ones_like(size) << order[:, i].clamp(0, 31), 0)
        mask |= torch.where((idx[None] >= i) & (idx[None] < end[:, i, None]), bit[:, None], 0)
    b = chosen.nonzero()
    a = parent[b[:, 0], b[:, 1]]
    gap = (pos[b[:, 0], b[:, 1]] - pos[b[:, 0], a]).double().norm(dim=1)
    mid = (pos.double() * there[..., None]).sum(1) / size[:, None]
    offset = [torch.zeros(n + 1, dtype=torch.long, device=device) for _ in range(2)]
    offset[0][1:] = size.cumsum(0)
    offset[1][1:] = bonds.cumsum(0)
    packed = pos[there]
    mask = mask[there]
    return dict(atom_offset=offset[0].int(), tors_offset=offset[1].int(), xyz=packed,
                frag_mask=torch.where(mask >= 1 << 31, mask - (1 << 32), mask).int(),
                tors_atoms=torch.stack([a, b[:, 1]], 1).reshape(-1).int(), inv_bond_len=(1 / gap).float(),
                ref_point=mid.float().reshape(-1))


def make_turns(count, g, device):
    """Uniform rotations as [count, 3, 3]."""
    q = torch.randn(count, 4, generator=g, device=device, dtype=torch.float64)
    w, x, y, z = (q / q.norm(dim=1, keepdim=True)).unbind(1)
    return torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                        2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                        2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], 1).reshape(count, 3, 3)


def make_offsets(count, g, device):
    d = torch.randn(count, 3, generator=g, device=device, dtype=torch.float64)
    return d / d.norm(dim=1, keepdim=True) * 2.0 * torch.rand(count, 1, generator=g, device=device,
                                                              dtype=torch.float64).pow(1 / 3)


def make_restarts(count, seed, device):
    g = generator(device, seed, 31)
    m, t = make_turns(count, g, device), make_offsets(count, g, device)
    m[0] = torch.eye(3, dtype=torch.float64, device=device)
    t[0] = 0
    return torch.cat([m.reshape(count, 9), t], 1).float()


def make_angles(count, device):
    """(cos, sin) of 2 pi j / count, exact at quarter turns and under their symmetry."""
    def pair(j):
        j, turns = (j, 0) if count % 4 else (j % (count // 4), j // (count // 4))
        c, s = math.cos(2 * math.pi * j / count), math.sin(2 * math.pi * j / count)
        for _ in range(turns):
            c, s = -s, c
        return c, s
    return torch.tensor([pair(j) for j in range(count)], dtype=torch.float32, device=device)


def make_poses(case, seed, device):
    """Rescoring inputs: a library of ligands, each turned and put down near the site's centre."""
    few = min(case["n"], 5000)                                           # conformers; repeated with other placements
    L = make_ligands(case["library"], few, seed, device)
    copies = -(-case["n"] // few)
    atoms, bonds = (L[k].long().diff() for k in ("atom_offset", "tors_offset"))
    atoms, bonds = atoms.repeat(copies)[:case["n"]], bonds.repeat(copies)[:case["n"]]
    total, tors = int(atoms.sum()), int(bonds.sum())
    g = generator(device, seed, 41)
    owner = torch.repeat_interleave(torch.arange(case["n"], device=device), atoms)
    turn, shift = make_turns(case["n"], g, device), make_offsets(case["n"], g, device)
    shift += torch.tensor(CENTER, dtype=torch.float64, device=device)
    ref = L["ref_point"].reshape(few, 3).repeat(copies, 1)[:case["n"]].double()
    x = L["xyz"].repeat(copies, 1)[:total].double() - ref[owner]
    x = torch.stack([(turn[owner, a] * x).sum(1) for a in range(3)], 1) + shift[owner]
    offset = [torch.zeros(case["n"] + 1, dtype=torch.long, device=device) for _ in range(2)]
    offset[0][1:] = atoms.cumsum(0)
    offset[1][1:] = bonds.cumsum(0)
    xyz = x.float()
    ends = L["tors_atoms"].reshape(-1, 2).repeat(copies, 1)[:tors]
    bond_owner = torch.repeat_interleave(torch.arange(case["n"], device=device), bonds)
    a, b = (offset[0][bond_owner] + ends[:, i].long() for i in range(2))
    return dict(atom_offset=offset[0].int(), tors_offset=offset[1].int(), xyz=xyz,
                frag_mask=L["frag_mask"].repeat(copies)[:total], tors_atoms=ends.reshape(-1).contiguous(),
                inv_bond_len=(1 / (xyz[b] - xyz[a]).double().norm(dim=1)).float(), ref_point=shift.float().reshape(-1))


def make_moves(case, P, seed, device):
    g = generator(device, seed, 53)
    n, tors = case["n"], int(P["tors_offset"][-1])
    return [0.3 * torch.randn(n, 3, generator=g, device=device), 0.2 * torch.randn(n, 3, generator=g, device=device),
            0.3 * torch.randn(tors, generator=g, device=device)]


# ------------------------------------------------------------------ cases
def load_site(grid, seed, device):
    values, origin = make_site(grid, seed, device)
    h = GRIDS[grid][1]
    return lg.Pocket(values, origin.tolist(), h, CENTER)


def host_arrays(L):
    a = {k: v.cpu().numpy() for k, v in L.items()}
    xyz = a.pop("xyz")
    a.update({c: np.ascontiguousarray(xyz[:, i]) for i, c in enumerate("xyz")})
    a["frag_mask"] = a["frag_mask"].view(np.uint32)
    return a


def search(case):
    return dict(sweeps=case["sweeps"], top_k=case["top"], trans_samples=case["shifts"],
                trans_step=2 * HALF_WIDTH / case["shifts"], clash_dist2=CLASH2)


def prepare(case, seed):
    device = torch.device("cuda")
    kind = case["kind"]
    if kind == "rank":
        g = generator(device, seed, 61)
        score = 8.0 + 6.0 * torch.randn(case["n"] * case["poses"], generator=g, device=device)
        return dict(case=case, pocket=load_site("tiny", seed, device), score=score)
    if kind in ("score", "moves"):
        P = make_poses(case, seed, device)
        state = dict(case=case, pocket=load_site(case["grid"], seed, device), poses=lg.device_ligands(**host_arrays(P)))
        if kind == "moves":
            state["moves"] = [m.requires_grad_(True) for m in make_moves(case, P, seed, device)]
            state["upstream"] = torch.ones(case["n"], device=device)
        return state
    arrays = host_arrays(make_ligands(case["library"], case["n"], seed, device))
    if kind == "refine":
        # the kept poses of a quick docking run
        k = case["poses"]
        pocket, ligands = load_site(case["grid"], seed, device), lg.device_ligands(**arrays)
        docked = lg.lg_dock_batch(pocket, ligands, make_restarts(64, seed, device), make_angles(64, device),
                                  sweeps=1, top_k=k, trans_samples=64, trans_step=2 * HALF_WIDTH / 64,
                                  clash_dist2=CLASH2)
        torch.cuda.synchronize()
        return dict(case=case, pocket=pocket, poses=lg.docked_poses(ligands, docked),
                    params=lg.refine_params(steps=case["steps"], clash_dist2=CLASH2, poses_per_ligand=k))
    state = dict(case=case, restarts=make_restarts(case["restarts"], seed, device),
                 angles=make_angles(case["angles"], device))
    if kind == "sites":
        state["pockets"] = [load_site(case["grid"], seed * 16 + s, device) for s in range(case["sites"])]
    else:
        state["pocket"] = load_site(case["grid"], seed, device)
    if kind == "stream":
        state["library"] = arrays
    else:
        state["ligands"] = lg.device_ligands(**arrays)
    if kind == "dock" and case["tuned"]:
        t = state["pocket"].get_tuning()
        t.restart_chunk = 2
        t.waves_per_block[0] = 2
        state["pocket"].set_tuning(t)
    return state


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "dock":
        return lg.lg_dock_batch(state["pocket"], state["ligands"], state["restarts"], state["angles"], **search(case))
    if kind == "sites":
        return lg.lg_dock_sites(state["pockets"], state["ligands"], state["restarts"], state["angles"], **search(case))
    if kind == "stream":
        return lg.lg_dock_stream(state["pocket"], **state["library"], restart_table=state["restarts"],
                                 angle_table=state["angles"], chunk=case["chunk"], **search(case))
    if kind == "refine":
        return lg.lg_refine(state["pocket"], state["poses"], state["params"])
    if kind == "score":
        return lg.lg_score(state["pocket"], state["poses"], lg.LG_TRILINEAR, grad=True, top_m=case["top"])
    if kind == "moves":
        score = autograd.RefineScore.apply(*state["moves"], state["pocket"], state["poses"])
        return [score.detach(), *torch.autograd.grad(score, state["moves"], state["upstream"])]
    return lg.lg_rank(state["pocket"], state["score"], case["poses"], case["top"])


def mean_sizes(library):
    lo, hi, median, most = LIBRARIES[library]
    atoms = median * math.exp(0.08) if median else 0.5 * (lo + hi)
    return atoms, min(0.18 * atoms, most)


def work(case):
    """Bytes: inputs read once, outputs written once.  Floating operations: for docking, one grid value
    added per atom and sample of a rigid scan, per moving atom (a third of a ligand) and sample of a
    torsion scan, each after the turn and the three node indices (12); for the trilinear score and its
    gradient about 60 per atom and evaluation, a local move about 20 per atom and bond."""
    n, kind = case["n"], case["kind"]
    if kind == "rank":
        return {"bytes": 4.0 * n * case["poses"] + 12.0 * case["top"], "flops": 1.0 * n * case["poses"]}
    atoms, bonds = mean_sizes(case["library"])
    nodes = GRIDS[case["grid"]][0] ** 3
    ligand = 16 * atoms + 12 * bonds + 20
    if kind in ("dock", "sites", "stream"):
        sites, k = case.get("sites", 1), case["top"]
        scans = case["angles"] * (3 * atoms + bonds * atoms / 3) + case["shifts"] * 3 * atoms
        return {"bytes": n * (ligand + sites * k * (12 * atoms + 20)) + 4.0 * nodes * sites,
                "flops": 12.0 * n * sites * case["restarts"] * case["sweeps"] * scans}
    if kind == "refine":
        return {"bytes": n * (ligand + case["poses"] * (24 * atoms + 16)) + 4.0 * nodes,
                "flops": n * case["poses"] * case["steps"] * atoms * (60.0 + 20.0 * bonds / 3)}
    per = 28 + 4 * bonds if kind == "score" else 28 + 8 * bonds + 24
    return {"bytes": n * (ligand + per) + 4.0 * nodes, "flops": n * atoms * (60.0 + 20.0 * bonds / 3)}


# ------------------------------------------------------------------ 64-bit values
def trilinear64(values, origin, h, x):
    """Grid values at x [m, 3] with their gradient, zero outside; values [n, n, n], x fastest."""
    n = values.shape[0]
    f = (x - origin) / h
    inside = ((f >= 0) & (f < n - 1)).all(1)
    i = f.detach().floor().clamp(0, n - 2).long()
    w = f - i
    flat = values.reshape(-1)

    def corner(a, b, c):
        return flat[((i[:, 2] + c) * n + i[:, 1] + b) * n + i[:, 0] + a]

    v = 0
    for a in (0, 1):
        for b in (0, 1):
            for c in (0, 1):
                v = v + corner(a, b, c) * ((w[:, 0] if a else 1 - w[:, 0]) * (w[:, 1] if b else 1 - w[:, 1]) *
                                           (w[:, 2] if c else 1 - w[:, 2]))
    return torch.where(inside, v, 0.0)


def turn64(w, v):
    """v [m, 3] turned by the rotation vectors w [m, 3]."""
    t2 = w.square().sum(1, keepdim=True) + 1e-300
    t = t2.sqrt()
    u = torch.linalg.cross(w, v)
    return v + torch.sin(t) / t * u + (1 - torch.cos(t)) / t2 * torch.linalg.cross(w, u)


def exact(case, seed):
    device = torch.device("cuda")
    kind = case["kind"]
    if kind == "rank":
        g = generator(device, seed, 61)
        score = 8.0 + 6.0 * torch.randn(case["n"] * case["poses"], generator=g, device=device)
        top = score.double().reshape(case["n"], case["poses"]).amax(1).topk(case["top"]).values
        return dict(top_idx=None, top_score=top, top_member=None)
    if kind not in ("score", "moves"):
        # searches: a comparison at every scan or step decides what follows, so that 64 bits take other ways
        return None
    P = make_poses(case, seed, device)
    values, origin = make_site(case["grid"], seed, device)
    values, origin, h = values.double(), origin.double(), GRIDS[case["grid"]][1]
    n = case["n"]
    ao, to = P["atom_offset"].long(), P["tors_offset"].long()
    owner = torch.repeat_interleave(torch.arange(n, device=device), ao.diff())
    bond_owner = torch.repeat_interleave(torch.arange(n, device=device), to.diff())
    mask = P["frag_mask"].long() & 0xFFFFFFFF
    a, b = (ao[bond_owner] + P["tors_atoms"][i::2].long() for i in range(2))
    bond = torch.arange(len(bond_owner), device=device) - to[bond_owner]
    x = P["xyz"].double()
    pivot = P["ref_point"].double().reshape(n, 3)
    if kind == "moves":
        q = [m.double() for m in make_moves(case, P, seed, device)]
    else:
        q = [torch.zeros(n, 3, dtype=torch.float64, device=device), torch.zeros(n, 3, dtype=torch.float64, device=device),
             torch.zeros(len(bond_owner), dtype=torch.float64, device=device)]
    q = [m.requires_grad_(True) for m in q]
    for k in range(int(to.diff().max()) - 1, -1, -1):
        # bond k of every ligand that has one, about its present axis
        number = to[:-1] + k
        has = k < to.diff()
        number = torch.where(has, number, 0)
        at, axis = x[a[number]], x[b[number]] - x[a[number]]
        axis = axis / axis.norm(dim=1, keepdim=True)
        moves = (((mask >> k) & 1) == 1) & has[owner]
        moves &= torch.arange(len(x), device=device) != b[number][owner]
        o = owner[moves]
        moved = at[o] + turn64(q[2][number][o, None] * axis[o], x[moves] - at[o])
        x = x.index_put((moves.nonzero()[:, 0],), moved)
    x = pivot[owner] + turn64(q[1][owner], x - pivot[owner]) + q[0][owner]
    score = torch.zeros(n, dtype=torch.float64, device=device).index_add(0, owner, trilinear64(values, origin, h, x))
    gt, gw, gth = torch.autograd.grad(score.sum(), q)
    if kind == "moves":
        return [score.detach(), gt, gw, gth]
    grad = torch.zeros(6 * n + len(bond_owner), dtype=torch.float64, device=device)
    base = 6 * torch.arange(n, device=device) + to[:-1]
    for d in range(3):
        grad[base + d] = gt[:, d]
        grad[base + 3 + d] = gw[:, d]
    grad[6 * bond_owner + 6 + to[bond_owner] + bond] = gth
    return dict(score=score.detach(), grad=grad, top_idx=None,
                top_score=score.detach().topk(case["top"]).values)
