"""Scans of every sample, several per lane, and bounded scans in launches that fill the
device: the oracle's selected samples for sample counts around the lanes' and the
groups' sizes, angle tables with and without turn symmetries, crowded torsions, ligand
sizes on both sides of every instance, runs longer than a wavefront, sites and plain
launches."""
import numpy as np
import pytest

import gen
import oracle
from gpu_common import compare_ligand, device_ligands, device_pocket, dock_gpu, say

pytestmark = pytest.mark.gpu

SMALL = [(1, 0), (2, 1), (12, 3), (31, 8), (32, 9)]
MIXED = [(33, 8), (64, 12), (63, 20), (40, 8)]
LARGE = [(65, 12), (100, 32), (128, 24)]
MANY = 2400   # restarts of the whole batch: more than eight per compute unit on 256 of them


def ligands(sizes, first):
    n, k = (np.array([s[i] for s in sizes], np.int32) for i in (0, 1))
    return gen.ligands_from_sizes(np.arange(len(sizes)) + first, 11, n, k)


def angle_table(A, turned):
    """The uniform table, or one whose samples are nobody's half or quarter turn."""
    a32, _ = gen.angles(A)
    if not turned or A == 1:
        return a32
    w = 2 * np.pi * (np.arange(A) + 0.3 * np.random.default_rng(A).uniform(-1, 1, A)) / A
    w[0] = 0
    return np.stack([np.cos(w), np.sin(w)], 1).astype(np.float32)


def check(pk, L, A, T, step, mode, R, rows, turned=False, S=2):
    pocket = device_pocket(pk)
    r32, _ = gen.restarts(R, 4)
    a32 = angle_table(A, turned)
    out = dock_gpu(pocket, L, r32, a32, T=T, S=S, top_k=1, mode=mode, trans_step=step)
    pick = np.linspace(0, R - 1, rows).astype(int)
    for i in range(L.n):
        ref = oracle.dock_ligand(L.ligand(i), pk, r32[pick].astype(np.float64), a32.astype(np.float64), T, S, step,
                                 oracle.CLASH2, bits=32)
        compare_ligand(out, L, i, ref, pick, 1, R, f"A={A} T={T} mode={mode}")
    pocket.free()


# angle samples, translation samples, step, nodes, spacing, table without symmetries
CASES = [
    (1, 1, 0.5, 48, 0.5, False), (64, 64, 0.0625, 48, 0.5, False), (33, 40, 0.1, 48, 0.5, True),
    (65, 66, 0.0625, 48, 0.5, False), (128, 128, 1 / 32, 64, 0.375, False), (128, 100, 0.04, 64, 0.375, True),
    (127, 128, -1 / 32, 64, 0.375, False), (64, 65, 0.0625, 48, 0.5, False),
    (256, 256, 1 / 64, 96, 0.2, False), (256, 200, 1 / 64, 48, 1.0, True), (130, 129, 1 / 32, 96, 0.1, False),
    (200, 70, 0.5, 128, 0.2, False),        # runs longer than a wavefront
    (256, 256, 1 / 64, 64, 0.375, False), (130, 100, 0.04, 64, 0.375, False), (257, 255, 1 / 64, 64, 0.375, False),
    (1000, 1024, 1 / 256, 48, 0.5, False),
]


@pytest.mark.parametrize("sizes", ["small", "mixed", "large"])
@pytest.mark.parametrize("A,T,step,nodes,spacing,turned", CASES)
def test_full_launches_match_oracle(sizes, A, T, step, nodes, spacing, turned):
    from paper_2303_06150_amd import lg
    group = {"small": SMALL, "mixed": SMALL + MIXED, "large": MIXED + LARGE}[sizes]
    L = ligands(group, 4_600_000)
    say(f"full launch: {sizes} A={A} T={T} step={step} {nodes}^3 @ {spacing}")
    check(gen.pocket(nodes, spacing, 60, 400, 3), L, A, T, step, lg.LG_BUCKETED, -(-MANY // L.n), 4, turned)


@pytest.mark.parametrize("A,T", [(64, 64), (100, 128), (200, 200), (256, 256)])
def test_plain_launches_match_oracle(A, T):
    from paper_2303_06150_amd import lg
    L = ligands(SMALL[1:4] + MIXED[:2] + LARGE, 4_700_000)
    for R in (20, 2100):
        say(f"plain: A={A} T={T} R={R}")
        check(gen.pocket(64, 0.375, 60, 400, 3), L, A, T, 2 / T, lg.LG_PLAIN, R, 5)


@pytest.mark.parametrize("A", [64, 128, 256])
def test_crowded_torsions(A):
    """A clash distance of 9 A: more risky pairs than a list holds, taken in several lists."""
    from paper_2303_06150_amd import lg
    import torch
    pk = gen.pocket(64, 0.2, 60, 400, 3)
    L = ligands(MIXED + LARGE, 4_800_000)
    r32, _ = gen.restarts(-(-MANY // L.n), 4)
    a32, _ = gen.angles(A)
    pocket = device_pocket(pk)
    kmax = int(L.n_tors.max())
    say(f"crowded torsions, A={A}")
    out = lg.lg_dock_batch(pocket, device_ligands(L), torch.from_numpy(r32).cuda(), torch.from_numpy(a32).cuda(), sweeps=2,
                           top_k=1, trans_samples=A, trans_step=2 / A, clash_dist2=81.0, want_all_scores=True,
                           trace_kmax=kmax)
    torch.cuda.synchronize()
    got = {k: v.cpu().numpy() for k, v in out.items()}
    pick = np.array([0, 1, len(r32) - 1])
    for i in range(L.n):
        ref = oracle.dock_ligand(L.ligand(i), pk, r32[pick].astype(np.float64), a32.astype(np.float64), A, 2, 2 / A, 81.0,
                                 bits=32)
        compare_ligand(got, L, i, ref, pick, 1, len(r32), f"crowded A={A}")
    pocket.free()


@pytest.mark.parametrize("A", [100, 256])
def test_sites_with_and_without_bounds(A):
    """Sites of one launch, one of them with a NaN in a far corner: each as docked alone."""
    import torch
    from paper_2303_06150_amd import lg
    pks = [gen.pocket(64, 0.375, 60, 400, s) for s in (3, 4)]
    odd = pks[1].grid.copy()
    odd[0, 0, 0] = np.nan
    pks.append(gen.Pocket(odd, pks[1].origin, pks[1].spacing, pks[1].center, pks[1].out_value))
    L = ligands(SMALL + MIXED + LARGE, 4_900_000)
    r32, _ = gen.restarts(100, 4)
    a32, _ = gen.angles(A)
    rt, at = torch.from_numpy(r32).cuda(), torch.from_numpy(a32).cuda()
    kw = dict(sweeps=2, top_k=3, trans_samples=A, trans_step=2 / A, clash_dist2=oracle.CLASH2)
    dl = device_ligands(L)
    for few in (pks[:2], pks):
        pockets = [device_pocket(p) for p in few]
        say(f"sites: {len(few)}, A={A}")
        outs = lg.lg_dock_sites(pockets, dl, rt, at, **kw)
        torch.cuda.synchronize()
        alone = [lg.lg_dock_batch(p, dl, rt, at, **kw) for p in pockets]
        torch.cuda.synchronize()
        for o, a in zip(outs, alone):
            for key in a:
                assert torch.equal(o[key], a[key]), key
        for p in pockets:
            p.free()
