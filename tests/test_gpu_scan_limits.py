"""Docking scans where their shortcuts end: one sample, positions far from the
origin, sums near the largest float, ligands far longer than the site, sizes known
on the device only.  Every selected sample is the oracle's, or that of scans without
bounds."""
import numpy as np
import pytest

import gen
import oracle
from gpu_common import compare_ligand, device_ligands, device_pocket, dock_gpu, say

pytestmark = pytest.mark.gpu


def moved(pk, by):
    """The site somewhere else."""
    by = np.asarray(by, np.float64)
    return gen.Pocket(pk.grid, (pk.origin + by).astype(np.float32), pk.spacing, (pk.center + by).astype(np.float32),
                      pk.out_value)


def sized(sizes, first, seed=5):
    n, k = (np.array([s[i] for s in sizes], np.int32) for i in (0, 1))
    return gen.ligands_from_sizes(np.arange(len(sizes)) + first, seed, n, k)


def against_oracle(pk, L, r32, a32, T, S, step, mode, label):
    pocket = device_pocket(pk)
    out = dock_gpu(pocket, L, r32, a32, T=T, S=S, top_k=1, mode=mode, trans_step=step)
    for i in range(L.n):
        ref = oracle.dock_ligand(L.ligand(i), pk, r32.astype(np.float64), a32.astype(np.float64), T, S, step,
                                 oracle.CLASH2, bits=32)
        compare_ligand(out, L, i, ref, np.arange(len(r32)), 1, len(r32), label)
    pocket.free()


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("step", [0.7, 7.0, 1e6])
def test_one_translation_sample(mode, step):
    """T = 1: no displacement, however long the step, for atoms on either side of the box faces."""
    pk = gen.pocket(16, 0.375, 20, 100, 3)
    L = sized([(1, 0), (20, 4), (70, 9)], 4_100_000)
    r32, _ = gen.restarts(40, 2)
    a32, _ = gen.angles(32)
    say(f"T = 1, step {step}, mode {mode}")
    against_oracle(pk, L, r32, a32, 1, 2, step, mode, f"step {step}")


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("angles", [64, 256])
def test_positions_rounded_by_more_than_nodes(mode, angles):
    """Coordinates past 2^24, two Angstrom apart, nodes of 0.12: a turned atom lands up to
    eight nodes beyond its exact place."""
    pk = moved(gen.pocket(128, 0.12, 60, 400, 3), (1.75e7, -1.76e7, 1.77e7))
    L = sized([(1, 0), (2, 0), (3, 0), (4, 0)], 4_200_000)
    r32, _ = gen.restarts(200, 2, 7.0)
    a32, _ = gen.angles(angles)
    say(f"far origin, {angles} angles, mode {mode}")
    against_oracle(pk, L, r32, a32, 64, 2, 1.0, mode, f"{angles} angles")


def test_plain_sizes_known_on_the_device_only():
    """Host offsets without the bond atoms: the batch is checked from the device copies,
    and the plain launches are sized by those too."""
    import torch
    from paper_2303_06150_amd import lg
    pk = gen.pocket(32, 0.5, 40, 300, 3)
    L = sized([(10, 2), (130, 9), (64, 5), (65, 5)], 4_300_000)
    r32, _ = gen.restarts(20, 2)
    a32, _ = gen.angles(64)
    pocket = device_pocket(pk)
    outs = []
    for trusted in (True, False):
        dl = device_ligands(L)
        if not trusted:
            dl.atom_offset_host = np.array([0, 130, 140, 205, 269], np.int32)
            dl.tors_atoms_host = None
        say(f"plain, host sizes {'right' if trusted else 'of another order'}")
        outs.append(lg.lg_dock_batch(pocket, dl, torch.from_numpy(r32).cuda(), torch.from_numpy(a32).cuda(), sweeps=2,
                                     top_k=3, trans_samples=64, trans_step=0.0625, clash_dist2=oracle.CLASH2,
                                     mode=lg.LG_PLAIN, want_all_scores=True))
        torch.cuda.synchronize()
    for key in outs[0]:
        assert torch.equal(outs[0][key], outs[1][key]), key
    pocket.free()


def spiky(nodes, spacing, seed):
    """A site of independent values, multiples of 2^-10 in [-5, 5]: a window a node off shows."""
    rng = np.random.default_rng(seed)
    grid = (rng.integers(-5120, 5121, (nodes,) * 3) / 1024).astype(np.float32)
    centre = np.array(gen.DEFAULT_CENTER, np.float32)
    return gen.Pocket(grid, (centre - 0.5 * spacing * (nodes - 1)).astype(np.float32), float(np.float32(spacing)), centre)


@pytest.mark.parametrize("far", [0.0, 1e4, 2e5])
def test_translation_groups_far_from_the_origin(far):
    """Steps that let a group of samples span just under one node: rounded positions may
    take a sample into the node after the next."""
    pk = moved(spiky(64, 0.365, 3), (far, -far, far))
    L = sized([(1, 0), (2, 0), (3, 0)], 4_400_000)
    r32, _ = gen.restarts(4000, 2)
    a32, _ = gen.angles(200)                                 # bounded scans
    say(f"translations near {far}")
    for T in (128, 256):                                     # 16 groups
        step = 0.9975 / (T // 16 - 1) * 0.365
        against_oracle(pk, L, r32, a32, T, 3, step, 1, f"T {T} far {far}")


def test_translation_groups_of_each_site():
    """One launch for a site at the origin, whose translation groups have bounds, and one so
    far away that they have none: each as docked alone."""
    import torch
    from paper_2303_06150_amd import lg
    near = spiky(64, 0.365, 3)
    L = sized([(1, 0), (2, 0), (3, 0)], 4_400_000)
    r32, _ = gen.restarts(2000, 2)
    a32, _ = gen.angles(200)
    rt, at = torch.from_numpy(r32).cuda(), torch.from_numpy(a32).cuda()
    kw = dict(sweeps=2, top_k=3, trans_samples=128, trans_step=0.9975 / 7 * 0.365, clash_dist2=oracle.CLASH2,
              want_all_scores=True)
    dl = device_ligands(L)
    pockets = [device_pocket(moved(near, by)) for by in ((0, 0, 0), (2e5, -2e5, 2e5))]
    for order in (pockets, pockets[::-1]):
        say("translations at two sites")
        outs = lg.lg_dock_sites(order, dl, rt, at, **kw)
        torch.cuda.synchronize()
        for p, o in zip(order, outs):
            alone = lg.lg_dock_batch(p, dl, rt, at, **kw)
            torch.cuda.synchronize()
            for key in alone:
                assert torch.equal(o[key], alone[key]), key
    for p in pockets:
        p.free()


def scattered(sizes, seed):
    """Rigid ligands whose atoms lie anywhere within 6 A."""
    rng = np.random.default_rng(seed)
    n = np.array(sizes, np.int32)
    total, zero = int(n.sum()), np.zeros(0)
    xyz = rng.uniform(-6, 6, (total, 3))
    x = xyz.astype(np.float32)
    return gen.Ligands(np.arange(len(n)), n, 0 * n, np.concatenate([[0], n.cumsum()]).astype(np.int32),
                       np.zeros(len(n) + 1, np.int32), x[:, 0].copy(), x[:, 1].copy(), x[:, 2].copy(), xyz,
                       np.zeros(total, np.int32), np.zeros(total, np.uint32), zero.astype(np.int32),
                       zero.astype(np.float32), zero, np.zeros(3 * len(n), np.float32), np.zeros(3 * len(n)))


@pytest.mark.parametrize("largest", [3e35, 1e38, 3.4e38])
def test_sums_that_overflow(largest):
    """Finite values whose sums over a ligand are not, of one sign in blocks of 12 nodes: the
    samples of scans without bounds (a NaN in a corner that no atom reaches switches
    them off)."""
    from paper_2303_06150_amd import lg
    pk = gen.pocket(96, 0.375, 120, 900, 4)
    signs = np.kron(np.random.default_rng(5).choice([-1.0, 1.0], (8, 8, 8)), np.ones((12, 12, 12)))
    grid = (signs * largest).astype(np.float32)
    L = scattered([3, 4, 5, 6, 8, 13, 64, 70], 6)
    r32, _ = gen.restarts(500, 2)
    a32, _ = gen.angles(256)
    outs = []
    for corner in (grid[0, 0, 0], np.float32("nan")):
        g = grid.copy()
        g[0, 0, 0] = corner
        pocket = device_pocket(gen.Pocket(g, pk.origin, pk.spacing, pk.center, pk.out_value))
        say(f"largest value {largest}, corner {corner}")
        outs.append(dock_gpu(pocket, L, r32, a32, T=256, S=2, top_k=4, mode=lg.LG_BUCKETED))
        pocket.free()
    for key in outs[0]:
        np.testing.assert_array_equal(outs[0][key], outs[1][key], err_msg=f"{largest}: {key}")


def test_sums_that_run_to_infinity_in_one_order_only():
    """Eight atoms and values of a third of the largest float, in blocks of either sign: the first
    translation scan compares the sums in atom order (a sum of both infinities orders
    lowest), also when the current pose's sum is infinite in another order."""
    from paper_2303_06150_amd import lg
    nodes, h, R, T, step = 128, np.float32(0.375), 500, 256, 1 / 16
    centre = np.array(gen.DEFAULT_CENTER, np.float32)
    signs = np.kron(np.random.default_rng(5).choice([-1.0, 1.0], (16, 16, 16)), np.ones((8, 8, 8)))
    grid = (signs * 1e38).astype(np.float32)
    pk = gen.Pocket(grid, (centre - 0.5 * h * (nodes - 1)).astype(np.float32), float(h), centre)
    L = scattered([8] * 8, 8)
    r32, _ = gen.restarts(R, 2)
    pocket = device_pocket(pk)
    say("sums infinite in one order only")
    out = dock_gpu(pocket, L, r32, np.array([[1.0, 0.0]], np.float32), T=T, S=1, top_k=1, mode=lg.LG_BUCKETED,
                   trans_step=step)
    pocket.free()
    inv = np.float64(pk.inv_spacing)
    c0 = np.array([np.float32(0.5 - np.float64(o) * inv) for o in pk.origin], np.float64)
    j = np.arange(T)
    d = (np.float32(step) * np.where(j < T // 2, j, j - T).astype(np.float32)).astype(np.float32)
    finite = 0
    for i in range(L.n):
        for r in range(R):
            x, _ = oracle.place(L.ligand(i), r32[r].astype(np.float64), centre.astype(np.float64), bits=32)
            pose = np.broadcast_to(x.astype(np.float32), (T, 8, 3)).copy()
            pose[..., 0] += d[:, None]
            node = np.floor((pose.astype(np.float64) * inv + c0).astype(np.float32)).astype(int)
            assert node.min() >= 0 and node.max() < nodes
            v = grid[node[..., 2], node[..., 1], node[..., 0]]
            score = np.zeros(T, np.float32)
            with np.errstate(all="ignore"):
                for a in range(8):
                    score = score + v[:, a]
            order = np.where(np.isnan(score), -1e39, np.nan_to_num(score.astype(np.float64), posinf=1e39, neginf=-9e38))
            finite += np.isfinite(score).any()
            assert out["trace"][i, r, 0, 3] == np.argmax(order), (i, r, score[0])
    assert finite > 100
