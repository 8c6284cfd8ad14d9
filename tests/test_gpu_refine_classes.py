"""Refinement of mixed batches: every size class by the launch that the batch's size
picks (one launch for all classes with the wide or the narrow gradient tile, or one
launch per class), ligand sizes and bond counts on both sides of the classes, of the
gradient's 16-atom runs and of its column passes; bit for bit against the oracle."""
import numpy as np
import pytest

import gen
import oracle
from gpu_common import device_ligands, device_pocket, say

pytestmark = pytest.mark.gpu

SIZES = [(1, 0), (16, 4), (17, 5), (31, 9), (32, 14), (40, 3), (48, 4), (49, 5), (64, 18), (65, 19), (100, 32),
         (128, 20), (129, 6), (192, 32), (193, 5), (256, 32)]
STEPS = 12


# poses per ligand, copies of the batch: 16 to 2 048 poses (wide tile), 4 800 to 48 000 (narrow), 66 000 (by class)
@pytest.mark.parametrize("kpl,copies", [(1, 1), (3, 1), (2, 64), (3, 100), (2, 1500), (1, 300), (3, 1400)])
def test_refined_classes_match_oracle(kpl, copies):
    import torch
    from paper_2303_06150_amd import lg
    n1 = len(SIZES)
    n, k = (np.array([s[i] for s in SIZES], np.int32) for i in (0, 1))
    L1 = gen.ligands_from_sizes(np.arange(n1) + 6_000_000, 6, n, k)
    pk = gen.pocket(64, 0.5, 60, 400, 3)
    rng = np.random.default_rng(7)
    shift = rng.normal(scale=1.5, size=(n1, kpl, 3))
    pivot1 = (pk.center + shift).astype(np.float32)
    poses1 = []
    for i in range(n1):
        xyz = L1.ligand(i)["xyz"] - L1.ligand(i)["ref"]
        poses1.append([(xyz + pivot1[i, m].astype(np.float64)).astype(np.float32) for m in range(kpl)])
    L = L1.subset(np.tile(np.arange(n1), copies)) if copies > 1 else L1
    flat1 = np.concatenate([p for ps in poses1 for p in ps])
    out = {d: torch.from_numpy(np.tile(flat1[:, j], copies)).cuda() for j, d in enumerate("xyz")}
    out["pivot"] = torch.from_numpy(np.tile(pivot1, (copies, 1, 1))).cuda()
    pocket = device_pocket(pk)
    say(f"refine classes: {copies * n1 * kpl} poses, {kpl} per ligand")
    res = lg.lg_refine(pocket, lg.docked_poses(device_ligands(L), out),
                       lg.refine_params(steps=STEPS, clash_dist2=oracle.CLASH2, poses_per_ligand=kpl))
    torch.cuda.synchronize()
    got = np.stack([res[d].cpu().numpy() for d in "xyz"], 1).reshape(copies, len(flat1), 3)
    score = res["score"].cpu().numpy().reshape(copies, n1 * kpl)
    assert np.array_equal(got, np.broadcast_to(got[:1], got.shape))
    assert np.array_equal(score, np.broadcast_to(score[:1], score.shape))
    at = 0
    for i in range(n1):
        for m in range(kpl):
            s, best, _ = oracle.refine(L1.ligand(i), pk, poses1[i][m].astype(np.float64),
                                       pivot1[i, m].astype(np.float64), bits=32, steps=STEPS)
            np.testing.assert_array_equal(got[0, at:at + n[i]].astype(np.float64), best, err_msg=f"{SIZES[i]} pose {m}")
            assert score[0, i * kpl + m] == s, (SIZES[i], m)
            at += n[i]
    pocket.free()
