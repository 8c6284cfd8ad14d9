"""lg_score without moves on poses of every size: one atom to 256, no bond to 32, around
the rows' and the instances' edges, mixed in one batch; batches whose largest pose and
length pick each instance.  Scores bit for bit, gradients as close to 64 bits as the
tests of the small library ask for."""
import numpy as np
import pytest

import gen
import oracle
from gpu_common import device_pocket, say

pytestmark = pytest.mark.gpu

SIZES = [(1, 0), (2, 1), (15, 1), (16, 4), (17, 3), (33, 12), (48, 16), (63, 17), (64, 18), (65, 17), (100, 32), (127, 16),
         (128, 31), (129, 1), (200, 32), (241, 17), (256, 32)]


# largest pose, copies of the batch (several poses each): the wavefront and the rows of each instance
@pytest.mark.parametrize("largest,copies", [(64, 1), (64, 31), (128, 1), (128, 29), (256, 1), (256, 30), (256, 150)])
def test_scores_and_gradients_match_oracle(largest, copies):
    import torch
    from paper_2303_06150_amd import lg
    sizes = [s for s in SIZES if s[0] <= largest]
    sizes += sizes[::-1][:3]
    n1 = len(sizes)
    n, k = (np.array([s[i] for s in sizes], np.int32) for i in (0, 1))
    L1 = gen.ligands_from_sizes(np.arange(n1) + 5_100_000, 13, n, k)
    pk = gen.pocket(64, 0.5, 60, 400, 3)
    rng = np.random.default_rng(3)
    shift = (pk.center + rng.uniform(-3, 3, size=(n1, 3))).astype(np.float32)
    owner = np.repeat(np.arange(n1), L1.n_atoms)
    for axis, name in enumerate("xyz"):
        setattr(L1, name, (getattr(L1, name) - L1.ref_point[axis::3][owner] + shift[owner, axis]).astype(np.float32))
    L1.ref_point = shift.reshape(-1)
    L = L1.subset(np.tile(np.arange(n1), copies)) if copies > 1 else L1
    dl = lg.device_ligands(L.atom_offset, L.tors_offset, L.x, L.y, L.z, L.frag_mask, L.tors_atoms, L.inv_bond_len,
                           L.ref_point)
    pocket = device_pocket(pk)
    say(f"score sizes: largest {largest}, {L.n} poses")
    near = lg.lg_score(pocket, dl, lg.LG_NEAREST)["score"].cpu().numpy().reshape(copies, n1)
    tri = lg.lg_score(pocket, dl, lg.LG_TRILINEAR, grad=True)
    plain = lg.lg_score(pocket, dl, lg.LG_TRILINEAR)["score"].cpu().numpy().reshape(copies, n1)
    torch.cuda.synchronize()
    score = tri["score"].cpu().numpy().reshape(copies, n1)
    grad = tri["grad"].cpu().numpy().reshape(copies, 6 * n1 + int(L1.tors_offset[-1]))
    for a in (near, score, plain, grad):
        assert np.array_equal(a, np.broadcast_to(a[:1], a.shape))
    for i in range(n1):
        a0, a1 = L1.atom_offset[i], L1.atom_offset[i + 1]
        xyz = np.stack([L1.x[a0:a1], L1.y[a0:a1], L1.z[a0:a1]], 1).astype(np.float64)
        assert near[0, i] == oracle.score(pk, xyz, 0, 32)
        assert score[0, i] == plain[0, i] == oracle.score(pk, xyz, 1, 32)
        _, g64 = oracle.pose_grad(L1.ligand(i), pk, xyz, shift[i].astype(np.float64))
        t0 = 6 * i + L1.tors_offset[i]
        g = grad[0, t0:t0 + 6 + int(L1.n_tors[i])]
        assert np.abs(g - g64).max() <= 1e-4 * max(np.abs(g64).max(), 1e-3), (sizes[i], np.abs(g - g64).max())
    pocket.free()
