"""Small calls of many sites under a workspace limit that leaves 64 bytes a site beside
scores, move records and bucket arrays, and calls of more sites after fewer."""
import numpy as np
import pytest
import torch

import gen
import oracle
from gpu_common import device_ligands, device_pocket, say

pytestmark = pytest.mark.gpu


def test_many_sites_in_a_small_workspace(monkeypatch):
    from paper_2303_06150_amd import lg
    pks = [gen.pocket(24, 0.5, 20, 100, s) for s in range(16)]
    L = gen.ligands_from_sizes(np.arange(2) + 5_500_000, 5, np.array([9, 20], np.int32), np.array([2, 4], np.int32))
    dl = device_ligands(L)
    r32, _ = gen.restarts(3, 4)
    a32, _ = gen.angles(64)
    rt, at = torch.from_numpy(r32).cuda(), torch.from_numpy(a32).cuda()
    kw = dict(sweeps=1, top_k=2, trans_samples=64, trans_step=0.0625, clash_dist2=oracle.CLASH2)
    pockets = [device_pocket(p) for p in pks]
    alone = [lg.lg_dock_batch(device_pocket(p), dl, rt, at, **kw) for p in pks]
    up = lambda b: -(-b // 256) * 256
    for sites in (1, 5, 16, 2):
        moves = 3 * (6 * L.n + int(L.tors_offset[-1]))
        limit = 256 + up(L.n * 3 * sites * 4) + up(moves * sites * 2) + 2 * up(4 * L.n) + up(17 * 4) + up(64 * sites)
        monkeypatch.setenv("LG_WORKSPACE_LIMIT", str(limit))
        say(f"{sites} sites, workspace limit {limit}")
        outs = lg.lg_dock_sites(pockets[:sites], dl, rt, at, **kw)
        torch.cuda.synchronize()
        monkeypatch.delenv("LG_WORKSPACE_LIMIT")
        for a, o in zip(alone, outs):
            for key in a:
                assert torch.equal(a[key], o[key]), key
    for p in pockets:
        p.free()
