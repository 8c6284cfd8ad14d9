"""A flat grid of 1024 x 1024 x 28 nodes: the longest node tables beside the largest
ligands' scan data in a block's LDS, for bounded scans, scans of every sample and plain
launches with four wavefronts a block."""
import numpy as np
import pytest

import gen
import oracle
from gpu_common import compare_ligand, device_pocket, dock_gpu, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("A", [100, 200, 600])
def test_longest_tables(A):
    from paper_2303_06150_amd import lg
    h = np.float32(0.25)
    centre = np.array(gen.DEFAULT_CENTER, np.float32)
    grid = (np.random.default_rng(1).integers(-5120, 5121, (28, 1024, 1024)) / 1024).astype(np.float32)
    size = np.array(grid.shape[::-1])
    pk = gen.Pocket(grid, (centre - 0.5 * h * (size - 1)).astype(np.float32), float(h), centre, -5.0)
    n, k = np.array([40, 120, 256], np.int32), np.array([6, 9, 12], np.int32)
    L = gen.ligands_from_sizes(np.arange(3) + 5_400_000, 5, n, k)
    a32, _ = gen.angles(A)
    pocket = device_pocket(pk)
    for mode, R in ((lg.LG_BUCKETED, 20), (lg.LG_BUCKETED, 800), (lg.LG_PLAIN, 20), (lg.LG_PLAIN, 2100)):
        r32, _ = gen.restarts(R, 4)
        say(f"longest tables: A={A} mode={mode} R={R}")
        out = dock_gpu(pocket, L, r32, a32, T=A, S=1, top_k=1, mode=mode, trans_step=2 / A)
        pick = np.array([0, R // 2, R - 1])
        for i in range(L.n):
            ref = oracle.dock_ligand(L.ligand(i), pk, r32[pick].astype(np.float64), a32.astype(np.float64), A, 1, 2 / A,
                                     oracle.CLASH2, bits=32)
            compare_ligand(out, L, i, ref, pick, 1, R, f"A={A} mode={mode}")
    pocket.free()
