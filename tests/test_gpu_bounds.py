"""The scans' upper bounds (groups of samples dropped unscored): docking must select
exactly the oracle's samples for sample counts on both sides of the group sizes,
translation ranges with and without a bound, grids whose nodes are too fine for
any window, and exactly what an unbounded scan selects on grids with any values."""
import numpy as np
import pytest

import gen
import oracle
from gpu_common import compare_ligand, device_ligands, device_pocket, dock_gpu, dock_oracle, say

pytestmark = pytest.mark.gpu

SIZES = [(1, 0), (12, 3), (40, 8), (63, 20), (64, 10), (65, 12), (130, 25), (256, 32)]


@pytest.fixture(scope="module")
def ligands():
    n, k = (np.array([s[i] for s in SIZES], np.int32) for i in (0, 1))
    return gen.ligands_from_sizes(np.arange(len(SIZES)) + 4_000_000, 5, n, k)


# angle samples, translation samples, translation step, grid nodes, spacing
CASES = [
    (64, 64, 0.0625, 48, 0.5), (65, 65, 0.0625, 48, 0.5), (128, 16, 0.25, 48, 0.5), (130, 100, 0.04, 64, 0.375),
    (257, 255, 1 / 64, 64, 0.375), (1000, 1024, 1 / 256, 48, 0.5),
    (256, 200, 0.2, 64, 0.375),        # groups of 64: one sample of each lane spans more than a node
    (256, 70, 0.5, 96, 0.375),         # runs longer than a wavefront: no stage, no bound
    (200, 256, -1 / 64, 64, 0.375),    # displacements in falling order
    (256, 256, 1 / 64, 96, 0.09375),   # fine nodes: most radii have no window, most places lie outside the box
]


@pytest.mark.parametrize("A,T,step,nodes,spacing", CASES)
def test_selected_samples_match_oracle(ligands, A, T, step, nodes, spacing):
    pk = gen.pocket(nodes, spacing, 60, 400, 3)
    R, S = 5, 2
    r32, _ = gen.restarts(R, 2)
    a32, _ = gen.angles(A)
    pocket = device_pocket(pk)
    from paper_2303_06150_amd import lg
    say(f"bounds: A={A} T={T} step={step} {nodes}^3 @ {spacing}")
    out = dock_gpu(pocket, ligands, r32, a32, T=T, S=S, top_k=3, mode=lg.LG_BUCKETED, trans_step=step)
    for i in range(ligands.n):
        ref = oracle.dock_ligand(ligands.ligand(i), pk, r32.astype(np.float64), a32.astype(np.float64), T, S, step,
                                 oracle.CLASH2, bits=32)
        compare_ligand(out, ligands, i, ref, np.arange(R), 3, R, f"A={A} T={T}")
    pocket.free()


@pytest.mark.parametrize("scale,lazy", [(1.0, 0), (1.0, 1), (1e-20, 0), (3e4, 0)])
def test_bounded_equals_unbounded_on_any_grid(ligands, scale, lazy):
    """Values whose sums round: a NaN in a far corner switches the bounds off and changes nothing else."""
    from paper_2303_06150_amd import lg
    pk = gen.pocket(80, 0.375, 120, 900, 4)
    rng = np.random.default_rng(5)
    grid = ((pk.grid + rng.normal(size=pk.grid.shape) * 0.05) * scale).astype(np.float32)
    r32, _ = gen.restarts(16, 2)
    a32, _ = gen.angles(256)
    outs = []
    for corner in (grid[0, 0, 0], np.float32("nan")):
        g = grid.copy()
        g[0, 0, 0] = corner
        pocket = device_pocket(gen.Pocket(g, pk.origin, pk.spacing, pk.center, pk.out_value))
        t = pocket.get_tuning()
        t.lazy_clash = lazy
        pocket.set_tuning(t)
        outs.append(dock_gpu(pocket, ligands, r32, a32, T=256, S=3, top_k=4, mode=lg.LG_BUCKETED))
        pocket.free()
    for key in outs[0]:
        np.testing.assert_array_equal(outs[0][key], outs[1][key], err_msg=f"scale {scale} lazy {lazy}: {key}")
