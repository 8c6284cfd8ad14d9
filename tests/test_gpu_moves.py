"""RefineScore with parameters of every layout: the scores and gradients of a dense
copy, bit for bit."""
import numpy as np
import pytest

import gen
from gpu_common import device_ligands, device_pocket, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 5])
@pytest.mark.parametrize("layout", ["slice", "column", "expanded"])
def test_strided_parameters_equal_dense_ones(n, layout):
    import torch
    from paper_2303_06150_amd.autograd import RefineScore
    pk = gen.pocket(32, 0.5, 40, 300, 3)
    L = gen.ligands_from_sizes(np.arange(n) + 7_000_000, 7, np.full(n, 30, np.int32), np.full(n, 7, np.int32))
    to_centre = pk.center - L.ref_point.reshape(-1, 3)[np.repeat(np.arange(n), L.n_atoms)]
    for axis, name in enumerate("xyz"):
        setattr(L, name, (getattr(L, name) + to_centre[:, axis]).astype(np.float32))
    L.ref_point = np.tile(pk.center, n).astype(np.float32)
    pocket, poses = device_pocket(pk), device_ligands(L)
    tors = poses.total_torsions
    g = torch.Generator().manual_seed(n)
    store = 0.3 * torch.randn(12 * max(n, tors), generator=g).cuda()

    def views():
        if layout == "slice":
            return store[:6 * n:2].view(n, 3), store[1:6 * n:2].view(n, 3), store[:3 * tors:3]
        if layout == "column":
            return store[:3 * n].view(3, n).t(), store[3 * n:6 * n].view(3, n).t(), store[:6 * tors].view(tors, 6)[:, 5]
        return store[:1].expand(n, 3), store[1:2].expand(n, 3), store[2:3].expand(tors)

    say(f"moves: {layout}, {n} poses")
    results = []
    for dense in (False, True):
        args = [(v.clone(memory_format=torch.contiguous_format) if dense else v.detach()).requires_grad_(True) for v in views()]
        score = RefineScore.apply(*args, pocket, poses)
        results.append([score.detach(), *torch.autograd.grad(score, args, torch.linspace(0.5, 1.5, n, device="cuda"))])
    torch.cuda.synchronize()
    for got, want in zip(*results):
        assert torch.equal(got, want)
    assert results[0][0].abs().max() > 0
    pocket.free()
