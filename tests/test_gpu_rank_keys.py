"""Ranking keys read as float4 (groups of whole, aligned fours) and through LDS or
value by value (the others): the oracle's order at odd counts of fours, at one group
past a grid's pass, and for a score array that starts between two float4."""
import numpy as np
import pytest

import oracle
from gpu_common import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,group,shift", [
    (4097, 4, 0), (4097, 4, 1), (4100, 12, 0), (4100, 12, 3), (5000, 8, 2), (4099, 68, 0), (4099, 20, 0),
    (524289, 4, 0), (524288, 8, 0), (786435, 4, 0)])
def test_groups_of_fours(n, group, shift):
    import torch
    from paper_2303_06150_amd import lg
    rng = np.random.default_rng(n + group)
    score = rng.normal(size=shift + n * group).astype(np.float32)
    score[rng.integers(0, len(score), len(score) // 50)] = 2.5      # equal bests, within groups and between
    score[rng.integers(0, len(score), 50)] = -np.inf
    score[-group:] = np.finfo(np.float32).min                       # the last group: the type's lowest value
    m = 1500
    pocket = lg.Pocket(torch.zeros(8, 8, 8).cuda(), [0, 0, 0], 0.5, [0, 0, 0], 0.0)
    say(f"rank keys: {n} groups of {group}, offset {shift}")
    out = lg.lg_rank(pocket, torch.from_numpy(score).cuda()[shift:], group, m)
    ids, vals, members = oracle.rank(score[shift:], group, m)
    np.testing.assert_array_equal(out["top_idx"].cpu().numpy(), ids)
    np.testing.assert_array_equal(out["top_score"].cpu().numpy().astype(np.float64), vals)
    np.testing.assert_array_equal(out["top_member"].cpu().numpy(), members)
    pocket.free()
