"""Rankings at the edges of their launches: long groups (rows of 16 lanes), the most
values that one launch takes, values that are not numbers, and a workspace limit that
leaves no more than the scratch of 12 bytes a group and 8 a place."""
import numpy as np
import pytest

from gpu_common import say

pytestmark = pytest.mark.gpu


def expected(s, group, m):
    """Top m groups by best value (the first of equal ones; a first value that is NaN stays),
    NaN above all, equal values by lower group."""
    g = s.reshape(-1, group)
    with np.errstate(invalid="ignore"):
        member = np.where(np.isnan(g[:, 0]), 0, np.argmax(np.where(np.isnan(g), -np.inf, g), axis=1))
        # a group of -inf and NaN only keeps its first value's place
    best = g[np.arange(len(g)), member]
    rank = np.where(np.isnan(best), np.inf, best).astype(np.float64)
    order = np.lexsort((np.arange(len(g)), -rank, ~np.isnan(best)))[:m]
    return order, best[order], member[order]


def fresh_pocket():
    import torch
    from paper_2303_06150_amd import lg
    return lg.Pocket(torch.zeros(8, 8, 8).cuda(), [0, 0, 0], 0.5, [0, 0, 0], 0.0)


def check(out, s, group, m):
    ids, vals, members = expected(s, group, m)
    np.testing.assert_array_equal(out["top_idx"].cpu().numpy(), ids)
    np.testing.assert_array_equal(out["top_score"].cpu().numpy(), vals)
    np.testing.assert_array_equal(out["top_member"].cpu().numpy(), members)


@pytest.mark.parametrize("n,group,shift", [
    (4096, 16, 0), (4096, 17, 0), (1000, 65, 0), (1000, 66, 1), (4096, 64, 0), (4095, 200, 3), (1, 70000, 0),
    (4097, 63, 0), (4097, 64, 0), (5000, 25, 1), (5000, 200, 0), (5000, 200, 2), (20000, 24, 1), (66000, 68, 0),
    (40000, 4, 0), (2049, 32, 0)])
@pytest.mark.parametrize("odd", [False, True])
def test_long_groups(n, group, shift, odd):
    import torch
    from paper_2303_06150_amd import lg
    rng = np.random.default_rng(n + group)
    s = rng.normal(size=shift + n * group).astype(np.float32)
    s[rng.integers(0, len(s), len(s) // 20 + 1)] = 2.25
    s[shift:shift + group] = -np.inf
    s[-group:] = np.finfo(np.float32).min
    if odd:
        first = shift + group * rng.integers(0, n, n // 50 + 1)
        s[rng.integers(0, len(s), len(s) // 30 + 1)] = np.nan
        s[first] = np.nan
        s[rng.integers(0, len(s), 3)] = np.inf
    m = min(n, 1200)
    pocket = fresh_pocket()
    say(f"rank: {n} groups of {group}, offset {shift}, {'NaN and infinities' if odd else 'numbers'}")
    check(lg.lg_rank(pocket, torch.from_numpy(s).cuda()[shift:], group, m), s[shift:], group, m)
    pocket.free()


@pytest.mark.parametrize("n,group,m", [(1, 1, 1), (100, 1, 10), (100, 700, 10), (4096, 8, 4096), (4096, 64, 10), (4097, 8, 1),
                                       (4097, 100, 4096), (4200, 1, 4097), (10000, 3, 1000), (10000, 8, 10000)])
def test_workspace_limit(n, group, m, monkeypatch):
    import torch
    from paper_2303_06150_amd import lg
    places = 1 << (m - 1).bit_length() if m > 1 else 1
    round_up = lambda b: -(-b // 256) * 256
    limit = 256 + 1024 + round_up(8 * n) + round_up(4 * n) + round_up(8 * places)
    s = np.random.default_rng(n).normal(size=n * group).astype(np.float32)
    pocket = fresh_pocket()
    monkeypatch.setenv("LG_WORKSPACE_LIMIT", str(limit))
    say(f"rank: {n} groups of {group}, top {m}, workspace limit {limit}")
    check(lg.lg_rank(pocket, torch.from_numpy(s).cuda(), group, m), s, group, m)
    monkeypatch.delenv("LG_WORKSPACE_LIMIT")
    pocket.free()
