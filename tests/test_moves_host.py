"""Parameter tensors on their way to the pack kernel (no GPU): every layout that
torch allows arrives as dense float32 values, and the binding refuses the others."""
import types

import pytest
import torch

from paper_2303_06150_amd import lg
from paper_2303_06150_amd.autograd import RefineScore, _parameter

CPU = torch.device("cpu")


def layouts(count):
    """Tensors of `count` values (or one for all) with every kind of stride, and the values they stand for."""
    base = torch.arange(6.0 * max(count, 1)) + 1
    rows = base.reshape(-1, 6)
    return {
        "dense": (base[:count], base[:count]),
        "slice": (base[:2 * count:2], base[:2 * count:2].clone()),
        "column": (rows[:count, 5], rows[:count, 5].clone()),
        "reversed": (base[:count].flip(0), base[:count].flip(0).clone()),
        "expanded": (torch.full((1,), 2.5).expand(count), torch.full((count,), 2.5)),
        "single": (torch.full((1, 1), 2.5), torch.full((count,), 2.5)),
        "scalar": (torch.tensor(2.5), torch.full((count,), 2.5)),
        "double": (base[:2 * count:2].double(), base[:2 * count:2].clone()),
    }


@pytest.mark.parametrize("count", [0, 1, 3, 17])
@pytest.mark.parametrize("kind", list(layouts(1)))
def test_parameters_arrive_dense(count, kind):
    if count == 0 and kind in ("single", "scalar"):
        v, want = layouts(0)[kind]
        assert _parameter(v, 0, CPU).numel() == 0
        return
    v, want = layouts(count)[kind]
    got = _parameter(v.requires_grad_(True) if v.is_leaf else v, count, CPU)
    assert got.is_contiguous() and got.dtype == torch.float32 and not got.requires_grad
    assert got.untyped_storage().nbytes() >= 4 * (got.storage_offset() + count)
    assert torch.equal(got, want)


@pytest.mark.parametrize("n", [1, 4])
def test_parameters_of_poses_arrive_dense(n):
    """t and w as [n, 3] views: a transposed matrix, an expanded row, a strided matrix."""
    m = torch.arange(24.0 * n).reshape(3, -1)
    for v in (m[:, :n].t(), torch.ones(1, 1).expand(n, 3), torch.arange(12.0 * n).reshape(n, 12)[:, ::4]):
        got = _parameter(v, 3 * n, CPU)
        assert got.is_contiguous() and torch.equal(got, v.clone().reshape(-1))


def test_binding_refuses_what_the_kernel_cannot_read():
    poses = types.SimpleNamespace(x=torch.zeros(1), n=2, total_torsions=3, tors_offset=torch.zeros(3, dtype=torch.int32))
    t, w, th = torch.zeros(6), torch.zeros(6), torch.zeros(3)
    for bad in ((torch.zeros(12)[::2], w, th), (t, torch.zeros(5), th), (t, w, torch.zeros(1).expand(3)),
                (t, w, th.double()), (t.to("meta"), w, th)):
        with pytest.raises(ValueError, match="contiguous float32"):
            lg.lg_pack_moves(poses, *bad)


def test_forward_runs_on_the_poses_device(monkeypatch):
    """Both library calls happen with the poses' device current, whatever the caller's is,
    and on its current stream."""
    current = []

    class Device:
        def __init__(self, dev):
            self.dev = dev

        def __enter__(self):
            current.append(self.dev)

        def __exit__(self, *exc):
            current.pop()

    calls = []

    def pack(poses, t, w, theta, stream):
        calls.append(("pack", list(current), stream))
        return (torch.zeros(9), *(torch.arange(3),) * 4)

    def score(pocket, poses, interp, grad, moves, stream):
        calls.append(("score", list(current), stream))
        return dict(score=torch.ones(1), grad=torch.ones(9))

    monkeypatch.setattr(torch.cuda, "device", Device)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: f"stream of {current[-1]}")
    monkeypatch.setattr(lg, "lg_pack_moves", pack)
    monkeypatch.setattr(lg, "lg_score", score)
    poses = types.SimpleNamespace(x=torch.zeros(1), n=1, total_torsions=3)
    RefineScore.apply(torch.zeros(1, 3), torch.zeros(1, 3), torch.zeros(3), None, poses)
    assert calls == [("pack", [CPU], "stream of cpu"), ("score", [CPU], "stream of cpu")] and current == []
