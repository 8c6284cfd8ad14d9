"""torch.autograd.Function over the library's moved-pose score and its adjoint.

RefineScore.apply(t, w, theta, pocket, poses) returns the trilinear score of
every pose of `poses` after the local move (t [n,3] translation, w [n,3]
axis-angle rotation about the pose's pivot, theta [total_torsions] bond angles,
torsions applied in reverse bond order).  Forward and backward are one lg_score
call (moves + gradient); this module only packs and unpacks the parameter layout
and applies the chain rule's upstream factor.
"""
from __future__ import annotations

import numpy as np
import torch

from . import lg


def move_layout(poses: lg.DeviceLigands):
    """Index tensors into the flat parameter layout 6 i + tors_offset[i]."""
    n = poses.n
    to = poses.tors_offset_host.astype(np.int64)
    base = 6 * np.arange(n, dtype=np.int64) + to[:-1]
    idx_t = (base[:, None] + np.arange(3)).reshape(-1)
    idx_w = (base[:, None] + 3 + np.arange(3)).reshape(-1)
    k = np.diff(to)
    pose_of_bond = np.repeat(np.arange(n, dtype=np.int64), k)
    idx_th = 6 * pose_of_bond + 6 + np.arange(int(to[-1]), dtype=np.int64)
    dev = poses.x.device
    as_t = lambda a: torch.from_numpy(a).to(dev)
    return as_t(idx_t), as_t(idx_w), as_t(idx_th), as_t(pose_of_bond), 6 * n + int(to[-1])


def _parameter(v, count, dev):
    """v as `count` contiguous float32 values (a single value stands for all of them).
    Slices, matrix columns and expanded values come with strides of their own: reshape
    and float keep them, the pack kernel reads densely."""
    v = v.detach().reshape(-1).float()
    if v.numel() == 1 and count != 1:
        v = v.to(dev).expand(count)
    if v.numel() != count or (count and v.device != dev):
        raise RuntimeError(f"{v.numel()} values on {v.device} given for {count} parameters on {dev}")
    return v.contiguous()


class RefineScore(torch.autograd.Function):
    @staticmethod
    def forward(ctx, t, w, theta, pocket, poses):
        dev = poses.x.device
        # the pack kernel runs on the current device, and both calls on its current
        # stream: the poses' device, whichever one the caller has current
        with torch.cuda.device(dev):
            stream = torch.cuda.current_stream()
            moves, idx_t, idx_w, idx_th, pose_of_bond = lg.lg_pack_moves(
                poses, _parameter(t, 3 * poses.n, dev), _parameter(w, 3 * poses.n, dev),
                _parameter(theta, poses.total_torsions, dev), stream=stream)
            res = lg.lg_score(pocket, poses, lg.LG_TRILINEAR, grad=True, moves=moves, stream=stream)
        ctx.save_for_backward(res["grad"])
        ctx.layout = (idx_t, idx_w, idx_th, pose_of_bond)
        ctx.n = poses.n
        return res["score"]

    @staticmethod
    def backward(ctx, g_score):
        (g,) = ctx.saved_tensors
        idx_t, idx_w, idx_th, pose_of_bond = ctx.layout
        n = ctx.n
        gs = g_score.reshape(n)
        gt = g[idx_t].reshape(n, 3) * gs[:, None]
        gw = g[idx_w].reshape(n, 3) * gs[:, None]
        gth = g[idx_th] * gs[pose_of_bond]
        return gt, gw, gth, None, None
