"""The copies that bound the scans: not made at load, made by the first docking call
that uses them (also of a site among others, from several threads), and docking the
same before and after."""
import threading

import numpy as np
import pytest

import gen
import oracle
from gpu_common import device_ligands, device_pocket, say

pytestmark = pytest.mark.gpu


def held():
    import torch
    torch.cuda.synchronize()
    free, total = torch.cuda.mem_get_info()
    return total - free


def test_loading_allocates_the_grid_only():
    import torch
    from paper_2303_06150_amd import lg
    nodes = 200
    g = torch.zeros(nodes, nodes, nodes, device="cuda")
    lg.Pocket(torch.zeros(8, 8, 8).cuda(), [0, 0, 0], 0.5, [0, 0, 0], 0.0).free()
    before = held()
    pocket = lg.Pocket(g, [0, 0, 0], 0.375, [30, 30, 30], 0.0)
    grown = held() - before
    say(f"load of {nodes}^3 nodes: {grown >> 20} MiB")
    assert grown < 3 * 4 * (nodes + 4) ** 3     # two copies of the grid
    score = lg.lg_rank(pocket, torch.arange(10.0).cuda(), 1, 3)
    torch.cuda.synchronize()
    assert score["top_idx"].tolist() == [9, 8, 7] and held() - before < 3 * 4 * (nodes + 4) ** 3
    pocket.free()


def dock(lg, pocket, dl, R, A, stream=None):
    import torch
    r32, _ = gen.restarts(R, 4)
    a32, _ = gen.angles(A)
    return lg.lg_dock_batch(pocket, dl, torch.from_numpy(r32).cuda(), torch.from_numpy(a32).cuda(), sweeps=2, top_k=2,
                            trans_samples=A, trans_step=2 / A, clash_dist2=oracle.CLASH2, want_all_scores=True,
                            stream=stream)


def same(a, b):
    import torch
    torch.cuda.synchronize()
    return all(torch.equal(a[k], b[k]) for k in a)


def test_calls_before_and_after_the_copies():
    """64 angles (no copies), 256 (made), 64 and 256 again on one handle: as on handles of their own."""
    from paper_2303_06150_amd import lg
    pk = gen.pocket(64, 0.375, 60, 400, 3)
    n, k = np.array([12, 40, 64, 100, 200], np.int32), np.array([3, 8, 12, 20, 32], np.int32)
    dl = device_ligands(gen.ligands_from_sizes(np.arange(5) + 5_200_000, 5, n, k))
    pocket = device_pocket(pk)
    for R in (30, 600):
        for A in (64, 256, 64, 256):
            say(f"copies: {A} angles, {R} restarts")
            out = dock(lg, pocket, dl, R, A)
            fresh = device_pocket(pk)
            assert same(out, dock(lg, fresh, dl, R, A))
            fresh.free()
    pocket.free()


def test_sites_share_a_handle_between_threads():
    """Two threads dock into two pairs of sites with one handle in common, on streams of their own."""
    import torch
    from paper_2303_06150_amd import lg
    pks = [gen.pocket(48, 0.5, 40, 300, s) for s in range(3)]
    n, k = np.array([12, 40, 64], np.int32), np.array([3, 8, 12], np.int32)
    dl = device_ligands(gen.ligands_from_sizes(np.arange(3) + 5_300_000, 5, n, k))
    r32, _ = gen.restarts(50, 4)
    a32, _ = gen.angles(200)
    rt, at = torch.from_numpy(r32).cuda(), torch.from_numpy(a32).cuda()
    kw = dict(sweeps=2, top_k=2, trans_samples=200, trans_step=0.01, clash_dist2=oracle.CLASH2)
    for turn in range(3):
        say(f"sites from two threads, {turn}")
        pockets = [device_pocket(p) for p in pks]
        pairs = ([pockets[0], pockets[1]], [pockets[2], pockets[1]])
        outs, streams = [None, None], [torch.cuda.Stream(), torch.cuda.Stream()]
        torch.cuda.synchronize()

        def work(i):
            with torch.cuda.stream(streams[i]):
                outs[i] = lg.lg_dock_sites(pairs[i], dl, rt, at, stream=streams[i], **kw)

        threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        torch.cuda.synchronize()
        for pair, out in zip(pairs, outs):
            for p, o in zip(pair, out):
                assert same(lg.lg_dock_batch(p, dl, rt, at, **kw), o)
        for p in pockets:
            p.free()
