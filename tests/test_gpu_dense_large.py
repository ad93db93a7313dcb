"""Coupled matrices of more than 2^32 entries, more than a launch has threads:
the windows of a problem together, and one evaluation's own matrix."""
import numpy as np
import pytest

import scenes.sums as ss
from helpers import build_gpu_sums

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(120)]


@pytest.fixture
def room():
    import torch
    import paper_2608_14266_amd as ba
    torch.cuda.empty_cache()
    ba.release_cached_memory()
    if torch.cuda.mem_get_info()[0] < 130 << 30:
        pytest.skip("needs 130 GB of device memory")
    yield
    torch.cuda.empty_cache()
    ba.release_cached_memory()


def test_windows_of_more_than_2e32_entries_together(room, monkeypatch):
    """Every window gives bitwise its run alone."""
    import torch
    import paper_2608_14266_amd as ba
    dev = torch.device("cuda:0")
    monkeypatch.setenv("BA_NO_GRAPH", "1")   # as served requests run: a failed launch is then the call's error
    n, W = 1000, 121
    assert W * (6 * n) ** 2 > 2 ** 32
    print(f"[gpu-case] {W} coupled windows of {n} poses", flush=True)
    sc = ss.batch_windows(seed=929, n_windows=1, poses=[n], vox_per_pose=4, vox_range=(20, 100000), workers=1)
    V = int(sc.voxel.max()) + 1
    P0 = torch.as_tensor(sc.poses_init, device=dev).contiguous()
    d = lambda a, dt: torch.as_tensor(np.ascontiguousarray(a), dtype=dt, device=dev)
    one = (d(sc.voxel, torch.int32), d(sc.scan, torch.int32), d(sc.count, torch.int64), d(sc.sum, torch.float64),
           d(sc.sumsq, torch.float64))

    def run(k):
        at = torch.arange(k, device=dev, dtype=torch.int32).repeat_interleave(one[0].numel())
        data = [a.repeat((k,) + (1,) * (a.dim() - 1)).contiguous() for a in one]
        data[0] += at * V
        data[1] += at * n
        win = np.repeat(np.arange(k, dtype=np.int32), n) if k > 1 else None
        pb = ba.build_clusters_from_sums(*data, k * n, k * V, n_windows=k, scan_window=win)
        P = P0.repeat(k, 1).contiguous()
        reps, _ = ba.iterate(pb, P, ba.MODE_COUPLED, max_iters=1)
        pb.close()
        return reps, P.view(k, n, 12)

    ref, P1 = run(1)
    assert ref[0]["n_accepted"] == 1
    reps, P = run(W)
    for w in range(W):
        assert torch.equal(P[w], P1[0]) and reps[w]["cost_final"] == ref[0]["cost_final"], w


def test_an_evaluation_clears_a_matrix_of_more_than_2e32_entries(room):
    """Entries of scans without a common voxel are zero, whatever the matrix
    held, and the diagonal blocks are symmetric."""
    import torch
    import paper_2608_14266_amd as ba
    dev = torch.device("cuda:0")
    n = 10950
    assert (6 * n) ** 2 > 2 ** 32
    print(f"[gpu-case] coupled evaluation of {n} poses", flush=True)
    sc = ss.batch_windows(seed=930, n_windows=1, poses=[n], vox_per_pose=2, vox_range=(20, 100000), workers=1)
    pb = build_gpu_sums(ba, sc, dev)
    P = torch.as_tensor(sc.poses_init, device=dev).contiguous()
    # the evaluation's matrix takes this block again
    old = torch.full((6 * n, 6 * n), float("nan"), dtype=torch.float64, device=dev)
    at = old.data_ptr()
    del old
    _, _, H, _ = ba.eval_residual_grad_hessian(pb, P, ba.MODE_COUPLED)
    assert H.data_ptr() == at
    band = 6 * 17   # a voxel's scans lie within 16 of each other
    for r in range(0, 6 * n, 6 * 365):
        rows = H[r:r + 6 * 365]
        assert not torch.isnan(rows).any().item(), r
        lo, hi = max(0, r - band), min(6 * n, r + 6 * 365 + band)
        assert not rows[:, :lo].any().item() and not rows[:, hi:].any().item(), r
    assert torch.equal(H[:600, :600], H[:600, :600].T) and torch.equal(H[-600:, -600:], H[-600:, -600:].T)
    pb.close()
