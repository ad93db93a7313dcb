"""Problems whose window, cluster count and scan take 65 bits together (the plan
sorts their voxels by two keys): bitwise the same scans under window ids that
take fewer."""
import numpy as np
import pytest

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(120)]


def test_plan_of_windows_counts_and_scans_beyond_64_bits():
    import torch
    import paper_2608_14266_amd as ba
    dev = torch.device("cuda:0")
    big, G = 1 << 20, 349_530
    N = big + 3 * G             # a voxel of 2^20 scans in window 0, then windows of three scans
    assert (N - 1).bit_length() + big.bit_length() + (10 * G).bit_length() == 65
    print(f"[gpu-case] plan of {N} scans, window ids to {10 * G}", flush=True)
    g = torch.arange(G, device=dev)
    s0 = big + 3 * g
    # per small window a voxel of three scans and one of two; four voxels of two in window 0
    scan = torch.cat([torch.arange(big, device=dev), (s0[:, None] + torch.tensor([0, 1, 2, 0, 2], device=dev)).view(-1),
                      torch.arange(8, device=dev) * 1000])
    voxel = torch.cat([torch.zeros(big, device=dev, dtype=torch.int64),
                       (1 + 2 * g[:, None] + torch.tensor([0, 0, 0, 1, 1], device=dev)).view(-1),
                       1 + 2 * G + torch.arange(8, device=dev) // 2])
    C, V = scan.numel(), 5 + 2 * G
    gen = torch.Generator(device=dev).manual_seed(8)
    mu = torch.randn(C, 3, generator=gen, device=dev, dtype=torch.float64)
    mu[:, 2] *= 0.01
    count = torch.full((C,), 50, device=dev, dtype=torch.int64)
    s2 = torch.stack([50.0 * mu[:, a] * mu[:, b] + (c if a == b else 0.0)
                      for a, b, c in ((0, 0, 4.0), (0, 1, 0), (0, 2, 0), (1, 1, 4.0), (1, 2, 0), (2, 2, 0.05))], 1)
    data = (voxel.int(), scan.int(), count, 50.0 * mu, s2.contiguous())
    pose = torch.tensor([1.0, 0, 0, 0, 1, 0, 0, 0, 1, 0, 0, 0], device=dev, dtype=torch.float64)
    P = pose.repeat(N, 1).contiguous()
    out = {}
    for step in (1, 10):
        win = np.zeros(N, np.int32)
        win[big:] = step * (1 + np.arange(G, dtype=np.int64)).repeat(3)
        pb = ba.build_clusters_from_sums(*data, N, V, n_windows=step * G + 1, scan_window=win)
        cost, grad, hess, _ = ba.eval_residual_grad_hessian(pb, P)
        Q = P.clone()
        reps, _ = ba.iterate(pb, Q, ba.MODE_MM, max_iters=2, trace=False)
        pb.close()
        out[step] = (cost[::step], grad, hess, Q, [r["cost_final"] for r in reps[::step]])
    for a, b in zip(out[1][:4], out[10][:4]):
        assert torch.equal(a, b)
    assert out[1][4] == out[10][4]
