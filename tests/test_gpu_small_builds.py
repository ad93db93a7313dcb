"""Builds whose sorts fit one tile and around it, and plans with more runs than
the host takes ahead: bitwise the clusters and results of the sorted input, and
of every window alone."""
import numpy as np
import pytest

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(120)]


def _sums(voxel, scan, dev, seed):
    import torch
    C = voxel.numel()
    g = torch.Generator(device=dev).manual_seed(seed)
    mu = torch.randn(C, 3, generator=g, device=dev, dtype=torch.float64)
    count = torch.randint(4, 90, (C,), generator=g, device=dev)
    s2 = torch.stack([count * mu[:, a] * mu[:, b] + (4.0 if a == b else 0.0)
                      for a, b in ((0, 0), (0, 1), (0, 2), (1, 1), (1, 2), (2, 2))], 1).contiguous()
    return [voxel.int(), scan.int(), count, count[:, None] * mu, s2]


@pytest.mark.parametrize("C", [1, 2, 63, 64, 65, 256, 257, 1023, 2047, 2048, 2049, 4095, 4096, 4097, 9000])
def test_permuted_sums_of_small_builds(C):
    """(voxel, scan) pairs over 5 to 17 key bits, in order, permuted and by scan."""
    import torch
    import paper_2608_14266_amd as ba
    dev = torch.device("cuda:0")
    print(f"[gpu-case] small builds of {C} clusters", flush=True)
    N, V = 7 + C // 5, 3 + C // 3
    g = torch.Generator(device=dev).manual_seed(C)
    key = torch.sort(torch.randperm(N * V, generator=g, device=dev)[:C]).values
    data = _sums(key // N, key % N, dev, C)
    pose = torch.tensor([1.0, 0, 0, 0, 1, 0, 0, 0, 1, 0.1, 0.2, 0.3], device=dev, dtype=torch.float64)
    P = pose.repeat(N, 1).contiguous()
    out = []
    for order in (torch.arange(C, device=dev), torch.randperm(C, generator=g, device=dev),
                  torch.argsort(key % N, stable=True)):
        pb = ba.build_clusters_from_sums(*[a[order].contiguous() for a in data], N, V)
        out.append(list(pb.export_clusters()) + list(ba.eval_residual_grad_hessian(pb, P)[:3]))
        pb.close()
    assert torch.equal(out[0][0].long() * N + out[0][1], key)
    for o in out[1:]:
        assert all(torch.equal(a, b) for a, b in zip(out[0], o))


@pytest.mark.parametrize("W", [1023, 1024, 1025, 3000])
def test_windows_of_more_runs_than_are_taken_ahead(W):
    """Two runs a window, 2048 of them taken ahead: every window as the first."""
    import torch
    import paper_2608_14266_amd as ba
    dev = torch.device("cuda:0")
    print(f"[gpu-case] {2 * W} runs of voxels", flush=True)
    n, V = 5, 6
    v0 = torch.tensor([0, 0, 1, 1, 1, 2, 2, 3, 3, 3, 4, 4, 5, 5], device=dev)
    s0 = torch.tensor([0, 1, 1, 2, 3, 3, 4, 0, 2, 4, 1, 4, 2, 3], device=dev)
    one = _sums(v0, s0, dev, 5)
    w = torch.arange(W, device=dev).repeat_interleave(len(v0))
    data = [a.repeat((W,) + (1,) * (a.dim() - 1)).contiguous() for a in one]
    data[0], data[1] = (data[0] + w * V).int(), (data[1] + w * n).int()
    pose = torch.tensor([1.0, 0, 0, 0, 1, 0, 0, 0, 1, 0.1, 0.2, 0.3], device=dev, dtype=torch.float64)
    P = pose.repeat(W * n, 1).contiguous()
    pb = ba.build_clusters_from_sums(*data, W * n, W * V, n_windows=W,
                                     scan_window=np.repeat(np.arange(W, dtype=np.int32), n))
    cost, grad, hess, _ = ba.eval_residual_grad_hessian(pb, P)
    pb.close()
    pb = ba.build_clusters_from_sums(*one, n, V)
    c1, g1, h1, _ = ba.eval_residual_grad_hessian(pb, P[:n].contiguous())
    pb.close()
    assert (cost == c1).all().item()
    assert (grad.view(W, n, 6) == g1).all().item() and (hess.view(W, n, 6, 6) == h1).all().item()
