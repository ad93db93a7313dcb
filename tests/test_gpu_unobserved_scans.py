"""Scans without clusters, before, between and behind the observed ones: bitwise
the problem without them, and a build that takes as long as one whose scans are
all over the range."""
import time

import numpy as np
import pytest

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(120)]


def _data(scan, seed):
    """One voxel per two entries of `scan`."""
    import torch
    dev = scan.device
    C = scan.numel()
    g = torch.Generator(device=dev).manual_seed(seed)
    mu = torch.randn(C, 3, generator=g, device=dev, dtype=torch.float64)
    count = torch.full((C,), 50, device=dev, dtype=torch.int64)
    s2 = torch.stack([50.0 * mu[:, a] * mu[:, b] + (4.0 if a == b else 0.0)
                      for a, b in ((0, 0), (0, 1), (0, 2), (1, 1), (1, 2), (2, 2))], 1).contiguous()
    voxel = torch.arange(C // 2, device=dev).repeat_interleave(2).int()
    return voxel, scan.int(), count, 50.0 * mu, s2


@pytest.mark.parametrize("used,gap,N", [([0, 1, 2], 1, 3), ([5, 6, 9], 1, 10), ([0, 300, 700], 1, 1000),
                                        ([63, 64, 65, 127, 128], 3, 600)])
def test_unobserved_scans_change_nothing(used, gap, N):
    import torch
    import paper_2608_14266_amd as ba
    dev = torch.device("cuda:0")
    print(f"[gpu-case] scans {used} x {gap} of {N}", flush=True)
    at = gap * torch.tensor(used, device=dev)
    k = len(used)
    local = torch.tensor([(i, i + 1) for i in range(k - 1)] * 40, device=dev).view(-1)
    pose = torch.tensor([1.0, 0, 0, 0, 1, 0, 0, 0, 1, 0.1, 0.2, 0.3], device=dev, dtype=torch.float64)
    out = []
    for scan, n in ((local, k), (at[local], N)):
        v, s, c, s1, s2 = _data(scan, 3)
        pb = ba.build_clusters_from_sums(v, s, c, s1, s2, n, len(v) // 2)
        out.append(ba.eval_residual_grad_hessian(pb, pose.repeat(n, 1).contiguous())[:3])
        pb.close()
    (c0, g0, h0), (c1, g1, h1) = out
    assert torch.equal(c0, c1) and torch.equal(g0, g1[at]) and torch.equal(h0, h1[at])
    rest = torch.ones(N, dtype=torch.bool, device=dev)
    rest[at] = False
    assert not g1[rest].any().item() and not h1[rest].any().item()


def test_a_build_does_not_wait_for_unobserved_scans():
    """4M scans of which 1000 are observed, against the same clusters spread over
    all of them: at most three times as long (it was six)."""
    import torch
    import paper_2608_14266_amd as ba
    dev = torch.device("cuda:0")
    print("[gpu-case] build with 4M scans", flush=True)
    N, V = 4_000_000, 50_000
    g = torch.Generator(device=dev).manual_seed(4)
    took = {}
    for used in (1000, N):
        a = torch.randint(0, used - 1, (V,), generator=g, device=dev)
        data = _data(torch.stack([a, a + 1], 1).view(-1), 5)
        t = []
        for _ in range(5):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            pb = ba.build_clusters_from_sums(*data, N, V)
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
            pb.close()
        took[used] = float(np.median(t))
    print(f"[gpu-case] {1e3 * took[1000]:.1f} and {1e3 * took[N]:.1f} ms", flush=True)
    assert took[1000] <= 3 * took[N]
