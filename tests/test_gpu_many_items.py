"""Lists whose kernels give every item a wave and whose items are more than one
launch of fewer than 2^32 threads holds (67M): they go in several."""
import pytest

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(120)]


def _room(gb):
    import torch
    import paper_2608_14266_amd as ba
    torch.cuda.empty_cache()
    ba.release_cached_memory()
    if torch.cuda.mem_get_info()[0] < gb << 30:
        pytest.skip(f"needs {gb} GB of device memory")


def test_points_of_more_clusters_than_a_launch_holds_waves():
    """68M clusters of one point: every centroid is its point."""
    import torch
    import paper_2608_14266_amd as ba
    _room(60)
    dev = torch.device("cuda:0")
    m, V, N = 4, 17_000_000, 100
    C = m * V
    assert C * 64 > 2 ** 32
    print(f"[gpu-case] {C} clusters from points", flush=True)
    voxel = torch.arange(V, device=dev, dtype=torch.int32).repeat_interleave(m)
    scan = torch.arange(m, device=dev, dtype=torch.int32).repeat(V) + voxel % (N - m)
    g = torch.Generator(device=dev).manual_seed(5)
    x, y, z = (torch.randn(C, generator=g, device=dev, dtype=torch.float64) for _ in range(3))
    pb = ba.build_clusters(x, y, z, scan, voxel, N, V)
    v, s, n, mu, S = pb.export_clusters()
    pb.close()
    assert torch.equal(v, voxel) and torch.equal(s, scan) and (n == 1).all().item()
    for k, p in enumerate((x, y, z)):
        assert torch.equal(mu[:, k], p)
    assert not S.any().item()
    del v, s, n, mu, S, x, y, z
    torch.cuda.empty_cache()
    ba.release_cached_memory()


def test_coupled_blocks_of_more_pose_pairs_than_a_launch_holds_waves():
    """A voxel that all 11,600 poses observe: 67.3M pose pairs.  Translations
    leave the residual as it is, so the rows of the last pairs sum to zero."""
    import torch
    import paper_2608_14266_amd as ba
    _room(140)
    dev = torch.device("cuda:0")
    N, V = 11600, 8
    assert N * (N + 1) // 2 * 64 > 2 ** 32
    print(f"[gpu-case] coupled pairs of {N} poses in a voxel", flush=True)
    f64 = dict(device=dev, dtype=torch.float64)
    # every pose in the first voxel, and the others in turn
    scan = torch.cat([torch.arange(N, device=dev)] * 2).int()
    voxel = torch.cat([torch.zeros(N, device=dev), 1 + torch.arange(N, device=dev) % (V - 1)]).int()
    C = 2 * N
    g = torch.Generator(device=dev).manual_seed(6)
    mu = torch.randn(C, 3, generator=g, **f64)
    mu[:, 2] *= 0.01
    mu[:, 2] += 5.0 * voxel
    count = torch.full((C,), 50, device=dev, dtype=torch.int64)
    s1 = 50.0 * mu
    s2 = torch.stack([50.0 * mu[:, a] * mu[:, b] + (c if a == b else 0.0)
                      for a, b, c in ((0, 0, 4.0), (0, 1, 0), (0, 2, 0), (1, 1, 4.0), (1, 2, 0), (2, 2, 0.05))], 1)
    pb = ba.build_clusters_from_sums(voxel, scan, count, s1, s2.contiguous(), N, V)
    pose = torch.cat([torch.eye(3, **f64).reshape(-1), torch.zeros(3, **f64)])
    _, _, H, _ = ba.eval_residual_grad_hessian(pb, pose.repeat(N, 1).contiguous(), ba.MODE_COUPLED)
    pb.close()
    # N u = 1.3e-12 of the absolute sum from the row's sum, and the diagonal block's own sum over N voxel terms
    for r in (0, 3 * N, 6 * N - 600):
        rows = H[r:r + 600]
        blocks = rows.view(600, N, 6)[:, :, 3:]   # the translation columns of every pose
        assert (blocks.abs().amax(2) > 0).all(1).all().item()
        scale = blocks.abs().sum(1)
        assert (blocks.sum(1).abs() <= 1e-11 * scale).all().item(), r
    assert torch.equal(H[-600:, :600], H[:600, -600:].T)
    del H, rows, blocks, scale
    torch.cuda.empty_cache()
    ba.release_cached_memory()
