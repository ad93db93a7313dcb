"""Export of a problem whose records hold more than 2^32 values (430M clusters),
more than a launch has threads: every record comes out."""
import pytest

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(120)]


def test_every_record_of_430m_clusters_is_exported():
    import torch
    import paper_2608_14266_amd as ba
    dev = torch.device("cuda:0")
    torch.cuda.empty_cache()
    ba.release_cached_memory()
    if torch.cuda.mem_get_info()[0] < 200 << 30:
        pytest.skip("needs 200 GB of device memory")
    m, V, N = 43, 10_000_000, 1000
    C = m * V
    assert 10 * C > 2 ** 32
    print(f"[gpu-case] export of {C} clusters", flush=True)
    f64 = dict(device=dev, dtype=torch.float64)
    voxel = torch.arange(V, device=dev, dtype=torch.int32).repeat_interleave(m)
    scan = torch.arange(m, device=dev, dtype=torch.int32).repeat(V) + voxel % (N - m)
    count = torch.full((C,), 4, device=dev, dtype=torch.int64)
    s1, s2 = torch.empty(C, 3, **f64), torch.empty(C, 6, **f64)   # four points with mean s1 / 4 and scatter I
    for a in range(3):
        s1[:, a] = 4.0 * (a + 1) + voxel % 1000
    for k, (a, b) in enumerate([(0, 0), (0, 1), (0, 2), (1, 1), (1, 2), (2, 2)]):
        s2[:, k] = s1[:, a] * s1[:, b] / 4 + (1.0 if a == b else 0.0)
    pose = torch.cat([torch.eye(3, **f64).reshape(-1), torch.zeros(3, **f64)])
    pb = ba.build_clusters_from_sums(voxel, scan, count, s1, s2, N, V, precision=ba.PREC_F32,
                                     ref_poses=pose.repeat(N, 1).contiguous())
    del s2, count
    torch.cuda.empty_cache()
    v, s, n, mu, S = pb.export_clusters()
    pb.close()
    unit = torch.tensor([1.0, 0.0, 0.0, 1.0, 0.0, 1.0], **f64)
    step = 10_000_000
    for a in range(0, C, step):
        b = a + step
        assert torch.equal(v[a:b], voxel[a:b]) and torch.equal(s[a:b], scan[a:b]), a
        assert (n[a:b] == 4).all().item() and torch.equal(mu[a:b], s1[a:b] / 4), a
        assert (S[a:b] == unit).all().item(), a
    del v, s, n, mu, S, s1, voxel, scan
    torch.cuda.empty_cache()
    ba.release_cached_memory()
