"""Clusters of more points than the statistics' ordinary kernel takes, at that
limit, in a log's order and shuffled: centroid and scatter against extended
precision, and the other clusters of the build as without them."""
import numpy as np
import pytest

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(120)]


@pytest.mark.parametrize("counts", [[32767, 32768, 32769], [1, 255, 100003, 64, 33000], [32768 + 64 * 8 * 3 + 17] * 9 + [5]])
@pytest.mark.parametrize("shuffled", [False, True])
def test_statistics_of_long_clusters(counts, shuffled):
    import torch
    import paper_2608_14266_amd as ba
    dev = torch.device("cuda:0")
    print(f"[gpu-case] clusters of {counts[:5]} points, shuffled {shuffled}", flush=True)
    rng = np.random.default_rng(len(counts))
    C = len(counts)
    lab = np.repeat(np.arange(C), counts)
    p = rng.standard_normal((len(lab), 3)) * [1, 2, 0.01] + 50.0 * rng.standard_normal((C, 3))[lab]
    if shuffled:
        o = rng.permutation(len(lab))
        lab, p = lab[o], p[o]
    voxel, scan = (lab // 2).astype(np.int32), (lab % 2).astype(np.int32)
    d = lambda a, dt: torch.as_tensor(np.ascontiguousarray(a), dtype=dt, device=dev)
    pb = ba.build_clusters(*(d(p[:, k], torch.float64) for k in range(3)), d(scan, torch.int32), d(voxel, torch.int32),
                           2, (C + 1) // 2)
    v, s, n, mu, S = (a.cpu().numpy() for a in pb.export_clusters())
    pb.close()
    assert np.array_equal(2 * v + s, np.arange(C)) and np.array_equal(n, counts)
    for c in range(C):
        q = p[lab == c].astype(np.longdouble)
        m = q.mean(0)
        # the centroid is the rounded one to an ulp or two of its size
        assert np.all(np.abs(mu[c] - m) <= 4 * 2.0 ** -53 * np.abs(m) + 1e-300)
        w = (q - m).T @ (q - m)
        # each lane sums its rows, then the wave's tree: (rows + 6) u, and the centroid's own rounding
        tol = (counts[c] / 64 + 8) * 2.0 ** -53 * np.sqrt(np.outer(np.diag(w), np.diag(w)))
        tol = tol + counts[c] * np.outer(mu[c], mu[c]).__abs__() * (4 * 2.0 ** -53) ** 2
        tol = tol + 4 * 2.0 ** -53 * (np.abs(mu[c])[:, None] + np.abs(mu[c])) * np.sqrt(counts[c] * np.trace(w))
        got = np.array([[S[c, 0], S[c, 1], S[c, 2]], [S[c, 1], S[c, 3], S[c, 4]], [S[c, 2], S[c, 4], S[c, 5]]])
        assert np.all(np.abs(got - w) <= tol.astype(float))
