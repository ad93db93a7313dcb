"""Voxels of more scans than a thread of the fill takes: every cluster is in the
voxel-major copy, at the counts around a thread's run and with several voxels of
a count, against the voxels' covariances formed in numpy."""
import numpy as np
import pytest

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(120)]


@pytest.mark.parametrize("counts", [[63, 64, 65], [64, 128, 129, 193], [200] * 70 + [3] * 5, [5000, 2, 4999]])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_residual_of_long_voxels(counts, prec):
    import torch
    import paper_2608_14266_amd as ba
    dev = torch.device("cuda:0")
    print(f"[gpu-case] voxels of {counts[:4]} scans {prec}", flush=True)
    rng = np.random.default_rng(len(counts))
    N = max(counts)
    scan = np.concatenate([np.sort(rng.permutation(N)[:m]) for m in counts]).astype(np.int32)
    voxel = np.repeat(np.arange(len(counts)), counts).astype(np.int32)
    C = len(scan)
    n = rng.integers(4, 60, C)
    mu = rng.standard_normal((C, 3)) * [1, 1, 0.02]
    s2 = np.stack([n * mu[:, a] * mu[:, b] + n * (c if a == b else 0.0)
                   for a, b, c in ((0, 0, 0.1), (0, 1, 0), (0, 2, 0), (1, 1, 0.1), (1, 2, 0), (2, 2, 1e-3))], 1)
    t = 0.05 * rng.standard_normal((N, 3))
    poses = np.concatenate([np.tile(np.eye(3).ravel(), (N, 1)), t], 1)
    d = lambda a, dt: torch.as_tensor(np.ascontiguousarray(a), dtype=dt, device=dev)
    P = d(poses, torch.float64)
    kw = {"precision": ba.PREC_F32, "ref_poses": P} if prec == "f32" else {}
    pb = ba.build_clusters_from_sums(d(voxel, torch.int32), d(scan, torch.int32), d(n, torch.int64),
                                     d(n[:, None] * mu, torch.float64), d(s2, torch.float64), N, len(counts), **kw)
    cost, _, _, eig = ba.eval_residual_grad_hessian(pb, P, derivatives=False, voxel_eig=True)
    pb.close()
    want = []
    for v in range(len(counts)):
        k = voxel == v
        w, p = n[k].astype(np.float64), mu[k] + t[scan[k]]
        m = (w[:, None] * p).sum(0) / w.sum()
        q = p - m
        A = (w[:, None, None] * (q[:, :, None] * q[:, None, :] + np.diag([0.1, 0.1, 1e-3]))).sum(0) / w.sum()
        want.append(np.linalg.eigvalsh(A)[0])
    want = np.array(want)
    # eps of the covariance's norm (about 1) by the sum's length; the precision form is specified to 1e-5
    tol = 1e-13 * max(counts) if prec == "f64" else 1e-5 * want.max()
    got = eig.cpu().numpy()[:, 0]
    assert np.abs(got - want).max() <= tol
    assert abs(cost.cpu().numpy()[0] - want.sum()) <= tol * len(counts)
