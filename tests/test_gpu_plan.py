"""The build plan formed on the device: group, block and chunk tables at the
edges (one cluster, group sizes round 64, split classes round 4 and 8 clusters
per voxel, windows without voxels, unobserved scans, unsorted input), checked
through the oracle's evaluation of the same clusters and through the plan's
own counts."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = 1e-12


@pytest.fixture(scope="module")
def ba():
    import torch
    torch.cuda.set_device(0)
    import paper_2608_14266_amd as m
    m.load()
    return m


def _clusters(rng, per_m, n_scans, scan0=0):
    """per_m: {observers per voxel: voxels}; every voxel's scans distinct, in random order."""
    vox, scan = [], []
    v = 0
    for m, k in per_m.items():
        for _ in range(k):
            scan += list(scan0 + rng.choice(n_scans, size=m, replace=False))
            vox += [v] * m
            v += 1
    vox, scan = np.array(vox, np.int32), np.array(scan, np.int32)
    perm = rng.permutation(len(vox))
    return vox[perm], scan[perm], v


def _payload(rng, n):
    count = rng.integers(5, 60, n).astype(np.int64)
    mu = rng.uniform(-20, 20, (n, 3))
    A = rng.normal(size=(n, 3, 3)) * 0.3
    S = (A @ A.transpose(0, 2, 1)) * count[:, None, None]
    Q = S + count[:, None, None] * mu[:, :, None] * mu[:, None, :]
    iu = ([0, 0, 0, 1, 1, 2], [0, 1, 2, 1, 2, 2])
    return count, mu * count[:, None], np.ascontiguousarray(Q[:, iu[0], iu[1]])


def _poses(rng, n):
    P = np.zeros((n, 12))
    for j in range(n):
        q, _ = np.linalg.qr(rng.normal(size=(3, 3)))
        q *= np.sign(np.linalg.det(q))
        P[j, :9], P[j, 9:] = q.ravel(), rng.uniform(-5, 5, 3)
    return P


CASES = {
    "one cluster": ({1: 1}, 1),
    "group edges": ({3: 63, 4: 64, 5: 65, 8: 129, 9: 1}, 12),
    "split classes": ({1: 5, 2: 300, 4: 257, 5: 200, 8: 64, 9: 70, 16: 3}, 20),
    "unobserved scans": ({2: 100}, 300),
    "long voxels": ({70: 3, 1: 10}, 90),
}


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("name", list(CASES))
def test_plan_tables_and_voxel_results(ba, orc, name, precision):
    import torch
    per_m, n_scans = CASES[name]
    rng = np.random.default_rng(77)
    vox, scan, V = _clusters(rng, per_m, n_scans)
    count, s1, s2 = _payload(rng, len(vox))
    P = _poses(rng, n_scans)
    print(f"[gpu-case] plan {name}: {len(vox)} clusters, {V} voxels, precision {precision}", flush=True)
    t = lambda a, dt: torch.as_tensor(a, dtype=dt, device="cuda")
    poses = t(P, torch.float64)

    def build(i):
        return ba.build_clusters_from_sums(t(vox[i], torch.int32), t(scan[i], torch.int32), t(count[i], torch.int64),
                                           t(s1[i], torch.float64), t(s2[i], torch.float64), n_scans, V,
                                           precision=precision, ref_poses=poses if precision else None)
    order = np.lexsort((scan, vox))
    prob, srt = build(np.arange(len(vox))), build(order)
    inf = prob.info()
    assert inf["n_clusters"] == len(vox) and inf["n_voxels"] == V and inf["max_m"] == max(per_m)
    assert inf["n_wave_groups"] == sum(-(-k // 64) for k in per_m.values())
    assert inf["padded_clusters"] == sum(64 * m * -(-k // 64) for m, k in per_m.items())
    per_scan = np.bincount(scan, minlength=n_scans)
    assert inf["n_pose_chunks"] == int(np.sum(-(-per_scan // 256)))
    ev, es, ec, _, _ = [a.cpu().numpy() for a in prob.export_clusters()]
    assert np.array_equal(ev, vox[order]) and np.array_equal(es, scan[order])
    assert np.array_equal(ec, count[order].astype(np.float64))
    mu, S = orc.center_raw_sums(count[order], s1[order], s2[order])
    lam = orc.voxel_stats(orc.Clusters(vox[order], scan[order], count[order], mu, S, V, n_scans), P)["lam"]
    # an eigenvalue is defined to rounding times the largest one, whatever the gaps
    tol = (1e-5 if precision else 1e-12) * lam[:, 2]
    for tuning in ({"vox_split": 4}, {"vox_split": 0}, {"vox_split": 1, "chunk_len": 32}):
        ba.problem_set_tuning(prob, tuning)
        ba.problem_set_tuning(srt, tuning)
        cost, grad, hess, eig = [a.cpu().numpy() for a in
                                 ba.eval_residual_grad_hessian(prob, poses, voxel_eig=True)]
        assert np.all(np.abs(eig[:, 0] - lam[:, 0]) <= tol)
        assert abs(cost[0] - lam[:, 0].sum()) <= tol.sum()
        # the input's order does not matter, bit for bit
        for a, b in zip((cost, grad, hess, eig), ba.eval_residual_grad_hessian(srt, poses, voxel_eig=True)):
            assert np.array_equal(a, b.cpu().numpy())
        # poses no cluster observes have empty blocks, the others do not
        assert np.array_equal(np.abs(hess).sum((1, 2)) > 0, per_scan > 0)


def test_windows_without_voxels(ba):
    """Windows 0, 2 and 4 of five hold the clusters; each equals its problem alone, bitwise."""
    import torch
    rng = np.random.default_rng(5)
    n_scans, win = 30, np.repeat(np.arange(5), 6).astype(np.int32)
    t = lambda a, dt: torch.as_tensor(np.ascontiguousarray(a), dtype=dt, device="cuda")
    parts, alone = [], []
    P = _poses(rng, n_scans)
    for w, per_m in ((0, {2: 70, 5: 3}), (2, {1: 1}), (4, {3: 130, 6: 65})):
        vox, scan, V = _clusters(rng, per_m, 6)
        pay = _payload(rng, len(vox))
        parts.append((w, vox, scan, V, pay))
        prob = ba.build_clusters_from_sums(t(vox, torch.int32), t(scan, torch.int32), t(pay[0], torch.int64),
                                           t(pay[1], torch.float64), t(pay[2], torch.float64), 6, V)
        ba.problem_set_tuning(prob, {"vox_split": 0})
        r = ba.eval_residual_grad_hessian(prob, t(P[6 * w:6 * w + 6], torch.float64))
        alone.append([a.cpu().numpy() for a in r[:3]])
    off = np.cumsum([0] + [p[3] for p in parts])
    vox = np.concatenate([p[1] + o for p, o in zip(parts, off)]).astype(np.int32)
    scan = np.concatenate([p[2] + 6 * p[0] for p in parts]).astype(np.int32)
    cnt, s1, s2 = [np.concatenate([p[4][k] for p in parts]) for k in range(3)]
    prob = ba.build_clusters_from_sums(t(vox, torch.int32), t(scan, torch.int32), t(cnt, torch.int64),
                                       t(s1, torch.float64), t(s2, torch.float64), n_scans, int(off[-1]), n_windows=5,
                                       scan_window=win)
    ba.problem_set_tuning(prob, {"vox_split": 0})
    cost, grad, hess, _ = [None if a is None else a.cpu().numpy() for a in
                           ba.eval_residual_grad_hessian(prob, t(P, torch.float64))]
    for (w, *_), (c, g, h) in zip(parts, alone):
        assert cost[w] == c[0]
        assert np.array_equal(grad[6 * w:6 * w + 6], g) and np.array_equal(hess[6 * w:6 * w + 6], h)
    assert cost[1] == 0.0 and cost[3] == 0.0


def test_voxel_across_windows_is_refused(ba):
    import torch
    t = lambda a, dt: torch.as_tensor(np.array(a), dtype=dt, device="cuda")
    rng = np.random.default_rng(6)
    pay = _payload(rng, 6)
    with pytest.raises(ba.BAError, match="voxel 7 is observed by scans of different windows"):
        ba.build_clusters_from_sums(t([3, 3, 7, 7, 9, 9], torch.int32), t([0, 1, 1, 2, 0, 3], torch.int32),
                                    t(pay[0], torch.int64), t(pay[1], torch.float64), t(pay[2], torch.float64), 4, 12,
                                    n_windows=2, scan_window=[0, 0, 1, 1])


@pytest.mark.parametrize("n", [1, 63, 64, 65, 2047, 2048, 2049, 4095, 4096, 4097, 20000])
def test_input_order_routes_agree(ba, n):
    """Points in log order, in (voxel, scan) order and in no order take different sorts (by voxel alone, none, by
    both); a cluster's own points keep their order in all three, so every output is bitwise the same."""
    import torch
    rng = np.random.default_rng(n)
    n_scans, V = 17, 300
    scan, vox = rng.integers(0, n_scans, n).astype(np.int32), rng.integers(0, V, n).astype(np.int32)
    xyz = rng.uniform(-30, 30, (3, n))
    P = _poses(rng, n_scans)
    t = lambda a, dt: torch.as_tensor(np.ascontiguousarray(a), dtype=dt, device="cuda")
    print(f"[gpu-case] input orders, {n} points", flush=True)
    builds, maps = [], []
    for order in (np.arange(n), np.argsort(scan, kind="stable"), np.lexsort((scan, vox))):
        x, y, z = (t(a[order], torch.float64) for a in xyz)
        sc, vx = t(scan[order], torch.int32), t(vox[order], torch.int32)
        prob = ba.build_clusters(x, y, z, sc, vx, n_scans, V)
        builds.append([a.cpu().numpy() for a in prob.export_clusters()])
        m = ba.voxelize(x, y, z, sc, t(P, torch.float64), 2.0, 3, 5.0)
        maps.append((m.info()["level_clusters"], {k: v.cpu().numpy() for k, v in m.export().items()}))
    key = np.unique(vox.astype(np.int64) * n_scans + scan, return_counts=True)
    assert np.array_equal(builds[0][0].astype(np.int64) * n_scans + builds[0][1], key[0])
    assert np.array_equal(builds[0][2], key[1].astype(np.float64))
    for b in builds[1:]:
        assert all(np.array_equal(a, c) for a, c in zip(builds[0], b))
    # log order against no order: a cell holds points of several voxels, in (voxel) order in the third
    assert maps[0][0] == maps[1][0] == maps[2][0]
    assert all(np.array_equal(maps[0][1][k], maps[1][1][k]) for k in maps[0][1])
