"""Windows of few poses whose poses have several chunks: the increment solve sums
the chunks itself up to 18 poses, bitwise as the general form does, alone and
with other small windows, in both precisions."""
from dataclasses import replace

import numpy as np
import pytest

import scenes.sums as ss
from helpers import build_gpu_sums

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(120)]

ITERS = 6


@pytest.mark.parametrize("chunk_len", [32, 100])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_sums_over_several_chunks_in_the_solve(prec, chunk_len):
    import torch
    import paper_2608_14266_amd as ba
    dev = torch.device("cuda:0")

    def run(sc, folded):
        P = torch.as_tensor(sc.poses_init, device=dev).contiguous()
        kw = {"precision": ba.PREC_F32, "ref_poses": P.clone()} if prec == "f32" else {}
        pb = build_gpu_sums(ba, sc, dev, chunk_len=chunk_len, **kw)
        assert pb.info()["n_pose_chunks"] >= 2 * sc.n_scans
        ba.profile_reset()
        ba.profile_enable(True)
        try:
            ba.iterate(pb, P.clone(), ba.MODE_MM, max_iters=ITERS)
        finally:
            ba.profile_enable(False)
        # the derivatives at the final poses are reduced by a launch of their own in both forms
        assert ba.profile_query("k_reduce_partials")[1] == (1 if folded else 1 + ITERS)
        ba.profile_reset()
        reps, tr = ba.iterate(pb, P, ba.MODE_MM, max_iters=ITERS)
        pb.close()
        return reps, np.asarray(tr), P.cpu().numpy()

    sizes = [2, 7, 17, 18]
    print(f"[gpu-case] folded chunks of {chunk_len} {prec}", flush=True)
    general = ss.batch_windows(seed=1131, n_windows=5, poses=sizes + [40], vox_per_pose=60, vox_range=(400, 8000),
                               workers=1)
    # the same windows without the last, which makes the batch take the general form
    n_s = sum(sizes)
    sel = general.scan < n_s
    small = replace(general, voxel=general.voxel[sel], scan=general.scan[sel], count=general.count[sel],
                    sum=general.sum[sel], sumsq=general.sumsq[sel], n_scans=n_s,
                    n_voxels=int(general.voxel[sel].max()) + 1, poses_true=general.poses_true[:n_s],
                    poses_init=general.poses_init[:n_s], n_windows=4, scan_window=general.scan_window[:n_s])
    reps, tr, P = run(general, False)
    reps_s, tr_s, P_s = run(small, True)
    s0 = 0
    for w, n in enumerate(sizes):
        one = run(ss.window_of(general, w), True)
        for r, t, Q in ((one[0][0], one[1][:, 0], one[2]), (reps_s[w], tr_s[:, w], P_s[s0:s0 + n])):
            assert np.array_equal(Q, P[s0:s0 + n]), f"window {w} poses"
            assert np.array_equal(t, tr[:, w]), f"window {w} trace"
            for k in ("iters", "n_accepted", "cost_final", "gnorm_final", "mu_final"):
                assert r[k] == reps[w][k], (w, k)
        s0 += n
