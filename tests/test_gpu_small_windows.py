"""Windows of few poses, whose increment solve reduces the derivatives itself,
at the widest size that does so and around it: bitwise the run of the same
window in a batch that takes the general form."""
import numpy as np
import pytest

import scenes.sums as ss
from helpers import build_gpu_sums

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(120)]


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_folded_reduction_equals_general_form(prec):
    import torch
    import paper_2608_14266_amd as ba
    dev = torch.device("cuda:0")
    kw = {"precision": ba.PREC_F32} if prec == "f32" else {}

    def run(sc):
        if prec == "f32":
            kw["ref_poses"] = torch.as_tensor(sc.poses_init, device=dev).contiguous()
        pb = build_gpu_sums(ba, sc, dev, **kw)
        P = torch.as_tensor(sc.poses_init, device=dev).contiguous()
        reps, tr = ba.iterate(pb, P, ba.MODE_MM, max_iters=8)
        pb.close()
        return reps, tr, P.cpu().numpy()

    sizes = [2, 7, 17, 18, 19, 40]   # the last makes the batch take the general form
    print(f"[gpu-case] folded reduction {prec} windows {sizes}", flush=True)
    sc = ss.batch_windows(seed=515, n_windows=len(sizes), poses=sizes, vox_per_pose=8, vox_range=(40, 8000),
                          workers=1)
    reps, tr, P = run(sc)
    s0 = 0
    for w in range(sc.n_windows):
        sw = ss.window_of(sc, w)
        r1, t1, Q = run(sw)
        assert np.array_equal(Q, P[s0:s0 + sw.n_scans]), f"window {w} poses"
        assert np.array_equal(t1[:, 0, :], tr[:, w, :]), f"window {w} trace"
        for k in ("iters", "n_accepted", "cost_final", "gnorm_final", "mu_final"):
            assert r1[0][k] == reps[w][k], (w, k)
        s0 += sw.n_scans
