"""Problems whose poses have one chunk each, whose derivative pass stores the
derivatives itself and sums the windows' residuals: bitwise the form with a
reduction, over window sizes around a block of the pass and window sums longer
than the summing block."""
import numpy as np
import pytest

import scenes.sums as ss
from helpers import build_gpu_sums

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(120)]


@pytest.mark.parametrize("sizes,vox_per_pose", [([2], 8), ([3, 4, 5, 9], 20), ([1200], 60)])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_direct_pass_equals_reduction(sizes, vox_per_pose, prec):
    import torch
    import paper_2608_14266_amd as ba
    dev = torch.device("cuda:0")
    print(f"[gpu-case] direct pass {prec} windows {sizes}", flush=True)
    sc = ss.batch_windows(seed=626, n_windows=len(sizes), poses=list(sizes), vox_per_pose=vox_per_pose,
                          vox_range=(20, 100000), workers=1)
    P = torch.as_tensor(sc.poses_init, device=dev).contiguous()
    kw = {"precision": ba.PREC_F32, "ref_poses": P} if prec == "f32" else {}
    pb = build_gpu_sums(ba, sc, dev, chunk_len=1024, **kw)
    assert pb.info()["n_pose_chunks"] == sum(sizes)
    modes = [ba.MODE_MM] + ([ba.MODE_COUPLED] if sizes == [2] else [])
    out = {}
    for grid in (0, 1):   # a persistent grid takes the form with a reduction
        ba.problem_set_tuning(pb, {"vox_split": 4, "vox_grid": 0, "pose_grid": grid, "chunk_len": 1024})
        out[grid] = [[a.cpu().numpy() for a in ba.eval_residual_grad_hessian(pb, P, mode)[:3]] for mode in modes]
        Q = P.clone()
        reps, tr = ba.iterate(pb, Q, ba.MODE_MM, max_iters=5)
        out[grid].append([Q.cpu().numpy(), np.asarray(tr)])
    pb.close()
    for a, b in zip(out[0], out[1]):
        for x, y in zip(a, b):
            assert np.array_equal(x, y)
