"""The autotuner times the derivative pass in the form each choice leads to:
with one chunk per pose, direct without a persistent grid and with the
reduction otherwise; the results stay those of the default choices."""
import pytest

import scenes.sums as ss
from helpers import build_gpu_sums

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(120)]


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_autotune_times_the_form_that_runs(prec):
    import torch
    import paper_2608_14266_amd as ba
    dev = torch.device("cuda:0")
    print(f"[gpu-case] tuner form {prec}", flush=True)
    sc = ss.batch_windows(seed=1030, n_windows=1, poses=[10], vox_per_pose=4, vox_range=(20, 100000), workers=1)
    P = torch.as_tensor(sc.poses_init, device=dev).contiguous()
    kw = {"precision": ba.PREC_F32, "ref_poses": P} if prec == "f32" else {}
    pb = build_gpu_sums(ba, sc, dev, chunk_len=64, **kw)
    assert pb.info()["n_pose_chunks"] == 10
    ref = ba.eval_residual_grad_hessian(pb, P)[:3]
    reps = 2
    ba.profile_reset()
    ba.profile_enable(True)
    try:
        best = ba.autotune(pb, P, reps)
        torch.cuda.synchronize()
    finally:
        ba.profile_enable(False)
    passes, reduced = ba.profile_query("k_pose")[1], ba.profile_query("k_reduce_partials")[1]
    ba.profile_reset()
    # five chunk lengths by four grids, three of them persistent; one untimed launch each
    assert passes == 5 * 4 * (reps + 1) and reduced == 5 * 3 * (reps + 1)
    assert ba.problem_get_tuning(pb) == {k: best[k] for k in ("vox_split", "vox_grid", "pose_grid", "chunk_len")}
    for split in (4, best["vox_split"]):
        ba.problem_set_tuning(pb, dict(best, vox_split=split))
        out = ba.eval_residual_grad_hessian(pb, P)[:3]
        if split == 4:   # the derivative pass's choices leave one chunk per pose: the same sums
            assert all(torch.equal(a, b) for a, b in zip(out, ref))
    pb.close()
