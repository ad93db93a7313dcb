"""The coupled form's buffers when they do not fit the device: every call fails
by itself, also after a first failure, and the problem stays usable."""
import numpy as np
import pytest

import scenes.sums as ss
from helpers import build_gpu_sums

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(120)]


def test_a_coupled_form_that_does_not_fit_fails_on_every_call():
    import torch
    import paper_2608_14266_amd as ba
    dev = torch.device("cuda:0")
    n = 60000   # a 360,000 x 360,000 matrix: 1 TB
    print(f"[gpu-case] coupled form of {n} poses", flush=True)
    sc = ss.batch_windows(seed=727, n_windows=1, poses=[n], vox_per_pose=1, vox_range=(20, 100000), workers=1)
    pb = build_gpu_sums(ba, sc, dev)
    P = torch.as_tensor(sc.poses_init, device=dev).contiguous()
    ref = [a.cpu().numpy() for a in ba.eval_residual_grad_hessian(pb, P)[:3]]
    for _ in range(3):
        Q = P.clone()
        with pytest.raises(ba.BAError) as e:
            ba.iterate(pb, Q, ba.MODE_COUPLED, max_iters=1)
        assert e.value.status == -6 and torch.equal(Q, P)
    for a, r in zip(ba.eval_residual_grad_hessian(pb, P)[:3], ref):
        assert np.array_equal(a.cpu().numpy(), r)
    pb.close()
