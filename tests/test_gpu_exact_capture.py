"""The first run with the exact form near convergence, whose vectors are
allocated ahead of the graph capture: memory that the library keeps between
calls stays kept through it and goes back on request."""
import pytest

import scenes
import scenes.sums as ss
from helpers import build_gpu, build_gpu_sums

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(120)]


def test_first_exact_run_leaves_the_kept_memory_alone():
    import torch
    import paper_2608_14266_amd as ba
    dev = torch.device("cuda:0")
    print("[gpu-case] first exact run with kept memory", flush=True)
    free = lambda: torch.cuda.mem_get_info()[0]
    big = scenes.scaled_window(seed=828, n_scans=60, n_planes=20000)   # the kept memory: 24 bytes a point and more
    sc = ss.batch_windows(seed=829, n_windows=1, poses=[100], vox_per_pose=1500, vox_range=(20, 200000), workers=1)
    ba.release_cached_memory()
    pb = build_gpu_sums(ba, sc, dev)
    P = torch.as_tensor(sc.poses_init, device=dev).contiguous()
    ba.iterate(pb, P.clone(), ba.MODE_COUPLED, max_iters=1)
    ba.release_cached_memory()
    # kept blocks, none as large as the exact vectors (144 bytes a cluster), so that these are allocated anew
    assert 144 * pb.info()["n_clusters"] > 8 * big.n_points
    build_gpu(ba, big, dev).close()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    kept = free()
    reps, _ = ba.iterate(pb, P.clone(), ba.MODE_COUPLED, max_iters=2, exact_below=1e30)
    assert reps[0]["iters"] == 2
    torch.cuda.synchronize()
    after = free()
    ba.release_cached_memory()
    given = free() - after
    print(f"[gpu-case] free {kept} before, {after} after the run, {given} given back on request", flush=True)
    assert given >= 24 * big.n_points
    assert after <= kept
    pb.close()
