"""Memory kept between calls (ba_release_cached_memory): calls that take kept
blocks give bitwise the results of calls that took fresh ones, from several
threads and streams at once, and what is kept goes back on request."""
import threading

import numpy as np
import pytest

import scenes
from helpers import build_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ba():
    import torch
    torch.cuda.set_device(0)
    import paper_2608_14266_amd as m
    m.load()
    return m


def _pass(ba, sc, dev):
    """Build, evaluate, voxelize (device and host): every output as numpy arrays."""
    import torch
    prob = build_gpu(ba, sc, dev)
    P = torch.as_tensor(sc.poses_init, dtype=torch.float64, device=dev)
    out = [t.cpu().numpy() for t in ba.eval_residual_grad_hessian(prob, P)[:3]]
    out += [t.cpu().numpy() for t in prob.export_clusters()]
    prob.close()
    t = lambda a, dt: torch.as_tensor(a, dtype=dt, device=dev)
    m = ba.voxelize(t(sc.x, torch.float64), t(sc.y, torch.float64), t(sc.z, torch.float64), t(sc.scan, torch.int32),
                    P, 0.5, 2, 0.1)
    out += [v.cpu().numpy() for _, v in sorted(m.export().items())]
    m.close()
    m = ba.voxelize_host(sc.x, sc.y, sc.z, sc.scan, P, 0.5, 2, 0.1, batch_points=max(1024, sc.n_points // 3))
    out += [v.cpu().numpy() for _, v in sorted(m.export().items())]
    m.close()
    return out


def _same(a, b):
    return len(a) == len(b) and all(np.array_equal(x, y) for x, y in zip(a, b))


def test_kept_blocks_threads_and_streams_change_nothing(ba):
    import torch
    dev = torch.device("cuda:0")
    sizes = [(12, 300), (40, 2500), (25, 900)]
    scs = [scenes.scaled_window(seed=2100 + i, n_scans=n, n_planes=p) for i, (n, p) in enumerate(sizes)]
    ba.release_cached_memory()
    fresh = []
    for sc in scs:
        fresh.append(_pass(ba, sc, dev))
        ba.release_cached_memory()
    for sc, ref in zip(scs, fresh):
        print(f"[gpu-case] kept blocks, one thread: {sc.n_points} points", flush=True)
        for _ in range(2):
            assert _same(_pass(ba, sc, dev), ref)
    bad = []

    def work(i):
        torch.cuda.set_device(0)
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(3):
                if not _same(_pass(ba, scs[i], dev), fresh[i]):
                    bad.append(i)

    print("[gpu-case] kept blocks, three threads on their own streams", flush=True)
    th = [threading.Thread(target=work, args=(i,)) for i in range(3)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    assert not bad


def test_kept_memory_is_given_back(ba):
    import torch
    dev = torch.device("cuda:0")
    sc = scenes.scaled_window(seed=2110, n_scans=60, n_planes=20000)
    ba.release_cached_memory()
    pts = sc.n_points
    _pass(ba, sc, dev)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    held = torch.cuda.mem_get_info()[0]
    ba.release_cached_memory()
    free = torch.cuda.mem_get_info()[0]
    # the build's sort alone takes 24 bytes a point
    print(f"[gpu-case] {pts} points: {free - held} bytes given back", flush=True)
    assert free - held >= 24 * pts
    ba.release_cached_memory()   # nothing kept: no error
