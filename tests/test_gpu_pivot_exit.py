"""A non-positive pivot in every row of the 64 x 64 diagonal factor: reported at
its place, with every wave of the workgroup leaving at the same block, so that
the workgroup's next tasks and the next solve are those of a fresh start."""
import numpy as np
import pytest

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(120)]


@pytest.mark.parametrize("n", [66, 198])
def test_every_failing_pivot_ends_the_factor_at_its_block(n):
    import torch
    import paper_2608_14266_amd as ba
    dev = torch.device("cuda:0")
    print(f"[gpu-case] failing pivots n={n}", flush=True)
    rng = np.random.default_rng(n)
    A = rng.standard_normal((n, n))
    H = torch.tensor(A @ A.T / n + np.diag(0.1 + rng.random(n)), device=dev)
    b = torch.tensor(rng.standard_normal(n), device=dev)
    ref, info = ba.solve_increment(ba.MODE_COUPLED, H, b, 0.0)
    assert info.item() == 0
    for bad in range(n):
        Hb = H.clone()
        Hb[bad, bad] = -1.0
        dx, info = ba.solve_increment(ba.MODE_COUPLED, Hb, b, 0.0)
        assert info.item() == bad + 1 and not dx.any().item()
        dx, info = ba.solve_increment(ba.MODE_COUPLED, H, b, 0.0)
        assert info.item() == 0 and torch.equal(dx, ref)
