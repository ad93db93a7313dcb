"""Dense systems at the edges of the factorization's tasks of two rows and two
columns: 79 tile rows, below which a task has one column, 80 and 81, and even
and odd numbers of tile rows whose last tile is nearly full or has a few rows."""
import numpy as np
import pytest

from helpers import dense_backward_error

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(300)]


@pytest.mark.parametrize("n", [5004, 5052, 5058, 5118, 5124, 5190, 6276])
def test_task_edges_against_lapack(n):
    """Backward error within 16 times LAPACK's own on the same system; a
    non-positive pivot in the last tile is reported at its place."""
    import torch
    import paper_2608_14266_amd as ba
    dev = torch.device("cuda:0")
    print(f"[gpu-case] task edges n={n}, {-(-n // 64)} tile rows, {(n - 1) % 64 + 1} in the last", flush=True)
    g = torch.Generator(device=dev).manual_seed(n)
    A = torch.randn(n, n, generator=g, dtype=torch.float64, device=dev)
    H = A @ A.T / n
    del A
    H.diagonal().add_(0.5 + torch.rand(n, generator=g, dtype=torch.float64, device=dev))
    H = (H + H.T) / 2
    b = torch.randn(n, generator=g, dtype=torch.float64, device=dev)
    dx, info = ba.solve_increment(ba.MODE_COUPLED, H, b, 0.0)
    assert info.item() == 0
    Hn, bn = H.cpu().numpy(), b.cpu().numpy()
    ref = np.linalg.solve(Hn, -bn)
    e_ref, e = dense_backward_error(Hn, ref, -bn), dense_backward_error(Hn, dx.cpu().numpy().ravel(), -bn)
    print(f"[gpu-case] backward error {e:.2e}, LAPACK {e_ref:.2e}", flush=True)
    assert e <= 16 * e_ref
    bad = n - 1
    H[bad, bad] = -1.0
    dx, info = ba.solve_increment(ba.MODE_COUPLED, H, b, 0.0)
    assert info.item() == bad + 1 and not dx.any().item()
