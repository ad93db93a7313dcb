"""The 64 x 64 diagonal factor of the dense solve at the edges of its 16 x 16
blocks, of its tiles and of the tile columns that the dataflow hands on."""
import numpy as np
import pytest

from helpers import dense_backward_error

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(120)]


@pytest.mark.parametrize("n", [6, 12, 18, 48, 54, 66, 78, 126, 132, 192, 198, 258, 390])
def test_diagonal_factor_against_lapack(n):
    """Backward error within the n u bound of a Cholesky solve (factor and two
    substitutions) plus LAPACK's own; a non-positive pivot is reported at its
    place in every block, and a system with a huge or tiny scale is solved as
    the unscaled one."""
    import torch
    import paper_2608_14266_amd as ba
    dev = torch.device("cuda:0")
    print(f"[gpu-case] diagonal factor n={n}", flush=True)
    rng = np.random.default_rng(n)
    A = rng.standard_normal((n, n))
    H = A @ A.T / n + np.diag(0.1 + rng.random(n))
    H = (H + H.T) / 2
    b = rng.standard_normal(n)
    bound = 3 * n * 2.0 ** -53 + 16 * dense_backward_error(H, np.linalg.solve(H, -b), -b)
    for scale in (1.0, 2.0 ** 1000, 2.0 ** -1000):
        dx, info = ba.solve_increment(ba.MODE_COUPLED, torch.tensor(H * scale, device=dev),
                                      torch.tensor(b, device=dev), 0.0)
        assert info.item() == 0
        e = dense_backward_error(H, dx.cpu().numpy().ravel() * scale, -b)
        assert e <= bound, (scale, e, bound)
    for bad in sorted({k for k in (0, 1, 15, 16, 31, 40, 47, 63, 64, 65, 90, 127, 128, 191, 250, n - 1) if k < n}):
        Hb = torch.tensor(H, device=dev)
        Hb[bad, bad] = -1.0
        dx, info = ba.solve_increment(ba.MODE_COUPLED, Hb, torch.tensor(b, device=dev), 0.0)
        assert info.item() == bad + 1 and not dx.any().item()
