"""GPU inverse by LU with pivoting where the square of a pivot leaves the range of the
type: blocks of two rows that only exchange each other, beside ordinary ones."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# 3074 rows: a panel that stays in global memory
@pytest.mark.parametrize("n", [2, 34, 260, 3074])
@pytest.mark.parametrize("x", [1e-150, 1e-155, 1e-158, 1e-161, 1e-300, 1e150, 1e155, 1e300])
def test_pivots_whose_square_leaves_the_range(x, n):
    import paper_2206_00808_amd as P
    # eps = I - chi: zero diagonal, eps[i, n-1-i] = x (3 + 4i) / 5 or (every third pair) 2
    i = np.arange(n)
    z = np.where(np.minimum(i, n - 1 - i) % 3 == 2, 2.0, x) * (0.6 + 0.8j)
    chi = np.eye(n) + 0j
    chi[i, n - 1 - i] = -z
    ctx = P.Context(0)
    out = torch.empty((1, n, n), dtype=torch.complex128, device="cuda")
    P.gw_epsinv_lu(ctx, n, 1, torch.from_numpy(chi[None]).cuda(),
                   torch.ones(n, dtype=torch.float64, device="cuda"), out)
    ctx.close()
    got = out[0].cpu().numpy()
    want = (0.6 - 0.8j) / np.where(np.minimum(i, n - 1 - i) % 3 == 2, 2.0, x)  # |0.6 + 0.8i| = 1
    # one reciprocal and one product per entry: a few roundings, and 0.6, 0.8 themselves
    assert np.all(np.abs(got[i, n - 1 - i] / want - 1) <= 32 * 2.0 ** -53)
    got[i, n - 1 - i] = 0
    assert not got.any()
