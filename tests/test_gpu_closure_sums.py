"""GPU closure gradients over many rows: the length of the single-precision sums."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _bias_gradient(P, neps, width, depth):
    """Gradient of the two output biases where every row is the same: (Y - T) whatever
    the number of rows, one term of (Y - T) / rows each."""
    from paper_2206_00808_amd.binding import Mlp, mlp_blob_unpack
    ctx = P.Context(0)
    net = Mlp(ctx, 7, width, depth, 2, seed=1)
    chi = torch.full((neps, neps), -0.75, dtype=torch.complex128, device="cuda")
    qg = torch.full((neps, 3), 0.4, dtype=torch.float64, device="cuda")
    full = chi + (-0.31 + 0.17j)
    P.binding.gw_chi0_closure(ctx, net, P.GW_CLOSURE_TRAIN_STEP, neps, qg, chi, 0.05, 0.6,
                              chi0_full=full, lr=0.0)
    m = mlp_blob_unpack(net.save())["m"].astype(np.float64)
    ctx.close()
    return m[-32:-30]


# 64 splits of a small network; 16 and 8 by the size of the partials alone
@pytest.mark.parametrize("width,depth", [(64, 1), (1024, 4), (2048, 3)])
@pytest.mark.parametrize("neps", [600, 1448])
def test_bias_sums_over_many_rows(neps, width, depth):
    import paper_2206_00808_amd as P
    rows = neps * (neps + 1) // 2
    # 32 rows, rows / 32 of a split (32 splits at least) and the splits are added one after
    # another; the terms and the moment are rounded a few times more
    tol = (32 + rows / 32 / 32 + 64 + 8) * 2.0 ** -24
    got, want = _bias_gradient(P, neps, width, depth), _bias_gradient(P, 1, width, depth)
    assert np.all(np.abs(want) > 1e-3)
    assert np.all(np.abs(got / want - 1) <= tol), (got / want - 1, tol)
