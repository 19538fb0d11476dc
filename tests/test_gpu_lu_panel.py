"""GPU eps^-1 by pivoted LU at the edges of its panels and row counts: below, at and
above one 32-column panel and one 256-row slice of a thread's rows, matrices whose
pivots move at every step, and a singular one."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("neps", [1, 2, 7, 8, 9, 31, 32, 33, 40, 255, 256, 257, 289, 513, 1100, 3105])
def test_lu_inverse(neps):
    import paper_2206_00808_amd as P
    rng = np.random.default_rng(neps)
    ctx = P.Context(0)
    nf = 2 if neps < 1000 else 1
    eps = rng.normal(size=(nf, neps, neps)) + 1j * rng.normal(size=(nf, neps, neps))
    eps[0] = eps[0, ::-1]
    if neps > 8:  # equal columns of candidates: the lowest row is taken
        eps[0, :, 0] = 1.0
    v = rng.uniform(0.5, 2.0, neps)
    chi = (np.eye(neps) - eps) / v[:, None]
    c = torch.from_numpy(np.ascontiguousarray(chi)).cuda()
    out = torch.empty_like(c)
    P.gw_epsinv_lu(ctx, neps, nf, c, torch.from_numpy(v).cuda(), out)
    e = torch.eye(neps, dtype=torch.complex128, device="cuda")
    for f in range(nf):
        m = e - torch.from_numpy(v).cuda()[:, None] * c[f]
        r = (m @ out[f] - e).abs().max()
        # partial pivoting: residual within n u times the norms (growth included by a
        # factor n^(1/2) for random matrices)
        bound = neps ** 1.5 * 2.0 ** -52 * m.abs().sum(1).max() * out[f].abs().max()
        assert float(r) <= max(float(bound), 2.0 ** -50)
    ctx.close()


def test_lu_reports_a_zero_pivot():
    import paper_2206_00808_amd as P
    rng = np.random.default_rng(5)
    n = 70
    eps = rng.normal(size=(n, n)) + 1j * rng.normal(size=(n, n))
    eps[:, 41] = 0.0
    chi = torch.from_numpy((np.eye(n) - eps)[None].copy()).cuda()
    ctx = P.Context(0)
    with pytest.raises(P.GwError) as err:
        P.gw_epsinv_lu(ctx, n, 1, chi, torch.ones(n, dtype=torch.float64, device="cuda"),
                       torch.empty_like(chi))
    assert err.value.status == P.GW_ESINGULAR
    ctx.close()
