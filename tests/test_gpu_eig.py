"""GPU eigenvectors for the reduced basis at the edges of leaves (32 rows), spans (256) and
of the sizes whose step vectors fit LDS (2048), over spectra that deflate not at all, in
part and entirely, against numpy."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _matrix(kind, n, rng):
    g = lambda *s: rng.standard_normal(s) + 1j * rng.standard_normal(s)
    if kind == "random":
        a = g(n, n)
        return a + a.conj().T
    if kind == "rank":  # most eigenvalues equal
        m = g(max(1, n // 4), n)
        return np.eye(n) + m.conj().T @ m
    if kind == "fourfold":
        q = np.linalg.qr(g(n, n))[0]
        h = (q * np.repeat(np.arange(1.0, n // 4 + 2), 4)[:n]) @ q.conj().T
        return (h + h.conj().T) / 2
    if kind == "wilkinson":  # pairs of eigenvalues equal to working precision
        o = np.ones(n - 1)
        return np.diag(np.abs(np.arange(n) - (n - 1) / 2)) + np.diag(o, 1) + np.diag(o, -1) + 0j
    return np.ones((n, n)) + 0j


@pytest.mark.parametrize("n", [1, 2, 3, 4, 32, 33, 65, 130, 257, 500])
@pytest.mark.parametrize("kind", ["random", "rank", "fourfold", "wilkinson", "ones"])
def test_eigenvectors(kind, n):
    _check(_matrix(kind, n, np.random.default_rng(n)), (n, max(1, n // 10)))


def test_eigenvectors_above_lds_size():
    _check(_matrix("random", 2055, np.random.default_rng(3)), (40,))


def _check(h, nbs):
    import paper_2206_00808_amd as P
    n = h.shape[0]
    ctx = P.Context(0)
    chi = np.ascontiguousarray(np.eye(n) - h)
    h = np.eye(n) - chi
    c, v = torch.from_numpy(chi).cuda(), torch.ones(n, dtype=torch.float64, device="cuda")
    w = np.linalg.eigvalsh(h)
    big = np.abs(w).max()
    # backward error of the reflections, rotations and products: a small multiple of
    # n 2^-53 of the norm
    tol = 16 * n * 2.0 ** -53
    hd = torch.from_numpy(h).cuda()
    for nb in nbs:
        u = torch.empty((n, nb), dtype=torch.complex128, device="cuda")
        ev = torch.empty(n, dtype=torch.float64, device="cuda")
        P.gw_lowrank_basis(ctx, n, c, v, nb, u, ev)
        lam = ev.cpu().numpy()
        assert np.abs(lam - w).max() <= tol * big
        top = ev.flip(0)[:nb]
        assert float((hd @ u - u * top[None, :]).abs().max()) <= tol * big
        assert float((u.conj().T @ u - torch.eye(nb, device="cuda")).abs().max()) <= tol
    ctx.close()


@pytest.mark.parametrize("n", [20, 150])
def test_matrix_that_has_no_such_basis_is_refused(n):
    import paper_2206_00808_amd as P
    rng = np.random.default_rng(n)
    ctx = P.Context(0)
    v = torch.ones(n, dtype=torch.float64, device="cuda")
    u = torch.empty((n, 2), dtype=torch.complex128, device="cuda")
    h = _matrix("random", n, rng)
    for bad in ("nan", "inf", "skew"):
        a = h.copy()
        if bad == "skew":
            a[1, 2] += 1e-3
        else:
            a[3, 5] = complex(float(bad), 0.0)
        with pytest.raises(P.GwError) as err:
            P.gw_lowrank_basis(ctx, n, torch.from_numpy(a).cuda(), v, 2, u)
        assert err.value.status == P.GW_EINVAL
    ctx.close()
