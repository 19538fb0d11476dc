"""GPU eigenvectors for the reduced basis where the squares of entries leave the range of
the type, and at further edges of the divide (leaves of at most 16 rows) and of the blocks
of 32 reflectors, against numpy."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _random(n, rng):
    a = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    return a + a.conj().T


def _matrix(kind, n, rng):
    if kind == "random":
        return _random(n, rng)
    if kind == "rank":  # three quarters of the eigenvalues equal
        m = _random(n, rng)[:max(1, n // 4)]
        return np.eye(n) + m.conj().T @ m
    if kind == "fourfold":
        q = np.linalg.qr(_random(n, rng))[0]
        h = (q * np.repeat(np.arange(1.0, n // 4 + 2), 4)[:n]) @ q.conj().T
        return (h + h.conj().T) / 2
    # graded: rows and columns from one down to 2^-40
    d = 2.0 ** np.linspace(0, -40, n)
    return d[:, None] * _random(n, rng) * d[None, :]


def _check(h, nb):
    import paper_2206_00808_amd as P
    n = h.shape[0]
    ctx = P.Context(0)
    chi = np.ascontiguousarray(np.eye(n) - h)
    h = np.eye(n) - chi
    c, v = torch.from_numpy(chi).cuda(), torch.ones(n, dtype=torch.float64, device="cuda")
    u = torch.empty((n, nb), dtype=torch.complex128, device="cuda")
    ev = torch.empty(n, dtype=torch.float64, device="cuda")
    P.gw_lowrank_basis(ctx, n, c, v, nb, u, ev)
    ctx.close()
    lam, u = ev.cpu().numpy(), u.cpu().numpy()
    w = np.linalg.eigvalsh(h)
    # backward error of the reflections, rotations and products: a small multiple of
    # n 2^-53 of the norm
    tol = 16 * n * 2.0 ** -53
    big = np.abs(w).max()
    assert np.abs(lam - w).max() <= tol * big
    assert np.abs(h @ u - u * lam[::-1][None, :nb]).max() <= tol * big
    assert np.abs(u.conj().T @ u - np.eye(nb)).max() <= tol


@pytest.mark.parametrize("x", [1e-150, 1e-157, 1e-158, 1e-160, 1e-161, 2.5e-162, 1e-170, 1e-300,
                               3e-324, 0.0])
@pytest.mark.parametrize("n", [3, 12, 300])
def test_subdiagonal_entry_whose_square_underflows(n, x):
    h = _random(n, np.random.default_rng(n))
    h[1, 0], h[0, 1] = x * (1 + 1j), x * (1 - 1j)
    _check(h, n)


@pytest.mark.parametrize("x", [1e-160, 1e-310, 3e-324])
def test_two_rows_with_a_vanishing_entry(x):
    _check(np.array([[2.0, x * (1 - 1j)], [x * (1 + 1j), -1.0]]), 2)


@pytest.mark.parametrize("n", [15, 16, 17, 34, 35])
@pytest.mark.parametrize("kind", ["random", "rank", "fourfold", "graded"])
def test_edges_of_leaves_and_blocks(kind, n):
    _check(_matrix(kind, n, np.random.default_rng(n)), n)


@pytest.mark.parametrize("kind,n", [("rank", 600), ("fourfold", 1100), ("graded", 600)])
def test_spectra_that_deflate_over_512_rows(kind, n):
    _check(_matrix(kind, n, np.random.default_rng(n)), 60)
