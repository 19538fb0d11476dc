"""GPU eps^-1 by blocked Gauss-Jordan at the edges of its 16- and 64-row blocks, 32-row
output tiles and of the LDS route (2048), for a chi0 that is Hermitian to the last bit (half
the blocks are kept) and for one that is so to rounding only (every block)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _chi(n, nf, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    b = torch.randn((nf, n, n + 9), dtype=torch.complex128, device="cuda", generator=g)
    x = -0.5 / (n + 9) * torch.matmul(b, b.conj().transpose(1, 2).contiguous())
    return 0.5 * (x + x.conj().transpose(1, 2))


@pytest.mark.parametrize("exact", [True, False])
@pytest.mark.parametrize("n,nf", [(1, 1), (15, 2), (16, 1), (17, 3), (63, 2), (64, 2), (65, 2),
                                  (128, 1), (129, 3), (191, 2), (321, 2), (2049, 1)])
def test_epsinv_blocks(n, nf, exact):
    import paper_2206_00808_amd as P
    if n == 1 and not exact:
        pytest.skip("one real number")
    ctx = P.Context(0)
    chi = _chi(n, nf, n)
    assert bool((chi == chi.conj().transpose(1, 2)).all())
    if not exact:  # one entry per matrix off by its last bit
        chi[:, 0, n - 1] = chi[:, 0, n - 1] * (1 + 2.0 ** -52)
        assert not bool((chi == chi.conj().transpose(1, 2)).all())
    v = torch.linspace(0.3, 4.0, n, dtype=torch.float64, device="cuda")
    out = torch.empty_like(chi)
    ctx.profile(True)
    P.gw_epsinv(ctx, n, nf, chi, v, out)
    torch.cuda.synchronize()
    assert "lu_panel" not in ctx.profile_table()
    ctx.profile(False)
    e = torch.eye(n, dtype=torch.complex128, device="cuda")
    for f in range(nf):
        m = e - v[:, None] * chi[f]
        r = (torch.matmul(m, out[f]) - e).abs().max()
        # eps~ is at most 1 + max v ||chi0|| < 20, its inverse at most 1: the elimination's
        # error and the residual's own, each a small multiple of n 2^-53 of the norms
        assert float(r) <= 16 * n * 2.0 ** -53 * 20
    ctx.close()
