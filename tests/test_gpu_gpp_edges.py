"""GPU plasmon-pole self-energy at the edges of its tiles (16 rows, 64 columns), chunks of
32 states and counts of occupied states and energies, against the sums in numpy."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [1, 15, 17, 64, 65])
@pytest.mark.parametrize("nn,nocc", [(1, 0), (1, 1), (32, 32), (65, 33), (40, 0)])
@pytest.mark.parametrize("ne", [1, 2, 3, 4])
def test_sigma_gpp_edges(n, nn, nocc, ne):
    import paper_2206_00808_amd as P
    rng = np.random.default_rng(1000 * n + 10 * nn + ne)
    nb = 2
    m = rng.standard_normal((nn, nb, n)) + 1j * rng.standard_normal((nn, nb, n))
    en = np.sort(rng.uniform(-0.5, 1.0, nn))
    v = rng.uniform(0.1, 3.0, n)
    amp = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    wt = rng.uniform(0.8, 3.0, (n, n)) + 1j * rng.uniform(-0.3, 0.3, (n, n))
    amp[0, 0], wt[0, 0] = 0.0, 1.0  # an element without a pole
    ee = rng.uniform(-0.2, 0.2, (nb, ne))
    ctx = P.Context(0)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    sx = torch.zeros((nb, ne), dtype=torch.complex128, device="cuda")
    coh = torch.zeros_like(sx)
    P.gw_sigma_gpp(ctx, nn, nocc, nb, n, dev(m), dev(en), dev(v), dev(amp), dev(wt), dev(ee), 0.7,
                   sx, coh)
    gx, gc = sx.cpu().numpy(), coh.cpu().numpy()
    for b in range(nb):
        c = np.conj(m[:, b, :, None]) * m[:, b, None, :] * v  # [nn][G][G']
        for k in range(ne):
            d = (ee[b, k] - en)[:, None, None]
            h = 0.35 * c * amp / (d - wt)
            x = -0.7 * c[:nocc] * (np.eye(n) + 0.5 * amp * (1 / (d - wt) - 1 / (d + wt))[:nocc])
            # every term to a few ulp (poles are at least 0.05 away), sums of nn n^2 terms
            assert abs(gc[b, k] - h.sum()) <= 1e-14 * np.abs(h).sum() * np.log2(4 + nn * n)
            if nocc == 0:
                assert gx[b, k] == 0
            else:
                mag = np.abs(c[:nocc]) * (np.eye(n) + np.abs(amp) * np.abs(1 / (d - wt))[:nocc]
                                          + np.abs(amp) * np.abs(1 / (d + wt))[:nocc])
                assert abs(gx[b, k] - x.sum()) <= 1e-14 * mag.sum() * np.log2(4 + nn * n)
    ctx.close()
