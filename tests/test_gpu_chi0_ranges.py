"""GPU chi0 in FP64 where fewer tiles than CUs make the pair sum split into ranges: whole
and short last ranges, pair counts at the edges of a range, one and several frequencies,
added to what the matrix holds."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("neps,nv,nc", [(1, 1, 1), (59, 1, 31), (59, 8, 8), (59, 5, 13), (64, 7, 37),
                                        (65, 16, 129), (200, 11, 91), (130, 3, 1367)])
@pytest.mark.parametrize("nf,dtype", [(1, "complex128"), (3, "complex64")])
def test_chi0_pair_ranges(neps, nv, nc, nf, dtype):
    import paper_2206_00808_amd as P
    dt = getattr(torch, dtype)
    g = torch.Generator(device="cuda").manual_seed(neps + nv * nc)
    m = torch.randn((nv, nc, neps), dtype=torch.complex128, device="cuda", generator=g).to(dt)
    ev = torch.sort(-0.1 - torch.rand(nv, dtype=torch.float64, device="cuda", generator=g)).values
    ec = torch.sort(0.1 + torch.rand(nc, dtype=torch.float64, device="cuda", generator=g)).values
    om = np.linspace(0.0, 2.0, nf)
    h = torch.randn((nf, neps, neps), dtype=torch.complex128, device="cuda", generator=g)
    chi = h + h.conj().transpose(1, 2)
    want = chi.clone()
    ctx = P.Context(0)
    P.gw_chi0_accumulate(ctx, nv, nc, neps, m, ev, ec, om, 0.7, P.GW_PREC_FP64, chi)
    d = (ec[None, :] - ev[:, None]).reshape(-1)
    x = m.reshape(-1, neps).to(torch.complex128)
    mag = torch.matmul(x.abs().t().contiguous(), x.abs())
    for f, w in enumerate(om):
        wt = -0.7 * 2.0 * d / (d * d + w * w)
        want[f] += torch.matmul((x.conj() * wt[:, None]).t().contiguous(), x)
        # each product and its weight to a few ulp, sums of P terms in whole chains
        tol = (8 + nv * nc) * 2.0 ** -52 * (float(wt.abs().max()) * mag + 6.0)
        assert bool(((chi[f] - want[f]).abs() <= tol).all())
    ctx.close()
