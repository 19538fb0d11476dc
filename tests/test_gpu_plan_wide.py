"""GPU plan over q-points of which some are too wide for the dense transforms, against
the oracle: shared and separate conduction bands, in a box whose own planes no kernel holds."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _sphere(rng, gmax, n):
    g = np.concatenate([np.stack([rng.integers(-m, m + 1, n) for m in gmax], axis=1),
                        [[0, 0, 0]], [gmax], [[-m for m in gmax]]])
    return np.unique(g, axis=0).astype(np.int32)


@pytest.mark.parametrize("shared", [True, False])
@pytest.mark.parametrize("order", [(0, 1, 0), (1, 0, 1), (1, 1, 1)])
def test_mixed_widths(order, shared):
    import paper_2206_00808_amd as P
    from paper_2206_00808_amd.binding import Plan
    rng = np.random.default_rng(10 * shared + sum(3 ** i * o for i, o in enumerate(order)))
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    box, nf, omega = (20, 120, 120), 2, [0.0, 0.3]
    gc = _sphere(rng, (2, 30, 31), 40)
    band = lambda n, g: (rng.normal(size=(n, 2, len(g))) + 1j * rng.normal(size=(n, 2, len(g)))) / 20
    cc0 = band(9, gc)
    d0, qs, host = dev(cc0), [], []
    for i, wide in enumerate(order):
        # valence, conduction and eps reach 67 and more points on two axes, or 45
        gv = _sphere(rng, (3, 33, 34) if wide else (3, 4, 5), 30 + i)
        ge = _sphere(rng, (1, 3, 4) if wide else (1, 3, 3), 12 + i)
        cc, nc = (cc0, 9 - i) if shared else (band(9, gc), 9 - i)
        cv, ne = band(4, gv), len(ge)
        ev, ec = np.sort(rng.uniform(-0.3, 0, 4)), np.sort(rng.uniform(0.1, 0.5, nc))
        v = rng.uniform(0.2, 1.0, ne)
        host.append((cv, gv, cc[:nc], gc, ge, ev, ec, v))
        qs.append(dict(gv=gv, gc=gc, geps=ge, cv=dev(cv), cc=d0 if shared else dev(cc), nc=nc,
                       ev=dev(ev), ec=dev(ec), vcoul=dev(v), head_index=-1,
                       chi0=dev(np.zeros((nf, ne, ne), complex)),
                       epsinv=dev(np.zeros((nf, ne, ne), complex))))
    ctx = P.Context(0)
    plan = Plan(ctx, box, 2, P.GW_C128, P.GW_PREC_FP64, omega, 1.0, qs)
    plan.compile()
    for _ in range(3):
        plan.launch()
        for q, (cv, gv, cc, g, ge, ev, ec, v) in zip(qs, host):
            m = oracle.mtxel_convolution(cv, gv, cc, g, ge)
            x = oracle.chi0(m, ev, ec, np.asarray(omega))
            e = oracle.epsilon_inverse(x, v)
            for f in range(nf):
                assert oracle.rel_f(q["chi0"][f].cpu().numpy(), x[f]) < 1e-12
                assert oracle.rel_f(q["epsinv"][f].cpu().numpy(), e[f]) < 1e-12
    plan.close()
    ctx.close()
