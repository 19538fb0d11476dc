"""GPU checks of the closure's products at the edges of their tiles: rows below,
at and above one 128-row tile and one split, widths that take the 64-, 128- and
256-column kernels (and several of them), one layer and many."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("neps,width,depth", [
    (1, 64, 1), (15, 64, 2), (16, 128, 1), (22, 192, 3), (23, 256, 1), (91, 256, 2),
    (130, 256, 4), (60, 320, 2), (37, 512, 3),
])
def test_loss_gradients_and_inference(neps, width, depth):
    import paper_2206_00808_amd as P
    from paper_2206_00808_amd.binding import Mlp, mlp_blob_pack, mlp_blob_unpack, mlp_layers
    rng = np.random.default_rng(100 * neps + width + depth)
    ctx = P.Context(0)
    net = Mlp(ctx, 7, width, depth, 2, seed=1)
    meta = mlp_blob_unpack(net.save())
    real = [7] + [width] * depth + [2]
    params = [(w, rng.normal(size=b.shape) * 0.05) for w, b in oracle.init_params(rng, real)]
    flat = []
    for (w, b), (din, dout) in zip(params, mlp_layers(meta)):
        wf, bf = np.zeros((dout, din)), np.zeros(dout)
        wf[:w.shape[0], :w.shape[1]], bf[:b.shape[0]] = w, b
        flat += [wf.ravel(), bf]
    net.load(mlp_blob_pack(meta, np.concatenate(flat).astype(np.float32)))
    b = rng.normal(size=(neps, neps + 3)) + 1j * rng.normal(size=(neps, neps + 3))
    chi_t = -(b @ b.conj().T) / (neps + 3)
    r = rng.normal(size=(neps, neps)) + 1j * rng.normal(size=(neps, neps))
    # targets of a few units, so that Y - T does not cancel
    chi_f = chi_t - 2.0 * (r + r.conj().T) - 3.0 * np.eye(neps)
    qg = rng.normal(size=(neps, 3))
    d = dict(qg=torch.from_numpy(qg).cuda(), t=torch.from_numpy(chi_t).cuda(),
             f=torch.from_numpy(chi_f).cuda())
    feat, _, s = oracle.closure_features(qg, chi_t, 0.05, 0.6)
    # each of the 2 (depth + 1) products on the way to a gradient rounds two
    # operands to bfloat16 (2^-9 each); a factor of two for the slope of SiLU'
    tol = 8 * (depth + 1) * 2.0 ** -9
    out = torch.empty_like(d["t"])
    P.binding.gw_chi0_closure(ctx, net, P.GW_CLOSURE_INFER, neps, d["qg"], d["t"], 0.05, 0.6,
                              chi0_out=out)
    y, _ = oracle.mlp_forward(params, feat)
    assert oracle.rel_f(out.cpu().numpy() - chi_t, oracle.closure_apply(chi_t, y, s) - chi_t) < tol
    _, loss = P.binding.gw_chi0_closure(ctx, net, P.GW_CLOSURE_TRAIN_STEP, neps, d["qg"], d["t"],
                                        0.05, 0.6, chi0_full=d["f"], lr=0.0)
    m = mlp_blob_unpack(net.save())["m"].astype(np.float64) / 0.1
    t = oracle.closure_target(chi_t, chi_f, s)
    ref_loss, ref = oracle.mlp_loss_and_grads(params, feat, t, nout=2)
    assert abs(loss - ref_loss) <= tol * ref_loss
    off = 0
    for l, (din, dout) in enumerate(mlp_layers(meta)):
        gw = m[off:off + din * dout].reshape(dout, din)
        gb = m[off + din * dout:off + din * dout + dout]
        off += din * dout + dout
        rw, rb = ref[l]
        assert oracle.rel_f(gw[:rw.shape[0], :rw.shape[1]], rw) < tol
        assert oracle.rel_f(gb[:rb.shape[0]], rb) < tol
        # the padding gets no gradient
        assert not gw[rw.shape[0]:].any() and not gw[:, rw.shape[1]:].any()
    ctx.close()
