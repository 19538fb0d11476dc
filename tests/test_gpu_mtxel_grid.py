"""GPU matrix elements at the edges of the dense-transform kernels' tiles, and where
spheres are too wide for them, against the plane-wave convolution of the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# max |g| of (valence, conduction, eps) per axis.  The grid has their sum plus one
# points; rows go in tiles of 16, entries in steps of 4, kept |g| in tiles of 8.
CASES = {
    "single_point": ((0, 0, 0), (0, 0, 0), (0, 0, 0)),
    "one_axis": ((3, 2, 3), (0, 0, 0), (0, 0, 0)),
    "rows_16": ((6, 6, 3), (2, 2, 2), (9, 9, 9)),
    "rows_17": ((6, 6, 4), (2, 2, 1), (9, 9, 8)),
    "kept_7_and_8": ((8, 8, 7), (8, 8, 8), (9, 8, 7)),
    "rows_32": ((12, 12, 7), (13, 12, 7), (14, 12, 6)),
    "rows_33": ((12, 12, 8), (13, 12, 7), (15, 15, 9)),
    "kept_15_and_16": ((14, 14, 15), (13, 13, 16), (6, 5, 3)),
    "rows_48_steps_12": ((17, 18, 12), (17, 18, 12), (17, 18, 11)),
    "long_axis": ((40, 36, 33), (3, 2, 3), (2, 4, 1)),
    # two axes beyond the built kernels: the general transforms
    "wide": ((21, 20, 9), (20, 21, 8), (2, 2, 2)),
    "wide_three": ((18, 19, 13), (19, 18, 12), (18, 18, 13)),
}


def _sphere(rng, gmax, n):
    """n distinct G inside the ranges, the largest |g| of every axis among them."""
    pts = {(0, 0, 0)}
    for a in range(3):
        for s in (-1, 1):
            g = [int(rng.integers(-m, m + 1)) for m in gmax]
            g[a] = s * gmax[a]
            pts.add(tuple(g))
    total = int(np.prod([2 * m + 1 for m in gmax]))
    while len(pts) < min(n, total):
        pts.add(tuple(int(rng.integers(-m, m + 1)) for m in gmax))
    return np.array(sorted(pts), dtype=np.int32)[rng.permutation(len(pts))]


def _box(need):
    while not _smooth(need):
        need += 1
    return need


def _smooth(n):
    for p in (2, 3, 5):
        while n % p == 0:
            n //= p
    return n == 1


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("nspinor", [1, 2])
@pytest.mark.parametrize("name", sorted(CASES))
def test_against_convolution(name, nspinor, dtype):
    import paper_2206_00808_amd as P
    axes = CASES[name]
    rng = np.random.default_rng(sum(map(ord, name)) + nspinor)
    gv, gc, ge = (_sphere(rng, [a[i] for a in axes], n) for i, n in ((0, 70), (1, 90), (2, 60)))
    nv, nc = 5, 9
    cv = rng.normal(size=(nv, nspinor, len(gv))) + 1j * rng.normal(size=(nv, nspinor, len(gv)))
    cc = rng.normal(size=(nc, nspinor, len(gc))) + 1j * rng.normal(size=(nc, nspinor, len(gc)))
    cdt = np.complex128 if dtype == "c128" else np.complex64
    cv, cc = cv.astype(cdt), cc.astype(cdt)
    box = [_box(max(sum(a), 2 * max(a)) + 1) for a in axes]
    ctx = P.Context(0)
    out = torch.full((nv, nc, len(ge)), float("nan"), device="cuda",
                     dtype=torch.complex128 if dtype == "c128" else torch.complex64)
    for _ in range(2):  # the second call runs on cached tables
        P.gw_mtxel_spinor(ctx, box, nspinor, gv, torch.from_numpy(cv).cuda(), gc,
                          torch.from_numpy(cc).cuda(), ge, out)
        ref = oracle.mtxel_convolution(cv.astype(np.complex128), gv, cc.astype(np.complex128), gc,
                                       ge)
        got = out.cpu().numpy()
        # an entry sums products of the two bands' coefficients; nine transforms of at
        # most 128 terms round each at u: |error| <= 9 * 128 u |cv| |cc|
        u = 2.0 ** -53 if dtype == "c128" else 2.0 ** -24
        scale = np.linalg.norm(cv.reshape(nv, -1), axis=1)[:, None, None] * \
            np.linalg.norm(cc.reshape(nc, -1), axis=1)[None, :, None]
        assert np.all(np.abs(got - ref) <= 9 * 128 * u * scale)
    ctx.close()
