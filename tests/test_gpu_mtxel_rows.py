"""GPU matrix elements of spheres whose planes are split over wavefronts by rows, and of
those beyond these kernels too, at the edges of their tiles, against the plane-wave
convolution of the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# max |g| of (valence, conduction, eps) per axis; the grid has their sum plus one points.
# Rows go in tiles of 16, entries in steps of 8 or more, kept |g| in tiles of 8.
CASES = {
    "29": ((9, 10, 9), (10, 9, 9), (10, 10, 8)),
    "32_kept_8": ((12, 12, 7), (11, 12, 8), (12, 11, 8)),
    "33_kept_7": ((13, 12, 7), (13, 13, 6), (12, 13, 7)),
    "41_and_48": ((16, 16, 8), (16, 16, 15), (16, 16, 15)),
    "49_one_output_tile": ((21, 21, 6), (22, 20, 6), (11, 3, 2)),
    "57_kept_16": ((20, 20, 16), (20, 20, 16), (3, 2, 1)),
    "64": ((24, 24, 15), (24, 24, 15), (9, 8, 7)),
    "64_long_third": ((24, 24, 15), (24, 24, 15), (40, 39, 7)),
    "kept_24": ((18, 18, 24), (18, 18, 23), (2, 2, 24)),
    "flat": ((0, 0, 0), (25, 26, 11), (26, 25, 8)),
    "kept_24_flat": ((6, 7, 14), (15, 9, 24), (0, 0, 0)),
    "33_by_13": ((10, 2, 20), (7, 1, 4), (0, 0, 4)),
    "38_by_21": ((0, 0, 0), (8, 10, 19), (6, 6, 8)),
    "one_tile_of_two_rows": ((23, 4, 1), (17, 13, 1), (0, 1, 0)),
    "needle": ((2, 2, 2), (1, 2, 2), (26, 25, 12)),
    # more than 64 points on two axes: the general transforms
    "65_general": ((24, 24, 16), (24, 24, 16), (3, 2, 1)),
    "65_three": ((26, 26, 13), (25, 26, 14), (24, 25, 16)),
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
    def smooth(n):
        for p in (2, 3, 5):
            while n % p == 0:
                n //= p
        return n == 1
    while not smooth(need):
        need += 1
    return need


# one pair; several workgroups' bands and valence ranges, the last ones short
@pytest.mark.parametrize("nv,nc", [(1, 1), (13, 5)])
@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("nspinor", [1, 2])
@pytest.mark.parametrize("name", sorted(CASES))
def test_against_convolution(name, nspinor, dtype, nv, nc):
    import paper_2206_00808_amd as P
    axes = CASES[name]
    rng = np.random.default_rng(sum(map(ord, name)) + nspinor + nv)
    gv, gc, ge = (_sphere(rng, [a[i] for a in axes], n) for i, n in ((0, 60), (1, 70), (2, 50)))
    cdt = np.complex128 if dtype == "c128" else np.complex64
    band = lambda n, g: (rng.normal(size=(n, nspinor, len(g)))
                         + 1j * rng.normal(size=(n, nspinor, len(g)))).astype(cdt)
    cv, cc = band(nv, gv), band(nc, gc)
    box = [_box(max(sum(a), 2 * max(a)) + 1) for a in axes]
    ctx = P.Context(0)
    out = torch.full((nv, nc, len(ge)), float("nan"), device="cuda",
                     dtype=torch.complex128 if dtype == "c128" else torch.complex64)
    P.gw_mtxel_spinor(ctx, box, nspinor, gv, torch.from_numpy(cv).cuda(), gc,
                      torch.from_numpy(cc).cuda(), ge, out)
    got = out.cpu().numpy()
    ctx.close()
    ref = oracle.mtxel_convolution(cv.astype(np.complex128), gv, cc.astype(np.complex128), gc, ge)
    # an entry sums products of the two bands' coefficients; nine transforms of at most
    # 128 terms round each at u: |error| <= 9 * 128 u |cv| |cc|
    u = 2.0 ** -53 if dtype == "c128" else 2.0 ** -24
    scale = np.linalg.norm(cv.reshape(nv, -1), axis=1)[:, None, None] * \
        np.linalg.norm(cc.reshape(nc, -1), axis=1)[None, :, None]
    assert np.all(np.abs(got - ref) <= 9 * 128 * u * scale)
