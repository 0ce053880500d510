"""LDS-resident chains at the edges of the workgroup variants.

The resident launch deals a chain's sites to its threads as 16-byte vectors and
picks a variant by the largest chain: one site a thread up to 256 sites (for at
most 1024 chains), else 64, 256, 1024 or 2 x 1024 vectors.  Around each edge, and
for the row lengths that pad most, a resident chain equals the tiled one bit for
bit (the two share per-site arithmetic and grouping of the exact sums).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SERIES = ("dH", "H_old", "H_new", "m", "abs_m", "m2c", "beta_eps", "accepted", "flipped", "psi_final")


@pytest.fixture(scope="module")
def ctxs():
    from paper_1912_03278_amd import ihmc
    res = ihmc.Context(arena_bytes=1 << 30)
    tiled = ihmc.Context(arena_bytes=1 << 30, resident=0)
    yield res, tiled
    res.close()
    tiled.close()


def run(ctx, L, prec, h, n=1, **kw):
    from paper_1912_03278_amd import ihmc
    lat = ihmc.Lattice(L, beta=0.4 if len(L) == 2 else 0.2, C=2 * len(L) + 0.1, h=h)
    return ctx.run_batch([lat] * n, [ihmc.Run(n_md=3, n_traj=3, precision=prec, seed=9, chain_id=i, **kw)
                                     for i in range(n)])


SHAPES = [
    # one site a thread: the smallest, a full workgroup, rows around 16 sites
    ((3, 3), 4), ((3, 3), 8), ((16, 16), 4), ((16, 16), 8), ((17, 15), 4), ((3, 3, 3), 8), ((8, 8, 4), 4),
    # past it: vectors of four (FP32) or two (FP64), 64 and 256 of them and one more
    ((257, 3), 4), ((16, 64), 4), ((16, 65), 4), ((20, 13), 8), ((32, 16), 8), ((16, 33), 8), ((9, 7, 12), 4),
    # 1024 vectors and one row more; the most padded rows (five and three sites) at the largest size
    ((64, 64), 4), ((64, 65), 4), ((32, 64), 8), ((34, 63), 8), ((5, 1004), 4), ((3, 837), 8), ((5, 10, 100), 4),
    ((17, 17, 17), 4), ((13, 13, 13), 8),
]


@pytest.mark.parametrize("L,prec", SHAPES)
def test_variant_edges_equal_tiled(ctxs, L, prec):
    rng = np.random.default_rng(5)
    N = int(np.prod(L))
    site = N * prec <= 4019 * 4
    for h, kw in ((None, {}), (rng.normal(0, 0.1, N) if site else 0.05, {"integrator": 1, "flip_every": 2})):
        a, b = (run(c, L, prec, h, **kw)[0] for c in ctxs)
        for k in SERIES:
            assert np.array_equal(a[k], b[k], equal_nan=True), (L, prec, k)


def test_many_small_chains_equal_alone(ctxs):
    """More than four chains a CU: vectors instead of one site a thread."""
    many = run(ctxs[0], (7, 9), 4, 0.02, n=1100)
    one = run(ctxs[0], (7, 9), 4, 0.02, n=3)
    for i in range(3):
        for k in SERIES:
            assert np.array_equal(many[i][k], one[i][k]), (i, k)
    big = run(ctxs[1], (7, 9), 4, 0.02, n=1100)
    for i in (0, 511, 1099):
        for k in SERIES:
            assert np.array_equal(many[i][k], big[i][k]), (i, k)
