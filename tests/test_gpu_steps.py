"""Fused middle steps (2D): every tile shape, ring and remainder against one step per launch.

A launch takes up to four middle steps on tiles that the plan chooses from the
lattices it covers: 16 x 16 tiles for a small lattice up to 64 x 64 ones, one to
three rows a thread.  Fused and single-step chains must be equal bit for bit for
lattices around the tile splits, smaller than the 8-wide halo, with ragged rows,
for every remainder of the step count, and in sets whose chains end at
different launches.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SERIES = ("dH", "H_old", "H_new", "m", "beta_eps", "accepted", "flipped", "psi_final")


@pytest.fixture(scope="module")
def ctxs():
    from paper_1912_03278_amd import ihmc
    cs = [ihmc.Context(arena_bytes=1 << 30, resident=0, fuse_steps=f) for f in (True, False)]
    yield cs
    for c in cs:
        c.close()


def both(ctxs, lats, runs):
    a, b = (c.run_batch(lats, runs) for c in ctxs)
    for l, x, y in zip(lats, a, b):
        for k in SERIES:
            assert np.array_equal(x[k], y[k], equal_nan=True), (l.L, k)


SHAPES = [(3, 3), (5, 70), (16, 16), (17, 15), (33, 16), (66, 62), (64, 61), (65, 62), (130, 257), (6, 300),
          (520, 510), (1030, 515)]


@pytest.mark.parametrize("prec", [4, 8])
@pytest.mark.parametrize("L", SHAPES)
def test_shapes_and_remainders(ctxs, L, prec):
    """One set per shape: chains of 1 .. 7 MD steps, the second integrator, fields of each kind."""
    from paper_1912_03278_amd import ihmc
    rng = np.random.default_rng(1)
    N = L[0] * L[1]
    lats, runs = [], []
    for i, n_md in enumerate((1, 2, 3, 4, 5, 6, 7, 3) if N < 40000 else (6,)):
        h = (None, 0.04, rng.normal(0, 0.1, N))[i % 3]
        lats.append(ihmc.Lattice(L, beta=0.42, C=4.1, h=h))
        runs.append(ihmc.Run(n_md=n_md, n_traj=2, precision=prec, seed=4, chain_id=i, integrator=i == 7,
                             flip_every=2 * (i == 1)))
    both(ctxs, lats, runs)


@pytest.mark.parametrize("prec", [4, 8])
def test_launch_of_many_tiles(ctxs, prec):
    """More than 1024 tiles: rows per thread chosen for a full chip."""
    from paper_1912_03278_amd import ihmc
    both(ctxs, [ihmc.Lattice((2100, 2050), beta=0.44, C=4.1)], [ihmc.Run(n_md=7, n_traj=1, precision=prec, seed=2)])


def test_uneven_set(ctxs):
    from paper_1912_03278_amd import ihmc
    rng = np.random.default_rng(3)
    lats, runs = [], []
    for i in range(90):
        L = tuple(int(v) for v in rng.integers(40, 260, 2))
        lats.append(ihmc.Lattice(L, beta=0.4, C=4.1, h=rng.normal(0, 0.05, L[0] * L[1]) if i % 2 else None))
        runs.append(ihmc.Run(n_md=int(rng.integers(1, 14)), n_traj=2, precision=4, seed=5, chain_id=i))
    both(ctxs, lats, runs)
