"""2D launches of two and of four steps, full and with fewer steps left, equal one step a launch.

Two steps a launch: FP64 sets of more than 1024 tiles, and chains of at most two middle
steps.  Where most chains have all steps or all but one left, a launch works on all rows.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,n,prec,n_md", [
    ((30, 25), 1100, 8, (2, 3, 4, 5, 7)),     # FP64, two a launch, every remainder in one launch
    ((2060, 1700), 1, 8, (6,)),               # 64-wide tiles, rows split 50 at most
    ((5, 3), 1030, 8, (4, 2)),                # smaller than the halo
    ((300, 40), 5, 4, (3, 2)), ((300, 40), 5, 8, (3, 2)),
    ((1256, 1250), 1, 8, (3,)), ((1024, 900), 1, 4, (3,)), ((3, 5), 7, 4, (3, 1)),
    ((70, 66), 40, 4, (9,)), ((70, 66), 40, 4, (9, 10, 6)), ((512, 512), 1, 4, (10,)),
    ((70, 66), 40, 4, (9, 9, 9, 9, 6)), ((33, 40), 60, 4, (9, 9, 9, 9, 9, 7)), ((5, 7), 30, 4, (5, 5, 5, 5, 3)),  # few with fewer left
])
def test_equal_one_step_a_launch(L, n, prec, n_md):
    from paper_1912_03278_amd import ihmc
    N = L[0] * L[1]
    h = np.random.default_rng(n).normal(0, 0.1, N)
    lats = [ihmc.Lattice(L, beta=0.42, C=4.1, h=(None, 0.04, h)[i % 3]) for i in range(n)]
    runs = [ihmc.Run(n_md=n_md[i % len(n_md)], n_traj=2, precision=prec, seed=4, chain_id=i) for i in range(n)]
    out = []
    for fuse in (True, False):
        with ihmc.Context(arena_bytes=2 << 30, resident=0, fuse_steps=fuse) as ctx:
            out.append(ctx.run_batch(lats, runs))
    for a, b in zip(*out):
        for k in ("dH", "H_old", "H_new", "m", "beta_eps", "accepted", "psi_final"):
            assert np.array_equal(a[k], b[k], equal_nan=True), k


@pytest.mark.parametrize("L,n,prec,n_md,steps", [
    ((64, 50), 3, 4, (9,), 4), ((30, 25), 1100, 8, (9,), 2), ((64, 50), 4, 4, (9, 4), (4 + 3) / 2),
])
def test_timed_launch_is_the_rounds_own(L, n, prec, n_md, steps):
    """The timed launch takes as many steps as a round's, at most what a chain has,
    counts a site once for each, and leaves the chains' results as they are."""
    from paper_1912_03278_amd import ihmc
    lats = [ihmc.Lattice(L, beta=0.42, C=4.1) for _ in range(n)]
    runs = [ihmc.Run(n_md=n_md[i % len(n_md)], n_traj=2, precision=prec, seed=4, chain_id=i) for i in range(n)]
    with ihmc.Context(arena_bytes=2 << 30, resident=0) as ctx:
        ref = ctx.run_batch(lats, runs)
        ch = ihmc.Chains(ctx, lats, runs)
        t = ch.time_pass(0, mode=ihmc.FUSED, reps=3)
        assert t["us"] > 0 and t["sites"] == steps * n * L[0] * L[1]
        ch.advance(2)
        for i, a in enumerate(ref):
            b = ch.result(i)
            assert np.array_equal(a["dH"], b["dH"]) and np.array_equal(a["m"], b["m"])
        with pytest.raises(ihmc.IhmcError):
            ch.time_pass(0, mode=ihmc.FUSED + 1, reps=1)
        ch.close()
