"""In 2D the tile class sets the first and last passes, so the tuner times those."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,site", [((131, 131), False), ((131, 131), True), ((24, 24), False)])
def test_tuned_class_is_fast_in_first_and_last(L, site):
    """Chosen by the middle pass, 131 x 131 ran its first and last passes 22 % longer and
    24 x 24 15 % longer than on the best class; 8 % is allowed to a choice within the tuner's
    3 % margin and to the spread of two timings."""
    from paper_1912_03278_amd import ihmc
    N = L[0] * L[1]
    n = max(1, (1 << 20) // N)
    lat = ihmc.Lattice(L, beta=0.44, C=4.1, h=np.random.default_rng(1).normal(0, 0.05, N) if site else None)
    us = []
    with ihmc.Context(arena_bytes=1 << 30, resident=0) as ctx:
        ctx.tune([lat] * n)
        t = ctx.tile_class(lat)
        assert t["source"] == ihmc.TUNE_MEASURED and all(0 < v < 10 for v in t["ns_per_site"][:3])
        for cls in range(3):
            ctx.pin_tile(lat, cls)
            ch = ihmc.Chains(ctx, [lat] * n, [ihmc.Run(n_md=5, n_traj=4, chain_id=i) for i in range(n)])
            us.append(sum(min(ch.time_pass(0, mode=m, reps=20)["us"] for _ in range(4)) for m in (0, 2)))
            ch.close()
    assert us[t["cls"]] <= 1.08 * min(us), (t, us)


def test_tuned_chains_keep_their_values():
    """A tuning run in the middle of a context's life leaves the chains on it alone."""
    from paper_1912_03278_amd import ihmc
    lat = ihmc.Lattice((70, 66), beta=0.44, C=4.1, h=0.02)
    run = ihmc.Run(n_md=6, n_traj=6, seed=2)
    with ihmc.Context(arena_bytes=256 << 20, resident=0) as ctx:
        want = ctx.run_lattice(lat, run)
        ch = ihmc.Chains(ctx, [lat], [run])
        ch.advance(3)
        used = ctx.memory()[0]
        ctx.tune([lat, ihmc.Lattice((3, 3), beta=0.4, C=4.1), ihmc.Lattice((5, 5), beta=0.4, C=4.1, h=np.ones(25))], sites=1)
        assert ctx.memory()[0] == used
        ch.advance(3)
        got = ch.result(0)
        ch.close()
    for k in ("dH", "H_new", "m", "psi_final"):
        assert np.array_equal(got[k], want[k]), k
