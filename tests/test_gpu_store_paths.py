"""Middle launches store plainly or through the L2 by their size: chains of sets on
either side of the limits equal the same chains run alone, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,m,prec", [
    ((30, 25), 250, 4), ((30, 25), 300, 4), ((131, 70), 150, 4), ((18, 17), 2100, 4), ((30, 25), 300, 8),
    ((24, 21, 14), 100, 4), ((24, 21, 14), 250, 4), ((24, 21, 14), 250, 8), ((35, 18, 9), 300, 4),
    ((16, 16, 16), 4, 4), ((160, 128, 100), 1, 4), ((160, 128, 100), 1, 8)])
def test_set_equals_chains_alone(L, m, prec):
    from paper_1912_03278_amd import ihmc
    N, d = int(np.prod(L)), len(L)
    rng = np.random.default_rng(m)
    h = rng.normal(0, 0.1, N)
    lats = [ihmc.Lattice(L, beta=0.3, C=2 * d + 0.1, h=(None, 0.04, h)[i % 3]) for i in range(m)]
    runs = [ihmc.Run(n_md=9 + i % 3, n_traj=2, precision=prec, seed=5, chain_id=i) for i in range(m)]
    with_fusion, single = (ihmc.Context(arena_bytes=3 << 30, resident=0, fuse_steps=f) for f in (True, False))
    try:
        a = with_fusion.run_batch(lats, runs)
        if m == 1:  # through the L2 alone, plainly among six
            more = [ihmc.Run(n_md=9, n_traj=2, precision=prec, seed=5, chain_id=i) for i in range(6)]
            b = with_fusion.run_batch(lats * 6, more)
            pairs = [(a[0], b[0])]
        else:
            pairs = [(a[i], single.run_batch([lats[i]], [runs[i]])[0]) for i in sorted({0, 1, 2, m // 2, m - 2, m - 1})]
        for x, y in pairs:
            for k in ("dH", "H_old", "H_new", "m", "beta_eps", "accepted", "psi_final"):
                assert np.array_equal(x[k], y[k]), k
    finally:
        with_fusion.close()
        single.close()
