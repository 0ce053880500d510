"""The largest chains that run resident, and the first that do not, equal the tiled passes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

KEYS = ("dH", "H_old", "H_new", "m", "beta_eps", "accepted", "psi_final")


@pytest.mark.parametrize("L,prec,site", [
    ((5, 1017), 4, False), ((5, 1018), 4, False), ((53, 96), 4, False), ((3, 848), 8, False), ((3, 849), 8, False),
    ((5, 814), 4, True), ((5, 815), 4, True), ((5, 407), 8, True), ((5, 408), 8, True), ((5, 7, 145), 4, False)])
def test_equal_tiled(L, prec, site):
    """5088 FP32 and 2544 FP64 sites, 4070 and 2035 with a per-site field; rows of five pad most."""
    from paper_1912_03278_amd import ihmc
    N = int(np.prod(L))
    with ihmc.Context(arena_bytes=256 << 20) as ctx:
        fit = dict(zip((4, 8), ctx.set_resident(-1)))
    assert fit == {4: 5088, 8: 2544}
    h = np.random.default_rng(2).normal(0, 0.1, N) if site else 0.03
    lat = ihmc.Lattice(L, beta=0.4 if len(L) == 2 else 0.2, C=2 * len(L) + 0.1, h=h)
    out = []
    for resident in (-1, 0):
        with ihmc.Context(arena_bytes=256 << 20, resident=resident) as ctx:
            ch = ihmc.Chains(ctx, [lat], [ihmc.Run(n_md=4, n_traj=4, precision=prec, seed=7)])
            if resident:
                limit = (4070 if prec == 4 else 2035) if site else fit[prec]
                assert (ch.group_info(0)["cls"] < 0) == (N <= limit)
            ch.advance(4)
            out.append(ch.result(0))
            ch.close()
    for k in KEYS:
        assert np.array_equal(out[0][k], out[1][k]), k
