"""A chain set whose arrays just fit the arena: its tile tables need no room of their own."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,short", [((256, 250), 256), ((256, 250), 4096), ((700, 300), 256)])
def test_tables_find_room_elsewhere(L, short):
    """`used` counts the tables, over 4 KiB here; an arena smaller by `short` holds the arrays."""
    from paper_1912_03278_amd import ihmc
    lat = ihmc.Lattice(L, beta=0.4, C=4.1)
    run = ihmc.Run(n_md=5, n_traj=4, seed=2)
    with ihmc.Context(arena_bytes=64 << 20, resident=0) as ctx:
        ch = ihmc.Chains(ctx, [lat], [run])
        used = ctx.memory()[0]
        ch.advance(4)
        want = ch.result(0, want_psi=False)
        ch.close()
    with ihmc.Context(arena_bytes=used - short, resident=0) as ctx:
        ch = ihmc.Chains(ctx, [lat], [run])
        ch.advance(4)
        got = ch.result(0, want_psi=False)
        ch.close()
    for k in ("dH", "H_new", "m", "beta_eps"):
        assert np.array_equal(got[k], want[k]), k
