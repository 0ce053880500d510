"""Serving with an arena that the requests' own memory fills.

Tile tables and the buffer that final fields are exported through are not part of a
request's budget: where the arena has no room for them a request still runs, and its
result is whole.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

KEYS = ("dH", "H_old", "H_new", "m", "beta_eps", "accepted", "psi_final")


def fill(ctx, leave):
    """A chain set that leaves about `leave` bytes of the arena (records take 64 each)."""
    from paper_1912_03278_amd import ihmc
    lat = ihmc.Lattice((4, 4), beta=0.4, C=4.1)
    before = ctx.memory()[0]
    one = ihmc.Chains(ctx, [lat], [ihmc.Run(n_md=2, n_traj=1)])
    fixed = ctx.memory()[0] - before
    one.close()
    used, total = ctx.memory()
    n = (total - used - fixed - leave) // 64
    return ihmc.Chains(ctx, [lat], [ihmc.Run(n_md=2, n_traj=int(n))])


@pytest.mark.parametrize("L,room", [((512, 500), 2048), ((64, 64, 40), 2048), ((512, 500), 10000)])
def test_request_that_fills_the_arena(L, room):
    from paper_1912_03278_amd import ihmc
    N = int(np.prod(L))
    lat = ihmc.Lattice(L, beta=0.4 if len(L) == 2 else 0.2, C=2 * len(L) + 0.1, h=0.01)
    runs = [ihmc.Run(n_md=6, n_traj=5, seed=3, chain_id=i) for i in range(3)]
    with ihmc.Context(arena_bytes=64 << 20) as ctx:
        alone = [ctx.run_lattice(lat, r) for r in runs]
    with ihmc.Context(arena_bytes=64 << 20) as ctx:
        srv = ihmc.Server(ctx, budget_bytes=64 << 20, max_active=1)
        filler = None
        try:
            before = ctx.memory()[0]
            probe = ihmc.Chains(ctx, [lat], [runs[0]])  # a chain set takes the chain, its tables and the descriptor
            chain = ctx.memory()[0] - before
            probe.close()
            filler = fill(ctx, chain + room)
            tickets = [srv.submit(lat, r) for r in runs]
            for t, a in zip(tickets, alone):
                srv.wait(t, 30.0)
                got = srv.fetch(t)
                for k in KEYS:
                    assert np.array_equal(got[k], a[k]), k
            assert srv.stats()["completed"] == 3
        finally:
            srv.close()
            if filler is not None:
                filler.close()
