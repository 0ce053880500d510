"""Allocation-free force of thin lattices: tiles four sites wide, their bits and their cost."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def call(ctx, L, prec, psi=None):
    import torch
    from paper_1912_03278_amd import ihmc
    lat = ihmc.Lattice(L, beta=0.3, C=2 * len(L) + 0.2, h=0.03)
    dt = torch.float32 if prec == 4 else torch.float64
    x = torch.randn(lat.N, dtype=dt, device="cuda") if psi is None else torch.tensor(psi, dtype=dt, device="cuda")
    F = torch.empty_like(x)
    torch.cuda.synchronize()
    return lat, x, F, lambda: ctx.force_noalloc(lat, x.data_ptr(), F.data_ptr(), precision=prec)


@pytest.mark.parametrize("prec", [4, 8])
@pytest.mark.parametrize("L", [(3, 64), (4, 65), (7, 129), (5, 16, 4), (3, 17, 9), (6, 40, 5), (4, 4, 16), (3, 5, 70),
                               (20, 3, 33)])
def test_bits_of_the_force_pass(prec, L):
    from paper_1912_03278_amd import ihmc
    with ihmc.Context(arena_bytes=64 << 20) as ctx:
        psi = np.random.default_rng(1).standard_normal(int(np.prod(L)))
        psi = psi.astype(np.float32).astype(np.float64) if prec == 4 else psi
        lat, _, F, f = call(ctx, L, prec, psi)
        f()
        ctx.sync()
        assert np.array_equal(F.cpu().numpy().astype(np.float64), ctx.force(lat, psi, precision=prec))


@pytest.mark.parametrize("thin,wide", [((4, 500000), (1414, 1414)), ((3, 3, 200000), (121, 122, 122))])
def test_thin_lattices_cost_about_what_wide_ones_do(thin, wide):
    """Two million sites in rows of four or three: 1.5 and 2.1 times as long as square and
    cubic ones; 10 and 23 times on tiles of 64 x 16 and 16 x 16 x 4."""
    from paper_1912_03278_amd import ihmc
    us = []
    with ihmc.Context(arena_bytes=64 << 20) as ctx:
        for L in (thin, wide):
            f = call(ctx, L, 4)[3]
            best = float("inf")
            for _ in range(6):
                ctx.sync()
                t = time.perf_counter()
                for _ in range(100):
                    f()
                ctx.sync()
                best = min(best, time.perf_counter() - t)
            us.append(1e4 * best)
    assert us[0] < 4.0 * us[1], us
