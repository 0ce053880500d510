"""Set-up solve of long, thin lattices: conjugate gradients where the transform would take longer."""
import time

import numpy as np
import pytest

from test_gpu_field_solve import expected

pytestmark = pytest.mark.gpu


# on either side of the line: 2^18 x 3 conjugate gradients, 3 x 3 x 5000 and 9000 x 5 the transform
@pytest.mark.parametrize("L,C", [((1 << 18, 3), 4.1), ((3, 150000), 40.0), ((3, 3, 5000), 6.1), ((9000, 5), 4.1)])
def test_constants(L, C):
    """Conjugate gradients stop at a relative residual of 1e-15; the transform's sums of L
    products err by about 3 L 2^-53 of the constant, 3e-12 at 9000.  The estimator holds a
    constant over 2 N beta; 1e-11 of it covers both."""
    from paper_1912_03278_amd import ihmc
    rng = np.random.default_rng(1)
    N, beta = int(np.prod(L)), 0.37
    h, psi = rng.normal(0.1, 0.3, N), rng.standard_normal(N)
    with ihmc.Context(arena_bytes=1 << 30) as ctx:
        got = ctx.action(ihmc.Lattice(L, beta=beta, C=C, h=h), psi, precision=ihmc.F64)
    m, e, scale = expected(L, beta, C, h, psi)
    assert abs(got["m"] - m) <= 1e-11 * (1 + abs(m))
    assert abs(got["beta_eps"] - e) <= 1e-11 * (1 + abs(scale))


def test_long_axis_takes_no_seconds():
    """2^19 x 3 at a large shift: six iterations, 0.1 s; 1.4 s by transform."""
    from paper_1912_03278_amd import ihmc
    L = (1 << 19, 3)
    lat = ihmc.Lattice(L, beta=0.4, C=1000.0, h=np.full(L[0] * L[1], 0.1))
    with ihmc.Context(arena_bytes=1 << 30) as ctx:
        best = float("inf")
        for _ in range(2):
            t = time.perf_counter()
            ihmc.Chains(ctx, [lat], [ihmc.Run(n_md=2, n_traj=1)]).close()
            best = min(best, time.perf_counter() - t)
    assert best < 0.8, best
