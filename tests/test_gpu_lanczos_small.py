"""Lanczos of small matrices in one workgroup: partly filled blocks of rows, its largest size and the
next one, runs that go on past its 64 steps."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [1, 3, 16, 33, 64, 65, 111, 112, 113, 129])
def test_lowest_eigenvalue(N):
    """At convergence the residual is at most 1e-10 (|theta| + 1), and the Ritz value lies
    within it of the lowest eigenvalue; numpy's is good to a few 1e-15."""
    from paper_1912_03278_amd import ihmc
    rng = np.random.default_rng(N)
    with ihmc.Context(arena_bytes=256 << 20) as ctx:
        for K in (rng.standard_normal((N, N)), np.ones((N, N)), np.diag(np.arange(N) - 0.5 * N)):
            K = 0.5 * (K + K.T)
            theta, resid, steps = ctx.min_eig(K)
            want = np.linalg.eigvalsh(K)[0]
            scale = abs(want) + 1.0
            assert resid <= 1.5e-10 * scale and 1 <= steps <= N
            assert abs(theta - want) <= 2e-10 * scale + 1e-14 * np.abs(K).sum(0).max()

