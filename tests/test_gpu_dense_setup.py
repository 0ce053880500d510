"""Set-up of dense chains on the device: the check of K's entries, the Lanczos
shift over row splits that do not come out even, conjugate gradients of one and of
two right-hand sides."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1912_03278_amd import ihmc
    c = ihmc.Context(arena_bytes=3 << 30)
    yield c
    c.close()


def rand_K(N, seed):
    rng = np.random.default_rng(seed)
    K = np.triu(rng.standard_normal((N, N)) / np.sqrt(N), 1)
    return K + K.T


@pytest.mark.parametrize("N", [2, 31, 32, 33, 65, 300])
def test_entries_are_refused_as_on_the_host(ctx, N):
    """Any non-finite entry and any pair that differs by more than 1e-12 of the
    largest is refused, the first in row order named; a pair at the bound passes."""
    from paper_1912_03278_amd import ihmc
    K = rand_K(N, N)
    K[0, 0] = -8.0  # the largest: the bound is 8e-12
    for i, k in sorted({(0, 1), (0, N - 1), (N // 2 - 1, N - 1), (N - 2, N - 1)}):
        for bad in (np.nan, np.inf, -np.inf):
            M = K.copy()
            M[k, i] = bad
            with pytest.raises(ihmc.IhmcError, match="non-finite"):
                ctx.min_eig(M)
            with pytest.raises(ihmc.IhmcError, match="non-finite"):
                ctx.dense_force(ihmc.Dense(M, beta=0.5, C=20.0), np.zeros((1, N)))
        M = K.copy()
        M[i, k], M[k, i] = 1e-12 * 8.0, 0.0
        ctx.min_eig(M)
        M[i, k] = np.nextafter(1e-12 * 8.0, 1.0)
        if (i, k) != (N - 2, N - 1):
            M[N - 2, N - 1] += 1.0
        with pytest.raises(ihmc.IhmcError, match=f"entry {i}, {k}"):
            ctx.min_eig(M)
        with pytest.raises(ihmc.IhmcError, match=f"entry {i}, {k}"):
            ctx.dense_force(ihmc.Dense(M, beta=0.5, C=20.0), np.zeros((1, N)), products=5)


# rows per block 16 (1 .. 128 blocks), 18, 34
@pytest.mark.parametrize("N", [1, 2, 17, 257, 2048, 2300, 4100])
def test_lowest_eigenvalue(ctx, N):
    """A reflected diagonal: every entry is non-zero, the eigenvalues are known to
    rounding.  At convergence the residual is at most 1e-10 (|theta| + 1), and the
    Ritz value lies within it of the lowest eigenvalue."""
    rng = np.random.default_rng(N + 1)
    d = rng.uniform(0.0, 1.0, N)
    d[N // 2] = -0.5
    v = rng.standard_normal(N)
    v /= np.linalg.norm(v)
    K = np.diag(d) - 2.0 * (np.outer(v, d * v) + np.outer(d * v, v)) + 4.0 * (v @ (d * v)) * np.outer(v, v)
    theta, resid, _ = ctx.min_eig(0.5 * (K + K.T))
    assert resid <= 1.5e-10
    assert abs(theta + 0.5) <= 2e-10


@pytest.mark.parametrize("N", [5, 300, 1025])
def test_constants_of_one_and_two_systems(ctx, N):
    """The magnetisation estimator of a cold field carries Kt^-1 h': uniform and
    per-site fields with the same values agree (one system and two) to the
    solver's 1e-13 residual times Kt's condition number, under 100 here."""
    from paper_1912_03278_amd import ihmc
    K = rand_K(N, 7)
    psi0 = np.random.default_rng(1).standard_normal(N)
    run = [ihmc.Run(n_md=4, n_traj=2, seed=3, chain_id=1, psi0=psi0, replay_accept=[1, 1])]
    a = ctx.run_dense(ihmc.Dense(K, beta=0.5, C=4.0, h=0.1), run)[0]
    b = ctx.run_dense(ihmc.Dense(K, beta=0.5, C=4.0, h=np.full(N, 0.1)), run)[0]
    for k in ("m", "beta_eps"):
        scale = np.max(np.abs(a[k])) + 1.0
        assert np.max(np.abs(np.asarray(a[k]) - np.asarray(b[k]))) <= 1e-10 * scale, k


def test_checkpoint_with_a_computed_shift(ctx):
    """A shift from Lanczos may differ in the last digits between builds; a given
    one is part of the chain's identity to the bit."""
    import struct

    from paper_1912_03278_amd import ihmc
    K, run = rand_K(64, 2), ihmc.Run(n_md=3, n_traj=4, seed=1)
    for C, moved, ok in ((-1.0, 1e-15, True), (-1.0, 1e-6, False), (4.0, 1e-15, False)):
        ch = ihmc.DenseChains(ctx, ihmc.Dense(K, beta=0.4, C=C), [run])
        ch.advance(2)
        blob, shift = ch.checkpoint(0), ch.info()["C"]
        at = blob.index(struct.pack("d", shift))
        other = shift * (1.0 + moved)
        assert other != shift
        blob = blob[:at] + struct.pack("d", other) + blob[at + 8:]
        if ok:
            ch.restore(0, blob)
        else:
            with pytest.raises(ihmc.IhmcError):
                ch.restore(0, blob)
        ch.close()
