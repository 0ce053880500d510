"""Tiles of the dense BF16-limb GEMM: every tile size, ragged site and chain
counts, both product sets."""
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


# (sites, chains): 2x1 blocks per wave with 1, 16 and 17 chains, 2x2, 4x2 (also
# with a partly filled last column tile), 4x4
@pytest.mark.parametrize("products", [6, 3])
@pytest.mark.parametrize("N,B", [(1, 1), (256, 16), (257, 17), (700, 65), (1024, 128), (2048, 161), (2048, 300)])
def test_tiles_against_oracle_and_alone(ctx, orc, N, B, products):
    """A force row is that of the chain alone, bit for bit (one accumulator per
    output runs over the slice in the same order in every tile), and agrees with
    the FP64 oracle to the product set's accuracy."""
    from paper_1912_03278_amd import ihmc
    rng = np.random.default_rng(N + B)
    K = rand_K(N, 5)
    m = dict(beta=0.6, C=3.0, h=0.05)
    psi = rng.standard_normal((B, N)).astype(np.float32).astype(np.float64)
    F = ctx.dense_force(ihmc.Dense(K, **m), psi, products=products)
    for i in sorted({0, min(15, B - 1), min(16, B - 1), B // 2, B - 1}):
        alone = ctx.dense_force(ihmc.Dense(K, **m), psi[i:i + 1], products=products)
        assert np.array_equal(F[i], alone[0]), i
        ref = orc.force(orc.Dense(K, **m), psi[i])
        err = np.linalg.norm(F[i] - ref) / np.linalg.norm(ref)
        assert err < (2e-6 if products == 6 else 2e-3), (i, err)


# FP64 product: 1x1 blocks per wave with 1, 16, 17 chains, 1x2, 2x2 (also with a
# partly filled last column tile)
@pytest.mark.parametrize("N,B", [(1, 1), (300, 17), (257, 16), (2048, 193), (2048, 256), (4096, 250)])
def test_action_against_numpy_and_alone(ctx, N, B):
    """H_old of a first trajectory is the FP64 action of the start plus the
    momenta's energy: bit for bit that of the chain alone, and against a product
    in numpy (both sum N terms of order one in FP64: 1e-15 sqrt(N) relative)."""
    from paper_1912_03278_amd import ihmc
    rng = np.random.default_rng(N * 3 + B)
    K = rand_K(N, 6)
    m = ihmc.Dense(K, beta=0.6, C=3.0)
    psi0 = rng.standard_normal((B, N)).astype(np.float32).astype(np.float64)
    runs = [ihmc.Run(n_md=1, n_traj=1, seed=9, chain_id=i, psi0=psi0[i]) for i in range(B)]
    full = ctx.run_dense(m, runs)
    # the momenta's part is the same for another field: it drops out of differences
    flip = [ihmc.Run(n_md=1, n_traj=1, seed=9, chain_id=i, psi0=0.5 * psi0[i]) for i in range(B)]
    half = ctx.run_dense(m, flip)

    def action(x):
        u = x @ K + 3.0 * x
        y = np.sqrt(0.6) * u
        return np.sum(0.5 * x * u - np.logaddexp(y, -y) + np.log(2.0), axis=-1)

    ref = action(psi0) - action(0.5 * psi0)
    got = np.array([full[i]["H_old"][0] - half[i]["H_old"][0] for i in range(B)])
    assert np.max(np.abs(got - ref)) <= 1e-12 * N
    for i in sorted({0, min(15, B - 1), min(16, B - 1), B - 1}):
        alone = ctx.run_dense(m, runs[i:i + 1])[0]
        assert alone["H_old"][0] == full[i]["H_old"][0] and alone["H_new"][0] == full[i]["H_new"][0], i
