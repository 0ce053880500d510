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
