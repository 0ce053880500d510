"""FP64 action and estimator sums where their evaluation can go wrong: fields from
nearly zero to where exp(-2|y|) underflows, ragged quads and slabs, with no, a
uniform and a per-site field, and non-finite fields."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctxs():
    from paper_1912_03278_amd import ihmc
    res = ihmc.Context(arena_bytes=1 << 30)
    tiled = ihmc.Context(arena_bytes=1 << 30, resident=0)
    yield res, tiled
    res.close()
    tiled.close()


@pytest.mark.parametrize("form", ["psi", "shifted"])
@pytest.mark.parametrize("scale", [0.0, 1e-9, 1e-2, 1.0, 30.0, 300.0])
@pytest.mark.parametrize("L", [(3, 3), (8, 4), (17, 5), (33, 6), (64, 64), (3, 3, 3), (4, 4, 4), (9, 5, 6), (16, 8, 7)])
def test_against_oracle(ctxs, orc, L, scale, form):
    """H_old of one trajectory and the measured estimators after it (rejected), in
    both kernels, bit-identical to each other.  A site's density is at most (12 psi^2
    + 20 |psi| + 1) here and carries a few ulp: 2e-15 of that, times the sites."""
    from paper_1912_03278_amd import ihmc
    N, d = int(np.prod(L)), len(L)
    rng = np.random.default_rng(N + d)
    psi0 = scale * rng.standard_normal(N)
    for h in (None, 0.07) + (() if form == "shifted" else (rng.normal(0, 0.2, N),)):
        m = dict(beta=0.3, C=2 * d + 0.1, h=h)
        run = ihmc.Run(n_md=1, n_traj=1, traj_len=1e-3, precision=8, seed=3, psi0=psi0, replay_accept=[0],
                       form=ihmc.FORM_SHIFTED if form == "shifted" else ihmc.FORM_PSI)
        a, b = (c.run_batch([ihmc.Lattice(L, **m)], [run])[0] for c in ctxs)
        ref = orc.run(orc.Lattice(tuple(L), **m), 1, 1, traj_len=1e-3, seed=3, psi0=psi0, replay_accept=[0],
                      form=form)
        bound = 2e-15 * float(np.sum(12 * psi0 ** 2 + 20 * np.abs(psi0) + 1)) + 1e-14 * N
        assert abs(a["H_old"][0] - ref.H_old[0]) <= bound, (h is None, a["H_old"][0], ref.H_old[0])
        for k in ("m", "beta_eps"):
            assert abs(a[k][0] - getattr(ref, k)[0]) <= 1e-10 * (abs(getattr(ref, k)[0]) + 1.0), k
        for k in ("dH", "H_old", "H_new", "m", "m2c", "beta_eps", "psi_final"):
            assert np.array_equal(a[k], b[k]), k


@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf, 1e200])
@pytest.mark.parametrize("prec", [4, 8])
@pytest.mark.parametrize("L", [(6, 5), (40, 36), (5, 4, 6)])
def test_non_finite_field_is_flagged(ctxs, L, prec, bad):
    """A proposal from a field that is not finite is recorded as such and refused."""
    from paper_1912_03278_amd import ihmc
    psi0 = np.zeros(int(np.prod(L)))
    psi0[len(psi0) // 2] = bad
    for c in ctxs:
        lat = ihmc.Lattice(L, beta=0.3, C=2 * len(L) + 0.1)
        r = c.run_batch([lat], [ihmc.Run(n_md=2, n_traj=2, precision=prec, seed=3, psi0=psi0)])[0]
        assert r["n_nonfinite"] == 2 and not r["accepted"].any() and np.isnan(r["dH"]).all()
