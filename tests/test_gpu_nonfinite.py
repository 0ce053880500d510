"""A field that is not finite stays visible in what a chain reports."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [(4, 4), (3, 4, 5)])
def test_phi_form_of_a_nan_site(L):
    """The phi form's m2c holds the plain sum of tanh^2(phi + h'): NaN with any NaN site,
    as tanh(NaN) is, and the trajectory is counted as non-finite."""
    from paper_1912_03278_amd import ihmc
    psi0 = np.linspace(-1.0, 1.0, int(np.prod(L)))
    with ihmc.Context(arena_bytes=64 << 20) as ctx:
        lat = ihmc.Lattice(L, beta=0.3, C=2 * len(L) + 0.1, h=0.1)
        run = ihmc.Run(n_md=3, n_traj=2, precision=ihmc.F64, form=ihmc.FORM_PHI, psi0=psi0)
        good = ctx.run_lattice(lat, run)
        assert np.all(np.isfinite(good["m2c"])) and good["n_nonfinite"] == 0
        psi0[5] = np.nan
        bad = ctx.run_lattice(lat, run)
    assert np.all(np.isnan(bad["m2c"])) and bad["n_nonfinite"] == 2 and not bad["accepted"].any()
    assert np.isnan(bad["psi_final"][5])
