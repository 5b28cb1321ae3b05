"""The refinement indicator and the network inputs for every block shape the
library is built for (the layer around a block from ghost slabs, finer and
equal neighbours), against the oracle on its own state."""
import numpy as np
import pytest

from oracle import mlp, solver, units
from synthetic import Cme, Wind, as_dict

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block,n,levels", [((4, 4, 4), (16, 8, 12), 2), ((8, 8, 8), (24, 16, 16), 2),
                                            ((12, 8, 12), (24, 16, 24), 2), ((12, 12, 12), (36, 12, 24), 2),
                                            ((16, 12, 12), (32, 24, 24), 2)])
def test_flags_and_features(block, n, levels):
    import paper_2211_12867_amd as ic
    grid = dict(geometry="spherical", x0=(0.1, 60.0, 0.0), x1=(1.1, 120.0, 90.0), n=n, block=block,
                stretched_r=True, max_level=levels, periodic=(False, False, False), gamma=1.5, cfl=0.4)
    wind = as_dict(Wind(seed=3))
    cme = as_dict(Cme(t_start_s=0.0, duration_s=6 * 3600.0, v_kms=1400.0, half_width_deg=35.0,
                      colat_deg=90.0, lon_deg=20.0, n_cm3=1500.0, T_K=0.8e6))
    amr = dict(eps_lohner=0.01, tol_refine=0.1, tol_coarsen=0.0125, w_rho=0.5, w_v=0.5,
               lon_earth_deg=0.0, clt_earth_deg=90.0, dlon_earth_deg=60.0, dclt_earth_deg=30.0,
               dlon_cme_deg=90.0, use_windows=True, regrid_every=2, buffer_blocks=1)
    ora = solver.Solver(grid, wind, cme, amr)
    for _ in range(3):
        ora.step()
    ora.regrid(ora.flags())
    for _ in range(2):
        ora.step()
    bl, U = ora.state()
    gpu = ic.Sim(grid, wind, [cme], amr)
    gpu.set_state(bl, U, ora.t * units.T0)
    ties = []
    f = ora.flags(ties)
    got = gpu.eval_flags()
    tied = {t[0] if isinstance(t, tuple) and isinstance(t[0], tuple) else t for t in ties}
    assert [int(x) for b, x in zip(bl, got) if b not in tied] == [f[b] for b in bl if b not in tied]
    ref = np.stack([mlp.features(u, ora.gamma) for u in U])
    np.testing.assert_allclose(gpu.features(), ref, rtol=3e-7, atol=1e-12)     # one float32 rounding
    gpu.close()
