"""Ghost modes that relax without noise (kT = 0, omega_ghost != 1): every site's
collision starts from its own ghost moments, in the D2Q9 halves on both tiles
(the wide one has two rows a thread) and in the 3-D flux form, against the FP64
oracle from populations with ghost moments of 1e-3 (bars of the parity tests);
in a pool whose residents put the group on the wide tile, a request keeps the
bits that it has alone."""
import numpy as np
import pytest

import oracle as O
from tests import harness as H
from tests.inputs import perturbed_populations

pytestmark = pytest.mark.gpu

FORMS = [dict(smol=H.FD), dict(smol=H.FV),
         dict(smol=H.FV, walls=1, u_wall=((0.02, 0, 0), (-0.01, 0, 0)))]
CASES = [(H.D2Q9, shape, k) for shape in ((33, 9, 1), (1473, 513, 1)) for k in range(len(FORMS))]
CASES += [(H.D3Q19, (33, 9, 6), 1), (H.D3Q15, (33, 9, 6), 2)]


def _start(c):
    p = H.oracle_params(c)
    f, psi = O.init(p, 0, 1e-3)
    f = perturbed_populations(f[:, 0], f.shape[1], 1e-3, 7)
    return f, psi


@pytest.mark.parametrize("lattice,shape,form", CASES)
@pytest.mark.parametrize("precision", [H.FP64, H.FP32DEV])
def test_noise_free_ghosts_match_oracle(lattice, shape, form, precision):
    from paper_1104_0078_amd import lbl
    c = H.config(lattice=lattice, precision=precision, shape=shape, a=-0.04, b=0.04, kT=0.0,
                 omega_ghost=0.7, **FORMS[form])
    print("noise-free ghosts:", lattice, shape, FORMS[form], precision, flush=True)
    f0, psi0 = _start(c)
    f_ref, psi_ref = H.oracle_run(c, 2, f0.copy(), psi0.copy())
    ini = lbl.make_init(lbl.LBL_INIT_USER, f0=f0, psi0=psi0)
    with lbl.Sim(H.lbl_params(c), ini) as sim:
        sim.step(2)
        f, psi = sim.observe(lbl.LBL_OBS_POP), sim.observe(lbl.LBL_OBS_PSI)
    tol = H.TOL[precision]
    assert H.rel_err(f, f_ref) <= tol and H.rel_err(psi, psi_ref) <= tol


@pytest.mark.parametrize("form", range(len(FORMS)))
@pytest.mark.parametrize("precision", [H.FP64, H.FP32DEV])
def test_noise_free_ghosts_in_a_wide_group(form, precision):
    """One request of 2 wide tiles among 49 of 32: more than the 1536 of the rule."""
    from paper_1104_0078_amd import lbl
    c = H.config(lattice=H.D2Q9, precision=precision, shape=(127, 13, 1), a=-0.04, b=0.04,
                 kT=0.0, omega_ghost=0.7, **FORMS[form])
    big = dict(c, shape=(127, 125, 1))
    f0, psi0 = _start(c)
    ini = lbl.make_init(lbl.LBL_INIT_USER, f0=f0, psi0=psi0)
    with lbl.Sim(H.lbl_params(c), ini) as sim:
        sim.step(8)
        psi = sim.observe(lbl.LBL_OBS_PSI)
    with lbl.Pool(1 << 31) as pool:
        rid = pool.submit(H.lbl_params(c), ini, 8, keep_psi=True)
        for _ in range(49):
            pool.submit(H.lbl_params(big), lbl.make_init(psi_std=1e-3), 8)
        while pool.run(4) > 0:
            pass
        np.testing.assert_array_equal(pool.result(rid, lbl.LBL_RES_PSI), psi)
