"""The two-launch Heun step on D2Q9 lattices whose populations outgrow the caches
in planes of whole 128-byte lines, which streams its stores, against the FP64
oracle (bars of the parity tests); u^n of a sampled step, which the same launch
stores; and a pool group past the same size, of lattices that alone are below it,
with the bits of one simulation."""
import numpy as np
import pytest

import oracle as O
from tests import harness as H

pytestmark = pytest.mark.gpu

FORMS = [dict(smol=H.FD), dict(smol=H.FV), dict(smol=H.FD, kT=0.0),
         dict(smol=H.FD, omega_ghost=0.8, omega_bulk=1.3),
         dict(smol=H.FV, walls=1, u_wall=((0.02, 0, 0), (-0.01, 0, 0)))]


def _size(precision):
    return 8 if precision == H.FP64 else 4


@pytest.mark.parametrize("form", range(len(FORMS)))
@pytest.mark.parametrize("precision", [H.FP64, H.FP32DEV])
def test_streamed_halves_match_oracle(form, precision):
    from paper_1104_0078_amd import lbl
    shape = (1376, 1376, 1) if precision == H.FP64 else (1952, 1952, 1)
    n = shape[0] * shape[1]
    assert 2 * 9 * n * _size(precision) > 1 << 28 and n * _size(precision) % 128 == 0
    c = H.config(lattice=H.D2Q9, precision=precision, shape=shape, a=-0.04, b=0.04, **FORMS[form])
    print("streamed halves:", shape, FORMS[form], precision, flush=True)
    p = H.oracle_params(c)
    f, psi = O.init(p, 0, 1e-3)
    O.run(p, f, psi, 0, 1)
    un = O.velocity(p, f, O.force(p, psi))
    O.run(p, f, psi, 1, 1)
    with lbl.Sim(H.lbl_params(c, sample_every=2), lbl.make_init(psi_std=1e-3)) as sim:
        sim.step(2)
        g, phi = sim.observe(lbl.LBL_OBS_POP), sim.observe(lbl.LBL_OBS_PSI)
        uk = sim.observe(lbl.LBL_OBS_UK_AXES)
    tol = H.TOL[precision]
    assert H.rel_err(g, f) <= tol and H.rel_err(phi, psi) <= tol
    if c["kT"] == 0.0:
        return  # |u| is 4e-8 after a step: populations of order 1 resolve it to 1e-9
    ref = np.zeros((2, 2, shape[0]))
    for b in range(2):
        ref[:, b, :] = O.axis_spectrum(p, un[b], shape[0])
    # the bars of the spectra's parity tests
    assert H.rel_err(uk, ref) < (1e-11 if precision == H.FP64 else 2e-5)


@pytest.mark.parametrize("form", [0, 1, 4])
@pytest.mark.parametrize("precision", [H.FP64, H.FP32DEV])
def test_streamed_group_has_the_bits_of_one(form, precision):
    from paper_1104_0078_amd import lbl
    shape = (512, 384, 1)
    count = (1 << 28) // (2 * 9 * shape[0] * shape[1] * _size(precision)) + 1
    c = H.config(lattice=H.D2Q9, precision=precision, shape=shape, a=-0.04, b=0.04, **FORMS[form])
    print("streamed group of", count, FORMS[form], precision, flush=True)
    with lbl.Sim(H.lbl_params(c), lbl.make_init(psi_std=1e-3)) as sim:
        sim.step(4)
        psi = sim.observe(lbl.LBL_OBS_PSI)
    with lbl.Pool(8 << 30) as pool:
        ids = [pool.submit(H.lbl_params(c), lbl.make_init(psi_std=1e-3), 4, keep_psi=True)
               for _ in range(count)]
        while pool.run(2) > 0:
            pass
        for rid in (ids[0], ids[-1]):
            np.testing.assert_array_equal(pool.result(rid, lbl.LBL_RES_PSI), psi)
