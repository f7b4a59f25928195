"""The passes over whole rows of e (the equilibrium start and the final
correction of a steady solve; a wavefront per cell, 16 bytes a lane where the
rows allow): band counts below, at and above the vector width and the
wavefront, rows that are no multiple of 16 bytes, a start off 16 bytes,
pores, two geometries of different materials.  One iteration of the
synthetic scheme from the diffusion guess against the oracle, FP64 1e-10
(the guess is solved to 1e-13 and the correction to 1e-12) and FP32 1e-5 of
the largest magnitude."""
import numpy as np
import pytest

import bte_inputs as I
import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2306_14181_amd import bte
    bte.load()
    return bte


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("nl,nth,off", [(1, 2, 0), (3, 2, 0), (4, 2, 0), (5, 4, 0), (70, 2, 0), (70, 2, 1), (3, 4, 1)])
def test_rows(B, prec, nl, nth, off):
    f64 = prec == "f64"
    n, geos, mats, refs = 21, [], [], []
    for g in range(2):
        solid = np.ones(n, dtype=np.uint8)
        if g:
            solid[9] = 0
        bc = [I.BC_THERMAL, I.BC_THERMAL] + [I.BC_SPECULAR] * 4
        geos.append(dict(dim=1, n=[n, 1, 1], len=[(1 + g) * 1e-7, 1.0, 1.0], bc=bc,
                         bcT=[301.0 + g, 299.5, 300, 300, 300, 300], solid=solid, pore_bc=I.BC_THERMAL))
        m = I.bands(11 + g, nl, 1e-12, 1e-10)
        m.update(n_theta=nth, n_phi=1, Tref=300.0)
        mats.append(m)
        refs.append(O.steady(O.Case(geos[g], m), scheme=1, tol_T=0.0, tol_q=0.0, max_iter=1)[0])
    prob = B.Problem(geos, mats, dict(precision=B.F64 if f64 else B.F32, scheme=B.SYNTHETIC, max_iter=1,
                                      residual_temp=0.0, residual_flux=0.0, cg_rtol=1e-12, cg_max_iter=2000),
                     geo_mat=[0, 1])
    buf = torch.zeros(prob.n_unknowns + off, dtype=prob.dtype, device="cuda")
    e = buf[off:]
    prob.steady_solve(e, init=True, allow_not_converged=True)
    eo = np.concatenate(refs)
    assert np.abs(e.double().cpu().numpy() - eo).max() <= (1e-10 if f64 else 1e-5) * np.abs(eo).max()
