"""The register-tile sweep (k_sweep2d): rows whose cells all have an interior
stencil next to rows that do not (walls, a pore, periodic faces, ragged
tiles), the moments of one, two and four tile rows per wavefront, lane chunks
that are not full, both launch forms and the form taken without a choice.  Two
source iterations of the sequential scheme (the second one reads the first
one's moments) against the oracle, FP64 1e-11 and FP32 1e-5 of the largest
magnitude."""
import numpy as np
import pytest

import bte_inputs as I
import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

T, S, D, P = I.BC_THERMAL, I.BC_SPECULAR, I.BC_DIFFUSE, I.BC_PERIODIC


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2306_14181_amd import bte
    bte.load()
    return bte


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n,bc,lim,pore", [((24, 24), [T, D, S, T], 0, 13), ((33, 17), [D, T, T, S], 1, -1),
                                           ((16, 40), [P, P, T, D], 2, 300), ((31, 32), [P, P, P, P], 0, 500),
                                           ((8, 1), [T, S, S, D], 0, -1)])
def test_sweep(B, prec, n, bc, lim, pore):
    f64 = prec == "f64"
    nc, h = n[0] * n[1], 20e-9
    solid = np.ones(nc, dtype=np.uint8)
    if pore >= 0:
        solid[pore] = 0
    g = dict(dim=2, n=[n[0], n[1], 1], len=[n[0] * h, n[1] * h, 1.0], bc=bc + [S, S],
             bcT=[301.0, 300.0, 299.5, 300.0, 300.0, 300.0], pdT=[0.7 if bc[0] == P else 0.0, 0.0, 0.0], solid=solid,
             pore_bc=D)
    mat = I.bands(17, 7, 1e-12, 1e-10)
    mat.update(n_theta=2, n_phi=5, Tref=300.0)      # 70 lanes a quadrant: a full chunk and one of 6
    gam, src = 1e11 * np.abs(I.random_field(1, nc)), 1e16 * np.abs(I.random_field(2, nc))
    case = O.Case(g, mat, P=src, gamma=gam, limiter=lim)
    c4 = mat["C"] / (4 * np.pi)
    e0 = (I.random_field(3, nc * case.na).reshape(nc, case.na, 1) * c4 * solid[:, None, None]).reshape(-1)
    dt = torch.float64 if f64 else torch.float32
    e0 = torch.as_tensor(e0, device="cuda").to(dt)
    eo = O.steady(case, scheme=0, tol_T=0.0, tol_q=0.0, max_iter=2, e=e0.double().cpu().numpy())[0]
    forms = [(None, None)] + [(k, t) for k in (B.TUNE_SWEEP, B.TUNE_SWEEP_ONE_LAUNCH)
                              for t in ((8, 8, 2), (8, 8, 1), (8, 8, 4)) if not (f64 and t[2] == 4)]
    for kind, tile in forms:
        prob = B.Problem(g, mat, dict(precision=B.F64 if f64 else B.F32, scheme=B.SEQUENTIAL, limiter=lim, max_iter=2,
                                      residual_temp=0.0, residual_flux=0.0))
        if tile:
            prob.set_tiles(kind, tile)
        prob.set_fields(torch.as_tensor(src, device="cuda"), torch.as_tensor(gam, device="cuda"))
        e = e0.clone()
        prob.steady_solve(e, init=False, allow_not_converged=True)
        err = np.abs(e.double().cpu().numpy() - eo).max() / np.abs(eo).max()
        assert err <= (1e-11 if f64 else 1e-5), (kind, tile, err)
