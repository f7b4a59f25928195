"""The 3D sweep (k_sweep3d: tiles of 4 x 4 columns, segments along z) at the
edges of its split: single cells and columns, ragged tiles, columns longer
than the longest segment, several segments, with pores, every wall kind and
periodic axes.  Two source iterations of the sequential scheme against the
oracle, FP64 1e-11 and FP32 1e-5 of the largest magnitude."""
import numpy as np
import pytest

import bte_inputs as I
import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

T, S, D, P = I.BC_THERMAL, I.BC_SPECULAR, I.BC_DIFFUSE, I.BC_PERIODIC
WALLS = [T, D, S, D, T, S]
PERIODIC = [P, P, T, S, P, P]


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2306_14181_amd import bte
    bte.load()
    return bte


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n,bc,lim,zseg", [((1, 1, 1), WALLS, 0, None), ((3, 5, 2), WALLS, 0, None),
                                           ((4, 4, 9), PERIODIC, 0, 8), ((5, 9, 50), WALLS, 0, 48),
                                           ((9, 5, 17), WALLS, 1, 16), ((13, 2, 11), PERIODIC, 2, 4),
                                           ((8, 7, 12), PERIODIC, 0, 12), ((2, 6, 10), WALLS, 0, 2)])
def test_sweep(B, prec, n, bc, lim, zseg):
    nc = int(np.prod(n))
    solid = np.ones(nc, dtype=np.uint8)
    if nc > 20:
        solid[(np.arange(nc) * 7919) % 13 == 5] = 0
    h = 20e-9
    g = dict(dim=3, n=list(n), len=[m * h for m in n], bc=bc, bcT=[301.0, 300.0, 299.5, 300.0, 299.0, 300.0],
             pdT=[0.7 if b == P else 0.0 for b in bc[::2]], solid=solid, pore_bc=D)
    mat = I.bands(17, 7, 1e-12, 1e-10)
    mat.update(n_theta=2, n_phi=3, Tref=300.0)      # 42 lanes an octant and a second octant's start off 64
    gam, src = 1e11 * np.abs(I.random_field(1, nc)), 1e16 * np.abs(I.random_field(2, nc))
    f64 = prec == "f64"
    prob = B.Problem(g, mat, dict(precision=B.F64 if f64 else B.F32, scheme=B.SEQUENTIAL, limiter=lim, max_iter=2,
                                  residual_temp=0.0, residual_flux=0.0))
    if zseg:
        prob.set_tiles(B.TUNE_SWEEP, (1, 1, zseg))
    prob.set_fields(torch.as_tensor(src, device="cuda"), torch.as_tensor(gam, device="cuda"))
    case = O.Case(g, mat, P=src, gamma=gam, limiter=lim)
    c4 = mat["C"] / (4 * np.pi)
    e0 = (I.random_field(3, nc * case.na).reshape(nc, case.na, 1) * c4 * solid[:, None, None]).reshape(-1)
    e = torch.as_tensor(e0, device="cuda").to(prob.dtype)
    e0 = e.double().cpu().numpy()
    prob.steady_solve(e, init=False, allow_not_converged=True)
    eo, _ = O.steady(case, scheme=0, tol_T=0.0, tol_q=0.0, max_iter=2, e=e0)
    assert np.abs(e.double().cpu().numpy() - eo).max() <= (1e-11 if f64 else 1e-5) * np.abs(eo).max()
