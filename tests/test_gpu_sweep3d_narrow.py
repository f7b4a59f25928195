"""The 3D sweep by blocks of 2 x 2 and of single columns, which geometries of a
small cross section (and, in FP64, many others) take: ragged tiles, pores, walls
and periodic axes, batches, and the transposed sweep.  Fields of two source
iterations against the oracle (FP64 1e-11, FP32 1e-5 of the largest magnitude),
gradients in FP64 to 1e-11, the bars of the wider geometries' tests."""
import numpy as np
import pytest

import bte_inputs as I
import oracle as O
from oracle.adjoint import keff_weights, steady_adjoint

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


def box(n, bc, pores=True):
    nc = int(np.prod(n))
    solid = np.ones(nc, dtype=np.uint8)
    if pores:
        solid[(np.arange(nc) * 7919) % 13 == 5] = 0
    return dict(dim=3, n=list(n), len=[m * 20e-9 for m in n], bc=bc, bcT=[301.0, 300.0, 299.5, 300.0, 299.0, 300.0],
                pdT=[0.7 if b == P else 0.0 for b in bc[::2]], solid=solid, pore_bc=D)


# single columns: the rods of 1 x 1 and 2 x 1; 2 x 2: the batches (of ten, both precisions), 5 x 9 and 9 x 5 in FP64
@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("ns,bc,lim", [([(1, 1, 60)], WALLS, 0), ([(2, 1, 100)], PERIODIC, 1), ([(1, 2, 53)], WALLS, 2),
                                       ([(5, 5, 60)] * 10, WALLS, 0), ([(7, 6, 40), (9, 3, 25)] * 5, PERIODIC, 0),
                                       ([(5, 9, 50)], PERIODIC, 1), ([(9, 5, 17)], WALLS, 2)])
def test_sweep(B, prec, ns, bc, lim):
    f64 = prec == "f64"
    mat = I.bands(17, 7, 1e-12, 1e-10)
    mat.update(n_theta=2, n_phi=3, Tref=300.0)
    geos = [box(n, bc, int(np.prod(n)) > 200) for n in ns]
    nc = sum(g["solid"].size for g in geos)
    gam, src = 1e11 * np.abs(I.random_field(1, nc)), 1e16 * np.abs(I.random_field(2, nc))
    prob = B.Problem(geos, mat, dict(precision=B.F64 if f64 else B.F32, scheme=B.SEQUENTIAL, limiter=lim, max_iter=2,
                                     residual_temp=0.0, residual_flux=0.0))
    prob.set_fields(torch.as_tensor(src, device="cuda"), torch.as_tensor(gam, device="cuda"))
    c4 = mat["C"] / (4 * np.pi)
    solid = np.concatenate([g["solid"] for g in geos])
    e0 = (I.random_field(3, nc * 48).reshape(nc, 48, 1) * c4 * solid[:, None, None])
    e = torch.as_tensor(e0.reshape(-1), device="cuda").to(prob.dtype)
    start = e.double().cpu().numpy().reshape(nc, -1)
    prob.steady_solve(e, init=False, allow_not_converged=True)
    got, c0 = e.double().cpu().numpy().reshape(nc, -1), 0
    for g in geos:
        c1 = c0 + g["solid"].size
        case = O.Case(g, mat, P=src[c0:c1], gamma=gam[c0:c1], limiter=lim)
        ref, _ = O.steady(case, scheme=0, tol_T=0.0, tol_q=0.0, max_iter=2, e=start[c0:c1].reshape(-1).copy())
        assert np.abs(got[c0:c1].reshape(-1) - ref).max() <= (1e-11 if f64 else 1e-5) * np.abs(ref).max()
        c0 = c1


@pytest.mark.parametrize("n,pores", [((2, 1, 100), False), ((5, 6, 20), True)])
def test_gradient(B, n, pores):
    g = box(n, [P, P, D, S, T, D], pores)
    mat = I.bands(9, 2, 1e-12, 1e-10)
    mat.update(n_theta=1, n_phi=1, Tref=300.0)
    gam = 1e11 * np.abs(I.random_field(1, int(np.prod(n))))
    case = O.Case(g, mat, gamma=gam)
    eo, _ = O.steady(case, scheme=1, tol_T=1e-15, tol_q=1e-15, max_iter=20000, cg_rtol=1e-14)
    _, ref = steady_adjoint(case, eo, keff_weights(case))
    ctl = dict(precision=B.F64, scheme=B.SYNTHETIC, limiter=B.LIM_NONE, adjoint=True, residual_temp=1e-13,
               residual_flux=1e-13, max_iter=20000, cg_rtol=1e-12, cg_max_iter=5000)
    prob = B.Problem(g, mat, ctl)
    prob.set_fields(None, torch.as_tensor(gam, device="cuda"))
    e = torch.as_tensor(eo, device="cuda")
    grad, st = prob.adjoint(e)
    assert st["converged"]
    assert np.abs(grad.cpu().numpy() - ref).max() <= 1e-11 * np.abs(ref).max()
