"""The diffusion solves: the one-launch CG (k_cg_solve) where its split of the
cells can go wrong (one block with and without full waves, one and two cells
past a block, ragged tiles, periodic wraps, pores, two geometries in one problem
with ghosts of both, and a problem past its largest grid: a launch per
iteration), and the solution by eigenvectors (bte_direct.hip) that geometries
without pores and scattering rates take instead (one cell, odd and even
periodic axes, every pair of ends, three axes).

One source iteration (sequential scheme, FP64) from the heat-diffusion guess
is compared with the oracle's: the guess is a CG solve to a relative residual
of 1e-13, so a field may differ by that times the operator's condition number,
at most (2 n / pi)^2 per axis, on either side."""
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


def material(nl=2):
    m = I.bands(11, nl, 1e-12, 1e-11)
    m.update(n_theta=1, n_phi=1, Tref=300.0)
    return m


def geometry(n, bc, bcT=None, pdT=(0.0, 0.0, 0.0), pores=False):
    h = 5e-9
    nc = int(np.prod(n))
    solid = None
    if pores:
        idx = np.arange(nc)
        solid = np.ones(nc, dtype=np.uint8)
        solid[(idx * 7919) % 11 == 3] = 0     # isolated pore cells
    return dict(dim=len(n), n=list(n) + [1] * (3 - len(n)), len=[m * h for m in n] + [1.0] * (3 - len(n)),
                bc=list(bc) + [S] * (6 - len(bc)), bcT=bcT or [301.0, 299.0] + [300.0] * 4, pdT=list(pdT),
                solid=solid, pore_bc=D)


CASES = {
    "line_1": geometry((1,), [T, T]),
    "line_63": geometry((63,), [T, T]),
    "line_512": geometry((512,), [T, S]),
    "line_513": geometry((513,), [T, T]),
    "line_2049": geometry((2049,), [T, T]),
    "plane_45x46": geometry((45, 46), [T, D, S, D]),
    "plane_33x17": geometry((33, 17), [D, D, T, S]),
    "plane_97x83": geometry((97, 83), [T, T, D, D]),
    "pores_periodic_47x47": geometry((47, 47), [P, P, P, P], pdT=(1.0, 0.0, 0.0), pores=True),
    "periodic_12x9": geometry((12, 9), [P, P, P, P], pdT=(0.5, 0.0, 0.0)),
    "box_plain": geometry((7, 6, 9), [T, S, D, T, P, P]),
    "box_walls": geometry((33, 4, 5), [T, T, T, T, T, D]),
    "box_13": geometry((13, 14, 13), [T, T, D, S, S, D], pores=True),
    "box_periodic": geometry((9, 17, 16), [P, P, T, T, P, P], pdT=(1.0, 0.0, 0.0), pores=True),
}


def one_iteration(B, geos, mat, Ps, scheme, init, e=None, rates=False, **ctl):
    prob = B.Problem(geos, mat, dict(precision=B.F64, scheme=scheme, residual_temp=0.0, residual_flux=0.0, **ctl))
    gam = torch.zeros(prob.n_cells, dtype=torch.float64, device="cuda") if rates else None
    prob.set_fields(torch.as_tensor(np.concatenate(Ps), device="cuda"), gam)
    e = prob.zeros() if e is None else torch.as_tensor(e, device="cuda")
    st = prob.steady_solve(e, init=init, allow_not_converged=True)
    return e.cpu().numpy(), st


def source(g, k):
    nc = int(np.prod(g["n"]))
    p = 1e16 * (1.0 + I.random_field(k, nc))
    if all(b != T for b in g["bc"][:2 * g["dim"]]):     # no wall: no net heat
        s = np.ones(nc, bool) if g["solid"] is None else g["solid"] != 0
        p -= p[s].mean()
    return p


@pytest.mark.parametrize("rates", [False, True])      # given (zero) scattering rates: CG
@pytest.mark.parametrize("name", sorted(CASES))
def test_guess_against_oracle(B, name, rates):
    g = CASES[name]
    mat, P_ = material(), source(g, 5)
    e, _ = one_iteration(B, [g], mat, [P_], B.SEQUENTIAL, True, rates=rates, max_iter=1)
    eo, _ = O.steady(O.Case(g, mat, P=P_), scheme=0, tol_T=0.0, tol_q=0.0, max_iter=1)
    bar = 2e-13 * sum((2 * n / np.pi) ** 2 + 1 for n in g["n"]) + 1e-11
    assert np.abs(e - eo).max() <= bar * np.abs(eo).max()


def test_two_geometries(B):
    """Two geometries in one problem: CG steps are shared, the guess is each one's own."""
    names = ["plane_45x46", "plane_97x83"]
    mat, Ps = material(), [source(CASES[n], k) for k, n in enumerate(names)]
    e, _ = one_iteration(B, [CASES[n] for n in names], mat, Ps, B.SEQUENTIAL, True, max_iter=1)
    at = 0
    for n, P_ in zip(names, Ps):
        eo, _ = O.steady(O.Case(CASES[n], mat, P=P_), scheme=0, tol_T=0.0, tol_q=0.0, max_iter=1)
        bar = 2e-13 * sum((2 * 97 / np.pi) ** 2 for _ in range(2)) + 1e-11
        assert np.abs(e[at:at + eo.size] - eo).max() <= bar * np.abs(eo).max()
        at += eo.size


@pytest.mark.parametrize("n", [(60, 37), (730, 730)])
def test_capped_correction(B, n):
    """Two synthetic iterations whose CG stops at its cap, one launch (2 220 cells) and a launch per iteration
    (532 900 cells, past the largest grid)."""
    g = geometry(n, [T, T, S, S])
    mat, P_ = material(1), source(g, 9)
    c4 = mat["C"] / (4 * np.pi)
    case = O.Case(g, mat, P=P_)
    e0 = (1e-3 * P_ / 1e16)[:, None, None] * c4 * np.ones((1, 8, 1))
    e, st = one_iteration(B, [g], mat, [P_], B.SYNTHETIC, False, e0.reshape(-1).copy(), max_iter=2, cg_rtol=1e-12,
                          cg_max_iter=25)
    eo, so = O.steady(case, scheme=1, tol_T=0.0, tol_q=0.0, max_iter=2, cg_rtol=1e-12, cg_maxit=25, e=e0.reshape(-1))
    assert st["cg_iters"] == so["cg_iters"] == 50
    assert np.abs(e - eo).max() <= 1e-10 * np.abs(eo).max()


@pytest.mark.parametrize("name", ["line_63", "plane_33x17", "periodic_12x9", "box_plain"])
def test_correction_by_eigenvectors(B, name):
    """Three synthetic iterations with a cap that CG cannot reach: no CG iteration is counted, and the fields are the
    oracle's, whose corrections are solved to 1e-13."""
    g = CASES[name]
    mat, P_ = material(), source(g, 7)
    e, st = one_iteration(B, [g], mat, [P_], B.SYNTHETIC, True, max_iter=3, cg_rtol=1e-8, cg_max_iter=5000)
    eo, _ = O.steady(O.Case(g, mat, P=P_), scheme=1, tol_T=0.0, tol_q=0.0, max_iter=3, cg_rtol=1e-13, cg_maxit=5000)
    assert st["cg_iters"] == 0
    bar = 1e-12 * sum((2 * n / np.pi) ** 2 + 1 for n in g["n"]) + 1e-11
    assert np.abs(e - eo).max() <= bar * np.abs(eo).max()
