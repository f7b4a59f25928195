"""What follows a one-launch sweep or CG solve that gave up waiting: the library
repeats the work with a launch per tile diagonal or per CG iteration.  The
abort words are set beforehand from the host (bte_internal_give_up), so waits
that find nothing at once end, and every kernel ends as usual."""
import ctypes as C

import numpy as np
import pytest

import bte_inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

T, S, D, P = I.BC_THERMAL, I.BC_SPECULAR, I.BC_DIFFUSE, I.BC_PERIODIC
SWEEP, CG, TAGS = 1, 2, 4


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2306_14181_amd import bte
    bte.load()
    return bte


def give_up(B, prob, what):
    n = (C.c_int * 2)()
    B.load().bte_internal_give_up(prob._h, what, n)
    return list(n)


def geometry(n, bc, pores=True, pdT=(0.0, 0.0, 0.0)):
    nc = int(np.prod(n))
    solid = np.ones(nc, dtype=np.uint8)
    if pores:
        solid[(np.arange(nc) * 7919) % 13 == 5] = 0
    return dict(dim=len(n), n=list(n) + [1] * (3 - len(n)), len=[m * 20e-9 for m in n] + [1.0] * (3 - len(n)),
                bc=list(bc) + [S] * (6 - len(bc)), bcT=[301.0, 299.0] + [300.0] * 4, pdT=list(pdT), solid=solid,
                pore_bc=D)


def problem(B, geo, prec=None, **ctl):
    mat = I.bands(23, 5, 1e-12, 1e-10)
    mat.update(n_theta=2, n_phi=2, Tref=300.0)
    control = dict(precision=B.F64 if prec is None else prec, scheme=B.SYNTHETIC, max_iter=5, residual_temp=0.0,
                   residual_flux=0.0, cg_rtol=1e-15, cg_max_iter=12)   # a CG solve takes its 12 iterations
    control.update(ctl)
    prob = B.Problem(geo, mat, control)
    e = torch.as_tensor(np.random.default_rng(4).uniform(-1, 1, prob.n_unknowns), device="cuda").to(prob.dtype)
    return prob, e


@pytest.mark.parametrize("graphs", [True, False])
@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("scheme", ["synthetic", "sequential"])
@pytest.mark.parametrize("geos", [[(61, 45)], [(30, 70), (17, 9), (64, 64)]])
def test_sweep(B, geos, scheme, prec, graphs):
    """The default form: the iteration again, by launches per diagonal from then on; bitwise the solve
    that was asked for them."""
    geo = [geometry(n, [T, T, S, D]) for n in geos]
    ctl = dict(prec=B.F64 if prec == "f64" else B.F32, scheme=B.SYNTHETIC if scheme == "synthetic" else B.SEQUENTIAL)
    ref, want = problem(B, geo, **ctl)
    ref.set_persistent(False)
    ref.set_graphs(graphs)
    rs = ref.steady_solve(want, init=False, allow_not_converged=True)
    prob, e = problem(B, geo, **ctl)
    prob.set_graphs(graphs)
    give_up(B, prob, SWEEP)
    st = prob.steady_solve(e, init=False, allow_not_converged=True)
    assert give_up(B, prob, 0) == [1, 0]
    assert torch.equal(e, want)
    for k in ("iters", "cg_iters", "sweep_launches", "updates", "eps_T", "eps_q"):
        assert st[k] == rs[k], k
    # the next solve waits again
    _, e = problem(B, geo, **ctl)
    st = prob.steady_solve(e, init=False, allow_not_converged=True)
    assert give_up(B, prob, 0) == [1, 0] and st["sweep_launches"] == 5
    assert torch.equal(e, want)


def test_sweep_asked_for(B):
    prob, e = problem(B, geometry((61, 45), [T, T, S, D]))
    prob.set_persistent(True)
    give_up(B, prob, SWEEP)
    with pytest.raises(B.BteError) as x:
        prob.steady_solve(e, init=False, allow_not_converged=True)
    assert x.value.status == B.BTE_ERR_HIP


# Either form runs the same recurrences in FP64, in another order of the sums: 12 steps on operators of a condition
# number below (2 * 80 / pi)^2 = 2600, five iterations: 60 * 2600 * 2^-53 = 2e-11.
@pytest.mark.parametrize("n,bc", [((700,), [T, T]), ((3000,), [T, D]), ((70, 80), [T, T, S, D]), ((20, 16, 18), [T, S])])
@pytest.mark.parametrize("init", [False, True])
def test_cg(B, n, bc, init):
    geo = geometry(n, bc)
    ref, want = problem(B, geo)
    rs = ref.steady_solve(want, init=init, allow_not_converged=True)
    assert give_up(B, ref, 0) == [0, 0]
    prob, e = problem(B, geo)
    give_up(B, prob, CG)
    st = prob.steady_solve(e, init=init, allow_not_converged=True)
    assert give_up(B, prob, 0)[1] == 1    # not tried again in the same call
    assert (e - want).abs().max() <= 1e-10 * want.abs().max()
    assert st["iters"] == rs["iters"] and st["sweep_launches"] == rs["sweep_launches"]
    assert st["cg_iters"] == rs["cg_iters"] == 5 * 12


def test_cg_of_the_gradient(B):
    geo = geometry((44, 60), [P, P, D, D], pdT=(1.0, 0.0, 0.0))
    ctl = dict(adjoint=1, max_iter=4)
    ref, e = problem(B, geo, **ctl)
    want, rs = ref.adjoint(e, allow_not_converged=True)
    prob, _ = problem(B, geo, **ctl)
    give_up(B, prob, CG)
    g, st = prob.adjoint(e, allow_not_converged=True)
    assert give_up(B, prob, 0)[1] == 1 and give_up(B, ref, 0) == [0, 0]
    assert (g - want).abs().max() <= 1e-10 * want.abs().max()
    assert st["iters"] == rs["iters"]
    assert st["cg_iters"] == rs["cg_iters"] > 0


@pytest.mark.parametrize("n,bc", [((700,), [T, T]), ((70, 80), [T, T, S, D])])
def test_tags_used_up(B, n, bc):
    """Room for two solves of 12 iterations: the third starts on cleared words."""
    geo = geometry(n, bc)
    ref, want = problem(B, geo)
    ref.steady_solve(want, init=False, allow_not_converged=True)
    prob, e = problem(B, geo)
    first = e.clone()
    prob.steady_solve(first, init=False, allow_not_converged=True)   # words hold tags of earlier solves
    give_up(B, prob, TAGS)
    prob.steady_solve(e, init=False, allow_not_converged=True)
    assert give_up(B, prob, 0) == [0, 0]
    assert torch.equal(e, want) and torch.equal(first, want)
