"""One-dimensional geometries (bte_line.hip) at the edges of their split: lines
of one to three cells, lengths around a thread's run of 4 cells, a block's
round of 256 cells and a step's tile, several rounds, ragged lane groups, pores, every wall kind, periodic lines
with a temperature drop, batches.  Two source iterations of the sequential
scheme and three explicit steps against the oracle, FP64 1e-11 and FP32 1e-5
of the largest magnitude."""
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


def line(n, ends, pores):
    solid = np.ones(n, dtype=np.uint8)
    if pores:
        solid[(np.arange(n) * 7919) % 17 == 5] = 0
    return dict(dim=1, n=[n, 1, 1], len=[n * 20e-9, 1.0, 1.0], bc=list(ends) + [S] * 4,
                bcT=[301.0, 299.0, 300, 300, 300, 300], pdT=[0.7 if ends[0] == P else 0.0, 0.0, 0.0], solid=solid,
                pore_bc=D)


def problem(B, lines, nl, nt, **ctl):
    mat = I.bands(17, nl, 1e-12, 1e-10)
    mat.update(n_theta=nt, n_phi=1, Tref=300.0)
    nc = sum(g["n"][0] for g in lines)
    src, gam = 1e16 * np.abs(I.random_field(2, nc)), 1e11 * np.abs(I.random_field(1, nc))
    prob = B.Problem(lines, mat, ctl)
    prob.set_fields(torch.as_tensor(src, device="cuda"), torch.as_tensor(gam, device="cuda"))
    cases, c0 = [], 0
    for g in lines:
        c1 = c0 + g["n"][0]
        cases.append(O.Case(g, mat, P=src[c0:c1], gamma=gam[c0:c1], limiter=ctl.get("limiter", 0)))
        c0 = c1
    solid = np.concatenate([g["solid"] for g in lines])
    c4 = mat["C"] / (4 * np.pi)
    e = (I.random_field(3, nc * cases[0].na).reshape(nc, -1, 1) * c4 * solid[:, None, None]).reshape(-1)
    e = torch.as_tensor(e, device="cuda").to(prob.dtype)
    host = e.double().cpu().numpy()
    cut = np.cumsum([0] + [c.size for c in cases])
    return prob, cases, e, [host[a:b].copy() for a, b in zip(cut[:-1], cut[1:])]


LINES = [([1], (T, S), 0), ([2], (P, P), 1), ([3], (D, T), 2), ([4], (P, P), 0), ([61], (S, D), 0), ([255], (T, D), 1),
         ([257], (P, P), 2), ([700], (D, S), 0), ([5, 64, 33], (T, T), 0)]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("ns,ends,lim", LINES + [([3, 63, 64, 65, 130, 1, 9, 40] * 8, (T, D), 0)])
def test_sweep(B, prec, ns, ends, lim):
    f64 = prec == "f64"
    # 21 lanes an octant (two groups of 16), 77 in the batch of 64 lines (five)
    prob, cases, e, host = problem(B, [line(n, ends, n > 8) for n in ns], 7, 11 if len(ns) > 8 else 3, limiter=lim,
                                   precision=B.F64 if f64 else B.F32, scheme=B.SEQUENTIAL, max_iter=2,
                                   residual_temp=0.0, residual_flux=0.0)
    st = prob.steady_solve(e, init=False, allow_not_converged=True)
    assert st["iters"] == 2
    ref = np.concatenate([O.steady(c, scheme=0, tol_T=0.0, tol_q=0.0, max_iter=2, e=h)[0] for c, h in zip(cases, host)])
    assert np.abs(e.double().cpu().numpy() - ref).max() <= (1e-11 if f64 else 1e-5) * np.abs(ref).max()


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("ns,ends,lim", LINES)
def test_steps(B, prec, ns, ends, lim):
    f64 = prec == "f64"
    dt = 2e-13
    for tile in (4, 16, 64):
        prob, cases, e, host = problem(B, [line(n, ends, n > 8) for n in ns], 7, 11, limiter=lim, dt=dt,
                                       precision=B.F64 if f64 else B.F32)
        prob.set_tiles(B.TUNE_TRANSIENT, (tile, 1, 1))
        prob.transient_step(e, 3, 0.0, (1e-12, 2e-12))
        ref = np.concatenate([O.transient(c, h, 3, dt, 0.0, (1e-12, 2e-12))[0] for c, h in zip(cases, host)])
        assert np.abs(e.double().cpu().numpy() - ref).max() <= (1e-11 if f64 else 1e-5) * np.abs(ref).max(), tile


def test_autotune_times_the_sweep_that_runs(B):
    # without an adjoint the forward sweep, which has no tiles; the transposed sweep of 1000 cells x 1280 lanes takes
    # 13 times as long
    prob, _, e, _ = problem(B, [line(1000, (T, T), False)], 20, 64, precision=B.F64, scheme=B.SEQUENTIAL, max_iter=50,
                            residual_temp=0.0, residual_flux=0.0)
    ent = [x for x in prob.autotune(reps=20) if x["kind"] == B.TUNE_SWEEP]
    prob.steady_solve(e, init=False, allow_not_converged=True)
    st = prob.steady_solve(e, init=False, allow_not_converged=True)
    assert len(ent) > 1 and sum(x["chosen"] for x in ent) == 1
    assert max(x["ms"] for x in ent) < 4.0 * st["ms_sweep"] / st["iters"], (ent, st["ms_sweep"] / st["iters"])
