"""Both forms of the 3D explicit step: the shapes of test_gpu_transient3d.py, most
of whose cells lie at walls and pores, by 2 x 2 columns and column by column,
and the form that the rule takes."""
import types

import numpy as np
import pytest

import bte_inputs as I
from tests import test_gpu_transient3d as base

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

T, S, P = I.BC_THERMAL, I.BC_SPECULAR, I.BC_PERIODIC
SHAPES = [m for m in base.test_steps.pytestmark if m.args[0] == "n,bc,lim,nl"][0].args[1]


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2306_14181_amd import bte
    bte.load()
    return bte


@pytest.mark.parametrize("quads", [1, 0])
@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n,bc,lim,nl", SHAPES)
def test_steps(B, prec, n, bc, lim, nl, quads):
    def problem(*args):
        p = B.Problem(*args)
        took = B.load().bte_internal_quads(p._h, quads)
        assert took == quads
        return p
    base.test_steps(types.SimpleNamespace(Problem=problem, F64=B.F64, F32=B.F32), prec, n, bc, lim, nl)


# 2 x 2 columns in (FP32, FP64 unlimited, FP64 limited)
@pytest.mark.parametrize("bc,pores,want", [([P, P, P, P, T, T], 0.0, (1, 1, 1)), ([T, T, S, S, S, S], 0.0, (1, 1, 0)),
                                           ([T, T, S, S, S, S], 0.02, (1, 1, 0)), ([T, T, S, S, S, S], 0.1, (0, 0, 0)),
                                           ([T, T, S, S, S, S], 0.3, (0, 0, 0))])
def test_rule(B, bc, pores, want):
    n = (26, 26, 4)
    solid = (np.random.default_rng(1).random(n[0] * n[1] * n[2]) >= pores).astype(np.uint8)
    g = dict(dim=3, n=list(n), len=[20e-9 * m for m in n], bc=bc, bcT=[300.0] * 6, pdT=[0.0] * 3, solid=solid,
             pore_bc=I.BC_DIFFUSE)
    mat = I.bands(2, 8, 1e-12, 1e-10)
    mat.update(n_theta=4, n_phi=8, Tref=300.0)
    got = []
    for prec, lim in ((B.F32, B.LIM_MC), (B.F64, B.LIM_NONE), (B.F64, B.LIM_MC)):
        p = B.Problem(g, mat, dict(precision=prec, limiter=lim, dt=1e-13))
        got.append(B.load().bte_internal_quads(p._h, -1))
    assert tuple(got) == want
