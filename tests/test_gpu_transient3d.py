"""The explicit step by 2 x 2 columns (k_transient3d_quad) at the edges of its
split: even and odd widths and depths (the last pair starts one column early),
two columns only, one to a few planes and more than the 64 of a record run,
pores, every wall kind, periodic axes with a temperature drop; enough lanes that
the wavefronts fill the chip, the last chunk not full.  Two steps against the
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
@pytest.mark.parametrize("n,bc,lim,nl", [((8, 8, 6), WALLS, 1, 70), ((7, 8, 5), WALLS, 0, 70), ((9, 7, 3), PERIODIC, 2, 50),
                                         ((5, 6, 70), PERIODIC, 1, 120), ((2, 2, 4), WALLS, 1, 250),
                                         ((18, 3, 1), WALLS, 0, 70), ((3, 19, 2), PERIODIC, 0, 60)])
def test_steps(B, prec, n, bc, lim, nl):
    f64 = prec == "f64"
    nc = int(np.prod(n))
    # 2 x 2 columns x 8 octants x chunks of 64 lanes: at least 4096 wavefronts
    quads = -(-n[0] // 2) * -(-n[1] // 2) * 8
    nphi = 1
    while quads * -(-(2 * nphi * nl + 63) // 64) < 4300:
        nphi += 1
    solid = np.ones(nc, dtype=np.uint8)
    if nc > 40:
        solid[(np.arange(nc) * 7919) % 23 == 5] = 0
    h = 20e-9
    g = dict(dim=3, n=list(n), len=[m * h for m in n], bc=bc, bcT=[301.0, 300.0, 299.5, 300.0, 299.0, 300.0],
             pdT=[0.7 if b == P else 0.0 for b in bc[::2]], solid=solid, pore_bc=D)
    mat = I.bands(17, nl, 1e-12, 1e-10)
    mat.update(n_theta=2, n_phi=nphi, Tref=300.0)
    gam, src = 1e11 * np.abs(I.random_field(1, nc)), 1e16 * np.abs(I.random_field(2, nc))
    dt = 2e-13
    prob = B.Problem(g, mat, dict(precision=B.F64 if f64 else B.F32, limiter=lim, dt=dt))
    prob.set_fields(torch.as_tensor(src, device="cuda"), torch.as_tensor(gam, device="cuda"))
    case = O.Case(g, mat, P=src, gamma=gam, limiter=lim)
    c4 = mat["C"] / (4 * np.pi)
    e0 = (I.random_field(3, nc * case.na).reshape(nc, case.na, 1) * c4 * solid[:, None, None]).reshape(-1)
    e = torch.as_tensor(e0, device="cuda").to(prob.dtype)
    ref = O.transient(case, e.double().cpu().numpy(), 2, dt, 0.0, (1e-12, 2e-12))[0]
    prob.transient_step(e, 2, 0.0, (1e-12, 2e-12))
    assert np.abs(e.double().cpu().numpy() - ref).max() <= (1e-11 if f64 else 1e-5) * np.abs(ref).max()
