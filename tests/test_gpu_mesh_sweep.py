"""The per-direction mesh sweep (k_mesh_sweep_dir) where its split can go wrong:
band counts with one, two and four bands per thread, groups of bands that do
not divide the count, few and many directions, steps with empty places, a
state that is not aligned for vector accesses, and a mesh whose live
increments do not fit the LDS (a launch per level).  Two source iterations
against the oracle, FP64 1e-11 and FP32 1e-5 of the largest magnitude as in
test_gpu_mesh.py."""
import numpy as np
import pytest

import bte_inputs as I
from oracle import mesh as M
from tests.helpers import rel_err

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2306_14181_amd import bte
    bte.load()
    return bte


def material(nl, nt, nphi):
    m = I.bands(31, nl, 1e-12, 1e-10)
    m.update(n_theta=nt, n_phi=nphi, Tref=300.0)
    return m


def check(B, mesh, mat, prec, offset=0, iters=2):
    case = (M.TetMeshCase if "xyz" in mesh else M.MeshCase)(mesh, mat)
    prob = B.MeshProblem(mesh, mat, dict(precision=prec, max_iter=iters, residual_temp=0.0))
    rng = np.random.default_rng(5)
    e0 = case.C4 * rng.uniform(-1, 1, (case.nc, case.na, 1))
    room = torch.zeros(prob.n_unknowns + 8, dtype=prob.dtype, device="cuda")
    eg = room[offset:offset + prob.n_unknowns]
    eg.copy_(torch.as_tensor(e0.reshape(-1)))
    e = eg.double().cpu().numpy()
    prob.steady_solve(eg, init=False, allow_not_converged=True)
    for _ in range(iters):
        e = M.sweep(case, e, M.moments(case, e)[1] - case.Tref)
    assert rel_err(eg.double().cpu().numpy(), e) < (1e-11 if prec == B.F64 else 1e-5)
    assert not room[:offset].any() and not room[offset + prob.n_unknowns:].any()


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("nl,nt,nphi,offset", [(1, 1, 1, 0), (2, 1, 2, 1), (3, 2, 2, 0), (4, 1, 1, 0), (5, 1, 3, 0),
                                               (6, 2, 2, 1), (7, 1, 1, 3), (12, 1, 2, 2), (20, 2, 2, 0), (20, 2, 2, 1),
                                               (36, 1, 1, 0)])
def test_bands_and_directions(B, prec, nl, nt, nphi, offset):
    mesh = I.mesh2d(41, 7, 6, 7 * 60e-9, 6 * 50e-9, jitter=0.3, quad_frac=0.4, bcT=(301.0, 299.0, 300.5, 299.5))
    check(B, mesh, material(nl, nt, nphi), B.F64 if prec == "f64" else B.F32, offset)


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_tetrahedra(B, prec):
    mesh = I.mesh3d(42, 3, 4, 3, 3 * 60e-9, 4 * 50e-9, 3 * 55e-9)
    check(B, mesh, material(10, 1, 2), B.F64 if prec == "f64" else B.F32)


def test_wide_front(B):
    """20 000 islands of two squares: every first cell's increment is live until the second cells' step."""
    n, h = 20000, 50e-9
    xy = np.array([[x, y] for x in (0.0, h, 2 * h) for y in (0.0, h)])
    xy = (xy[None] + np.stack([np.arange(n) % 200, np.arange(n) // 200], 1)[:, None, :] * 5 * h).reshape(-1, 2)
    one = np.array([[0, 2, 3, 1], [2, 4, 5, 3]])
    vtx = (one.reshape(-1)[None] + 6 * np.arange(n)[:, None]).reshape(-1)
    tag = np.tile([0, -1, 0, 0, 0, 0, 0, -1], n)
    mesh = dict(xy=xy, cell_ptr=4 * np.arange(2 * n + 1), cell_vtx=vtx, edge_tag=tag, tag_bc=[I.BC_THERMAL], tag_T=[301.0])
    check(B, mesh, material(2, 1, 1), B.F64, iters=1)
