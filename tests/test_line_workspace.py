"""Workspace of large one-dimensional problems (host set-up, no GPU), and their
sweeps by folded groups of lanes (GPU, against the oracle)."""
import ctypes as C

import numpy as np
import pytest

import bte_inputs as I
from tests.helpers import geo, mat


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n,nfilm,nl,nt", [(200, 100, 200, 128), (200, 1000, 20, 64), (20000, 4, 64, 64), (100, 8000, 8, 16)])
def test_partials(n, nfilm, nl, nt, prec):
    """Beside the state's copy, five FP64 moments per 64 lanes and octant."""
    from paper_2306_14181_amd import bte
    lib = bte.load()
    g = geo(1, (n,), (n * 1e-9,), [I.BC_THERMAL] * 2 + [I.BC_SPECULAR] * 4)
    s, keep = bte._geometry_struct(g)
    arr = (bte.Geometry * nfilm)(*[s] * nfilm)
    m = mat(I.bands(0, nl), nt)
    b = [np.ascontiguousarray(m[k]) for k in ("C", "v", "tau")]
    mm = bte.Material()
    mm.n_bands, mm.n_theta, mm.n_phi, mm.T_ref, mm.material_dim = nl, nt, 1, 300.0, 3
    mm.C, mm.v, mm.tau = [x.ctypes.data_as(C.POINTER(C.c_double)) for x in b]
    ctl = bte.Control()
    ctl.precision = prec
    h = C.c_void_p()
    assert lib.bte_setup(arr, nfilm, C.byref(mm), C.byref(ctl), C.byref(h)) == 0
    size, nel, nc = lib.bte_workspace_bytes(h), lib.bte_num_unknowns(h), lib.bte_num_cells(h)
    lib.bte_destroy(h)
    parts = 2 * -(-nl * nt // 64)
    # fields, tables and work lists: under 1000 bytes a cell; rows of zeros, walls and bands by lane
    assert size < nel * (8 if prec else 4) + nc * (40 * parts + 1000) + 8 * nfilm * nl * nt * 16 + (1 << 20)


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_folded_sweep(prec):
    """200 equal lines of 30 cells x 2 x 9999 lanes against one of them alone, whose blocks are not folded: the same
    arithmetic, but for the order of the moments' sums (2^-53 x 10^4 terms at most)."""
    import torch

    from paper_2306_14181_amd import bte as B
    from tests.test_gpu_line import line
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    m = mat(I.bands(17, 99, 1e-12, 1e-10), 101)
    ctl = dict(precision=B.F64 if prec == "f64" else B.F32, scheme=B.SEQUENTIAL, max_iter=3, residual_temp=0.0,
               residual_flux=0.0)
    lone = line(30, (I.BC_THERMAL, I.BC_DIFFUSE), 1)
    one = B.Problem(lone, m, ctl)
    c4 = np.tile(m["C"] / (4 * np.pi), 202)
    e = (np.random.default_rng(0).uniform(-1, 1, (30, c4.size)) * c4 * lone["solid"][:, None]).reshape(-1)
    e1 = torch.as_tensor(e, device="cuda").to(one.dtype)
    many = B.Problem([lone] * 200, m, ctl)
    em = e1.repeat(200)
    assert many.workspace.numel() < em.numel() * em.element_size() * (1.4 if prec == "f32" else 1.2)
    one.steady_solve(e1, init=False, allow_not_converged=True)
    many.steady_solve(em, init=False, allow_not_converged=True)
    err = (em.view(200, -1) - e1).abs().max().item()
    assert err <= (1e-11 if prec == "f64" else 1e-6) * e1.abs().max().item()
