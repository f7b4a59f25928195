"""Long strips.  Workspace of a mesh problem, from the host set-up: a table entry per
(direction, cell) beside the arrays of the state's size, whatever the mesh's
shape.  Long strips have thousands of sweep steps of a few cells each."""
import ctypes as C

import numpy as np
import pytest

import bte_inputs as I


@pytest.mark.parametrize("nx,ny,nl", [(24, 24, 1), (1000, 4, 1), (3000, 1, 1), (1000, 4, 20), (1, 800, 3)])
@pytest.mark.parametrize("prec", [0, 1])
def test_strips(nx, ny, nl, prec):
    from paper_2306_14181_amd import bte
    lib = bte.load()
    mesh, keep = bte.mesh_struct(I.mesh2d(3, nx, ny, nx * 20e-9, ny * 20e-9))
    b = {k: np.ascontiguousarray(v) for k, v in I.bands(7, nl, 1e-12, 1e-10).items()}
    m = bte.Material()
    m.n_bands, m.n_theta, m.n_phi, m.T_ref, m.material_dim = nl, 2, 4, 300.0, 3
    m.C, m.v, m.tau = [b[k].ctypes.data_as(C.POINTER(C.c_double)) for k in ("C", "v", "tau")]
    ctl = bte.Control()
    ctl.precision, ctl.scheme, ctl.limiter = prec, bte.SEQUENTIAL, bte.LIM_NONE
    h = C.c_void_p()
    assert lib.bte_mesh_setup(C.byref(mesh), C.byref(m), C.byref(ctl), C.byref(h)) == 0, lib.bte_mesh_last_error(h)
    nc, na = lib.bte_mesh_num_cells(h), lib.bte_mesh_num_directions(h)
    size = lib.bte_mesh_workspace_bytes(h)
    lib.bte_mesh_destroy(h)
    # 64 bytes of schedule per (direction, cell), gradients (two) and residual, and per cell the
    # geometry: at most 4 faces of 92 bytes, 24 stencil neighbours of 28 bytes, 110 bytes of scalars
    assert size < nc * na * (64 + 3 * nl * (8 if prec else 4)) + nc * 1200 + 40 * 256 + 64 * na


@pytest.mark.gpu
@pytest.mark.parametrize("nx,ny,nl", [(300, 1, 1), (2, 150, 20)])
def test_sweep_of_strips(nx, ny, nl):
    """Many steps of few cells against the oracle, two source iterations as in test_gpu_mesh_sweep.py."""
    import torch

    from paper_2306_14181_amd import bte
    from tests.test_gpu_mesh_sweep import check, material
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    mesh = I.mesh2d(6, nx, ny, nx * 40e-9, ny * 40e-9, bcT=(301.0, 299.0, 300.5, 299.5))
    check(bte, mesh, material(nl, 1, 2), bte.F64)
