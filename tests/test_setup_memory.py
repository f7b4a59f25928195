"""Set-up in too little memory: an error from the C entry, not an exception
through it (which would end the process).  The call runs in a process of its
own whose address space is limited first."""
import os
import subprocess
import sys

import pytest

COMMON = r"""
import ctypes as C, resource, sys
import numpy as np
import bte_inputs as I
from paper_2306_14181_amd import bte
lib = bte.load()
b = {k: np.ascontiguousarray(v) for k, v in I.bands(7, 2, 1e-12, 1e-10).items()}
m = bte.Material()
m.n_bands, m.n_theta, m.n_phi, m.T_ref, m.material_dim = 2, 4, 4, 300.0, 3
m.C, m.v, m.tau = [b[k].ctypes.data_as(C.POINTER(C.c_double)) for k in ("C", "v", "tau")]
ctl = bte.Control()
ctl.precision, ctl.limiter = bte.F64, bte.LIM_NONE
h = C.c_void_p()

def limit(more):
    used = int(open("/proc/self/statm").read().split()[0]) * resource.getpagesize()
    resource.setrlimit(resource.RLIMIT_AS, (used + more, used + more))
"""

MESH = COMMON + r"""
mesh, keep = bte.mesh_struct(I.mesh2d(3, 120, 120, 1e-6, 1e-6))
ctl.scheme = bte.SEQUENTIAL
limit(int(sys.argv[1]) << 20)
st = lib.bte_mesh_setup(C.byref(mesh), C.byref(m), C.byref(ctl), C.byref(h))
assert st == 1 and b"memory" in lib.bte_mesh_last_error(h), st
assert lib.bte_mesh_bind(h, C.c_void_p(4096), C.c_size_t(1 << 40)) == 7
lib.bte_mesh_destroy(h)
print("refused")
"""

GRID = COMMON + r"""
g, keep = bte._geometry_struct(dict(dim=3, n=[300, 300, 300], len=[1e-6] * 3, bc=[I.BC_THERMAL] * 6, bcT=[300.0] * 6,
                                    pdT=[0.0] * 3, solid=None, pore_bc=I.BC_DIFFUSE))
arr = (bte.Geometry * 1)(g)
ctl.scheme = bte.SYNTHETIC
limit(int(sys.argv[1]) << 20)
st = lib.bte_setup(arr, 1, C.byref(m), C.byref(ctl), C.byref(h))
assert st == 1 and b"memory" in lib.bte_last_error(h), st
assert lib.bte_bind(h, C.c_void_p(4096), C.c_size_t(1 << 40)) == 7
lib.bte_destroy(h)
print("refused")
"""


@pytest.mark.parametrize("code,mb", [(MESH, 130), (MESH, 200), (GRID, 100), (GRID, 600)],
                         ids=["mesh130", "mesh200", "grid100", "grid600"])
def test_refused(code, mb):
    r = subprocess.run([sys.executable, "-c", code, str(mb)], capture_output=True, text=True, timeout=300,
                       env=dict(os.environ, MALLOC_ARENA_MAX="1"))
    assert r.returncode == 0 and "refused" in r.stdout, (r.returncode, r.stderr[-500:])
