"""The workspace-size functions (host code): they answer 0, and never end the process, for
options that every other call refuses."""

import subprocess
import sys

import pytest

CALL = """
import ctypes
from paper_1411_4283_amd import _lib
from paper_1411_4283_amd.api import make_opts
lib = _lib.load()
o = make_opts({dim}, {n}, 0.25, 2, 2)
sizes = _lib.Sizes(n_vol=10, n_eb=0, n_box=4, n_phi=14, n_face=20, nnz=100, max_rows=5, n_geom=1)
print(lib.cutcell_workspace_bytes(ctypes.byref(o), 1),
      lib.cutcell_backward_workspace_bytes(ctypes.byref(o), ctypes.byref(sizes)))
"""


@pytest.mark.parametrize("dim,n", [(2, (-4, 4)), (2, (4, 0)), (2, (-4, -4)), (3, (4, 4, 0)), (3, (4, -4, 4))])
def test_grids_without_cells_need_no_workspace(dim, n):
    """A grid with an extent below 1, in a process of its own: the answer is 0 and the process lives."""
    r = subprocess.run([sys.executable, "-c", CALL.format(dim=dim, n=n)], capture_output=True, text=True)
    assert r.returncode == 0, (r.returncode, r.stderr)
    assert r.stdout.split() == ["0", "0"]
