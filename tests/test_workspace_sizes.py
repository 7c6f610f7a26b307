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


def _al(x):
    return (x + 255) // 256 * 256


def _former_solve(n, n_phi, n_face, m):
    """Bytes that a solve of n volumes with restart m took with 512 partial sums per inner
    product, five vectors and three blocks of coefficients: what callers brought."""
    nv = max(n, 1)
    return (2 * _al(8 * n_phi) + _al(8 * max(n_face, 1)) + 5 * _al(8 * nv) + _al(4 * nv) + _al(8 * nv * (m + 1))
            + _al(8 * 512 * (m + 2)) + _al(8 * (2 * m + 5)) + _al(8 * (m + 1)))


def _former_ritz(n, n_phi, n_face, k, inner):
    nv = max(n, 1)
    return (2 * _al(8 * n_phi) + _al(8 * max(n_face, 1)) + _al(8 * nv) + _al(4 * nv) + _al(8 * nv * (k + 1))
            + _al(8 * 512 * (k + 2)) + _al(8 * (2 * k + 5)) + (_former_solve(n, n_phi, n_face, inner) if inner else 0))


def test_krylov_workspaces_ask_for_no_more_than_they_did():
    """Solves and Ritz values take every buffer of the former size, at the sizes where the
    numbers of tiles and of elements per thread change and for every depth."""
    import ctypes

    from paper_1411_4283_amd import _lib

    lib = _lib.load()
    edges = [256 * t * e for e in (1, 2, 4, 8, 16) for t in (1, 2, 127, 128, 129, 223, 224, 225, 251, 252, 253, 254,
                                                             255, 256, 257, 384, 511, 512, 513)]
    vols = sorted({max(e + d, 0) for e in edges + [0, 30, 100, 3000, 30000, 600000, 2000000] for d in (-1, 0, 1)})
    depths = [1, 2, 3, 7, 8, 9, 20, 63, 64, 65, 100, 400, 1023, 1024]
    for n in vols:
        for n_phi, n_face in ((n, 0), (n + n // 9, 3 * n)):
            z = _lib.Sizes(n_vol=n, n_phi=n_phi, n_face=n_face, n_geom=1)
            for m in depths:
                need = lib.cutcell_solve_workspace_bytes(ctypes.byref(z), m)
                assert 0 < need <= _former_solve(n, n_phi, n_face, m), (n, n_phi, m)
                for inner in (0, 1, 50, 1024):
                    need = lib.cutcell_ritz_workspace_bytes(ctypes.byref(z), m, 1 if inner else 0, inner)
                    assert 0 < need <= _former_ritz(n, n_phi, n_face, m, inner), (n, n_phi, m, inner)
