"""The transpose on made-up face rows whose row_ptr ends before, at or after the number of
nonzeros in the sizes: every nonzero's face is the last one that starts at or before it, and
nothing past the caller's arrays is written."""

import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_1411_4283_amd import _lib  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_face,rows,extra", [(500, 88, 0), (500, 40, -977), (500, 40, 311), (3, 700, -1500),
                                               (1, 5, 0), (1, 20, -19), (0, 0, 37), (4000, 1, -1)])
def test_faces_of_the_listed_nonzeros(n_face, rows, extra):
    rng = np.random.default_rng(n_face + rows)
    n_phi = 1000
    ptr = np.concatenate([[0], np.cumsum(rng.integers(0, 2 * rows + 1, n_face))]).astype(np.int64)
    if n_face == 1:
        ptr[1] = rows
    nnz = int(ptr[-1]) + extra
    assert nnz > 0
    col = rng.integers(0, n_phi, max(nnz, int(ptr[-1]))).astype(np.int32)
    pad = 4096                      # words past every output that have to stay
    row_ptr, cols = torch.from_numpy(ptr).cuda(), torch.from_numpy(col).cuda()
    z = _lib.Sizes(n_phi=n_phi, n_face=n_face, nnz=nnz, n_geom=1)
    lib = _lib.load()
    need = lib.cutcell_transpose_workspace_bytes(ctypes.byref(z))
    ws = torch.full((need + 4 * pad,), 77, dtype=torch.uint8, device="cuda")
    out = {k: torch.full((n + pad,), -7, dtype=dt, device="cuda")
           for k, n, dt in (("col_ptr", n_phi + 1, torch.int64), ("nz", nnz, torch.int32), ("nz_face", nnz, torch.int32))}
    arr, tr = _lib.StencilArrays(), _lib.TransposeArrays()
    for name in ("val", "status", "vol_face", "vol_scale"):
        setattr(arr, name, ws.data_ptr())     # required, not read
    arr.row_ptr, arr.col = row_ptr.data_ptr(), cols.data_ptr()
    for k, v in out.items():
        setattr(tr, k, v.data_ptr())
    print(f"transpose: {n_face} faces, {nnz} nonzeros, row_ptr ends at {ptr[-1]}", flush=True)
    rc = lib.cutcell_build_transpose(ctypes.byref(z), ctypes.byref(arr), ctypes.byref(tr), ws.data_ptr(), need, None)
    torch.cuda.synchronize()
    assert rc == 0, lib.cutcell_last_error()
    nz = np.argsort(col[:nnz], kind="stable")
    face = np.maximum(np.searchsorted(ptr[:n_face], nz, side="right") - 1, 0)
    got = {k: v.cpu().numpy() for k, v in out.items()}
    assert np.array_equal(got["nz"][:nnz], nz) and np.array_equal(got["nz_face"][:nnz], face)
    assert np.array_equal(got["col_ptr"][: n_phi + 1], np.searchsorted(np.sort(col[:nnz]), np.arange(n_phi + 1)))
    assert all((v[-pad:] == -7).all() for v in got.values()) and bool((ws[need:] == 77).all())
