"""Stencils of one face of every row count that a small geometry has: from as many rows as
monomials to the 128-row limit, on both sides of 64 rows, where a lane starts to hold two
rows, and with row counts that are no multiple of the eights the kernels read them in."""

import numpy as np
import pytest

import cutgeom as cg
import oracle

pytest.importorskip("torch")
import paper_1411_4283_amd as cc  # noqa: E402
from test_gpu_parity import _host  # noqa: E402

pytestmark = pytest.mark.gpu

BAR = 1e-11   # of the largest entry of the stencil, as everywhere: cond(B) eps at the routing bound


@pytest.mark.parametrize("D,Q,R,n,bc", [(2, 2, 2, 12, "dirichlet"), (2, 2, 4, 20, "dirichlet"),
                                        (2, 4, 3, 16, "neumann"), (2, 4, 4, 24, "dirichlet"),
                                        (3, 2, 2, 8, "neumann"), (3, 2, 3, 14, "dirichlet"),
                                        (3, 4, 3, 14, "dirichlet"), (3, 4, 3, 16, "neumann")])
def test_one_face_of_every_row_count(D, Q, R, n, bc):
    shape = cg.ball_outside((0.47, 0.52, 0.55)[:D], 0.27)
    g = cg.make_geometry(shape, n, Q)
    st = cc.Builder(cc.DeviceGeometry.from_host(g, "cuda"), R, eb_bc=bc).build()
    en = oracle.enumerate_geometry(g)
    rp, col, val, status = _host(st)
    counts = np.diff(rp)
    M = cc.api.n_monomials(D, Q)
    faces = {}
    for f in np.flatnonzero(counts >= M):
        faces.setdefault(int(counts[f]), int(f))
    worst, seen = 0.0, []
    for N, f in sorted(faces.items()):
        idx, s, so = oracle.face_stencil(g, en, f, R, eb_bc=bc)
        a, e = rp[f], rp[f + 1]
        assert np.array_equal(col[a:e], idx) and status[f] == so
        if so != oracle.STATUS_OK:
            continue
        err = np.abs(val[a:e] - s).max() / np.abs(s).max()
        assert err <= BAR, (f, N, err)
        worst, seen = max(worst, err), seen + [N]
    print(f"[gpu] D{D} Q{Q} R{R}: rows {seen[0]}..{seen[-1]} ({len(seen)} counts), worst rel err {worst:.2e}")
    if (D, R) == (3, 3):
        assert seen[0] <= 64 < seen[-1]


@pytest.mark.parametrize("D,Q,R,n", [(2, 2, 4, 14), (2, 4, 3, 14), (3, 2, 2, 8), (3, 4, 3, 12)])
def test_rows_of_many_small_cells(D, Q, R, n):
    """A layer of slivers (kappa below 1e-3, their box faces as small): faces with one small
    row and with more than are formed at a time, volume and box-face rows among them, in the
    first 64 rows and past them."""
    shape = cg.halfspace((1.0, 0.0, 0.0)[:D], 0.5 - 2e-5)
    g = cg.make_geometry(shape, n, Q)
    st = cc.Builder(cc.DeviceGeometry.from_host(g, "cuda"), R).build()
    en = oracle.enumerate_geometry(g)
    rp, col, val, status = _host(st)
    kappa = np.concatenate([g.vol_mom[en.vol_cell, 0], g.eb_mom[:, 0]] +
                           [[g.face_mom[d][f, 0]] for d, f in zip(en.box_dir, en.box_face)])
    small = np.array([(kappa[col[rp[f]:rp[f + 1]]] < 1e-3).sum() for f in range(en.n_face)])
    M = cc.api.n_monomials(D, Q)
    ok = np.diff(rp) >= M
    assert small[ok].max() > 8
    faces = [int(np.flatnonzero(ok & (small == s))[0]) for s in np.unique(small[ok]) if s > 0]
    faces += [int(f) for f in np.flatnonzero(ok & (small > 0))[:: max(1, int((small > 0).sum()) // 25)]]
    worst = 0.0
    for f in faces:
        idx, s, so = oracle.face_stencil(g, en, f, R)
        a, e = rp[f], rp[f + 1]
        assert np.array_equal(col[a:e], idx) and status[f] == so, f
        if so != oracle.STATUS_OK:
            continue
        err = np.abs(val[a:e] - s).max() / np.abs(s).max()
        assert err <= BAR, (f, int(small[f]), err)
        worst = max(worst, err)
    print(f"[gpu] D{D} Q{Q}: {len(faces)} faces of up to {small.max()} small rows, worst rel err {worst:.2e}")
