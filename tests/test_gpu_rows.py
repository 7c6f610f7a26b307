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
