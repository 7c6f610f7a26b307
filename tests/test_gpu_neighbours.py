"""Rows (Phi indices) of every face against the oracle's breadth-first search, bit for bit,
over every dimension and path radius: windows of one and of two lines per lane, several
faces per wave, windows wider than the box, bodies that block paths, Neumann EB faces."""

import numpy as np
import pytest

import cutgeom as cg
import oracle

pytest.importorskip("torch")
import paper_1411_4283_amd as cc  # noqa: E402
from test_gpu_parity import _host  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,R,n,shape,bc", [
    (2, 1, 7, cg.ball_outside((0.5, 0.45), 0.3), "dirichlet"),
    (2, 2, 33, cg.star2_outside((0.5, 0.5), 0.25, 0.05, 6), "neumann"),
    (2, 3, 3, cg.halfspace((0.3, 1.0), 0.4), "dirichlet"),
    (2, 4, 21, cg.ball_inside((0.52, 0.48), 0.4), "dirichlet"),
    (3, 1, 9, cg.ball_outside((0.5, 0.45, 0.55), 0.3), "neumann"),
    (3, 2, 11, cg.ball_inside((0.5, 0.52, 0.49), 0.45), "dirichlet"),
    (3, 3, 14, cg.ball_outside((0.5, 0.45, 0.55), 0.3), "dirichlet"),
    (3, 3, 5, cg.halfspace((0.2, 0.1, 1.0), 0.75), "dirichlet"),
    (3, 4, 4, cg.halfspace((0.1, 0.05, 1.0), 0.62), "dirichlet"),
    (3, 4, 5, cg.halfspace((1.0, 0.02, 0.05), 0.87), "neumann"),
])
def test_rows_of_every_face(D, R, n, shape, bc):
    g = cg.make_geometry(shape, n, 2)
    st = cc.Builder(cc.DeviceGeometry.from_host(g, "cuda"), R, eb_bc=bc).build()
    en = oracle.enumerate_geometry(g)
    rp, col, _, _ = _host(st)
    assert st.sizes.n_face == en.n_face and len(rp) == en.n_face + 1
    first_eb = en.n_face - en.n_eb
    for f in range(en.n_face):
        ref = oracle.neighbours(en, f, R)
        if bc == "neumann" and f >= first_eb:
            ref = np.array([en.n_vol + f - first_eb])
        assert np.array_equal(col[rp[f]:rp[f + 1]], ref), f
    print(f"[gpu] D{D} R{R} n{n}: {en.n_face} faces, {np.diff(rp).min()}..{np.diff(rp).max()} rows")


@pytest.mark.parametrize("D,R,n", [(2, 2, 460), (2, 3, 640), (3, 2, 60), (3, 1, 64)])
def test_rows_where_a_wave_takes_many_faces(D, R, n):
    """Grids with so many faces that a wave takes chunks of 32 or 64 of them, several at a
    time: all faces of seeded stretches of 64 and of the last ones, and every face's count
    through the row pointers of a build (rows ascending, in range)."""
    g = cg.make_geometry(cg.ball_outside((0.48, 0.53, 0.51)[:D], 0.31), n, 2)
    st = cc.Builder(cc.DeviceGeometry.from_host(g, "cuda"), R).build()
    en = oracle.enumerate_geometry(g)
    rp, col, _, _ = _host(st)
    assert st.sizes.n_face == en.n_face and en.n_face > 262144
    inner = np.ones(len(col), bool)
    inner[rp[:-1]] = False
    assert col.min() >= 0 and col.max() < st.sizes.n_phi
    assert np.all(np.diff(col.astype(np.int64))[inner[1:]] > 0)
    starts = 64 * np.random.default_rng(n).choice(en.n_face // 64, 25, replace=False)
    eb = np.arange(en.n_face - en.n_eb, en.n_face)
    for f in np.concatenate([*(np.arange(a, a + 64) for a in starts), eb[:64], eb[-64:]]):
        assert np.array_equal(col[rp[f]:rp[f + 1]], oracle.neighbours(en, int(f), R)), f
