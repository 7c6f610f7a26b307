"""The buckets of the processing order: counts against the rows' histogram, and every face
solved exactly where it belongs (no status or value of a prefilled output left over), on
grids of one cell, of one tile and less, batches whose tiles span geometries, several steps
per workgroup, and with template copies."""

import ctypes

import numpy as np
import pytest

import cutgeom as cg
import oracle

torch = pytest.importorskip("torch")
import paper_1411_4283_amd as cc  # noqa: E402
from paper_1411_4283_amd._lib import load  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,n,Q,R,batch,reuse", [
    (2, 3, 2, 2, 1, False),
    (2, 1, 2, 1, 1, False),
    (2, 17, 2, 3, 3, False),
    (2, 61, 4, 3, 5, True),
    (2, 760, 2, 2, 1, False),       # 2257 tiles' worth of cells: two steps per workgroup
    (3, 7, 2, 2, 5, False),
    (3, 24, 4, 3, 2, True),
])
def test_every_face_has_its_place(D, n, Q, R, batch, reuse):
    geoms = [cg.make_geometry(cg.ball_outside((0.5, 0.47, 0.52)[:D], 0.2 + 0.03 * i), n, Q) for i in range(batch)]
    b = cc.Builder([cc.DeviceGeometry.from_host(g, "cuda") for g in geoms], R, reuse_templates=reuse)
    st = b.build()
    first = st.val[: st.sizes.nnz].clone()
    st.status.fill_(99)
    st.val.fill_(float("nan"))
    b.build(out=st)
    assert int(st.status[: st.sizes.n_face].max()) < 99
    assert torch.equal(st.val[: st.sizes.nnz], first) and bool(torch.isfinite(first).all())
    rows = np.diff(st.row_ptr.cpu().numpy())
    M = {(2, 2): 6, (2, 4): 15, (3, 2): 10, (3, 4): 35}[D, Q]
    solved = rows[rows >= M]
    hist = np.bincount((solved - 1) // 16, minlength=8)
    counts = (ctypes.c_int64 * 8)()
    load().cutcell_last_bin_faces(counts, 8)
    bins, reused = np.array(counts), load().cutcell_last_reused_faces()
    assert bins.sum() + reused == len(solved) and np.all(bins <= hist)
    if not reuse:
        assert reused == 0 and np.array_equal(bins, hist)
    print(f"[gpu] D{D} n{n} x{batch}: bins {bins.tolist()}, copies {reused}, short {int((rows < M).sum())}")


@pytest.mark.parametrize("D,R,n", [(2, 1, 24), (2, 4, 51), (2, 3, 52), (3, 1, 12), (3, 2, 12), (3, 3, 20)])
def test_regular_cells_and_short_scans(D, R, n):
    """Rows of every face against the oracle's search on grids whose inner cells are regular
    out to the path radius, with flag spaces of one to five scan tiles (the one-workgroup
    scan takes up to four) and more."""
    g = cg.make_geometry(cg.ball_outside((0.5, 0.47, 0.52)[:D], 0.15), n, 2)
    st = cc.Builder(cc.DeviceGeometry.from_host(g, "cuda"), R).build()
    en = oracle.enumerate_geometry(g)
    rp, col = st.row_ptr.cpu().numpy(), st.col.cpu().numpy()
    assert st.sizes.n_face == en.n_face
    for f in range(en.n_face):
        assert np.array_equal(col[rp[f]:rp[f + 1]], oracle.neighbours(en, f, R)), f


@pytest.mark.parametrize("batch", [1, 32, 33])
def test_batches_on_both_sides_of_the_argument_limit(batch):
    """Geometries reach the device as a kernel argument (up to 32) or by a copy: a batch's
    stencils are those of its geometries built alone, bit for bit."""
    geoms = [cg.make_geometry(cg.ball_outside((0.5, 0.48), 0.2 + 0.004 * i), 9, 2) for i in range(batch)]
    dev = [cc.DeviceGeometry.from_host(g, "cuda") for g in geoms]
    st = cc.Builder(dev, 2).build()
    val, rows, phi = [], [], 0
    for d in dev:
        s = cc.Builder(d, 2).build()
        val.append(s.val[: s.sizes.nnz])
        rows.append(s.col[: s.sizes.nnz] + phi)
        phi += s.sizes.n_phi
    assert torch.equal(st.val[: st.sizes.nnz], torch.cat(val))
    assert torch.equal(st.col[: st.sizes.nnz], torch.cat(rows).to(st.col.dtype))
    assert int(st.phi_off[-1]) == phi
