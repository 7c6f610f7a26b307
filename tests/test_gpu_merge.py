"""The volume matrix on made-up face rows, which reach what no geometry does: merged rows of
up to 1,024 entries (the large hash table), rows longer than the 128 a wave loads at once,
disjoint and identical rows, empty ones, and columns that collide in the table."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
import paper_1411_4283_amd as cc  # noqa: E402
from paper_1411_4283_amd._lib import Sizes  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,rows,span,stride", [(2, 41, 90, 1), (2, 1, 3, 1), (3, 88, 140, 1), (3, 64, 600, 1),
                                                (3, 65, 10**6, 1), (3, 128, 10**6, 1024), (3, 146, 2000, 1),
                                                (2, 204, 4000, 1), (3, 0, 1, 1)])
def test_merge_of_made_up_rows(D, rows, span, stride):
    rng = np.random.default_rng(D * 1000 + rows)
    S, n_vol = 2 * D + 1, 70
    n_face = S * n_vol
    n_phi = span * stride + 8
    lens = np.where(rng.random(n_face) < 0.1, 0, np.minimum(rows, span))
    ptr = np.concatenate([[0], np.cumsum(lens)])
    col = np.concatenate([np.sort(rng.choice(span, k, replace=False)) * stride for k in lens] or [[]]).astype(np.int32)
    val = rng.standard_normal(len(col))
    vf = rng.permutation(n_face).reshape(n_vol, S).astype(np.int32)
    vf[rng.random(vf.shape) < 0.1] = -1
    scale = rng.uniform(0.5, 2.0, n_vol)

    def t(a, dt):
        return torch.from_numpy(np.concatenate([a, [0]]) if len(a) == 0 else np.ascontiguousarray(a)).to("cuda", dt)

    z = Sizes()
    z.n_vol, z.n_phi, z.n_face, z.nnz, z.n_geom = n_vol, n_phi, n_face, len(col), 1
    i64 = torch.int64
    st = cc.Stencils(dim=D, sizes=z, row_ptr=t(ptr, i64), col=t(col, torch.int32), val=t(val, torch.float64),
                     status=t(np.zeros(n_face), torch.int8), vol_face=t(vf.ravel(), torch.int32),
                     vol_scale=t(scale, torch.float64), phi_off=t(np.array([0, n_phi]), i64),
                     vol_off=t(np.array([0, n_vol]), i64), face_off=t(np.array([0, n_face]), i64))
    lap = cc.build_laplacian(st)
    lp, lc, lv = lap.row_ptr.cpu().numpy(), lap.col.cpu().numpy(), lap.val.cpu().numpy()
    longest = 0
    for v in range(n_vol):
        acc = {}
        for k in range(S):
            if vf[v, k] >= 0:
                sg = -1.0 if k < 2 * D and k % 2 == 0 else 1.0
                for j in range(ptr[vf[v, k]], ptr[vf[v, k] + 1]):
                    acc[col[j]] = acc.get(col[j], 0.0) + sg * val[j]   # the order of the faces
        keys = sorted(acc)
        longest = max(longest, len(keys))
        a, b = lp[v], lp[v + 1]
        assert np.array_equal(lc[a:b], keys)
        assert np.array_equal(lv[a:b], [scale[v] * acc[k] for k in keys])
    print(f"[gpu] merge D{D}: {rows} per row, longest merged row {longest}")
