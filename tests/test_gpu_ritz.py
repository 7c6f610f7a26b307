"""Ritz values at depths around the 64 steps between two reads of the coefficients, through
the volume matrix and through the faces, and with inner solves: converged ones against the
eigenvalues of the dense matrix."""

import numpy as np
import pytest

import cutgeom as cg

torch = pytest.importorskip("torch")
import paper_1411_4283_amd as cc  # noqa: E402

pytestmark = pytest.mark.gpu

CONVERGED = 1e-9


def _dense(st, lap):
    n = st.sizes.n_vol
    ptr, col, val = lap.row_ptr.cpu().numpy(), lap.col.cpu().numpy(), lap.val.cpu().numpy()
    A = np.zeros((n, st.sizes.n_phi))
    for v in range(n):
        A[v, col[ptr[v]:ptr[v + 1]]] = val[ptr[v]:ptr[v + 1]]
    return A[:, :n]


@pytest.mark.parametrize("mode,steps,least", [(0, 1, 0), (0, 20, 2), (0, 63, 10), (0, 64, 10), (0, 65, 10),
                                              (0, 128, 30), (0, 129, 30), (0, 150, 50), (1, 1, 0), (1, 40, 3)])
def test_depths_around_the_batch(mode, steps, least):
    """A converged value (residual estimate below 1e-9) is within cond(eigenvectors) times its
    residual of an eigenvalue (Bauer and Fike), with n eps |A| for the rounding of the steps."""
    g = cg.make_geometry(cg.ball_outside((0.47, 0.52), 0.27), 14, 2)
    st = cc.Builder(cc.DeviceGeometry.from_host(g, "cuda"), 2).build()
    lap = cc.build_laplacian(st)
    A = _dense(st, lap)
    n = len(A)
    assert n > 150
    B = A if mode == 0 else np.linalg.inv(A)
    ev, vec = np.linalg.eig(B)
    kappa, size = np.linalg.cond(vec), np.linalg.norm(B, 2)
    for use in (lap, None):
        theta, res, ok = cc.ritz(st, mode, steps, use, inner_rtol=1e-12)
        assert len(theta) == steps and ok
        theta = theta if mode == 0 else 1.0 / theta
        conv = theta[res < CONVERGED]
        print(f"mode {mode}, {steps} steps: {len(conv)} converged", flush=True)
        assert len(conv) >= least
        slack = n * 2.2e-16 * size if mode == 0 else 1e-12 * np.linalg.cond(A) * size
        for t in conv:
            assert np.abs(ev - t).min() <= kappa * (CONVERGED * abs(t) + slack), (t, np.abs(ev - t).min())
