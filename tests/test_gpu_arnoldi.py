"""The Arnoldi steps of the Poisson solve at the sizes where their tiles change (256, 512,
1,024 and 2,048 elements per block, more tiles than blocks) and at restarts around the
chunks of inner products: the solution against a dense solve (small) and the true residual."""

import numpy as np
import pytest

import cutgeom as cg

torch = pytest.importorskip("torch")
import paper_1411_4283_amd as cc  # noqa: E402

pytestmark = pytest.mark.gpu


def _problem(D, n, Q, R, seed=5):
    g = cg.make_geometry(cg.ball_outside((0.47, 0.52, 0.55)[:D], 0.27), n, Q)
    st = cc.Builder(cc.DeviceGeometry.from_host(g, "cuda"), R).build()
    rng = np.random.default_rng(seed)
    bc = torch.from_numpy(rng.standard_normal(st.sizes.n_phi)).cuda()
    rhs = torch.from_numpy(rng.standard_normal(st.sizes.n_vol) / g.h**2).cuda()
    return st, bc, rhs, cc.build_laplacian(st)


def _residual(st, lap, bc, rhs, x):
    phi = bc.clone()
    phi[: st.sizes.n_vol] = x
    phi0 = bc.clone()
    phi0[: st.sizes.n_vol] = 0.0
    b = rhs - cc.apply_laplacian(lap, phi0)
    return float((rhs - cc.apply_laplacian(lap, phi)).norm() / b.norm())


@pytest.mark.parametrize("restart", [1, 7, 8, 9, 63, 64, 65, 200])
def test_small_problem_at_restarts(restart):
    st, bc, rhs, lap = _problem(2, 20, 2, 2)
    n = st.sizes.n_vol
    iters = 4000 if restart == 1 else 2000
    res = cc.solve(st, bc, rhs, restart=restart, max_iters=iters, rtol=1e-11, lap=lap)
    assert res.iters <= iters
    assert abs(_residual(st, lap, bc, rhs, res.x) - res.relres) <= 1e-13 + 1e-3 * res.relres
    if restart >= 63:
        assert res.converged
        ptr, col, val = lap.row_ptr.cpu().numpy(), lap.col.cpu().numpy(), lap.val.cpu().numpy()
        A = np.zeros((n, st.sizes.n_phi))
        for v in range(n):
            A[v, col[ptr[v]:ptr[v + 1]]] = val[ptr[v]:ptr[v + 1]]
        ref = np.linalg.solve(A[:, :n], rhs.cpu().numpy() - A[:, n:] @ bc.cpu().numpy()[n:])
        assert np.linalg.norm(res.x.cpu().numpy() - ref) <= 1e-7 * np.linalg.norm(ref)
    # the step limit is kept, whatever steps were launched ahead
    few = cc.solve(st, bc, rhs, restart=restart, max_iters=5, rtol=1e-30, lap=lap)
    assert few.iters == 5 and not few.converged


@pytest.mark.parametrize("D,n", [(2, 256), (2, 300), (2, 400), (2, 760), (2, 1300)])
def test_tile_sizes(D, n):
    st, bc, rhs, lap = _problem(D, n, 2, 2)
    one = cc.solve(st, bc, rhs, restart=20, max_iters=60, rtol=1e-9, lap=lap)
    print(f"[gpu] {st.sizes.n_vol} volumes: {one.iters} steps, relres {one.relres:.3e}")
    assert one.iters == 60
    assert abs(_residual(st, lap, bc, rhs, one.x) - one.relres) <= 1e-12
    again = cc.solve(st, bc, rhs, restart=20, max_iters=60, rtol=1e-9, lap=lap)
    assert torch.equal(one.x, again.x)   # deterministic
