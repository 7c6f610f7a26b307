"""A build that flags most of its faces: 3D second order at path radius 1, where a regular face
has 12 rows for 10 monomials and no cross terms, so that 70 thousand faces of 32^3 are left to
the Householder QR path and found rank deficient there."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
import cutgeom as cg  # noqa: E402
import oracle  # noqa: E402
import paper_1411_4283_amd as cc  # noqa: E402

pytestmark = pytest.mark.gpu


def test_flagged_faces_and_their_cost():
    """Statuses against the oracle's on a small grid; and the counters of flagged and routed
    faces must not slow down the faces themselves: with QR the build stays below 3 times the
    build without it (both read the same rows and form the same Gram matrices; the QR kernel
    takes about as long as the Gram kernel, and took four times as long while its counter
    shared a cache line with what every face reads)."""
    g = cg.make_geometry(cg.ball_outside((0.5, 0.5, 0.5), 0.3), 10, 2)
    st = cc.Builder(cc.DeviceGeometry.from_host(g, "cuda"), 1).build()
    want = oracle.build(g, 1)[4]
    assert np.array_equal(st.status.cpu().numpy()[: len(want)], want) and (want == 2).sum() > 100
    dg = cc.DeviceGeometry.from_host(cg.make_geometry(cg.ball_outside((0.5, 0.5, 0.5), 0.3), 32, 2), "cuda")
    ms = {}
    for fac in ("gram", "auto"):
        b = cc.Builder(dg, 1, factorization=fac)
        out = b.build()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        times = []
        for _ in range(8):
            e0.record()
            b.build(out=out)
            e1.record()
            torch.cuda.synchronize()
            times.append(e0.elapsed_time(e1))
        ms[fac] = min(times)
        print(f"{fac}: {ms[fac]:.2f} ms, {out.qr_faces} faces by QR", flush=True)
    assert out.qr_faces > 60000
    assert ms["auto"] < 3 * ms["gram"]
