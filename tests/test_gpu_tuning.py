"""Launch schedules per bin: stencils under schedules that part the launch of a kernel width,
and what the autotuner chooses."""

import pytest

torch = pytest.importorskip("torch")
import cutgeom as cg  # noqa: E402
import paper_1411_4283_amd as cc  # noqa: E402
from paper_1411_4283_amd._lib import Tuning  # noqa: E402

pytestmark = pytest.mark.gpu

WIDTHS = (range(0, 4), range(4, 6), range(6, 8))   # bins of up to 64, 96 and 128 rows


def _builder(D, order, n, R, **kw):
    g = cg.make_geometry(cg.ball_outside((0.483, 0.512, 0.531)[:D], 0.3), n, order)
    b = cc.Builder(cc.DeviceGeometry.from_host(g, "cuda"), R, **kw)
    return b, b.build()


@pytest.mark.parametrize("D,order,n,R,kw", [(3, 4, 20, 3, {}), (3, 2, 16, 3, {}), (2, 4, 40, 4, {}),
                                            (3, 4, 16, 3, dict(eb_bc="neumann")),
                                            (3, 4, 16, 3, dict(reuse_templates=True))])
def test_bins_of_one_width_with_different_schedules(D, order, n, R, kw):
    b, st = _builder(D, order, n, R, **kw)
    val, status = st.val.clone(), st.status.clone()
    for kinds in ([(1, 0), (8, 0)], [(8, 3), (1, 0), (3, 5)], [(1, 7), (8, 2)]):
        t = Tuning()
        for i in range(8):
            t.xcd_chunks[i], t.blocks_per_xcd[i] = kinds[i % len(kinds)]
        b.set_tuning(t)
        st.val.zero_()
        b.build(out=st)
        torch.cuda.synchronize()
        assert torch.equal(st.val, val) and torch.equal(st.status, status), kinds


def _ms(b, st, reps):
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    best = 1e300
    for _ in range(reps):
        e0.record()
        b.build(out=st)
        e1.record()
        torch.cuda.synchronize()
        best = min(best, e0.elapsed_time(e1))
    return best


@pytest.mark.parametrize("D,order,n,R,kw", [(3, 4, 24, 3, {}), (3, 4, 48, 3, {}), (3, 2, 32, 3, {}),
                                            (3, 2, 24, 2, dict(eb_bc="neumann")),
                                            (3, 2, 12, 2, dict(factorization="qr"))])
def test_tuned_builds_keep_their_launches_and_their_time(D, order, n, R, kw):
    """The bins of a width get one schedule, empty bins no time, and the tuned build is no slower
    than the untuned one (by more than a tenth, the spread of short builds)."""
    b, st = _builder(D, order, n, R, **kw)
    val = st.val.clone()
    tuning, best = b.autotune(out=st)
    torch.cuda.synchronize()
    assert torch.equal(st.val, val)
    chosen = [(tuning.xcd_chunks[i], tuning.blocks_per_xcd[i]) for i in range(8)]
    print(f"chosen {chosen}, best {best}", flush=True)
    for bins in WIDTHS:
        assert len({chosen[i] for i in bins}) == 1
        assert len({best[i] for i in bins if best[i] >= 0}) <= 1
    assert any(t > 0 for t in best)
    tuned = _ms(b, st, 20)
    b.set_tuning(None)
    plain = _ms(b, st, 20)
    print(f"tuned {tuned:.3f} ms, untuned {plain:.3f} ms", flush=True)
    assert tuned < 1.1 * plain
