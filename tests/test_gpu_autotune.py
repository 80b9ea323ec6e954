"""Autotuned plans: whatever settings win, the transforms are those of the untuned
plan up to FP32 rounding, both ways, and the reported times belong to them."""
import numpy as np
import pytest

from gpu_helpers import assert_close

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def lf2():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1508_05610_amd as m
    m.load()
    return m


# small planes (one launch for x and y, timed against the two passes) of every
# layout; run-time-schedule axes; 64-point complex rows; wide and register tiles
@pytest.mark.parametrize("shape,kind,ncomp,kw", [
    ((32, 24, 16), 0, 1, {}), ((16, 12, 10), 0, 1, {"halo": 1}), ((24, 16, 12), 0, 2, {"paper_layout": True}),
    ((16, 16, 8), 0, 1, {"in_place": True}), ((64, 16, 8), 1, 1, {}), ((12, 20, 6), 1, 3, {"halo": 2}),
    ((16, 8, 32), 1, 1, {"paper_layout": True}), ((300, 200, 90), 0, 1, {}), ((90, 300, 144), 1, 2, {}),
    ((64, 256, 320), 0, 1, {}), ((32, 1024, 160), 1, 1, {}), ((16, 40, 2048), 0, 3, {})])
def test_tuned_plan_is_the_untuned_one(lf2, shape, kind, ncomp, kw):
    print(f"case autotuned {shape} kind={kind} ncomp={ncomp} {kw}", flush=True)
    p, q = lf2.Plan(shape, kind, ncomp=ncomp, **kw), lf2.Plan(shape, kind, ncomp=ncomp, autotune=True, **kw)
    print("  ", [q.tuning(a) for a in range(3)], flush=True)
    for axis in (1, 2):
        v, c, us0, us = q.tuning(axis)
        assert 0 < us <= us0 and c in (4, 16, 64)
    g = torch.Generator(device="cuda:0")
    g.manual_seed(62)
    x = torch.randn(p.x_shape, generator=g, device="cuda:0",
                    dtype=torch.complex64 if kind else torch.float32)
    F, Fq = p.forward(x), q.forward(x)
    b, bq = p.backward(F), q.backward(F)
    torch.cuda.synchronize()
    assert_close(Fq.cpu().numpy(), F.cpu().numpy(), shape, "forward")
    assert_close(bq.cpu().numpy(), b.cpu().numpy(), shape, "backward")
    if kind == 0 and ncomp == 1:
        for nb in (0, 8):
            a, aq = (pl.poisson(x, nbins=nb) for pl in (p, q))
            a, aq = (a, aq) if nb == 0 else (a[0], aq[0])
            assert_close(aq.cpu().numpy(), a.cpu().numpy(), shape, f"phi {nb}")
