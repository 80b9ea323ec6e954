"""Small lattices' x and y passes in one launch per direction (whole z planes in
LDS): against the oracle and against the two passes, which a plan runs once a
tile setting or a schedule of its y pass has been asked for.  The default gate of the parity
tests holds both; bins and Parseval sums, whose forward spectrum has the two
passes' bits, differ from theirs by the order of the sums of squares alone."""
import numpy as np
import pytest

import oracle
from gpu_helpers import assert_close, complex_field, real_field

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def lf2():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1508_05610_amd as m
    m.load()
    return m


def dev():
    return torch.device("cuda:0")


def _inner(a, h):
    return a[h:a.shape[0] - h, h:a.shape[1] - h, h:a.shape[2] - h] if h else a


def _kernels(lf2, fn):
    """Names of the kernels a call launches."""
    from paper_1508_05610_amd import _lib
    _lib.lf2_profile_enable(1)
    try:
        fn()
        return " ".join(_lib.profile_table())
    finally:
        _lib.lf2_profile_enable(0)


def _two_pass(lf2, *args, **kw):
    p = lf2.Plan(*args, **kw)
    radices, runtime = p.schedule(1)
    if runtime:
        p.set_schedule(1, radices)
    else:
        p.set_tuning(1, 0, 16)
    return p


# the smallest planes; one plane; planes on both sides of 256; the largest
# planes (128 x 128, which one launch takes from 256 planes on; 120 x 120); many factors; odd halo offsets; a field at the size limit
R2C = [((4, 2, 3), 1, 0), ((16, 12, 1), 1, 0), ((8, 6, 256), 1, 0), ((8, 6, 270), 1, 0),
       ((128, 128, 256), 1, 0), ((120, 120, 4), 1, 0), ((36, 81, 5), 1, 0), ((16, 12, 10), 1, 1), ((12, 10, 6), 3, 1),
       ((32, 24, 16), 6, 0), ((20, 40, 8), 2, 2), ((96, 16, 3072), 1, 0)]


@pytest.mark.parametrize("paper", [False, True])
@pytest.mark.parametrize("shape,ncomp,halo", R2C)
def test_r2c_pair(lf2, shape, ncomp, halo, paper):
    print(f"case plane r2c {shape} ncomp={ncomp} halo={halo} paper={paper}", flush=True)
    f = real_field(shape, seed=91, ncomp=ncomp)[0]
    p = lf2.Plan(shape, lf2.LF2_R2C, ncomp=ncomp, halo=halo, paper_layout=paper)
    q = _two_pass(lf2, shape, lf2.LF2_R2C, ncomp=ncomp, halo=halo, paper_layout=paper)
    x = torch.full(p.x_shape, float("nan"), device=dev())
    _inner(x, halo).copy_(torch.from_numpy(f if ncomp > 1 else f[..., 0]).to(dev()))
    F = p.forward(x)
    assert "k_plane<r2c" in _kernels(lf2, lambda: p.forward(x, out=F))
    assert "k_plane" not in _kernels(lf2, lambda: q.forward(x))
    back = torch.full(p.x_shape, 7.0, device=dev())
    p.backward(F, out=back)
    torch.cuda.synchronize()
    if halo:  # halo sites stay as they were
        rim = back.clone()
        _inner(rim, halo).fill_(7.0)
        assert bool((rim == 7.0).all())
    Fq, bq = q.forward(x).cpu().numpy(), _inner(q.backward(F), halo).cpu().numpy()
    F, back = F.cpu().numpy(), _inner(back, halo).cpu().numpy()
    assert_close(F, Fq, shape, "forward, two passes")
    assert_close(back, bq, shape, "backward, two passes")
    if not paper and np.prod(shape) <= 1 << 20:
        for c in range(ncomp):
            Fc = F[..., c] if ncomp > 1 else F
            assert_close(Fc, oracle.r2c(f[..., c].astype(np.float64)), shape, f"r2c {c}")
            assert_close(back[..., c] if ncomp > 1 else back,
                         oracle.c2r(Fc.astype(np.complex128), shape[0]), shape, f"c2r {c}")


@pytest.mark.parametrize("shape,ncomp,halo", [((2, 2, 2), 1, 0), ((16, 16, 16), 1, 0), ((64, 60, 9), 1, 0),
                                              ((12, 18, 300), 3, 0), ((25, 27, 6), 2, 1), ((80, 16, 5), 6, 0)])
@pytest.mark.parametrize("direction", [-1, 1])
@pytest.mark.parametrize("in_place", [False, True])
def test_c2c(lf2, shape, ncomp, halo, direction, in_place):
    if in_place and halo:
        return
    print(f"case plane c2c {shape} ncomp={ncomp} halo={halo} dir={direction} in place={in_place}", flush=True)
    z = complex_field(shape, seed=92, ncomp=ncomp)
    p = lf2.Plan(shape, lf2.LF2_C2C, ncomp=ncomp, halo=halo, in_place=in_place)
    src = torch.from_numpy(z if ncomp > 1 else z[..., 0]).to(dev())
    if direction < 0:
        x = torch.zeros(p.x_shape, dtype=torch.complex64, device=dev())
        _inner(x, halo).copy_(src)
        got = p.forward_(x) if in_place else p.forward(x)
    else:
        k = src.contiguous().clone()
        got = p.backward_(k) if in_place else _inner(p.backward(k), halo)
    got = got.cpu().numpy()
    for c in range(ncomp):
        assert_close(got[..., c] if ncomp > 1 else got,
                     oracle.c2c(z[..., c].astype(np.complex128), direction), shape, f"comp {c}")


@pytest.mark.parametrize("shape,nbins", [((32, 32, 32), 16), ((64, 64, 40), 32), ((48, 36, 30), 24),
                                         ((96, 40, 20), 16), ((16, 4, 300), 8), ((60, 50, 45), 0)])
def test_poisson_bins_equal_two_passes(lf2, shape, nbins):
    print(f"case plane poisson {shape} nbins={nbins}", flush=True)
    f = real_field(shape, seed=93)[0][..., 0]
    x = torch.from_numpy(f).to(dev())
    p, q = lf2.Plan(shape), _two_pass(lf2, shape)
    a, b = (pl.poisson(x, nbins=nbins, parseval=True) for pl in (p, q))
    torch.cuda.synchronize()
    assert_close(a[0].cpu().numpy(), oracle.poisson(f.astype(np.float64)), shape, "phi")
    assert np.all(np.abs(a[4].cpu().numpy() - b[4].cpu().numpy()) <= 1e-12 * np.abs(b[4].cpu().numpy()))
    if nbins:
        assert torch.equal(a[3], b[3])
        pa, pb = a[1].cpu().numpy(), b[1].cpu().numpy()
        assert np.max(np.abs(pa - pb)) <= 1e-12 * np.max(pb)


@pytest.mark.parametrize("kind,shape,halo", [
    (1, (32, 32, 32), 0), (1, (64, 64, 24), 0), (1, (12, 24, 24), 0), (1, (6, 8, 300), 0),
    (1, (36, 36, 20), 0), (1, (8, 64, 40), 0), (0, (36, 40, 20), 1), (0, (64, 32, 30), 1)])
def test_bins_of_a_field_equal_two_passes(lf2, kind, shape, halo):
    """P(k) of more rows than one x tile of the two passes holds: the same
    spectrum bit for bit, whichever way the plan takes."""
    print(f"case plane bins kind={kind} {shape} halo={halo}", flush=True)
    p, q = (mk(lf2, shape, kind, halo=halo) for mk in (lambda m, *a, **k: m.Plan(*a, **k), _two_pass))
    g = torch.Generator(device=dev())
    g.manual_seed(95)
    x = torch.randn(p.x_shape, generator=g, device=dev(),
                    dtype=torch.complex64 if kind else torch.float32)
    pa, pb = p.power_spectrum(x, 8), q.power_spectrum(x, 8)
    assert torch.equal(pa[2], pb[2]) and float(pb[0].max()) > 0
    assert "k_plane" not in _kernels(lf2, lambda: q.power_spectrum(x, 8))
    # the binned sums are the same numbers added in the same order
    assert float((pa[0] - pb[0]).abs().max()) <= 1e-13 * float(pb[0].max())


def test_workspace_of_the_two_passes_is_enough(lf2):
    """A solve given a workspace that holds the two passes' sums of squares but
    not one per plane still runs (300 planes, 5 x tiles)."""
    from paper_1508_05610_amd import _lib
    shape = (16, 4, 300)
    f = real_field(shape, seed=94)[0][..., 0]
    x = torch.from_numpy(f).to(dev())
    p, ref = lf2.Plan(shape), lf2.Plan(shape).poisson(x, nbins=4, parseval=True)
    # spectrum, 1024 rows of 5 doubles, 5 doubles, 5 sums of squares, one sum,
    # each rounded up to 256 bytes
    need = sum((v + 255) // 256 * 256 for v in (8 * 9 * 4 * 300, 1024 * 5 * 8, 5 * 8, 5 * 8)) + 256
    ws = torch.empty(need, dtype=torch.uint8, device=dev())
    _lib.lf2_plan_set_workspace(p.handle, ws.data_ptr(), need)
    got = p.poisson(x, nbins=4, parseval=True)
    torch.cuda.synchronize()
    for a, b in zip(got, ref):
        assert_close(a.cpu().numpy(), b.cpu().numpy(), shape)


def test_graph_replay(lf2):
    """One launch per direction under graph capture, replayed between eager work."""
    shape = (32, 24, 20)
    f = real_field(shape, seed=95)[0][..., 0]
    x = torch.from_numpy(f).to(dev())
    p = lf2.Plan(shape)
    F, back = p.forward(x), torch.empty_like(x)
    p.backward(F, out=back)  # the shared workspace exists
    want_F, want_b = F.clone(), back.clone()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        p.forward(x, out=F)
        p.backward(F, out=back)
    for _ in range(3):
        F.zero_()
        back.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(torch.view_as_real(F), torch.view_as_real(want_F))
        assert torch.equal(back, want_b)
