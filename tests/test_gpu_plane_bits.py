"""Small lattices whose planes run x and y in one launch: what a call asks for beside phi
does not change phi, and where bins are taken from the planes' spectrum it is the two
passes' bit for bit."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def lf2():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1508_05610_amd as m
    m.load()
    return m


def _random(shape, dtype, seed):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(seed)
    return torch.randn(shape, generator=g, device="cuda:0", dtype=dtype)


# planes whose forward spectrum has the two passes' bits and planes (factors of 16
# along x or y, of 5 along y) whose spectrum does not
@pytest.mark.parametrize("shape", [(32, 32, 32), (64, 64, 24), (96, 40, 20), (32, 16, 12), (24, 80, 8),
                                   (256, 48, 5), (20, 10, 40), (60, 50, 45), (16, 4, 300)])
def test_phi_does_not_depend_on_bins(lf2, shape):
    print(f"case phi with and without bins {shape}", flush=True)
    p = lf2.Plan(shape)
    x = _random(p.x_shape, torch.float32, 63)
    phi = p.poisson(x)
    for kw in ({"nbins": 8}, {"nbins": 0, "parseval": True}, {"nbins": 20, "parseval": True}):
        assert torch.equal(p.poisson(x, **kw)[0], phi), kw


def _kernels(fn):
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


LENGTHS = sorted({2 ** a * 3 ** b * 5 ** c for a in range(11) for b in range(7) for c in range(5)
                  if 1 < 2 ** a * 3 ** b * 5 ** c <= 1024})


@pytest.mark.parametrize("axis,kind", [("x", 0), ("x", 1), ("y", 0), ("y", 1)])
def test_binned_planes_have_the_two_passes_bits(lf2, axis, kind):
    """Every line length along x and y, real and complex fields, 432 rows (an x tile and
    part of a second at the shortest lines): where P(k) runs the plane kernel, the
    spectrum is the two passes'."""
    dtype = torch.complex64 if kind else torch.float32
    taken, differ = [], []
    for n in LENGTHS:
        # the other axis: 3 points (x) or 6 (y), whose stages have the bits
        shape = ((n if kind else 2 * n), 6, 72) if axis == "x" else ((3 if kind else 6), n, 72)
        p, q = lf2.Plan(shape, kind), _two_pass(lf2, shape, kind)
        x = _random(p.x_shape, dtype, 64)
        if "k_plane" not in _kernels(lambda: p.power_spectrum(x, 4)):
            continue
        taken.append(n)
        assert "k_plane" not in _kernels(lambda: q.forward(x))
        if not torch.equal(torch.view_as_real(p.forward(x)), torch.view_as_real(q.forward(x))):
            differ.append(n)
    print(f"case plane bits {axis} kind={kind}: {len(taken)} lengths {taken}", flush=True)
    assert not differ and len(taken) >= 20


# 128 x 128 real planes take a CU alone: one launch where they fill three quarters of
# the 256 CUs up to all of them
@pytest.mark.parametrize("planes,one", [(160, False), (192, True), (225, True), (256, True), (270, False)])
def test_large_planes_run_in_one_launch_where_they_fill_the_chip(lf2, planes, one):
    print(f"case large planes {planes}", flush=True)
    shape = (128, 128, planes)
    p, q = lf2.Plan(shape), _two_pass(lf2, shape)
    x = _random(p.x_shape, torch.float32, 65)
    F, Fq = p.forward(x), q.forward(x)
    assert ("k_plane<r2c" in _kernels(lambda: p.forward(x))) == one
    assert ("k_plane<c2r" in _kernels(lambda: p.backward(F))) == one
    # two FP32 transforms of 2^22 points, each within 3e-7 of the exact one
    assert float(torch.linalg.vector_norm(F - Fq) / torch.linalg.vector_norm(Fq)) <= 6e-7
    b, bq = p.backward(F), q.backward(F)
    assert float(torch.linalg.vector_norm(b - bq) / torch.linalg.vector_norm(bq)) <= 6e-7
