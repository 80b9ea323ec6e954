"""Tiles that a plan's y and z passes take by default over long lines and large
spectra: forward transforms are those of the narrow tiles bit for bit, backward ones
as near to the FP64 transform, so that a plan's error does not depend on the lattice's
size."""
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


def dev():
    return torch.device("cuda:0")


def _random(shape, dtype, seed):
    g = torch.Generator(device=dev())
    g.manual_seed(seed)
    return torch.randn(shape, generator=g, device=dev(), dtype=dtype)


# spectra of 256 to 520 MiB, past the memory-side cache: z lines of every length
# with a default of its own, rows a multiple of 64 KB apart (complex) and not
# (real); long y lines
@pytest.mark.parametrize("shape,kind,ncomp", [
    ((256, 256, 1024), 0, 1), ((128, 320, 1024), 1, 1), ((256, 128, 2048), 0, 1),
    ((64, 320, 2048), 1, 1), ((320, 384, 640), 0, 1), ((256, 320, 640), 1, 1),
    ((256, 384, 768), 0, 1), ((128, 128, 768), 1, 3), ((256, 320, 512), 1, 1),
    ((512, 512, 512), 0, 1), ((128, 1024, 320), 0, 1), ((96, 768, 320), 1, 2)])
def test_rounds_as_narrow_tiles(lf2, shape, kind, ncomp):
    print(f"case default tiles {shape} kind={kind} ncomp={ncomp}", flush=True)
    p, q = (lf2.Plan(shape, kind, ncomp=ncomp) for _ in range(2))
    for axis in (1, 2):
        if not q.schedule(axis)[1]:
            q.set_tuning(axis, 0, 16)
    x = _random(p.x_shape, torch.complex64 if kind else torch.float32, 61)
    F = p.forward(x)
    assert torch.equal(torch.view_as_real(F), torch.view_as_real(q.forward(x)))
    del x
    # the same butterflies in the same order, of which the compiler may fuse
    # other products: one rounding of the about sixty along a line's path
    b, bq = p.backward(F), q.backward(F)
    if not torch.equal(b, bq):
        axes = (0, 1, 2)
        ref = (torch.fft.ifftn(F.to(torch.complex128), dim=axes, norm="forward") if kind else
               torch.fft.irfftn(F.to(torch.complex128), s=p.x_shape[:3], dim=axes, norm="forward"))
        e, eq = (float(torch.linalg.vector_norm(t - ref) / torch.linalg.vector_norm(ref))
                 for t in (b, bq))
        print(f"  backward error {e:.4e}, narrow tiles {eq:.4e}", flush=True)
        assert e <= 1.02 * eq


def _kernels(fn):
    """Names of the kernels a call launches."""
    from paper_1508_05610_amd import _lib
    _lib.lf2_profile_enable(1)
    try:
        fn()
        return " ".join(_lib.profile_table())
    finally:
        _lib.lf2_profile_enable(0)


# backward z passes: nontemporal in narrow tiles of 320 to 512 points past 430 MB,
# normal over lengths that take run-time schedules and over 640 and 768 points
# (rows not a multiple of 64 KB apart)
@pytest.mark.parametrize("shape,kernel", [
    ((320, 640, 540), "k_strided<540,1,0,0> z"), ((360, 640, 540), "k_strided<540,1,0,0> z"),
    ((600, 400, 480), "k_strided<480,1,0,0> z"), ((384, 640, 512), "k_strided<512,1,0,1> z"),
    ((320, 384, 640), "k_strided<640,1,0,0> z"), ((256, 384, 768), "k_strided<768,1,0,0> z")])
def test_backward_z_kernel(lf2, shape, kernel):
    print(f"case default backward z {shape}", flush=True)
    p = lf2.Plan(shape)
    F = torch.zeros(p.k_shape, dtype=torch.complex64, device=dev())
    names = _kernels(lambda: p.backward(F))
    assert kernel in names, names


# long y lines: wide tiles past 256 MB only
@pytest.mark.parametrize("shape,kind,ncomp,kernel", [
    ((96, 1024, 96), 1, 1, "k_strided<1024,%d,0,0> y"), ((512, 1024, 64), 1, 1, "k_strided<1024,%d,0,0> y"),
    ((96, 768, 320), 1, 2, "k_strided_w<768,%d,0> y")])
def test_y_kernel(lf2, shape, kind, ncomp, kernel):
    print(f"case default y {shape}", flush=True)
    p = lf2.Plan(shape, kind, ncomp=ncomp)
    x = torch.zeros(p.x_shape, dtype=torch.complex64, device=dev())
    F = p.forward(x)
    assert kernel % -1 in _kernels(lambda: p.forward(x))
    assert kernel % 1 in _kernels(lambda: p.backward(F))
