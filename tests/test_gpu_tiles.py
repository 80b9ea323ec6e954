"""Edges of the pass tiles: rows and columns that do not fill a tile, tiles whose
rows span several planes or start inside one, tables fetched ahead of or behind a
tile's loads, binning passes of more tiles than blocks, and the derivative's
planes per block."""
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


def _passes(lf2, *args, **kw):
    """A plan that runs its x and y passes one by one."""
    p = lf2.Plan(*args, **kw)
    radices, runtime = p.schedule(1)
    if runtime:
        p.set_schedule(1, radices)
    else:
        p.set_tuning(1, 0, 16)
    return p


# x lines of one, a few and many stages, with a factor of 16 beside 3 or 5
# (table first) and without; y lines likewise
SHAPES = [(2, 3, 5), (96, 5, 12), (160, 6, 3), (192, 3, 9), (54, 5, 9), (1024, 3, 5), (256, 18, 2),
          (12, 80, 5), (10, 48, 8), (6, 512, 3), (300, 45, 2)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("ncomp,halo", [(1, 0), (1, 1), (1, 2), (3, 0), (3, 1)])
def test_real_pair(lf2, shape, ncomp, halo):
    if halo >= min(shape):
        return
    print(f"case tiles r2c {shape} ncomp={ncomp} halo={halo}", flush=True)
    f = real_field(shape, seed=71, ncomp=ncomp)[0]
    p = _passes(lf2, shape, lf2.LF2_R2C, ncomp=ncomp, halo=halo)
    x = torch.full(p.x_shape, float("nan"), device=dev())
    _inner(x, halo).copy_(torch.from_numpy(f if ncomp > 1 else f[..., 0]).to(dev()))
    F = p.forward(x)
    back = _inner(p.backward(F), halo).cpu().numpy()
    F = F.cpu().numpy()
    for c in range(ncomp):
        Fc = F[..., c] if ncomp > 1 else F
        assert_close(Fc, oracle.r2c(f[..., c].astype(np.float64)), shape, f"r2c {c}")
        assert_close(back[..., c] if ncomp > 1 else back,
                     oracle.c2r(Fc.astype(np.complex128), shape[0]), shape, f"c2r {c}")


@pytest.mark.parametrize("shape", [(48, 5, 8), (80, 3, 9), (512, 3, 2), (27, 5, 4), (16, 80, 3)])
@pytest.mark.parametrize("ncomp,halo", [(1, 0), (3, 1)])
@pytest.mark.parametrize("direction", [-1, 1])
def test_complex(lf2, shape, ncomp, halo, direction):
    print(f"case tiles c2c {shape} ncomp={ncomp} halo={halo} dir={direction}", flush=True)
    z = complex_field(shape, seed=72, ncomp=ncomp)
    p = _passes(lf2, shape, lf2.LF2_C2C, ncomp=ncomp, halo=halo)
    src = torch.from_numpy(z if ncomp > 1 else z[..., 0]).to(dev())
    if direction < 0:
        x = torch.zeros(p.x_shape, dtype=torch.complex64, device=dev())
        _inner(x, halo).copy_(src)
        got = p.forward(x)
    else:
        got = _inner(p.backward(src.contiguous()), halo)
    got = got.cpu().numpy()
    for c in range(ncomp):
        assert_close(got[..., c] if ncomp > 1 else got,
                     oracle.c2c(z[..., c].astype(np.complex128), direction), shape, f"comp {c}")


# fewer tiles than blocks; one more than a round of two blocks a CU, of three;
# a line past the rule's limit; a spectrum past the k-space pass's limit
@pytest.mark.parametrize("shape", [(16, 4, 8), (256, 128, 256), (300, 216, 300), (40, 300, 640), (512, 512, 540)])
def test_binning_passes_agree(lf2, shape):
    """P(k) from the field (z pass), from the solve's fused pass, and from the
    spectrum (k-space pass): the same modes, powers of one FP32 transform
    rounded in at most two ways."""
    print(f"case tiles bins {shape}", flush=True)
    p = lf2.Plan(shape)
    g = torch.Generator(device=dev())
    g.manual_seed(73)
    x = torch.randn(p.x_shape, generator=g, device=dev())
    field = p.power_spectrum(x, 24)
    solve = p.poisson(x, nbins=24, parseval=True)
    spec = p.power_spectrum(p.forward(x), 24, field_is_kspace=True)
    assert torch.equal(field[2], spec[2]) and torch.equal(field[2], solve[3])
    assert float(field[2].sum()) == np.prod(shape) - 1
    # FP32 transforms of 2^26 points are within 1e-6 of each other in norm, a
    # bin's power within twice that of the largest
    top = float(field[0].max())
    assert float((field[0] - spec[0]).abs().max()) <= 4e-6 * top
    assert float((field[0] - solve[1]).abs().max()) <= 4e-6 * top
    pv = solve[4].cpu().numpy()
    assert abs(pv[0] - pv[1]) <= 1e-5 * pv[0]


# 32, 16, 8 and 4 planes a block (12288 waves in the grid or fewer), the last
# block of each ragged
@pytest.mark.parametrize("shape,nc", [((128, 2048, 40), 6), ((128, 2048, 20), 6), ((128, 1024, 18), 6),
                                      ((128, 300, 18), 6)])
def test_gradient_planes(lf2, shape, nc):
    print(f"case tiles gradient {shape} nc={nc}", flush=True)
    h = 1
    g = torch.Generator(device=dev())
    g.manual_seed(74)
    t = torch.randn((shape[2] + 2, shape[1] + 2, shape[0] + 2, nc), generator=g, device=dev())
    lf2.update_halo(t, shape, h)
    out = torch.full(t.shape[:3] + (3 * nc,), float("nan"), device=dev())
    lf2.gradient(t, shape, h, dx=0.5, out=out)
    got = _inner(out, h)
    f = _inner(t, h).double()
    for i, axis in enumerate((2, 1, 0)):
        ref = (torch.roll(f, -1, axis) - f) / 0.5
        # one FP32 subtraction and one product
        assert float((got[..., i::3] - ref).abs().max()) <= 1e-6 * float(ref.abs().max())
