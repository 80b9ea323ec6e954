"""Compiled tiles of the line lengths 2^a 3^b 5^c that also take run-time
radix schedules: against the oracle, and against the default schedule run by
the run-time kernels.  Forward transforms are equal bit for bit (the compiled
stages spell out the run-time kernels' rounding); the way back and the Poisson
factor may round differently, so they are held to the oracle alone."""
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


# smallest and longest lines of each axis, pairs of factors in the first,
# middle and last stage, a 16 beside pairs, column counts that leave a
# remainder in the last tile
R2C = [((18, 9, 15), 1, 0), ((30, 25, 27), 3, 0), ((50, 36, 135), 1, 1), ((288, 10, 144), 2, 0),
       ((90, 270, 4), 6, 0), ((2000, 3, 5), 1, 0), ((6, 972, 3), 1, 0), ((4, 6, 1000), 1, 0),
       ((10, 625, 12), 1, 0), ((8, 240, 729), 1, 0)]


def _runtime_plan(lf2, plan, shape, kind, ncomp, halo):
    """The same plan with every run-time axis set to the schedule it reports."""
    p = lf2.Plan(shape, kind, ncomp=ncomp, halo=halo)
    for a in range(3):
        r, rt = plan.schedule(a)
        if rt:
            p.set_schedule(a, r)
    return p


def _inner(a, h):
    return a[h:a.shape[0] - h, h:a.shape[1] - h, h:a.shape[2] - h] if h else a


@pytest.mark.parametrize("shape,ncomp,halo", R2C)
def test_r2c_pair(lf2, shape, ncomp, halo):
    print(f"case ragged r2c {shape} ncomp={ncomp} halo={halo}", flush=True)
    f = real_field(shape, seed=81, ncomp=ncomp)[0]
    p = lf2.Plan(shape, lf2.LF2_R2C, ncomp=ncomp, halo=halo)
    x = torch.zeros(p.x_shape, device=dev())
    src = torch.from_numpy(f if ncomp > 1 else f[..., 0]).to(dev())
    _inner(x, halo).copy_(src)
    F = p.forward(x)
    back = p.backward(F)
    Fr = _runtime_plan(lf2, p, shape, lf2.LF2_R2C, ncomp, halo).forward(x)
    torch.cuda.synchronize()
    assert torch.equal(torch.view_as_real(F), torch.view_as_real(Fr))
    F, back = F.cpu().numpy(), _inner(back, halo).cpu().numpy()
    for c in range(ncomp):
        Fc = F[..., c] if ncomp > 1 else F
        bc = back[..., c] if ncomp > 1 else back
        assert_close(Fc, oracle.r2c(f[..., c].astype(np.float64)), shape, f"r2c {c}")
        assert_close(bc, oracle.c2r(Fc.astype(np.complex128), shape[0]), shape, f"c2r {c}")


@pytest.mark.parametrize("shape,ncomp", [((9, 15, 25), 1), ((45, 12, 18), 3), ((1000, 3, 9), 2),
                                         ((144, 50, 6), 6), ((4, 900, 27), 1)])
@pytest.mark.parametrize("direction", [-1, 1])
def test_c2c(lf2, shape, ncomp, direction):
    print(f"case ragged c2c {shape} ncomp={ncomp} dir={direction}", flush=True)
    z = complex_field(shape, seed=82, ncomp=ncomp)
    p = lf2.Plan(shape, lf2.LF2_C2C, ncomp=ncomp)
    zin = torch.from_numpy(z if ncomp > 1 else z[..., 0]).to(dev())
    run = p.forward if direction < 0 else p.backward
    out = run(zin)
    if direction < 0:
        ref = _runtime_plan(lf2, p, shape, lf2.LF2_C2C, ncomp, 0).forward(zin)
        assert torch.equal(torch.view_as_real(out), torch.view_as_real(ref))
    got = out.cpu().numpy()
    for c in range(ncomp):
        assert_close(got[..., c] if ncomp > 1 else got,
                     oracle.c2c(z[..., c].astype(np.complex128), direction), shape, f"comp {c}")


@pytest.mark.parametrize("shape,nbins,discrete,of_phi", [
    ((36, 20, 90), 12, 0, False), ((16, 9, 375), 4096, 0, False), ((30, 27, 50), 0, 1, False),
    ((24, 18, 225), 40, 1, True), ((8, 4, 1000), 64, 0, False)])
def test_poisson(lf2, shape, nbins, discrete, of_phi):
    """The fused last-axis pass: bins, Parseval sums and phi; P(k) of rho comes
    from the same spectrum bits as the run-time kernels', so its FP64 sums
    differ by their order alone (at most 1e-12 of the largest bin)."""
    print(f"case ragged poisson {shape} nbins={nbins} discrete={discrete}", flush=True)
    f = real_field(shape, seed=83)[0][..., 0]
    f64 = f.astype(np.float64)
    p = lf2.Plan(shape, lf2.LF2_R2C)
    q = _runtime_plan(lf2, p, shape, lf2.LF2_R2C, 1, 0)
    x = torch.from_numpy(f).to(dev())
    flags = (lf2.LF2_POISSON_DISCRETE_K2 if discrete else 0) | (lf2.LF2_PK_OF_PHI if of_phi else 0)
    a = p.poisson(x, nbins=nbins, flags=flags, parseval=not of_phi)
    b = q.poisson(x, nbins=nbins, flags=flags, parseval=not of_phi)
    torch.cuda.synchronize()
    assert_close(a[0].cpu().numpy(), oracle.poisson(f64, k2mode=oracle.K2_DISCRETE if discrete else oracle.K2_CONTINUOUS), shape, "phi")
    if not of_phi:
        va, vb = a[4].cpu().numpy(), b[4].cpu().numpy()
        assert np.all(np.abs(va - vb) <= 1e-12 * np.abs(vb))
    if nbins:
        assert torch.equal(a[3], b[3])  # counts
        pa, pb = a[1].cpu().numpy(), b[1].cpu().numpy()
        tol = 1e-5 * np.log2(f.size) if of_phi else 1e-12
        assert np.max(np.abs(pa - pb)) <= tol * np.max(pb)
