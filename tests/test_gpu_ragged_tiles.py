"""The compiled tiles of ragged line lengths by themselves: lattices whose planes do
not run x and y in one launch (an extent of 1, or planes too large for it), against the
oracle and, forward, bit for bit against the run-time kernels."""
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


def _kernels(fn):
    """Names of the kernels a call launches."""
    from paper_1508_05610_amd import _lib
    _lib.lf2_profile_enable(1)
    try:
        fn()
        return " ".join(_lib.profile_table())
    finally:
        _lib.lf2_profile_enable(0)


def _runtime_plan(lf2, plan, *args, **kw):
    """The same plan with every run-time axis set to the schedule it reports."""
    p = lf2.Plan(*args, **kw)
    for a in range(3):
        r, rt = plan.schedule(a)
        if rt:
            p.set_schedule(a, r)
    return p


RAGGED = {9, 15, 25, 27, 45, 50, 135, 243, 250, 270, 432, 480, 500, 540, 625, 729, 900, 960, 972, 1000}


def _check_names(names, shape, lens, x_kernel):
    """The passes' kernels: compiled tiles over every ragged axis, no plane kernel and no
    run-time one."""
    assert "k_plane" not in names and "k_gx" not in names and "k_gs" not in names, names
    assert f"{x_kernel}<{lens[0]}" in names or f"{x_kernel}_v<{lens[0]}" in names, names
    for axis, nm in ((1, "y"), (2, "z")):
        if lens[axis] in RAGGED:
            assert any(n.startswith(f"k_strided<{lens[axis]},") and f" {nm} " in n
                       for n in names.replace(" k_", "\nk_").splitlines()), names


# x lines of one stage (pairs of factors: 9, 15, 25), of two and of many, dense and
# with odd halo offsets, one component and several; y lines from one stage to 1000
# points; row counts that leave the last x tile and column counts that leave the
# last strided tile unfilled
R2C = [((18, 900, 3), 1, 0), ((18, 900, 3), 1, 1), ((18, 540, 3), 3, 0), ((30, 625, 4), 1, 0),
       ((30, 625, 4), 3, 1), ((50, 540, 3), 1, 0), ((50, 540, 3), 1, 1), ((50, 250, 3), 3, 0),
       ((54, 432, 2), 2, 0), ((270, 135, 2), 1, 0), ((500, 50, 9), 1, 1), ((540, 45, 5), 1, 0),
       ((2000, 9, 15), 1, 0), ((2000, 9, 4), 3, 0), ((1944, 15, 2), 1, 1), ((1920, 1, 25), 1, 0),
       ((90, 1, 27), 6, 0), ((16, 1000, 1), 1, 0), ((24, 972, 2), 1, 0)]


@pytest.mark.parametrize("shape,ncomp,halo", R2C)
def test_r2c_pair(lf2, shape, ncomp, halo):
    print(f"case ragged tiles r2c {shape} ncomp={ncomp} halo={halo}", flush=True)
    f = real_field(shape, seed=84, ncomp=ncomp)[0]
    p = lf2.Plan(shape, lf2.LF2_R2C, ncomp=ncomp, halo=halo)
    q = _runtime_plan(lf2, p, shape, lf2.LF2_R2C, ncomp=ncomp, halo=halo)
    x = torch.full(p.x_shape, float("nan"), device=dev())
    _inner(x, halo).copy_(torch.from_numpy(f if ncomp > 1 else f[..., 0]).to(dev()))
    F, Fq = p.forward(x), q.forward(x)
    back = torch.full(p.x_shape, 7.0, device=dev())
    p.backward(F, out=back)
    lens = (shape[0] // 2, shape[1], shape[2])
    _check_names(_kernels(lambda: p.forward(x)), shape, lens, "k_x_r2c")
    _check_names(_kernels(lambda: p.backward(F, out=back)), shape, lens, "k_x_c2r")
    names = _kernels(lambda: q.forward(x))
    assert "k_plane" not in names and ("k_gx" in names or "k_gs" in names)
    assert torch.equal(torch.view_as_real(F), torch.view_as_real(Fq))
    if halo:  # halo sites stay as they were
        rim = back.clone()
        _inner(rim, halo).fill_(7.0)
        assert bool((rim == 7.0).all())
    F, back = F.cpu().numpy(), _inner(back, halo).cpu().numpy()
    for c in range(ncomp):
        Fc = F[..., c] if ncomp > 1 else F
        assert_close(Fc, oracle.r2c(f[..., c].astype(np.float64)), shape, f"r2c {c}")
        assert_close(back[..., c] if ncomp > 1 else back,
                     oracle.c2r(Fc.astype(np.complex128), shape[0]), shape, f"c2r {c}")


@pytest.mark.parametrize("shape,ncomp,halo", [
    ((9, 1000, 3), 1, 0), ((9, 500, 3), 3, 1), ((15, 729, 4), 1, 0), ((15, 432, 3), 3, 0),
    ((25, 432, 3), 1, 1), ((25, 243, 3), 3, 0), ((1000, 27, 3), 1, 0), ((960, 9, 4), 3, 0),
    ((972, 1, 15), 2, 0), ((480, 50, 3), 1, 1)])
@pytest.mark.parametrize("direction", [-1, 1])
def test_c2c(lf2, shape, ncomp, halo, direction):
    print(f"case ragged tiles c2c {shape} ncomp={ncomp} halo={halo} dir={direction}", flush=True)
    z = complex_field(shape, seed=85, ncomp=ncomp)
    p = lf2.Plan(shape, lf2.LF2_C2C, ncomp=ncomp, halo=halo)
    src = torch.from_numpy(z if ncomp > 1 else z[..., 0]).to(dev())
    if direction < 0:
        x = torch.zeros(p.x_shape, dtype=torch.complex64, device=dev())
        _inner(x, halo).copy_(src)
        q = _runtime_plan(lf2, p, shape, lf2.LF2_C2C, ncomp=ncomp, halo=halo)
        got = p.forward(x)
        assert torch.equal(torch.view_as_real(got), torch.view_as_real(q.forward(x)))
        names = _kernels(lambda: p.forward(x))
    else:
        k = src.contiguous()
        got = _inner(p.backward(k), halo)
        names = _kernels(lambda: p.backward(k))
    _check_names(names, shape, shape, "k_x_c2c")
    got = got.cpu().numpy()
    for c in range(ncomp):
        assert_close(got[..., c] if ncomp > 1 else got,
                     oracle.c2c(z[..., c].astype(np.complex128), direction), shape, f"comp {c}")
