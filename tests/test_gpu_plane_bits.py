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
