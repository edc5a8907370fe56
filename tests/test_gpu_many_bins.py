"""More bins than one launch of a workgroup each holds (2^32 threads): the sort
(1024 threads a bin, both key types, one grid) and the fit of short bins (256),
with bins of one point, whose k(g) is the point and whose fit its logarithm."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hk = pytest.importorskip("paper_1503_03806_amd")


@pytest.fixture(scope="module")
def ctx():
    c = hk.Context(0)
    yield c
    c.close()


def values(n):
    return torch.rand(n, dtype=torch.float64, device="cuda", generator=torch.Generator(device="cuda").manual_seed(n)) + 1.0


@pytest.mark.parametrize("precision", [hk.HK_F64, hk.HK_F32_KAHAN])
def test_sort(ctx, precision):
    k = values((1 << 22) + 3).to(torch.float64 if precision == hk.HK_F64 else torch.float32)
    out = torch.zeros_like(k)
    kg = ctx.kdist(k, 1, [0.5], precision=precision, sorted_out=out)
    assert torch.equal(kg[:, 0], k.double()) and torch.equal(out, k)


def test_fit(ctx):
    k = values((1 << 24) + 3)
    c = ctx.resample(k, 1, 1)
    # (the factor of one point is 1; the logarithms differ by a rounding or two)
    assert bool(((c[:, 0] - k.log()).abs() <= 4 * 2.0 ** -53).all())
