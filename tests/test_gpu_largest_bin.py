"""A fit of one bin of 2^28 points, whose design matrix has more rows than a
launch of a thread per coefficient of 64 rows can count (2^32 threads): values
of a known exponential, so that the coefficients are known.

Tolerance: 1e-9 of the largest coefficient, the bar of the fit."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hk = pytest.importorskip("paper_1503_03806_amd")


def test_fit_of_a_bin_of_2_28_points():
    m = 1 << 28
    t = (torch.arange(m, dtype=torch.float64, device="cuda") + 0.5).mul_(2.0 / m).sub_(1.0)
    k = t.mul_(3.0).sub_(40.0).exp_()  # ln kappa = 3 t - 40
    ctx = hk.Context(0)
    try:
        c = ctx.resample(k, m, 3).cpu()
    finally:
        ctx.close()
        del k, t
        torch.cuda.empty_cache()
    want = torch.tensor([[-40.0, 3.0, 0.0]], dtype=torch.float64)
    assert bool(((c - want).abs() <= 1e-9 * 40.0).all()), c
