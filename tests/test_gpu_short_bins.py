"""The direct transmission of short bins (a thread per bin and mass, where there
are enough of them) and the fitted one of many bins (a wavefront per bin and 64
masses): sizes around both rules, values and masses of 0, infinite, NaN and
negative, and counts that need more than one launch.

Tolerance: a transmission's terms are positive and both sides form the same
product kappa m; the exponentials and the sums err by ~2 + 15 roundings: 1e-14;
1e-13 is asserted, above 1e-300 (denormal terms keep an absolute error).  The
fitted one as elsewhere: kappa at a node is an exponential of a sum of size
~60, ~60 * 20 roundings: 1e-12."""
import numpy as np
import pytest

from oracle import resample as R

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hk = pytest.importorskip("paper_1503_03806_amd")


@pytest.fixture(scope="module")
def ctx():
    c = hk.Context(0)
    yield c
    c.close()


def compare(got, ref):
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    inf = np.isinf(ref)
    assert np.array_equal(got[inf], ref[inf])
    ok = np.isfinite(ref)
    assert np.all(np.abs(got[ok] - ref[ok]) <= 1e-13 * np.abs(ref[ok]) + 1e-300)


@pytest.mark.parametrize("ppb", [1, 3, 4, 5, 63, 64, 65, 128, 255, 256, 257])
@pytest.mark.parametrize("n_m", [1, 65, 300])
@pytest.mark.parametrize("f32", [False, True])
def test_short_bins(ctx, ppb, n_m, f32):
    r = np.random.default_rng(ppb + n_m)
    n = 1000 * ppb + ppb // 2 if ppb < 100 or n_m == 300 else 3 * ppb + ppb // 2
    k = (10.0 ** r.uniform(-28, -16, n)).astype(np.float32 if f32 else np.float64)
    for i in range(0, n, ppb):
        k[i:i + ppb].sort()
    for bin, v in ((1, 0.0), (2, np.inf), (n // ppb - 1, np.nan), (n // ppb // 2, -1e-22)):
        k[bin * ppb + ppb - 1] = v
    m = np.concatenate([np.logspace(10, 30, n_m)[:max(n_m - 4, 1)], [0.0, 1e300, np.inf, -1e20]])[:n_m]
    with np.errstate(all="ignore"):
        ref = np.stack([R.transmission_direct(k[i:i + ppb].astype(np.float64), m) for i in range(0, n, ppb)])
    got = ctx.transmission_direct(torch.from_numpy(k).cuda(), ppb, torch.from_numpy(m).cuda(),
                                  precision=hk.HK_F32_KAHAN if f32 else hk.HK_F64).cpu().numpy()
    compare(got, ref)


@pytest.mark.parametrize("n_bins,n_m", [(1, 1), (3, 64), (4, 65), (5, 63), (1001, 10)])
def test_fitted_of_many_bins(ctx, n_bins, n_m):
    r = np.random.default_rng(n_bins)
    c = np.concatenate([r.uniform(-50, -40, (n_bins, 1)), r.normal(size=(n_bins, 7))], axis=1)
    if n_bins > 3:
        c[1, 3], c[2, 0] = np.nan, 800.0  # exp overflows
    m = np.logspace(14, 26, n_m)
    with np.errstate(all="ignore"):
        ref = np.stack([R.transmission_fit(x, m) for x in c])
    got = ctx.transmission(torch.from_numpy(c).cuda(), torch.from_numpy(m).cuda()).cpu().numpy()
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    ok = np.isfinite(ref)
    assert np.all(np.abs(got[ok] - ref[ok]) <= 1e-12 * np.maximum(np.abs(ref[ok]), 1.0))


@pytest.mark.parametrize("n_bins,n_m", [((1 << 23) + 5, 2), (1100000, 1000)])
def test_more_bins_than_a_launch_holds(ctx, n_bins, n_m):
    g = torch.Generator(device="cuda").manual_seed(1)
    k = torch.rand(n_bins, dtype=torch.float64, device="cuda", generator=g)
    m = torch.logspace(-3, 2, n_m, dtype=torch.float64, device="cuda")
    T = ctx.transmission_direct(k, 1, m)
    for b in range(0, n_bins, 1 << 17):
        ref = torch.exp(-k[b:b + (1 << 17), None] * m)
        assert bool(((T[b:b + (1 << 17)] - ref).abs() <= 1e-13 * ref).all())


def test_more_fits_than_a_launch_holds(ctx):
    n = (1 << 25) + 3
    c = torch.rand(n, 1, dtype=torch.float64, device="cuda", generator=torch.Generator(device="cuda").manual_seed(2))
    T = ctx.transmission(c, torch.ones(1, dtype=torch.float64, device="cuda"))
    assert bool(((T - torch.exp(-torch.exp(c))).abs() <= 1e-12).all())
