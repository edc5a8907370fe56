"""The fit by matrix products and the transmissions with their saturated
exponentials left out, at the sizes where their dispatch changes: bins just
below, at and above 512 rows and the chunks' ends, bin counts around a group
of 16, coefficient counts around a 16-wide tile, a last bin shorter than a
chunk; few and many column masses and bins (segmented bins); masses and values
of 0, infinite, NaN, negative, tiny and huge.

Tolerances: coefficients 1e-9 of their largest, as for the fit elsewhere (the
two sides' QR factors differ by ~1e-13).  A transmission's terms are positive
and both sides form the same product kappa m; the exponentials and the sums of
up to 3e4 of them err by ~2 + 15 roundings: 1e-14; 1e-13 is asserted, above
1e-300 (denormal terms keep an absolute error)."""
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


def sorted_bins(n, ppb, seed):
    r = np.random.default_rng(seed)
    k = 10.0 ** r.uniform(-28, -16, n)
    for i in range(0, n, ppb):
        k[i:i + ppb].sort()
    return k


@pytest.mark.parametrize("n_bins,ppb,last", [(1, 511, 0), (1, 512, 0), (1, 513, 0), (2, 767, 0), (15, 768, 0),
                                             (16, 769, 40), (17, 1024, 1023), (33, 600, 33), (3, 5000, 64)])
@pytest.mark.parametrize("nc", [1, 16, 17, 32])
def test_fit_at_the_products_edges(ctx, n_bins, ppb, last, nc):
    n = n_bins * ppb + last
    k = sorted_bins(n, ppb, n + nc)
    c = ctx.resample(torch.from_numpy(k).cuda(), ppb, nc).cpu().numpy()
    ref = R.fit(k, ppb, nc)
    assert c.shape == ref.shape
    err = (np.abs(c - ref) / np.abs(ref).max(axis=1, keepdims=True)).max()
    print("bins %d x %d + %d, %d coefficients: %.2e" % (n_bins, ppb, last, nc, err), flush=True)
    assert err <= 1e-9


def compare(got, ref):
    bad = np.isnan(ref)
    assert np.array_equal(np.isnan(got), bad)
    inf = np.isinf(ref)
    assert np.array_equal(got[inf], ref[inf])
    ok = ~bad & ~inf
    assert np.all(np.abs(got[ok] - ref[ok]) <= 1e-13 * np.abs(ref[ok]) + 1e-300)


@pytest.mark.parametrize("n,ppb", [(1, 1), (63, 64), (65, 64), (4000, 511), (30000, 30000), (50001, 3000)])
@pytest.mark.parametrize("n_m", [1, 63, 65, 300])
def test_direct_transmission_splits(ctx, n, ppb, n_m):
    k = sorted_bins(n, ppb, n + n_m)
    m = np.logspace(-18, 30, n_m)
    got = ctx.transmission_direct(torch.from_numpy(k).cuda(), ppb, torch.from_numpy(m).cuda()).cpu().numpy()
    compare(got, np.stack([R.transmission_direct(k[i:i + ppb], m) for i in range(0, n, ppb)]))


@pytest.mark.parametrize("special", ["plain", "zero", "inf", "nan", "unsorted"])
def test_transmissions_of_special_values(ctx, special):
    ppb, n = 700, 2100
    k = sorted_bins(n, ppb, 5)
    if special == "zero":
        k[:3] = 0.0
    elif special == "inf":
        k[ppb - 2:ppb] = np.inf
    elif special == "nan":
        k[2 * ppb - 1] = np.nan
    elif special == "unsorted":
        k = k[np.random.default_rng(1).permutation(n)]
    m = np.concatenate([[0.0, 1e-320, 1e300, np.inf], np.logspace(10, 30, 90), [-1e20, 1e19]])
    with np.errstate(all="ignore"):
        ref = np.stack([R.transmission_direct(k[i:i + ppb], m) for i in range(0, n, ppb)])
        got = ctx.transmission_direct(torch.from_numpy(k).cuda(), ppb, torch.from_numpy(m).cuda()).cpu().numpy()
        compare(got, ref)
        if special in ("plain", "zero"):
            coef = R.fit(k, ppb, 20)
            tf = ctx.transmission(torch.from_numpy(coef).cuda(), torch.from_numpy(m).cuda()).cpu().numpy()
            want = np.stack([R.transmission_fit(c, m) for c in coef])
            ok = np.isfinite(want)
            assert np.array_equal(np.isnan(tf), np.isnan(want))
            # (kappa at a node is an exponential of a 20-term sum of size ~60:
            # ~60 * 20 roundings, times the exponent where it matters, <= ~1)
            assert np.all(np.abs(tf[ok] - want[ok]) <= 1e-12 * np.maximum(np.abs(want[ok]), 1.0))
