"""Bins above one LDS sort: sorted chunks merged two, four or eight runs at a
time, at the edges of chunks, runs and groups, with a merge's windows larger
than its LDS (runs of very different ranges), with equal keys, a short last
bin and n_points below a bin.  Sorting keys is exact: every comparison is
bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hk = pytest.importorskip("paper_1503_03806_amd")


@pytest.fixture(scope="module")
def ctx():
    c = hk.Context(0)
    yield c
    c.close()


def keys(kind, n, r):
    x = 10.0 ** r.uniform(-28, -16, n)
    if kind == "apart":  # every eighth run of 2048 spans the others, which are narrow
        x = 1e-20 * (1.0 + 1e-9 * r.uniform(size=n))
        run = np.arange(n) // 2048 % 8 == 0
        x[run] = 10.0 ** r.uniform(-28, -16, int(run.sum()))
    elif kind == "equal":
        x = r.choice(x[:7], n)
    elif kind == "special":
        x[r.permutation(n)[:n // 9]] = 0.0
        x[r.permutation(n)[:5]] = np.inf
        x[r.permutation(n)[:300]] = np.nan
    return x


@pytest.mark.parametrize("n,ppb", [(16385, 16385), (2 * 16385, 16385), (17001, 20000), (3000, 20000), (20480, 20480),
                                   (20481, 20481), (40961, 20000), (131072, 131072), (131073, 131073),
                                   (262144 + 77, 65537), (600001, 600001)])
@pytest.mark.parametrize("kind", ["plain", "apart", "equal", "special"])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_large_bins_sort_exactly(ctx, n, ppb, kind, dtype):
    x = torch.from_numpy(keys(kind, n, np.random.default_rng(n))).to(dtype).cuda()
    precision = hk.HK_F64 if dtype == torch.float64 else hk.HK_F32_KAHAN
    as_int = torch.int64 if dtype == torch.float64 else torch.int32
    g = np.array([0.01, 0.3, 0.5, 0.9, 0.9999])
    ref = x.view(as_int).cpu().numpy().copy()
    want = []
    for i in range(0, n, ppb):
        ref[i:i + ppb].sort()  # (non-negative keys: signed order is the order of the bits)
        m = min(ppb, n - i)
        want.append(ref[i + np.maximum(np.ceil(g * m).astype(int) - 1, 0)])
    want = torch.from_numpy(np.stack(want)).view(dtype).double()
    out = torch.empty_like(x)
    k = ctx.kdist(x, ppb, g, precision, out)
    assert np.array_equal(out.view(as_int).cpu().numpy(), ref)
    assert torch.equal(torch.nan_to_num(k.cpu(), nan=-1.0), torch.nan_to_num(want, nan=-1.0))
    k2 = ctx.kdist(x, ppb, g, precision)  # without the sorted keys
    assert torch.equal(torch.nan_to_num(k2, nan=-1.0), torch.nan_to_num(k, nan=-1.0))
    ctx.kdist(x, ppb, g, precision, x)  # in place
    assert torch.equal(x.view(as_int), out.view(as_int))
