"""The order of an unordered device list, (nu, input index), at the sizes where
its sort changes: one chunk, chunk edges, two to nine runs, a second merge pass;
with equal centres within and across chunks, an ordered and a reversed list,
and centres close together beside a few far away (merge windows beyond LDS).
The opacity of the device list equals that of the same list ordered on the host
by a stable sort, bit for bit: lines of equal centre have different
intensities, so their order shows in the sums."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hk = pytest.importorskip("paper_1503_03806_amd")

STATE = {"T": 700.0, "P": 0.3, "P_self": 0.1, "q_ratio": 0.5}
GRID = {"nu_min": 0.0, "dnu": 0.05, "n_points": 20000, "cutoff": 5.0}


@pytest.fixture(scope="module")
def ctx():
    c = hk.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("n", [1, 2, 255, 2047, 2048, 2049, 4097, 8193, 16385, 18433, 131073, 270001])
@pytest.mark.parametrize("kind", ["plain", "equal", "reversed", "apart"])
def test_device_order_equals_a_stable_host_sort(ctx, n, kind):
    L = synth.line_list(n, 1000.0, seed=n)
    r = np.random.default_rng(n)
    nu = r.permutation(L["nu"])
    if kind == "equal":
        nu = np.round(nu, 1 if n < 10000 else 0) + 0.5
    elif kind == "reversed":
        nu = np.sort(nu)[::-1].copy()
    elif kind == "apart":
        far = np.arange(n) // 2048 % 8 == 0
        nu = np.where(far, nu, 500.0 + 1e-4 * r.uniform(size=n))
    L["nu"] = nu
    order = np.argsort(nu, kind="stable")
    out = []
    for d in ({k: torch.from_numpy(np.ascontiguousarray(v)).cuda() for k, v in L.items()},
              {k: np.ascontiguousarray(v[order]) for k, v in L.items()}):
        ctx.load_lines(d, 18.0)
        out.append(ctx.opacity(STATE, GRID, hk.HK_F32_KAHAN).cpu().numpy())
    assert np.array_equal(out[0], out[1])
    assert out[0].max() > 0.0


def test_order_of_a_list_beyond_the_merges(ctx):
    n = (1 << 24) + 4099
    g = torch.Generator(device="cuda").manual_seed(1)
    u = lambda a, b: torch.rand(n, dtype=torch.float64, device="cuda", generator=g) * (b - a) + a
    L = {"nu": torch.round(u(1.0, 60000.0), decimals=2), "S_ref": u(1e-28, 1e-22), "E_lower": u(0.0, 3000.0),
         "gamma_air": u(0.02, 0.1), "n_air": u(0.4, 0.8)}
    order = torch.sort(L["nu"], stable=True).indices
    out = []
    for d in (L, {k: v[order].contiguous() for k, v in L.items()}):
        ctx.load_lines(d, 18.0)
        out.append(ctx.opacity(STATE, GRID, hk.HK_F32_KAHAN).cpu().numpy())
    assert np.array_equal(out[0], out[1]) and out[0].max() > 0.0
