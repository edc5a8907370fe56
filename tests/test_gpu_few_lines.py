"""Work items of few lines in the binary64 opacity, taken a run of 256 points at a
time (up to 48 lines in blocks of 1024 points, 96 in blocks of 256), at those
limits, on grids that end inside a run, with windows, rules and series that end
inside it, lines outside the grouping range, and added to a grid.  Every point
against the oracle.

Tolerance: as for the wing's nodes elsewhere, 400 * 2^-53 of each (positive)
term on both sides together: 1e-13.  The grids are dyadic."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hk = pytest.importorskip("paper_1503_03806_amd")


@pytest.fixture(scope="module")
def ctx():
    c = hk.Context(0)
    yield c
    c.close()


def check(ctx, lines, cond, grid, tol=1e-13):
    ctx.load_lines(lines, cond["mass_amu"], cond["T0"])
    st = {k: cond[k] for k in ("T", "P", "P_self", "q_ratio")}
    got = ctx.opacity(st, grid, hk.HK_F64)
    ref, _ = oracle.opacity(lines, cond, grid)
    k = got.cpu().numpy()
    assert np.all(k[ref == 0] == 0)
    ok = ref != 0
    err = np.abs(k[ok] / ref[ok] - 1).max() if ok.any() else 0.0
    print("lines %d points %d: max rel err %.2e" % (len(lines["nu"]), grid["n_points"], err), flush=True)
    assert err <= tol
    # added to a grid: one rounding more
    base = torch.full_like(got, float(ref.max()))
    ctx.opacity(st, grid, hk.HK_F64, out=base, accumulate=True)
    want = ref.max() + ref
    assert np.abs(base.cpu().numpy() / want - 1).max() <= tol
    return got


def spread(n, lo, hi, seed):
    d = synth.line_list(n, 1.0, seed=seed)
    d["nu"] = np.random.default_rng(seed).uniform(lo, hi, n)
    d["nu"][:2] = (lo, hi)[:n]
    return d


FORMS = {
    "window_ends": (3.0, 900.0, 0.5, 28.0),
    "no_cutoff": (1e9, 1500.0, 1.0, 18.0),
    "wide_cores": (3.0, 3000.0, 1e-4, 1.0),
    "no_cores": (3.0, 300.0, 60.0, 44.0),
}


@pytest.mark.parametrize("form", sorted(FORMS))
@pytest.mark.parametrize("n_points", [1, 255, 256, 257, 700])
@pytest.mark.parametrize("n_lines", [1, 3, 95, 96, 97])
def test_blocks_of_256(ctx, form, n_points, n_lines):
    cut, T, P, mass = FORMS[form]
    grid = {"nu_min": 2000.0, "dnu": 0.0078125, "n_points": n_points, "cutoff": cut}
    lines = spread(n_lines, 1998.0, 2002.0 + n_points * 0.0078125, n_lines)
    check(ctx, lines, dict(synth.conditions(T, P), mass_amu=mass), grid)


@pytest.mark.parametrize("form", ["window_ends", "no_cutoff"])
@pytest.mark.parametrize("n_lines", [2, 47, 48, 49])
def test_blocks_of_1024(ctx, form, n_lines):
    cut, T, P, mass = FORMS[form]
    grid = {"nu_min": 2000.0, "dnu": 0.0078125, "n_points": 450001, "cutoff": cut}
    check(ctx, spread(n_lines, 2001.0, 5510.0, n_lines), dict(synth.conditions(T, P), mass_amu=mass), grid)


@pytest.mark.parametrize("n_lines", [5, 40])
def test_lines_outside_the_grouping_range(ctx, n_lines):
    """Centres within 1e-5 of zero: Doppler widths below 1e-11."""
    grid = {"nu_min": 0.0, "dnu": 2.0 ** -20, "n_points": 600, "cutoff": 2e-4}
    check(ctx, spread(n_lines, 1e-7, 1e-5, n_lines), synth.conditions(900.0, 1e-4), grid)
