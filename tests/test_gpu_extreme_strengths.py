"""Line strengths at the ends of binary64's range in the binary64 opacity: a
line whose strength overflows (or is NaN) at the state makes the points of its
own window infinite (or NaN) and changes no other; lists so weak that kappa lies
near 1e-285 keep their precision.  Every point against the oracle.

Tolerance: as for the wing's nodes elsewhere, 400 * 2^-53 of each (positive)
term on both sides together: 1e-13.  The grids are dyadic."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hk = pytest.importorskip("paper_1503_03806_amd")

GRID = {"nu_min": 2000.0, "dnu": 0.0078125, "n_points": 6000, "cutoff": 9.0}


def both(lines, cond, grid):
    ctx = hk.Context(0)
    try:
        ctx.load_lines(lines, cond["mass_amu"], cond["T0"])
        got = ctx.opacity({k: cond[k] for k in ("T", "P", "P_self", "q_ratio")}, grid, hk.HK_F64).cpu().numpy()
    finally:
        ctx.close()
    with np.errstate(all="ignore"):
        ref, _ = oracle.opacity(lines, cond, grid)
    return got, ref


def compare(got, ref):
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(np.isinf(got), np.isinf(ref))
    ok = np.isfinite(ref) & (ref > 0)
    assert np.all(got[ref == 0] == 0)
    err = np.abs(got[ok] / ref[ok] - 1).max()
    print("%d of %d points finite, max rel err %.2e" % (np.isfinite(ref).sum(), ref.size, err), flush=True)
    assert err <= 1e-13


@pytest.mark.parametrize("n_lines", [20, 2500])
@pytest.mark.parametrize("special", ["inf", "nan", "1e200"])
def test_one_line_out_of_range(n_lines, special):
    lines = synth.line_list(n_lines, 60.0, seed=n_lines)
    lines["nu"] = lines["nu"] + 1992.0
    cond = dict(synth.conditions(250.0, 0.5), q_ratio=1e12)
    at = n_lines // 2
    lines["nu"][at] = 2020.123
    lines["S_ref"][at], lines["E_lower"][at] = {"inf": (1e300, 0.0), "nan": (0.0, -1e8), "1e200": (1e188, 0.0)}[special]
    got, ref = both(lines, cond, dict(GRID, cutoff=2.0 if special == "nan" else 9.0))
    assert special == "1e200" or 0 < (~np.isfinite(ref)).sum() < 4000
    compare(got, ref)


@pytest.mark.parametrize("cutoff", [9.0, 25.0])
@pytest.mark.parametrize("scale", [1e-258, 1e-264])
def test_weak_lists(cutoff, scale):
    """Strengths of cold states' highest levels: kappa near 1e-280 and 1e-286."""
    lines = synth.line_list(2500, 60.0, seed=9)
    lines["nu"] = lines["nu"] + 1992.0
    lines["S_ref"] = lines["S_ref"] * scale
    lines["E_lower"] = np.zeros(2500)
    got, ref = both(lines, synth.conditions(1500.0, 0.5), dict(GRID, cutoff=cutoff))
    compare(got, ref)
