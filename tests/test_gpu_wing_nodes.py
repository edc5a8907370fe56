"""The binary64 wing takes a line at Chebyshev nodes of the largest tile (1024,
256 or 64 points) that admits it and point by point elsewhere.  Grids that end
at and around the tiles' edges, lists of one line to more than a wavefront's
list holds, and the forms that decide where a line is admitted (cutoff, none,
in Lorentz widths, shorter than a tile; pressures with and without a core;
coarse and fine grids; grids too fine for the nodes), every point against the
oracle.

Tolerance: all terms are positive, so a per-term relative error bounds the
sum's.  A term's: S(T) takes an exponent of size <= 100 (100 * 2^-53 on either
side), widths and the rules' rationals ~40 roundings on either side, the
interpolation 4e-17 of the value and ~3 * 24 roundings of the node sums:
together below 400 * 2^-53 = 4.5e-14; 1e-13 is asserted.  The grids are dyadic,
so that both sides hold the same nu_j (else nu_j differs by an ulp of 2000,
2.3e-13, against widths of 0.005: 1e-9 near the cores)."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hk = pytest.importorskip("paper_1503_03806_amd")

TOL = 1e-13


@pytest.fixture(scope="module")
def ctx():
    c = hk.Context(0)
    yield c
    c.close()


def check(ctx, n_lines, grid, T, P, tol=TOL, seed=31, extra=None, margin=8.0):
    lo, hi = grid["nu_min"], grid["nu_min"] + grid["n_points"] * grid["dnu"]
    lines = synth.line_list(n_lines, hi - lo + 2 * margin, seed=seed)
    lines["nu"] = lines["nu"] + lo - margin
    lines.update(extra or {})
    cond = synth.conditions(T, P)
    ctx.load_lines(lines, cond["mass_amu"], cond["T0"])
    st = {k: cond[k] for k in ("T", "P", "P_self", "q_ratio")}
    got = ctx.opacity(st, grid, hk.HK_F64).cpu().numpy()
    ref, _ = oracle.opacity(lines, cond, grid)
    zero = ref == 0
    assert np.all(got[zero] == 0)
    err = np.abs(got[~zero] / ref[~zero] - 1).max() if (~zero).any() else 0.0
    print("lines %d points %d dnu %g T %g P %g: max rel err %.2e" % (n_lines, grid["n_points"], grid["dnu"], T, P, err),
          flush=True)
    assert err <= tol


@pytest.mark.parametrize("n_points", [1, 63, 64, 65, 255, 256, 257, 1023, 1024, 1025, 2048 + 17, 5000])
@pytest.mark.parametrize("n_lines", [1, 24, 25, 900])
def test_grid_ends_and_list_sizes(ctx, n_points, n_lines):
    check(ctx, n_lines, {"nu_min": 2000.0, "dnu": 0.0078125, "n_points": n_points, "cutoff": 6.0}, 1500.0, 0.5)


FORMS = {
    "no_cutoff": ({"cutoff": 1e9}, 0.0078125, 1500.0, 1.0),
    "short_cutoff": ({"cutoff": 0.11}, 0.0078125, 1500.0, 1.0),
    "lorentz_widths": ({"cutoff": 0.0, "cutoff_lorentz": 500.0}, 0.0078125, 2000.0, 0.3),
    "high_pressure": ({"cutoff": 20.0}, 0.0078125, 400.0, 100.0),
    "low_pressure": ({"cutoff": 20.0}, 0.0078125, 2000.0, 1e-5),
    "coarse_grid": ({"cutoff": 25.0}, 0.5, 1500.0, 1.0),
    "fine_grid": ({"cutoff": 1.5}, 2.0 ** -12, 1500.0, 0.1),
}


@pytest.mark.parametrize("form", sorted(FORMS))
def test_forms(ctx, form):
    cut, dnu, T, P = FORMS[form]
    n = 6000 if dnu > 2.0 ** -12 else 20000
    check(ctx, 2500, dict(cut, nu_min=2000.0, dnu=dnu, n_points=n), T, P)


def test_shifted_and_natural_widths(ctx):
    r = np.random.default_rng(5)
    extra = {"gamma_self": r.uniform(0.1, 0.5, 2500), "delta": r.uniform(-0.02, 0.02, 2500),
             "A21": 10.0 ** r.uniform(0, 8, 2500)}
    check(ctx, 2500, {"nu_min": 2000.0, "dnu": 0.0078125, "n_points": 6000, "cutoff": 9.0}, 1200.0, 2.0, extra=extra)


def test_dense_list_fills_the_near_lists(ctx):
    """5e4 lines within 3 cm^-1: thousands of lines near every leaf."""
    check(ctx, 50000, {"nu_min": 2000.0, "dnu": 0.0078125, "n_points": 300, "cutoff": 4.0}, 1500.0, 0.5, margin=0.3)


def test_grids_too_fine_for_the_nodes(ctx):
    """Spacings near an ulp of the wavenumber, where positions within a tile
    are no longer evenly spaced: every line point by point."""
    check(ctx, 100, {"nu_min": 2000.0, "dnu": 2.0 ** -38, "n_points": 3000, "cutoff": 4.0}, 1500.0, 0.5, margin=2.0)
