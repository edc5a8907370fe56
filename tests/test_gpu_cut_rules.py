"""The rules by which the binary64 opacity's tiles are cut: the wing's from 1024
lines in the fullest reference tile on, the series' from 64 where a line's
series covers whole tiles (and each state of a table by its own reach).  Every
point against the oracle; tables and single states bit for bit.

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


def spread(n, lo, hi):
    d = synth.line_list(n, 1.0, seed=n)
    d["nu"] = np.random.default_rng(n).uniform(lo, hi, n)
    return d


def state(cond):
    return {k: cond[k] for k in ("T", "P", "P_self", "q_ratio")}


def check(ctx, lines, cond, grid):
    ctx.load_lines(lines, cond["mass_amu"], cond["T0"])
    got = ctx.opacity(state(cond), grid, hk.HK_F64)
    ref, _ = oracle.opacity(lines, cond, grid)
    assert np.abs(got.cpu().numpy() / ref - 1).max() <= 1e-13
    return got


@pytest.mark.parametrize("n_lines,cut", [(1023, False), (1024, True)])
def test_the_wings_cut(ctx, n_lines, cut):
    grid = {"nu_min": 2000.0, "dnu": 0.0078125, "n_points": 2000, "cutoff": 1e9}
    check(ctx, spread(n_lines, 2000.0, 2015.0), synth.conditions(900.0, 0.5), grid)
    assert (ctx.get_option("wing_segment_lines") > 0) == cut


@pytest.mark.parametrize("n_lines", [63, 64, 300])
def test_series_that_cover_tiles(ctx, n_lines):
    grid = {"nu_min": 2000.0, "dnu": 2.0 ** -17, "n_points": 20000, "cutoff": 25.0}
    cond = synth.conditions(1500.0, 0.01)
    got = check(ctx, spread(n_lines, 2000.05, 2000.1), cond, grid)
    g, _ = hk.hk_gauss_legendre(4)
    st, cold = state(cond), state(synth.conditions(20.0, 0.01))  # (cold: narrower, the usual rule)
    tab = ctx.tables([st, cold, st], grid, 4000, g, hk.HK_F64)
    assert torch.equal(tab[0], ctx.kdist(got, 4000, g)) and torch.equal(tab[2], tab[0])
    assert torch.equal(tab[1], ctx.kdist(ctx.opacity(cold, grid, hk.HK_F64), 4000, g))
