"""The binary64 wing's block size follows the grid points between the first
and the last line centre: lists on a small part of a large grid, at its ends
and outside it, of one line, and just below and above the limit of 400000
points, every point against the oracle; and the same bits from a list loaded
from the host and from device memory, in order and not, from hk_tables and
from a stream of one chunk.

Tolerance: as for the interpolated wing elsewhere, all terms are positive and
a term errs by less than 400 * 2^-53 = 4.5e-14 on both sides together; 1e-13 is
asserted.  The grids are dyadic, so that both sides hold the same nu_j."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hk = pytest.importorskip("paper_1503_03806_amd")

DNU = 0.0078125
GRID = {"nu_min": 2000.0, "dnu": DNU, "n_points": 450000, "cutoff": 3.0}


@pytest.fixture(scope="module")
def ctx():
    c = hk.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("n_lines,first,last", [
    (1, 2100.0, 2100.0),
    (700, 2000.0, 2040.0),
    (700, 5470.0, 5515.0),  # the grid ends at 5515.6
    (300, 1990.0, 1999.0),  # left of the grid
    (300, 5516.0, 5530.0),  # right of it
    (900, 1900.0, 6000.0),
    (500, 2100.0, 2100.0 + 399990 * DNU),
    (500, 2100.0, 2100.0 + 400010 * DNU),
])
def test_lists_on_a_part_of_the_grid(ctx, n_lines, first, last):
    lines = synth.line_list(n_lines, 1.0, seed=n_lines)
    nu = first + (last - first) * np.random.default_rng(3).uniform(size=n_lines)
    nu[:2] = (first, last)[:n_lines]
    lines["nu"] = nu
    cond = synth.conditions(900.0, 0.4)
    st = {k: cond[k] for k in ("T", "P", "P_self", "q_ratio")}
    order = np.argsort(nu, kind="stable")
    ordered = {k: np.ascontiguousarray(v[order]) for k, v in lines.items()}
    got = []
    for d in (lines, ordered, {k: torch.from_numpy(v).cuda() for k, v in lines.items()}):
        ctx.load_lines(d, cond["mass_amu"], cond["T0"])
        got.append(ctx.opacity(st, GRID, hk.HK_F64).cpu().numpy())
    g, _ = hk.hk_gauss_legendre(4)
    k_tab = ctx.tables([st, st], GRID, 10000, g, hk.HK_F64).cpu().numpy()
    k_one = ctx.kdist(torch.from_numpy(got[0]).cuda(), 10000, g).cpu().numpy()
    assert np.array_equal(got[1], got[0]) and np.array_equal(got[2], got[0])
    assert np.array_equal(k_tab[0], k_one) and np.array_equal(k_tab[1], k_one)
    stream = ctx.opacity_stream([lines], cond["mass_amu"], st, GRID, hk.HK_F64, T_ref=cond["T0"]).cpu().numpy()
    assert np.array_equal(stream, got[0])
    ref, _ = oracle.opacity(ordered, cond, GRID)
    zero = ref == 0
    assert np.all(got[0][zero] == 0)
    if (~zero).any():
        assert np.abs(got[0][~zero] / ref[~zero] - 1).max() <= 1e-13
