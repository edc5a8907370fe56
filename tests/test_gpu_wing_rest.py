"""Lines near one leaf (64 points) of the binary64 wing: whole batches of 64 lie
a line per lane, a rest of up to 48 a point per lane, and both add to the
leaf's points in turn.  Counts around both limits, every point against the
oracle.

Tolerance: as for the wing's nodes elsewhere, 400 * 2^-53 of each (positive)
term on both sides together: 1e-13.  The grid is dyadic."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hk = pytest.importorskip("paper_1503_03806_amd")


@pytest.mark.parametrize("n_lines", [25, 48, 49, 63, 64, 65, 111, 112, 113, 128, 129, 1000])
def test_batches_and_a_rest(n_lines):
    grid = {"nu_min": 2000.0, "dnu": 0.0078125, "n_points": 64, "cutoff": 3.0}
    lines = synth.line_list(n_lines, 0.5, seed=n_lines)
    lines["nu"] = lines["nu"] + 2000.0
    cond = synth.conditions(900.0, 0.05)
    ctx = hk.Context(0)
    try:
        ctx.load_lines(lines, cond["mass_amu"], cond["T0"])
        got = ctx.opacity({k: cond[k] for k in ("T", "P", "P_self", "q_ratio")}, grid, hk.HK_F64).cpu().numpy()
    finally:
        ctx.close()
    ref, _ = oracle.opacity(lines, cond, grid)
    assert np.abs(got / ref - 1).max() <= 1e-13
