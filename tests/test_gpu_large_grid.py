"""Lines beyond grid index 1e9 of a grid near the largest (2^30 points), narrow
against a tile of the wing: the index of a line's centre decides which tiles
take it at their nodes, so it has to be the true one there too.  The points
around the lines against the oracle on a grid of their own.

Tolerance: binary64 as for the wing's nodes elsewhere, 400 * 2^-53 of each
(positive) term on both sides together: 1e-13; binary32 its bar of 1e-4.  The
spacing is 2^-17, so both grids hold the same nu_j."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hk = pytest.importorskip("paper_1503_03806_amd")

DNU, NU_MIN, POINTS = 2.0 ** -17, -7600.0, 1060000000


@pytest.mark.parametrize("precision,tol", [(hk.HK_F64, 1e-13), (hk.HK_F32_KAHAN, 1e-4)])
@pytest.mark.parametrize("at", [1050000000, 999000000])
def test_lines_beyond_1e9(precision, tol, at):
    n = 8192
    r = np.random.default_rng(at)
    lo = NU_MIN + (at - n // 2) * DNU
    lines = {"nu": np.sort(r.uniform(lo, lo + n * DNU, 40)), "S_ref": 10.0 ** r.uniform(-22, -20, 40),
             "E_lower": np.zeros(40), "gamma_air": np.full(40, 25.0 * DNU), "n_air": np.zeros(40)}
    # Doppler widths of ~2 points, Lorentz widths of 25: no series points
    cond = {"T": 4.0, "P": 1.0, "P_self": 0.0, "q_ratio": 1.0, "mass_amu": 500.0, "T0": 296.0}
    st = {k: cond[k] for k in ("T", "P", "P_self", "q_ratio")}
    ref, _ = oracle.opacity(lines, cond, {"nu_min": lo, "dnu": DNU, "n_points": n, "cutoff": 0.02})
    ctx = hk.Context(0)
    try:
        ctx.load_lines(lines, cond["mass_amu"], cond["T0"])
        grid = {"nu_min": NU_MIN, "dnu": DNU, "n_points": POINTS, "cutoff": 0.02}
        kap = ctx.opacity(st, grid, precision)
        got = kap[at - n // 2:at + n // 2].cpu().numpy()
        del kap
        assert ctx.stats()["evals_core"] == 0
    finally:
        ctx.close()
        torch.cuda.empty_cache()
    err = np.abs(got / ref - 1).max()
    print("precision %d, lines near point %d: max rel err %.2e" % (precision, at, err), flush=True)
    assert np.all(ref > 0) and err <= tol
