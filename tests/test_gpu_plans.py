"""A pass's work plans are made by one workgroup each where they are small (up
to 16 states, 16384 (state, tile) pairs) and by parallel passes beyond; cut
tiles' partial sums are added in the finish.  hk_tables of 3 states (one
workgroup) and of 17 (parallel passes) against hk_opacity of each state (one
workgroup), bit for bit, on a list that crowds into part of a ragged grid (so
that tiles of the wing and of the series are cut) and on an even one, and
against the oracle at the precisions' bars (1e-6, 1e-4)."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hk = pytest.importorskip("paper_1503_03806_amd")

GRID = {"nu_min": 0.0, "dnu": 0.01, "n_points": 60011, "cutoff": 10.0}


@pytest.fixture(scope="module")
def ctx():
    c = hk.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("n_states", [3, 17])
@pytest.mark.parametrize("crowded", [True, False])
@pytest.mark.parametrize("prec,bar", [(hk.HK_F64, 1e-6), (hk.HK_F32_KAHAN, 1e-4)])
def test_tables_equal_single_calls_across_the_plans(ctx, n_states, crowded, prec, bar):
    lines = synth.line_list(8000, 40.0 if crowded else 600.0, seed=61)
    if crowded:
        lines["nu"] = lines["nu"] + 300.0
    conds = [synth.conditions(400.0 + 150.0 * i, 10.0 ** (-2 + 0.2 * i)) for i in range(n_states)]
    states = [{k: c[k] for k in ("T", "P", "P_self", "q_ratio")} for c in conds]
    ctx.load_lines(lines, conds[0]["mass_amu"], conds[0]["T0"])
    g, _ = hk.hk_gauss_legendre(20)
    tab = ctx.tables(states, GRID, 5000, g, prec).cpu().numpy()
    for i, st in enumerate(states):
        kap = ctx.opacity(st, GRID, prec)
        if crowded:
            assert ctx.get_option("wing_segment_lines") > 0
        one = ctx.kdist(kap, 5000, g).cpu().numpy()
        assert np.array_equal(one.view(np.uint64), tab[i].view(np.uint64)), i
        if i in (0, n_states - 1):
            ref, _ = oracle.opacity(lines, conds[i], GRID)
            k = kap.cpu().numpy()
            nz = ref > 0
            assert np.all(k[~nz] == 0)
            err = np.abs(k[nz] / ref[nz] - 1).max()
            print("states %d crowded %d precision %d state %d: %.2e" % (n_states, crowded, prec, i, err), flush=True)
            assert err <= bar
