"""Tables of more states than one launch holds the work items of (a narrow list
whose tiles are cut: 3 items of 256 threads per tile, 240 tiles, 23500 states:
more than 2^32 threads): every state's k(g) is that of its own opacity, bit for
bit, whichever batch it falls in."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hk = pytest.importorskip("paper_1503_03806_amd")


def test_more_states_than_a_launch_holds():
    n, n_states = 61440, 23500
    lines = synth.line_list(1100, n * 0.01, seed=3)
    lines["nu"] = lines["nu"] + 2000.0
    states = []
    for T, P in ((900.0, 0.3), (1500.0, 1.0)):
        c = synth.conditions(T, P)
        states.append({k: c[k] for k in ("T", "P", "P_self", "q_ratio")})
    grid = {"nu_min": 2000.0, "dnu": 0.01, "n_points": n, "cutoff": 1e9}
    g, _ = hk.hk_gauss_legendre(4)
    ctx = hk.Context(0)
    try:
        ctx.load_lines(lines, c["mass_amu"], c["T0"])
        want = []
        for st in states:
            kap = ctx.opacity(st, grid, hk.HK_F64)
            assert ctx.get_option("wing_items") >= 3 * (n // 256)
            want.append(ctx.kdist(kap, 8192, g))
        tab = ctx.tables([states[i % 2] for i in range(n_states)], grid, 8192, g, hk.HK_F64)
        for x in range(2):
            assert bool((tab[x::2] == want[x]).all())
    finally:
        ctx.close()
        torch.cuda.empty_cache()
