"""A binary64 stream whose chunks take both block sizes of the wing (line centres
on more and on fewer than 400000 points): each lane is sized for the smallest
tiles of all chunks, so that a second stream alike allocates nothing (growing a
buffer waits for the device) though its chunks fall on the other lanes; and the
result is that of the chunks one call at a time, bit for bit."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hk = pytest.importorskip("paper_1503_03806_amd")


def test_second_stream_allocates_nothing():
    n = 1 << 26
    grid = {"nu_min": 2000.0, "dnu": 2.0 ** -12, "n_points": n, "cutoff": 0.5}
    cond = synth.conditions(900.0, 0.4)
    st = {k: cond[k] for k in ("T", "P", "P_self", "q_ratio")}
    chunks = []
    for lo, hi in ((2000.0, 12000.0), (5000.0, 5050.0)):
        d = synth.line_list(300, 1.0, seed=int(lo))
        d["nu"] = np.sort(np.random.default_rng(int(lo)).uniform(lo, hi, 300))
        chunks.append(d)
    ctx = hk.Context(0)
    try:
        out = torch.empty(n, dtype=torch.float64, device="cuda")
        free = []
        for _ in range(2):
            ctx.opacity_stream(chunks, cond["mass_amu"], st, grid, hk.HK_F64, T_ref=cond["T0"], out=out)
            torch.cuda.synchronize()
            free.append(torch.cuda.mem_get_info()[0])
        assert free[0] == free[1]
        want = torch.empty_like(out)
        for c, d in enumerate(chunks):
            ctx.load_lines(d, cond["mass_amu"], cond["T0"])
            ctx.opacity(st, grid, hk.HK_F64, out=want, accumulate=c > 0)
        assert torch.equal(out, want)
    finally:
        ctx.close()
        torch.cuda.empty_cache()
