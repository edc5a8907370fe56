"""The radix sort's short cut after the high words of binary64 keys, at its
limits: runs of 31 to 34 keys with one high word that are all alike, or alike
but for one key that is less or more (in the first, the middle or the last
place of the input), alone and among other keys, in bins of one workgroup and in
chunks that are merged; and the same runs as line centres, whose order carries
the input index.  Bit for bit against a stable host sort."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hk = pytest.importorskip("paper_1503_03806_amd")


@pytest.fixture(scope="module")
def ctx():
    c = hk.Context(0)
    yield c
    c.close()


def runs(length, odd, scale, rng):
    """Runs of `length` keys of one high word each: two low words apart at the
    place `odd` (None: all alike), by less and by more."""
    out = []
    for sign in (-1, 1):
        for base in rng.uniform(1.0, 2.0, 6):
            k = np.full(length, np.float64(base * scale)).view(np.uint64)
            k = (k & ~np.uint64(0xFFFFFFFF)) | np.uint64(0x7FFFFFFF)
            if odd is not None:
                k[odd] = np.uint64(int(k[odd]) + sign * int(rng.integers(1, 1 << 30)))
            out.append(k.view(np.float64))
    return out


@pytest.mark.parametrize("length", [2, 16, 17, 31, 32, 33, 34, 65])
@pytest.mark.parametrize("place", ["none", "first", "middle", "last"])
@pytest.mark.parametrize("others", [0, 2000, 40000])
def test_runs_of_one_high_word(ctx, length, place, others):
    rng = np.random.default_rng(length + others)
    odd = {"none": None, "first": 0, "middle": length // 2, "last": length - 1}[place]
    parts = runs(length, odd, 1e-20, rng)
    if others:
        # whole runs between other keys, and some zeros (a long run of equal keys)
        rest = np.array_split(10.0 ** rng.uniform(-28, -16, others), len(parts))
        rest[0][: others // 40] = 0.0
        parts = [x for pair in zip(parts, rest) for x in pair]
    k = np.concatenate(parts)
    out = torch.empty(k.size, dtype=torch.float64, device="cuda")
    kg = ctx.kdist(torch.from_numpy(k).cuda(), k.size, [0.25, 0.5, 0.999], sorted_out=out).cpu().numpy()
    want = np.sort(k)
    assert np.array_equal(out.cpu().numpy().view(np.uint64), want.view(np.uint64))
    rank = np.ceil(np.array([0.25, 0.5, 0.999]) * k.size).astype(int) - 1
    assert np.array_equal(kg[0], want[rank])


@pytest.mark.parametrize("length", [31, 32, 33, 34])
@pytest.mark.parametrize("place", ["none", "first", "middle", "last"])
def test_line_centres(ctx, length, place):
    rng = np.random.default_rng(length)
    odd = {"none": None, "first": 0, "middle": length // 2, "last": length - 1}[place]
    nu = np.concatenate(runs(length, odd, 1500.0, rng) + [rng.uniform(1400.0, 3100.0, 500)])
    lines = synth.line_list(nu.size, 1.0, seed=length)
    lines["nu"] = nu
    cond = synth.conditions(900.0, 0.3)
    st = {k: cond[k] for k in ("T", "P", "P_self", "q_ratio")}
    grid = {"nu_min": 1400.0, "dnu": 0.125, "n_points": 13600, "cutoff": 20.0}
    order = np.argsort(nu, kind="stable")
    got = []
    for d in (lines, {k: np.ascontiguousarray(v[order]) for k, v in lines.items()}):
        ctx.load_lines(d, cond["mass_amu"], cond["T0"])
        got.append(ctx.opacity(st, grid, hk.HK_F64).cpu().numpy())
    assert np.array_equal(got[0], got[1])
