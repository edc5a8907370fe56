"""The fit and the direct transmission of one context on two streams that
nothing orders, and in captured graphs.  Both split work over partial sums in
scratch of the context; a call on one stream must not disturb one in flight on
another, and a graph must hold no scratch that a later call grows, nor need an
allocation while it is captured.

Two streams: the same kernels on the same inputs, so the bits of a call alone.
Graphs: a captured call takes the kernels without scratch, whose sums are
associated otherwise: 1e-9 of the largest coefficient (the bar of the fit) and
1e-13 (positive terms), as for these calls elsewhere; replays are bitwise alike."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
hk = pytest.importorskip("paper_1503_03806_amd")

PPB = 27000


def bins(n, seed, ppb=PPB):
    r = np.random.default_rng(seed)
    k = np.sort(10.0 ** r.uniform(-28, -16, (n, ppb)), axis=1)
    return torch.from_numpy(k.reshape(-1)).cuda()


CALLS = {
    "direct": lambda c, k, m: c.transmission_direct(k, PPB, m),
    "fit": lambda c, k, m: c.resample(k, PPB, 20),
}


@pytest.fixture
def ctx():
    c = hk.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


@pytest.mark.parametrize("first,second", [("direct", "direct"), ("direct", "fit"), ("fit", "direct"), ("fit", "fit")])
@pytest.mark.parametrize("default_first", [True, False])
def test_calls_on_two_streams(ctx, first, second, default_first):
    m = [torch.logspace(15, 27, 37, dtype=torch.float64, device="cuda"),
         torch.logspace(18, 24, 40, dtype=torch.float64, device="cuda")]
    k = [bins(3, 1), bins(5, 2)]
    f = [CALLS[first], CALLS[second]]
    ctx.use_current_stream()
    alone = [f[x](ctx, k[x], m[x]) for x in range(2)]  # (also makes the factors)
    s = [torch.cuda.default_stream() if default_first else torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    got = []
    for _ in range(20):
        for x in range(2):
            with torch.cuda.stream(s[x]):
                ctx.use_current_stream()
                got.append(f[x](ctx, k[x], m[x]))
    torch.cuda.synchronize()
    ctx.use_current_stream()
    for i, g in enumerate(got):
        assert torch.equal(g, alone[i % 2]), i


@pytest.mark.parametrize("default_first", [True, False])
def test_fits_of_two_sizes_on_two_streams(ctx, default_first):
    """A bin size of its own has factors of its own: making them must not
    disturb a fit that is still reading the others'."""
    size = [20000, 9000]
    k = [bins(200, 5, size[0]), bins(300, 6, size[1])]
    ctx.use_current_stream()
    alone = [ctx.resample(k[x], size[x], 20) for x in range(2)]
    s = [torch.cuda.default_stream() if default_first else torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    got = []
    for _ in range(10):
        for x in range(2):
            with torch.cuda.stream(s[x]):
                ctx.use_current_stream()
                got.append(ctx.resample(k[x], size[x], 20))
    torch.cuda.synchronize()
    ctx.use_current_stream()
    for i, g in enumerate(got):
        assert torch.equal(g, alone[i % 2]), i


def close(kind, a, b):
    if kind == "fit":
        return bool(((a - b).abs() <= 1e-9 * b.abs().amax(dim=1, keepdim=True)).all())
    return bool(((a - b).abs() <= 1e-13 * b.abs() + 1e-300).all())


@pytest.mark.parametrize("kind", ["direct", "fit"])
def test_captured_calls(ctx, kind):
    m = torch.logspace(15, 27, 37, dtype=torch.float64, device="cuda")
    k, more = bins(3, 3), bins(40, 4)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    if kind == "fit":  # the factors of a bin size are made by its first call
        ctx.use_current_stream()
        CALLS[kind](ctx, k, m)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        ctx.use_current_stream()
        out = CALLS[kind](ctx, k, m)
    ctx.use_current_stream()
    want = CALLS[kind](ctx, k, m)
    first = None
    for _ in range(3):
        graph.replay()
        CALLS[kind](ctx, more, m)  # the scratch grows (40 bins against 3)
        eager = CALLS[kind](ctx, k, m)
        torch.cuda.synchronize()
        assert torch.equal(eager, want)
        assert close(kind, out, want)
        first = out.clone() if first is None else first
        assert torch.equal(out, first)
        out.zero_()
