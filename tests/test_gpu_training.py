"""Surrogate training batches around a workgroup's 64 samples and around the
sample list's end."""
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


@pytest.mark.parametrize("n,batch", [(100, 64), (100, 65), (100, 63), (300, 257), (64, 200), (5000, 4096)])
def test_training_wraps_its_samples_like_gradients_of_the_gathered_batch(ctx, n, batch):
    """Steps take consecutive samples cyclically: after a first step, the
    second step's loss and update equal those of a plain gradient over the
    gathered samples, bit for bit (the same kernel, from sample 0)."""
    x, y = synth.surrogate_samples(n, seed=9)
    x, y = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    z = ctx.surrogate_labels(x, y)
    ctx.surrogate_set_params(synth.mlp_init(3))
    ctx.surrogate_train(x, y, z, batch, 1, 1e-3)
    idx = torch.arange(batch, 2 * batch, device="cuda") % n
    _, want = ctx.surrogate_grad(x[idx].contiguous(), y[idx].contiguous(), z[idx].contiguous())
    hist = ctx.surrogate_train(x, y, z, batch, 1, 1e-3)
    assert torch.equal(hist, want)
