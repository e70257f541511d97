"""The convolutions pick their tile height, and the weight gradients their
splits, by the number of workgroups: one image alone and the same image
repeated in a batch run different tilings of the same products."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _net(ctx):
    from paper_1903_07441_amd import learn, twg
    p = learn.he_init(3)
    p += 0.01 * np.random.default_rng(4).standard_normal(p.size).astype(np.float32)  # biases too
    return twg.UNet(ctx, p)


@pytest.mark.parametrize("shape", [(8, 8), (24, 40), (64, 136), (256, 264)])
def test_forward_bits_do_not_depend_on_the_tiling(ctx, shape):
    import torch
    H, W = shape
    net = _net(ctx)
    x = torch.as_tensor(np.random.default_rng(H).random((1, H, W, 3)), dtype=torch.float32).cuda()
    alone = net.forward(x)
    for n in (2, 5, 40):
        y = net.forward(x.expand(n, H, W, 3).contiguous())
        assert torch.equal(y, alone.expand(n, H, W)), n


@pytest.mark.parametrize("shape", [(8, 8), (24, 40), (64, 136), (128, 160)])
def test_gradients_do_not_depend_on_the_splits(ctx, shape):
    """The mean over n copies of an image has the gradients of the image.
    FP32 sums in other groupings: a chain of at most a few hundred additions
    of 2^-24 each stays within 2e-5 of the vector's norm."""
    import torch
    H, W = shape
    net = _net(ctx)
    rng = np.random.default_rng(W)
    x = torch.as_tensor(rng.random((1, H, W, 3)), dtype=torch.float32).cuda()
    t = torch.as_tensor(rng.random((1, H, W)), dtype=torch.float32).cuda()
    c = torch.as_tensor((rng.random((1, H, W)) < 0.2).astype(np.uint8)).cuda()
    got = []
    for n in (1, 8, 32):  # powers of two: the per-pixel gradients keep their bits
        g = torch.zeros(net.n_params, device="cuda")
        net.loss_grad(*(a.expand(n, *a.shape[1:]).contiguous() for a in (x, t, c)), None, g)
        got.append(g.double())
    for g in got[1:]:
        assert float((g - got[0]).norm() / got[0].norm()) < 2e-5
