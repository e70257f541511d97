"""The network's inputs and outputs on maps whose rows are aligned for wide
loads and on the same maps at other pitches and bases: equal bits; and the
inputs' counts against their definitions."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1903_07441_amd import twg
    c = twg.Context(0)
    yield c
    c.close()


def _at(a, pitch, shift, fill):
    """a copied to the device at a pitch, `shift` elements past an aligned base"""
    ny, nx = a.shape
    buf = torch.full((ny * pitch + shift,), fill, dtype=a.dtype, device="cuda")
    t = buf[shift:].view(ny, pitch)[:, :nx]
    t.copy_(a)
    return t


@pytest.mark.parametrize("nx,ny", [(8, 8), (64, 40), (61, 67), (521, 33), (1024, 16)])
def test_rows_aligned_or_not_give_the_same(ctx, nx, ny):
    from paper_1903_07441_amd import learn, twg
    rng = np.random.default_rng(nx)
    c = torch.as_tensor(rng.choice(np.array([0, 0, 0, 1, 2, 3, 4], np.uint8), (ny, nx)))
    r = torch.as_tensor(rng.integers(0, 1000, (ny, nx)).astype(np.int16))
    r[-1, -1] = 1234  # the largest, in the last cell
    goal = (nx // 2, ny // 2)
    net = twg.UNet(ctx, learn.he_init(5))
    got = []
    for pitch, shift in [((nx + 15) // 16 * 16, 0), (nx + 3, 0), ((nx + 15) // 16 * 16, 1)]:
        cls, ring = _at(c, pitch, shift, 1), _at(r, pitch, shift, 30000).view(torch.uint16)
        out = [net.features(cls, ring, goal)]
        for f in (4, 8):
            out += list(net.features_coarse(cls, ring, goal, f))
            psi = _at(torch.zeros(ny, nx), pitch, shift, 9.0)
            net.warm_start_coarse(cls, ring, goal, psi, f)
            out.append(psi.contiguous())
        psi = _at(torch.zeros(ny, nx), pitch, shift, 9.0)
        net.warm_start(cls, ring, goal, psi)
        out.append(psi.contiguous())
        got.append(out)
    for other in got[1:]:
        assert all(torch.equal(a, b) for a, b in zip(got[0], other))
    # occupancy shares and masks of the coarse blocks, by their definition
    for k, f in ((1, 4), (4, 8)):
        x, cc = got[0][k].cpu().numpy(), got[0][k + 1].cpu().numpy()
        full = np.ones((x.shape[0] * f, x.shape[1] * f), np.float32)
        full[:ny, :nx] = np.isin(c.numpy(), (1, 2))
        free = np.zeros(full.shape, bool)
        free[:ny, :nx] = c.numpy() == 0
        blocks = lambda a: a.reshape(x.shape[0], f, x.shape[1], f)
        assert np.array_equal(x[..., 0], blocks(full).sum((1, 3)) / np.float32(f * f))
        assert np.array_equal(cc == 0, blocks(free).any((1, 3)))
    net.close()
