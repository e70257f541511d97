"""Set-up of a field's cells on narrow grids (several rows a wave) and at wide,
odd pitches."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,pad", [(1, 5000, 0), (2, 300, 1), (3, 1100, 0), (8, 513, 3), (33, 129, 0), (63, 200, 2),
                                       (64, 257, 0), (65, 257, 0), (4099, 300, 1)])
def test_every_cell_is_set_once(ctx, nx, ny, pad):
    from paper_1903_07441_amd import twg
    g = torch.Generator(device="cuda").manual_seed(nx + ny)
    cls = torch.randint(0, 5, (ny, nx + pad), dtype=torch.uint8, device="cuda", generator=g)
    u = torch.rand((ny, nx + pad), device="cuda", generator=g)
    want = torch.where(cls == twg.FREE, 0.5, torch.where(cls == twg.GOAL, 1.0, torch.where(cls == twg.FIXED, u, 0.0)))
    want[:, nx:] = u[:, nx:]
    psi = u.clone()
    ctx.init_field(cls[:, :nx], psi[:, :nx], init=twg.INIT_HALF)
    assert torch.equal(psi, want)
    # the mask, by a solve of no sweeps and by one sweep against the untiled one
    a, b = psi.clone(), psi.clone()
    ctx.sweeps(cls[:, :nx], a[:, :nx], 1.2, 1)
    ctx.sweeps(cls[:, :nx], b[:, :nx], 1.2, 1, tiled=False)
    assert torch.equal(a, b)
    c = u.clone()
    ctx.relax(cls[:, :nx], c[:, :nx], tol=1e30, init=twg.INIT_HALF)
    assert torch.equal(c, want)
