"""Streamed tiles of every height around a turn of their register ring: the
row loop opens with a turn that fills the pipeline and ends at the tile's last
row, so each remainder of the height is a path of its own.  Tiled and untiled
sweeps give the same bits."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [32, 64])
@pytest.mark.parametrize("nx", [150, 149])
@pytest.mark.parametrize("S", [1, 4, 6, 8])
def test_every_tile_height_matches_untiled(ctx, S, nx, bits):
    import torch
    from paper_1903_07441_amd import twg
    turn = 2 * (2 * S + 2)
    rng = np.random.default_rng(100 * S + nx)
    for RH in range(2, turn + turn // 2 + 4, 2):
        ny = 2 * RH + RH // 2 + 1  # two full tiles and a shorter, odd or even one
        cls = np.where(rng.random((ny, nx)) < 0.2, twg.OBST, twg.FREE).astype(np.uint8)
        u0 = torch.as_tensor(rng.random((ny, nx)), dtype=torch.float64 if bits == 64 else torch.float32)
        c = torch.as_tensor(cls).cuda()
        c2 = twg.Context(0)
        c2.set_graphs(False)
        c2.set_tiling(nx, ny, S, RH, 0.0, S, RH)
        tiled, plain = u0.cuda(), u0.cuda()
        for u, t in ((tiled, True), (plain, False)):
            if bits == 64:
                c2.sweeps64(c, u, 1.9, 2 * S, tiled=t)
            else:
                c2.sweeps(c, u, 1.9, 2 * S, tiled=t)
        assert torch.equal(tiled, plain), (S, RH, ny, nx)
        c2.close()
