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


@pytest.mark.parametrize("bits", [32, 64])
@pytest.mark.parametrize("pad", [0, 1, 2])
@pytest.mark.parametrize("nx", [1, 2, 3, 104, 129, 255])
def test_any_width_and_pitch_match_untiled(ctx, nx, pad, bits):
    """Two columns per access at any width, pitch and alignment: the cells
    between the rows (NaN here) are neither used nor written."""
    import torch
    from paper_1903_07441_amd import twg
    ny, n = 37, 13  # 13 sweeps: a pass of 8 and the rest
    rng = np.random.default_rng(nx + 10 * pad)
    dt = torch.float64 if bits == 64 else torch.float32
    cls = np.where(rng.random((ny, nx)) < 0.2, twg.OBST, twg.FREE).astype(np.uint8)
    u0 = torch.as_tensor(rng.random((ny, nx)), dtype=dt)
    out = []
    for tiled in (True, False):
        flat = torch.full((1 + ny * (nx + pad),), float("nan"), dtype=dt, device="cuda")
        u = flat[1:].view(ny, nx + pad)[:, :nx]  # starts one element into its allocation
        u.copy_(u0)
        c = torch.full((ny, nx + pad), twg.FREE, dtype=torch.uint8, device="cuda")[:, :nx]
        c.copy_(torch.as_tensor(cls))
        f = ctx.sweeps64 if bits == 64 else ctx.sweeps
        f(c, u, 1.7, n, tiled=tiled)
        out.append(u.cpu())
        gaps = flat[1:].view(ny, nx + pad)[:, nx:]
        assert torch.isnan(flat[0]) and torch.isnan(gaps).all()
    assert torch.equal(*out)


@pytest.mark.parametrize("S", [2, 4])
@pytest.mark.parametrize("shape", [(60, 61), (333, 200), (520, 505)])
def test_fused_passes_match_single_passes(ctx, shape, S):
    """A blocking solve does several passes per launch between its checks;
    with the caller's own tile height it does one.  The same field, sweeps
    and checks, with and without a polish and a sweep budget."""
    import torch
    from paper_1903_07441_amd import twg
    nx, ny = shape
    rng = np.random.default_rng(nx)
    cls = np.where(rng.random((ny, nx)) < 0.01, twg.OBST, twg.FREE).astype(np.uint8)
    cls[0, :] = cls[-1, :] = cls[:, 0] = cls[:, -1] = twg.WALL
    cls[ny // 2, nx // 3] = twg.GOAL
    c = torch.as_tensor(cls).cuda()
    for kw in (dict(), dict(polish=1, tol_cert=1e-8), dict(max_sweeps=37 * S), dict(check_passes=5)):
        got = []
        for rows in (0, 16):
            u = torch.zeros((ny, nx), device="cuda")
            v = torch.zeros((ny, nx), dtype=torch.float64, device="cuda")
            st = ctx.relax(c, u, v if kw.get("polish") else None, sweeps_per_pass=S, rows_per_tile=rows, **kw)
            got.append((u, v, st))
        assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1]), kw
        assert got[0][2] == got[1][2], kw
