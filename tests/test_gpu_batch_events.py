"""The batch's control launches (only where a check can be): solves that end
at every distance from the checks' quantum, at a sweep budget or at a fixed
number of slots, and the residual a check reports; and the heights the device
chooses for the tiles."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

SIDES = [(64, 40), (97, 33), (130, 70)]
S = 2


@pytest.fixture(scope="module")
def ctx():
    from paper_1903_07441_amd import twg
    c = twg.Context(0)
    yield c
    c.close()


def _pack():
    rng = np.random.default_rng(5)
    descs, cls, at = [], [], 0
    for nx, ny in SIDES:
        c = np.zeros((ny, nx), np.uint8)
        c[0, :] = c[-1, :] = c[:, 0] = c[:, -1] = 2
        c[rng.integers(2, ny - 2, 12), rng.integers(2, nx - 2, 12)] = 1
        c[ny // 2, nx // 2] = 3
        descs.append((nx, ny, nx, at))
        cls.append(c)
        at += c.size
    return descs, cls, np.concatenate([c.ravel() for c in cls])


def _residual(c, u):
    """max |avg4(u) - u| over the free cells, in float64."""
    p = np.pad(u.astype(np.float64), 1)
    r = ((p[1:-1, 2:] + p[1:-1, :-2]) + (p[2:, 1:-1] + p[:-2, 1:-1])) * 0.25 - p[1:-1, 1:-1]
    return np.abs(r[c == 0]).max()


@pytest.mark.parametrize("asynchronous", [False, True])
@pytest.mark.parametrize("passes", [1, 2, 3, 4, 5, 6, 7, 8, 9, 21])
def test_budget_ends_between_events(ctx, passes, asynchronous):
    from paper_1903_07441_amd import twg
    descs, cls, flat = _pack()
    dc = torch.as_tensor(flat).cuda()
    psi = torch.zeros(flat.size, dtype=torch.float32, device="cuda")
    kw = dict(tol=1e-30, max_sweeps=S * passes, omega=1.7, sweeps_per_pass=S)
    if asynchronous:
        # a few slots more than the budget: the budget's event ends the solve
        stats = twg.batch_stats_from_device(ctx.relax_batched(dc, psi, descs, slots=passes + 3, **kw), len(descs))
    else:
        stats = ctx.relax_batched(dc, psi, descs, **kw)
    got = psi.cpu().numpy()
    for (nx, ny, _, at), c, st in zip(descs, cls, stats):
        one = torch.where(torch.as_tensor(c).cuda() == 3, 1.0,
                          torch.where(torch.as_tensor(c).cuda() == 0, 0.5, 0.0)).float()
        ctx.sweeps(torch.as_tensor(c).cuda(), one, 1.7, S * passes, tiled=False)
        u = got[at:at + nx * ny].reshape(ny, nx)
        assert st["sweeps"] == S * passes and st["status"] != 0, (passes, st)
        assert np.array_equal(u, one.cpu().numpy()), passes
        # every operation of the check is the reference's: the same bits
        assert st["residual"] == _residual(c, u), (passes, st)


# the least height, below and at the first and second heights of whole windows
# (2 (S + 1) k - 4 S rows), and more rows than any grid has
@pytest.mark.parametrize("S,rows", [(8, 2), (8, 20), (8, 22), (8, 24), (8, 40), (8, 42), (8, 128), (8, 2000), (1, 2),
                                    (1, 8), (1, 10), (1, 500), (3, 12), (3, 14), (3, 128), (4, 0), (7, 0)])
def test_chosen_tile_heights_give_the_same_bits(ctx, S, rows):
    rng = np.random.default_rng(S * 1000 + rows)
    descs, flat, at = [], [], 0
    for nx, ny in [(64, 64), (33, 201), (300, 7), (130, 257), (128, 1)] * 3:
        c = np.zeros((ny, nx), np.uint8)
        c[rng.random(c.shape) < 0.05] = 1
        c[ny // 2, nx // 2] = 3
        descs.append((nx, ny, nx, at))
        flat.append(c)
        at += c.size
    dc = torch.as_tensor(np.concatenate([c.ravel() for c in flat])).cuda()
    psi = torch.zeros(at, dtype=torch.float32, device="cuda")
    stats = ctx.relax_batched(dc, psi, descs, tol=1e-6, omega=1.5, sweeps_per_pass=S, rows_per_tile=rows)
    for (nx, ny, _, o), c, st in zip(descs, flat, stats):
        dcl = torch.as_tensor(c).cuda()
        one = torch.where(dcl == 3, 1.0, torch.where(dcl == 0, 0.5, 0.0)).float()
        ctx.sweeps(dcl, one, 1.5, st["sweeps"], tiled=False)
        assert st["status"] == 0 and torch.equal(one.view(-1), psi[o:o + nx * ny]), (nx, ny, st)


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_check_reports_what_is_not_finite(ctx, bad):
    """A NaN in one grid's fixed cells stops the batch as an error, an
    infinity (whose differences become NaN after a sweep) as well."""
    from paper_1903_07441_amd import twg
    descs, cls, flat = _pack()
    nx, ny, _, at = descs[1]
    flat = flat.copy()
    k = at + 5 * nx + 70
    flat[k] = 4  # FIXED: keeps its value
    psi = torch.zeros(flat.size, dtype=torch.float32, device="cuda")
    psi[k] = bad
    with pytest.raises(twg.TwgError):
        ctx.relax_batched(torch.as_tensor(flat).cuda(), psi, descs, tol=1e-5, omega=1.7, sweeps_per_pass=S)
