"""Small grids solved in one workgroup's registers: fields and statistics equal,
bit for bit, to the same solve run by slots (the asynchronous call)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# block heights (8, 16 and 24 rows), rows of 32 and 64 lanes, their edges and
# the first sizes past each; the last three run by slots in both calls
SIZES = [(1, 1), (2, 3), (3, 2), (5, 128), (32, 8), (63, 64), (64, 63), (64, 64), (64, 65), (61, 127), (64, 128),
         (65, 32), (65, 33), (127, 31), (128, 32), (128, 63), (128, 64), (96, 9), (128, 65), (101, 95),
         (128, 96), (128, 97), (65, 128), (64, 129)]


@pytest.fixture(scope="module")
def ctx():
    from paper_1903_07441_amd import twg
    c = twg.Context(0)
    yield c
    c.close()


def _grid(nx, ny, pad, seed):
    rng = np.random.default_rng(seed)
    c = np.zeros((ny, nx + pad), np.uint8)
    c[rng.random(c.shape) < 0.06] = 1
    c[rng.random(c.shape) < 0.03] = 4  # FIXED: keeps its value
    c[ny // 2, nx // 2] = 3
    u = rng.random(c.shape).astype(np.float32)
    cls = torch.as_tensor(c).cuda()[:, :nx]
    return cls, torch.as_tensor(u).cuda()[:, :nx]


def _both(ctx, cls, u, S, polish, **kw):
    from paper_1903_07441_amd import twg
    out = []
    slots = 0
    for _ in range(2):
        psi = torch.empty((u.shape[0], u.stride(0)), dtype=torch.float32, device="cuda")[:, :u.shape[1]]
        psi.copy_(u)
        p64 = torch.zeros((u.shape[0], u.stride(0)), dtype=torch.float64, device="cuda")[:, :u.shape[1]]
        p64 = p64 if polish else None
        if slots:
            st = ctx.relax_async(cls, psi, p64, slots=slots, sweeps_per_pass=S, polish=polish, **kw)
            torch.cuda.synchronize()
            st = twg.stats_from_device(st)
        else:
            st = ctx.relax(cls, psi, p64, sweeps_per_pass=S, polish=polish, **kw)
            # a slot a pass, a check, a defect and an update, and a few more
            slots = (st["sweeps"] + st["polish_sweeps"]) // S + 2 * st["checks"] + 3 * st["polish_rounds"] + 16
        out.append((psi, p64, st))
    (pa, da, sa), (pb, db, sb) = out
    assert sa == sb, (sa, sb)
    assert torch.equal(pa, pb)
    if polish:
        assert torch.equal(da, db)
    return sa


@pytest.mark.parametrize("pad", [0, 5])
@pytest.mark.parametrize("size", SIZES, ids=lambda s: f"{s[0]}x{s[1]}")
def test_equals_slots(ctx, size, pad):
    from paper_1903_07441_amd import twg
    nx, ny = size
    cls, u = _grid(nx, ny, pad, nx * 131 + ny)
    # FP32 to a tolerance; certified from a fresh and from a kept field
    _both(ctx, cls, u, 2, 0, tol=1e-5, init=twg.INIT_HALF)
    _both(ctx, cls, u, 4, 1, tol=1e-5, tol_cert=1e-9, init=twg.INIT_KEEP)
    _both(ctx, cls, u, 2, 1, tol=1e-7, init=twg.INIT_ZERO)


@pytest.mark.parametrize("kw", [dict(check_passes=1), dict(max_sweeps=1), dict(max_sweeps=37), dict(check_passes=3),
                                dict(max_sweeps=9000, omega=1.0, tol=1e-30)], ids=str)
def test_checks_and_budgets_equal_slots(ctx, kw):
    """Every pass checked, budgets that are no multiple of a pass, and more
    sweeps than one launch does."""
    from paper_1903_07441_amd import twg
    cls, u = _grid(64, 50, 0, 7)
    st = _both(ctx, cls, u, 2, 0, **{"tol": 1e-6, "init": twg.INIT_HALF, **kw})
    if kw.get("max_sweeps") == 9000:
        assert st["sweeps"] > 256


def test_not_finite_is_an_error(ctx):
    from paper_1903_07441_amd import twg
    cls, u = _grid(64, 64, 0, 9)
    cls[20, 20] = 4
    u[20, 20] = float("nan")
    with pytest.raises(twg.TwgError):
        ctx.relax(cls, u, tol=1e-6, init=twg.INIT_HALF)
