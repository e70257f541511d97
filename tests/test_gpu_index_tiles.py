"""The index matrix and descents where rows are read four cells at a time and
where they are not (pitch, bases and sides off multiples of four), with values
that compare with nothing, and with more tiles than workgroups."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _index(cls, u):
    """Eq. 3 cell by cell of whole arrays: E, W, S, N, the first best one."""
    ny, nx = cls.shape
    best, bv = np.full(cls.shape, 4, np.uint8), np.zeros_like(u)
    for d, (dy, dx) in enumerate(((0, 1), (0, -1), (1, 0), (-1, 0))):
        ok, v = np.zeros(cls.shape, bool), np.zeros_like(u)
        to = (slice(max(0, -dy), ny - max(0, dy)), slice(max(0, -dx), nx - max(0, dx)))
        frm = (slice(max(0, dy), ny - max(0, -dy)), slice(max(0, dx), nx - max(0, -dx)))
        ok[to] = (cls[frm] == 0) | (cls[frm] == 3)
        v[to] = u[frm]
        ok &= (best == 4) | (v > bv)
        best[ok], bv[ok] = d, v[ok]
    best[~(bv > u)] = 4
    return best


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("nx,ny,pitch,shift", [(31, 40, 31, 0), (32, 33, 36, 0), (66, 70, 68, 0), (64, 96, 64, 1),
                                               (97, 64, 100, 2), (35, 35, 36, 3), (96, 32767, 96, 0)])
def test_index_matrix_of_any_layout(ctx, nx, ny, pitch, shift, f64):
    from paper_1903_07441_amd import twg
    rng = np.random.default_rng(nx * 7 + shift)
    cls = rng.choice([0, 0, 0, 0, 1, 2, 3, 4], (ny, nx)).astype(np.uint8)
    u = rng.choice(17, (ny, nx)).astype(np.float64 if f64 else np.float32) / 16.0  # many ties
    u[rng.random(u.shape) < 0.02] = np.nan
    u[rng.random(u.shape) < 0.02] = np.inf
    u[rng.random(u.shape) < 0.02] = -np.inf

    def put(a, fill):
        flat = torch.full((ny * pitch + shift + 8,), fill, dtype=torch.from_numpy(a).dtype, device="cuda")
        t = flat[shift:shift + ny * pitch].view(ny, pitch)
        t[:, :nx] = torch.as_tensor(a).cuda()
        return t

    c, t, idx = put(cls, 0), put(u, 5.0), put(np.full((ny, nx), 77, np.uint8), 77)
    kw = dict(psi64=t[:, :nx]) if f64 else dict(psi=t[:, :nx])
    ctx.index_matrix(c[:, :nx], idx=idx[:, :nx], **kw)
    got, want = idx.cpu().numpy(), _index(cls, u)
    assert np.array_equal(got[:, :nx], want)
    assert (got[:, nx:] == 77).all()
    # one descent, cell by cell
    walk = np.argwhere((cls == 0) | (cls == 3))
    y, x = walk[rng.integers(len(walk))]
    path, info = ctx.descend(c[:, :nx], start=(x, y), cap=ny * nx, **kw)
    cells = [(x, y)]
    while cls[y, x] != 3 and want[y, x] < 4:
        x, y = x + (1, -1, 0, 0)[want[y, x]], y + (0, 0, 1, -1)[want[y, x]]
        cells.append((x, y))
    assert info.tolist() == [len(cells), twg.OK if cls[y, x] == 3 else twg.NO_PATH]
    assert np.array_equal(path[:len(cells)].cpu().numpy(), np.array(cells))
