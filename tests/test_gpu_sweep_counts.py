"""Fixed sweep counts of the library's own passes (an even number of them, of
unequal depth, after graph replays): the bits of one launch a colour."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

COUNTS = [0, 1, 2, 3, 7, 8, 9, 13, 16, 17, 24, 25, 41, 512, 513, 521]


@pytest.mark.parametrize("kind", ["f32", "source", "f64"])
@pytest.mark.parametrize("nx,ny,pitch", [(70, 45, 70), (129, 64, 131)])
def test_counts_equal_untiled(ctx, nx, ny, pitch, kind):
    rng = np.random.default_rng(nx)
    c = (rng.random((ny, pitch)) < 0.08).astype(np.uint8)
    c[ny // 2, nx // 2] = 3
    cls = torch.as_tensor(c).cuda()[:, :nx]
    dtype = torch.float64 if kind == "f64" else torch.float32
    u = torch.as_tensor(rng.random((ny, pitch))).to(dtype).cuda()
    f = torch.as_tensor(rng.normal(0.0, 1e-3, (ny, pitch))).float().cuda()[:, :nx] if kind == "source" else None
    for n in COUNTS:
        out = []
        for tiled in (True, False):
            t = u.clone()
            if kind == "f64":
                ctx.sweeps64(cls, t[:, :nx], 1.7, n, tiled=tiled)
            else:
                ctx.sweeps(cls, t[:, :nx], 1.7, n, tiled=tiled, f=f)
            out.append(t)
        assert torch.equal(*out), n
