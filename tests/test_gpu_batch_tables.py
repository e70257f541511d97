"""A batch's device tables when their buffer grows under the same grids (more,
lower tiles): they are uploaded again, whatever address the new buffer has."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lds", [False, True])
def test_grown_buffer_gets_its_tables(lds):
    from paper_1903_07441_amd import twg
    rng = np.random.default_rng(11)
    sides, descs, at = [(1024, 1024), (40, 30), (513, 700)], [], 0
    for nx, ny in sides:
        descs.append((nx, ny, nx, at))
        at += nx * ny
    cls = torch.as_tensor((rng.random(at) < 0.05).astype(np.uint8)).cuda()  # OBST
    for nx, ny, _, off in descs:
        cls[off + (ny // 2) * nx + nx // 2] = 3
    kw = dict(tol=1e-30, max_sweeps=32, omega=1.6, sweeps_per_pass=8, lds=lds)
    ctx, fields = twg.Context(0), []
    # the tables of the first call fit 3 waves a SIMD; 2-row tiles need more
    for rows in (128, 2, 128):
        psi = torch.zeros(at, device="cuda")
        st = ctx.relax_batched(cls, psi, descs, rows_per_tile=rows, **kw)
        assert [s["sweeps"] for s in st] == [32] * 3
        fields.append(psi)
    fresh = twg.Context(0)
    psi = torch.zeros(at, device="cuda")
    fresh.relax_batched(cls, psi, descs, rows_per_tile=2, **kw)
    for f in fields:
        assert torch.equal(f, psi)
    ctx.close()
    fresh.close()
