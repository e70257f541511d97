"""A descent captured into a graph in a context that has only run
descent_all: nothing is left to allocate."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,pitch", [(33, 70, 36), (300, 170, 300)])
def test_descend_is_captured_after_descent_all(nx, ny, pitch):
    from paper_1903_07441_amd import twg
    ctx = twg.Context(0)
    ys, xs = np.mgrid[0:ny, 0:pitch]
    u = 1.0 / (1.0 + np.hypot(xs - nx // 2, ys - ny // 3))
    c = np.zeros((ny, pitch), np.uint8)
    c[ny // 3, nx // 2] = twg.GOAL
    cls, psi64 = torch.as_tensor(c).cuda()[:, :nx], torch.as_tensor(u).cuda()[:, :nx]
    start = (nx - 1, ny - 1)
    steps = ctx.descent_all(cls, psi64=psi64)
    path = torch.full((nx * ny, 2), -7, dtype=torch.int32, device="cuda")
    info = torch.zeros(2, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    g, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        g.capture_begin()
        ctx.descend(cls, psi64=psi64, start=start, path=path, info=info)
        g.capture_end()
    torch.cuda.current_stream().wait_stream(side)
    want, want_info = ctx.descend(cls, psi64=psi64, start=start)
    n = want_info.tolist()[0]
    assert want_info.tolist() == [int(steps[start[1], start[0]]) + 1, twg.OK]
    for _ in range(3):
        path.fill_(-7)
        info.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(info, want_info)
        assert torch.equal(path[:n], want[:n]) and bool((path[n:] == -7).all())
        ctx.descend(cls, psi64=psi64, start=(0, 0))  # eager work on the same scratch
    ctx.close()
