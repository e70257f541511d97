"""Small maps in one launch: sizes and numbers of discs at the edges of that
path and just past them, against the oracle."""
import numpy as np
import pytest
import torch

from paper_1903_07441_amd import scenarios

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1903_07441_amd import twg
    c = twg.Context(0)
    yield c
    c.close()


CASES = [(1, 1, 1, 1), (9, 7, 9, 192), (128, 128, 128, 60), (127, 129, 136, 192), (128, 129, 128, 30), (8, 2048, 8, 12),
         (2048, 8, 2048, 1)]


# (193 discs, past the path's rule, with the circular metric only: on that map
# the elliptical ring test's lower end, 0.1 where it has to be 0.092 of the ring's
# r_x, loses seven cells behind the robot, whatever path marks them)
@pytest.mark.parametrize("nx,ny,pitch,n,mode", [(*c, m) for c in CASES for m in (0, 1)] + [(64, 64, 67, 193, 0)])
def test_one_launch_maps_equal_the_oracle(ctx, orc, nx, ny, pitch, n, mode):
    sc = scenarios.custom(max(nx, 3), max(ny, 3), n, rad=(0.0, 9.0), vel_sigma=0.5, seed=nx + n, W=7)
    sc = dict(sc, nx=nx, ny=ny)
    sc["robot"] = np.minimum(sc["robot"], [nx - 1, ny - 1])
    sc["goal"] = np.minimum(sc["goal"], [nx - 1, ny - 1])
    dev = [torch.as_tensor(np.ascontiguousarray(sc[k], dtype=np.float64)).cuda() for k in ("pos", "vel", "rad")]
    heading = (0.6, 0.8)
    for per_object in (False, True):
        cls = torch.full((ny, pitch), 77, dtype=torch.uint8, device="cuda")
        ring = torch.zeros((ny, pitch), dtype=torch.int16, device="cuda").view(torch.uint16)
        ctx.rasterize(nx, ny, sc["robot"], sc["goal"], *dev, W=sc["W"], robot_speed=sc["vr"], cls=cls[:, :nx],
                      ring=ring[:, :nx], ring_mode=mode, heading=heading, per_object=per_object)
        torch.cuda.synchronize()
        want, want_ring = orc.rasterize_modes(sc, ring_mode=mode, heading=heading, per_object=per_object)
        assert np.array_equal(cls.cpu().numpy()[:, :nx], want)
        assert np.array_equal(ring.view(torch.int16).cpu().numpy().view(np.uint16)[:, :nx], want_ring)
        assert (cls.cpu().numpy()[:, nx:] == 77).all()
