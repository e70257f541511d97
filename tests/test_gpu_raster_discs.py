"""Discs of every size against the oracle: wider than the 32 columns from which
a row is cut to the disc's chord and the ring's intervals, on both sides of the
radius where squares leave 32 bits, shared by 1 to 16 waves, and cut by the
tiles of a small map."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# (nx, ny, pitch, obstacles, W): small maps around their tiles' sides, then two
# launches with many and with few pairs
CASES = [(65, 70, 65, 12, 9), (64, 72, 72, 5, 300), (128, 128, 131, 190, 400), (1, 600, 3, 20, 31), (40, 300, 40, 9, 50),
         (200, 150, 200, 1, 1000), (300, 221, 304, 7, 8), (257, 380, 260, 40, 3), (640, 500, 640, 3, 64)]


def _check(orc, sc, pitch, **kw):
    from paper_1903_07441_amd import twg
    ctx = twg.Context(0)
    nx, ny = sc["nx"], sc["ny"]
    dev = [torch.as_tensor(np.ascontiguousarray(sc[k], dtype=np.float64)).cuda() for k in ("pos", "vel", "rad")]
    cls = torch.full((ny, pitch), 77, dtype=torch.uint8, device="cuda")
    ctx.rasterize(nx, ny, sc["robot"], sc["goal"], *dev, W=sc["W"], robot_speed=sc["vr"], cls=cls[:, :nx],
                  want_ring=False, **kw)
    want, _ = orc.rasterize_modes(sc, **kw)
    got = cls.cpu().numpy()
    assert np.array_equal(got[:, :nx], want)
    assert (got[:, nx:] == 77).all()
    ctx.close()


def _scenario(nx, ny, n, W, rng, rad, vel):
    sc = dict(nx=nx, ny=ny, W=W, vr=1.0, robot=np.array([nx // 2, ny // 3], np.int32),
              goal=np.array([nx // 4, ny // 4], np.int32))
    sc.update(pos=rng.uniform([-0.2 * nx, -0.2 * ny], [1.2 * nx, 1.2 * ny], (n, 2)), rad=rad,
              vel=rng.normal(0.0, vel, (n, 2)) if vel else np.zeros((n, 2)))
    return sc


@pytest.mark.parametrize("per_object", [False, True])
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0]}x{c[1]}")
def test_discs_of_every_size(orc, case, per_object):
    nx, ny, pitch, n, W = case
    rng = np.random.default_rng(nx + ny)
    for rad in (rng.uniform(0.0, 16.0, n), rng.uniform(16.0, 60.0, n), rng.uniform(253.5, 254.5, n),
                10.0 ** rng.uniform(0.0, 5.5, n)):
        pos = _scenario(nx, ny, n, W, rng, rad, 0.3)
        if rad.max() > 60.0:  # centres at the radius: the edge crosses the map
            a = rng.uniform(0.0, 2.0 * np.pi, n)
            pos["pos"] = pos["robot"] + (rad * rng.uniform(0.97, 1.03, n))[:, None] * np.stack([np.cos(a), np.sin(a)], 1)
        _check(orc, pos, pitch, ring_mode=0, per_object=per_object)
        _check(orc, pos, pitch, ring_mode=1, heading=(0.6, 0.8), per_object=True)


@pytest.mark.parametrize("nx,ny,n,W", [(65, 70, 2, 60), (200, 150, 1, 500), (200, 150, 6, 8), (120, 90, 30, 3)])
def test_elliptical_rings_of_large_discs(orc, nx, ny, n, W):
    """Discs that end beyond the map's farthest cell."""
    rng = np.random.default_rng(n)
    far = np.hypot(nx, ny)
    sc = _scenario(nx, ny, n, W, rng, rng.uniform(0.6, 2.0, n) * far, 0.0)
    a = rng.uniform(0.0, 2.0 * np.pi, n)
    sc["pos"] = sc["robot"] + (sc["rad"] * rng.uniform(0.9, 1.0, n))[:, None] * np.stack([np.cos(a), np.sin(a)], 1)
    _check(orc, sc, nx + 3, ring_mode=1, heading=(-0.6, 0.8), per_object=False)
