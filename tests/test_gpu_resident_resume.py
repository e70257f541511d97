"""A small grid's solve that needs several launches of the resident kernel: a
launch does 4096 sweeps' work, a check counting 16, so slow solves that check
after every pass are handed over between launches many times, in the FP32 stage
and in correction solves, and equal the same solve by slots bit for bit."""
import numpy as np
import pytest
import torch

import test_gpu_resident as resident

pytestmark = pytest.mark.gpu

WORK, CHECK = 4096, 16


@pytest.fixture(scope="module")
def ctx():
    from paper_1903_07441_amd import twg
    c = twg.Context(0)
    yield c
    c.close()


def _open(nx, ny, pad):
    """A free grid around one goal: as slow as its size gets."""
    c = np.zeros((ny, nx + pad), np.uint8)
    c[ny // 2, nx // 3] = 3
    u = np.random.default_rng(nx * ny).random(c.shape).astype(np.float32)
    return torch.as_tensor(c).cuda()[:, :nx], torch.as_tensor(u).cuda()[:, :nx]


# every block height (8, 16, 24 rows), rows of 32 and of 64 lanes
SIZES = [(60, 61), (63, 120), (127, 30), (101, 64), (128, 96)]


@pytest.mark.parametrize("S", [1, 2, 5])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_fp32_stage_over_several_launches(ctx, nx, ny, S):
    from paper_1903_07441_amd import twg
    cls, u = _open(nx, ny, 3)
    st = resident._both(ctx, cls, u, S, 0, tol=1e-30, omega=1.0, max_sweeps=2500, check_passes=1, init=twg.INIT_HALF)
    assert st["sweeps"] + CHECK * st["checks"] > 2 * WORK


@pytest.mark.parametrize("keep", [False, True])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_corrections_over_several_launches(ctx, nx, ny, keep):
    from paper_1903_07441_amd import twg
    cls, u = _open(nx, ny, 0)
    st = resident._both(ctx, cls, u, 1, 1, tol=1e-5, tol_cert=1e-8, omega=1.4, check_passes=1,
                        init=twg.INIT_KEEP if keep else twg.INIT_HALF)
    assert st["status"] == twg.OK and st["polish_rounds"] > 0
    # the corrections alone: a check a sweep
    assert (CHECK + 1) * st["polish_sweeps"] > 2 * WORK
