"""Streamed tiles of every height at the pass depths that test_gpu_tile_rows
leaves out (an autotuner may keep any of them)."""
import pytest

import test_gpu_tile_rows as rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [32, 64])
@pytest.mark.parametrize("nx", [150, 149])
@pytest.mark.parametrize("S", [2, 3, 5, 7])
def test_every_tile_height_at_other_depths(ctx, S, nx, bits):
    rows.test_every_tile_height_matches_untiled(ctx, S, nx, bits)
