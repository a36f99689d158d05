"""Minimum cut across tile borders (push tiles of 16, relabel tiles of 32) against the integer
oracle, bit for bit: frames at, below and just above a tile, one row, one column; strong n-links
and few sinks, so that excess travels through many tiles and rounds; nothing to push at all."""
import numpy as np
import pytest

from test_gpu_mincut import _compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W", [(16, 16), (17, 33), (32, 64), (33, 31), (1, 70), (70, 1), (64, 200)])
@pytest.mark.parametrize("kind", ["far", "noise", "none"])
def test_tiles(H, W, kind):
    print(f"\n[case] min cut {kind} {H}x{W}", flush=True)
    rng = np.random.default_rng(H * 1000 + W)
    unary = rng.integers(0, 9, (2, H, W)).astype(np.float32)
    pairwise = rng.integers(0, 30, (4, H, W)).astype(np.float32)
    if kind == "far":     # sources at one end, sinks at the other, everything between neutral
        unary[:] = 0
        q = max(1, W // 8) if W > 1 else 0
        if W > 1:
            unary[0, :, :q], unary[1, :, -q:] = 50, 60
        else:
            unary[0, :8], unary[1, -8:] = 50, 60
    elif kind == "none":  # no pixel has excess
        unary[0] = 0
    _compare(unary, pairwise, 1.0, f"{kind} {H}x{W}")
