"""The reverse step on frames with tiles wholly inside the frame and off its border ring (plain
taps, no test per pixel) beside edge tiles: one such tile, several, quads and single loads of the
next adjoint.  Oracle and tolerance of test_gpu_sweep."""
import pytest

from test_gpu_sweep import test_reverse_step as reverse_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W", [(103, 104), (130, 163), (161, 200)])
@pytest.mark.parametrize("c_max", [1, 2, 3])
def test_inner_tiles(c_max, H, W):
    reverse_step(c_max, H, W)
