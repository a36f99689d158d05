"""Colour likelihood on both sides of its launch rule (tiles halved for one or four components up to two
workgroups a CU; the fit inside the next pass up to 512 tiles, 256 with four components), against the
FP64 oracle; bars as in test_gpu_gmm."""
import pytest

from paper_1008_0502_amd import synth

from test_gpu_gmm import _check, _prior, _torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,M", [(1024, 512, 1), (1025, 512, 1), (1024, 1024, 1), (1025, 1024, 1), (513, 1024, 2),
                                   (1025, 1024, 3), (1025, 512, 4)])
def test_rule(H, W, M):
    _torch()
    print(f"\n[case] gmm rule {H}x{W} M={M}", flush=True)
    spec = synth.single_ellipse_spec(H=H, W=W, T=1, seed=H + M)
    spec.axes = (W / 5, H / 6)
    frames, masks = synth.Clip(spec).stack()
    _check(frames[0], _prior(masks[0], 3 * H + W), M, 2, 1e-4, f"{H}x{W}")
