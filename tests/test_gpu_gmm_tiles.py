"""Colour likelihood at the edges of its tiles (256 pixels a workgroup up to 256 workgroups, then as
many as keep it there, 2048 from 524288 pixels on) and on both sides of the rule that puts the fit
into the next pixel pass (256 tiles), against the FP64 oracle; bars as in test_gpu_gmm."""
import numpy as np
import pytest

from paper_1008_0502_amd import synth

from test_gpu_gmm import _check, _gpu, _prior, _torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,M,iters", [(16, 16, 1, 1), (17, 19, 2, 2), (120, 160, 4, 3), (256, 256, 3, 0), (257, 256, 3, 2),
                                         (513, 640, 2, 1), (721, 1001, 1, 2), (600, 1024, 3, 1), (600, 1024, 4, 0)])
def test_tiles(H, W, M, iters):
    _torch()
    print(f"\n[case] gmm {H}x{W} M={M} iters={iters}", flush=True)
    spec = synth.single_ellipse_spec(H=H, W=W, T=1, seed=H + M)
    spec.axes = (W / 5, H / 6)
    frames, masks = synth.Clip(spec).stack()
    _check(frames[0], _prior(masks[0], 3 * H + W), M, iters, 1e-4, f"{H}x{W}")


@pytest.mark.parametrize("H,W", [(64, 96), (600, 1024)])
def test_a_label_without_weight_keeps_its_costs(H, W):
    _torch()
    from paper_1008_0502_amd.api import Params
    print(f"\n[case] gmm one label {H}x{W}", flush=True)
    rng = np.random.default_rng(H)
    frame = rng.integers(0, 256, (H, W, 3), dtype=np.uint8)
    U, prm = _gpu(frame, np.ones((H, W), np.float32), Params(gmm_components=2, gmm_iters=2))
    assert np.all(U[0] == 0.0) and np.all(prm[0] == 0.0)
    assert np.all(np.isfinite(U[1])) and np.any(U[1] != 0.0)
