"""Moments of the colour mixtures where heavy samples (black, weight 1) and light ones (white, weight
1e-7) alternate every 1024 pixels: a thread's FP32 sum of both kinds would round the light ones away
(half a unit in the last place of 4 is 2.4e-7), sums of four samples joined in FP64 keep them.  The
start's means against the FP64 oracle: their average is the label's mean, about 1e-7, from FP32 means of
about 3e-4 (spacing 3e-11): bar 1e-9, against an error of 5e-8 and more when the light samples are lost."""
import numpy as np
import pytest

from oracle import gmm as Gm

from test_gpu_gmm import _gpu, _torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,M", [(512, 1024, 2), (1024, 1024, 2), (1024, 1024, 3), (1024, 1024, 4), (1536, 1024, 2)])
def test_light_samples_are_kept(H, W, M):
    _torch()
    from paper_1008_0502_amd.api import Params
    print(f"\n[case] gmm light samples {H}x{W} M={M}", flush=True)
    light = (np.arange(H * W).reshape(H, W) // 1024) % 2 == 1
    frame = np.repeat(np.where(light, 255, 0).astype(np.uint8)[:, :, None], 3, 2)
    prior = np.where(light, 1e-7, 1.0).astype(np.float32)
    _, prm = _gpu(frame, prior, Params(gmm_components=M, gmm_iters=0))
    _, mixes = Gm.colour_likelihood(frame, prior.astype(np.float64), M=M, iters=0)
    got = prm[1, :, 1:4].astype(np.float64).mean(0)
    want = np.mean([mixes[1]["mu"][m] for m in range(M)], axis=0)
    print(f"[parity] mean {got} oracle {want}", flush=True)
    assert np.max(np.abs(got - want)) <= 1e-9
