"""Covariance of a plain frame (one colour, random weights): the regularisation alone.  The rounding of a
sample's weighted difference (2^-24 of at most 0.25 in the second moment) varies with its weight, so over
12707 samples the moments' ratio is off by about 2^-24 * 0.25 / sqrt(12707) = 1.3e-10 of 1; bar 4e-10,
where products of differences rounded alike for every sample leave up to 2^-25 * 0.25 = 7.5e-9."""
import numpy as np
import pytest

from test_gpu_gmm import _gpu, _torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("colour", [(77, 77, 77), (200, 33, 9), (250, 3, 101), (1, 254, 129)])
def test_plain_frame(colour):
    _torch()
    from paper_1008_0502_amd.api import Params
    print(f"\n[case] plain frame {colour}", flush=True)
    H, W, reg = 97, 131, 1e-4
    frame = np.empty((H, W, 3), np.uint8)
    frame[:] = colour
    prior = np.random.default_rng(sum(colour)).uniform(0.1, 0.9, (H, W)).astype(np.float32)
    _, prm = _gpu(frame, prior, Params(gmm_components=1, gmm_iters=0, gmm_reg=reg))
    err = np.max(np.abs(prm[:, 0, 4:].astype(np.float64) - reg * np.array([1, 0, 0, 1, 0, 1])))
    print(f"[parity] covariance off by {err:.1e}", flush=True)
    assert err <= 4e-10
