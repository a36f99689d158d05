"""Distance-transform prediction at tile edges (32x32 tiles, four pixels a load) against the
FP64 oracle: widths that are and are not multiples of 4, frames of one tile and just over,
objects far from most tiles, at a corner, scattered, none; every source (segmentation bytes, an
unaligned segmentation, the prior above 1/2).  Bar: 1e-4 of the peak, as for the other variants."""
import numpy as np
import pytest

from oracle import variants as V
from paper_1008_0502_amd import synth

from _util import oracle_params
from test_gpu_variants import _check, _run, _torch

pytestmark = pytest.mark.gpu


def _seg(kind, H, W, rng):
    s = np.zeros((H, W), np.uint8)
    if kind == "corner":
        s[-1, -1] = 1
    elif kind == "scattered":
        s[rng.random((H, W)) < 0.01] = 3   # any nonzero byte is object
    elif kind == "edge":
        s[:, 0] = 1
    return s


@pytest.mark.parametrize("H,W", [(32, 32), (33, 36), (31, 131), (64, 65), (100, 200)])
@pytest.mark.parametrize("kind,sigma", [("corner", 4.0), ("scattered", 2.0), ("edge", 1.0), ("none", 2.0)])
def test_tiles(H, W, kind, sigma):
    _torch()
    from paper_1008_0502_amd.api import Params
    print(f"\n[case] dt {kind} {H}x{W}", flush=True)
    rng = np.random.default_rng(H + W)
    frames, _ = synth.Clip(synth.single_ellipse_spec(H=H, W=W, T=3, seed=1)).stack()
    segs = [None] + [_seg(kind, H, W, rng) for _ in range(2)]
    pp = Params(f_mode=1, dt_sigma=sigma)
    ref = V.run_clip_variant(frames, oracle_params(pp), f_mode=1, dt_sigma=sigma,
                             segs=[None if s is None else (s != 0).astype(np.uint8) for s in segs])
    _check(_run(frames, pp, segs=segs), ref, label=f"dt {kind} {H}x{W}")


def test_unaligned_sources():
    torch = _torch()
    from paper_1008_0502_amd.api import Context, Params
    H, W = 64, 96
    rng = np.random.default_rng(5)
    frames = torch.from_numpy(synth.Clip(synth.single_ellipse_spec(H=H, W=W, T=2, seed=1)).stack()[0]).cuda()
    seg = torch.from_numpy((rng.random((H, W)) < 0.02).astype(np.uint8)).cuda()
    shifted = torch.zeros(H * W + 1, dtype=torch.uint8, device="cuda")[1:].view(H, W)
    shifted.copy_(seg)
    out = []
    for s in (seg, shifted):
        ctx = Context(H, W, Params(f_mode=1))
        out.append(ctx.run_clip(frames, segs=[None, s])["pi"])
        ctx.close()
    assert torch.equal(out[0], out[1])


def test_stand_in_with_ragged_rows():
    _torch()
    from paper_1008_0502_amd.api import Params
    frames, _ = synth.Clip(synth.single_ellipse_spec(H=97, W=131, T=4, seed=7)).stack()
    pp = Params(f_mode=1, dt_sigma=2.0)
    ref = V.run_clip_variant(frames, oracle_params(pp), f_mode=1, dt_sigma=2.0)
    margin = min(float(np.min(np.abs(ref["pi"][t] - 0.5))) for t in range(3))
    assert margin > 1e-5   # the threshold of the stand-in is out of rounding's reach on this clip
    _check(_run(frames, pp), ref, label="dt stand-in 97x131")
