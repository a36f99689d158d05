"""Pixel-level adjoint with frames side by side: more frames than slots (the motion part crosses
from one launch to the next), a level that is both centre and surround, unused levels in the
pyramid, other Gabor radii, levels smaller than a tile; and the same call under graph capture.
Against the FP64 oracle with the bar of the other pixel-adjoint tests (1e-3 of the peak)."""
import pytest

from paper_1008_0502_amd import synth

from test_gpu_pixel_adjoint import _check, _torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,T,kw", [
    (64, 80, 11, {}), (50, 47, 17, dict(depth=4, centers=(1, 2), deltas=(1, 2))),
    (70, 130, 2, dict(depth=5, centers=(2, 3), deltas=(2,))), (49, 64, 3, dict(gabor_radius=4)),
    (49, 81, 2, dict(gabor_radius=8, gabor_sigma=2.5)), (64, 66, 1, dict(depth=4, centers=(1, 3), deltas=(1,)))])
def test_slots_match_oracle(H, W, T, kw):
    from paper_1008_0502_amd.api import Params
    print(f"\n[case] pixel adjoint {H}x{W} T={T} {kw}", flush=True)
    spec = synth.single_ellipse_spec(H=H, W=W, T=T, seed=4)
    spec.axes = (9.0, 6.0)
    frames, masks = synth.Clip(spec).stack()
    _check(frames, masks, Params(q=2e-3, r=5e-2, **kw), f"{H}x{W}x{T}")


def test_captured():
    torch = _torch()
    from paper_1008_0502_amd.api import Context, Params
    H, W, T = 96, 120, 10
    frames, masks = synth.Clip(synth.single_ellipse_spec(H=H, W=W, T=T, seed=6)).stack()
    fr, mk = torch.from_numpy(frames).cuda(), torch.from_numpy(masks).cuda()
    ctx = Context(H, W, Params(record_tape=T))
    _, g = ctx.mse_mask_loss(ctx.run_clip(fr)["pi"], mk)
    ctx.saliency_backward(g)
    ref = ctx.saliency_backward_frames(fr)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = ctx.saliency_backward_frames(fr)
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref)
        assert torch.equal(ctx.saliency_backward_frames(fr), ref)
        torch.cuda.synchronize()
    ctx.close()
