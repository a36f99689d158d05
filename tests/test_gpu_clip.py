"""A whole clip in one call (sp_run_clip): with a tape, frames side by side in slots (whole
chunks, a shorter last one, fewer frames than the tape); without, step by step.  Same kernels
and inputs as one sp_step per frame, so every output agrees bit for bit, gradients included;
also when the call is captured into a graph and replayed."""
import numpy as np
import pytest

from paper_1008_0502_amd import synth

from test_gpu_adjoint import _torch

pytestmark = pytest.mark.gpu


def _steps(ctx, fr, segs, mrf):
    import torch
    T, H, W = fr.shape[:3]
    g = ctx.geometry
    new = lambda *s: torch.empty((T, *s), device="cuda")   # noqa: E731
    o = {"S": new(g.Hc, g.Wc), "C": new(8, g.Hc, g.Wc), "pi": new(H, W)}
    if mrf:
        o.update(unary=new(2, H, W), pairwise=new(4, H, W), beta=new(1))
    ctx.reset()
    for t in range(T):
        ctx.step(fr[t], fr[t - 1] if t else None, None if segs is None else segs[t], o["S"][t], o["C"][t], o["pi"][t],
                 *((o["unary"][t], o["pairwise"][t], o["beta"][t]) if mrf else ()))
    return o


@pytest.mark.parametrize("H,W,T,cap,kw", [
    (97, 131, 7, 7, {}), (120, 160, 70, 100, {}), (240, 322, 5, 9, dict(centers=(2, 3), deltas=(2, 3))),
    (96, 128, 6, 6, dict(centers=(1, 3), deltas=(1, 2))), (600, 900, 11, 11, {}), (120, 160, 5, 0, {})])
@pytest.mark.parametrize("mrf,seg", [(False, False), (True, True)])
def test_clip_equals_steps(H, W, T, cap, kw, mrf, seg):
    torch = _torch()
    from paper_1008_0502_amd.api import Context, Params
    print(f"\n[case] clip {H}x{W}x{T} tape {cap} mrf {mrf}", flush=True)
    frames, masks = synth.Clip(synth.single_ellipse_spec(H=H, W=W, T=T, seed=T)).stack()
    fr, mk = torch.from_numpy(frames).cuda(), torch.from_numpy(masks).cuda()
    segs = [mk[t] if t % 2 else None for t in range(T)] if seg else None
    pp = Params(record_tape=cap, **kw)
    a, b = Context(H, W, pp), Context(H, W, pp)
    ref = _steps(a, fr, segs, mrf)
    for rep in range(2):   # a second clip on the same slots and tape
        out = b.run_clip(fr, with_mrf=mrf, want_C=True, segs=segs)
        for k, v in ref.items():
            assert torch.equal(v, out[k]), (k, rep)
    assert a.step_index == b.step_index == T
    if cap:
        g = torch.randn((T, H, W), device="cuda", generator=torch.Generator("cuda").manual_seed(1))
        for x, y in zip(a.saliency_backward(g), b.saliency_backward(g)):
            assert torch.equal(x, y)
    # the step after the clip continues from the same state
    if T < cap or not cap:
        for c in (a, b):
            c.step(fr[0], fr[-1], S_out=ref["S"][0], prior_out=ref["pi"][0 if c is a else 1])
        assert torch.equal(ref["pi"][0], ref["pi"][1])
    a.close()
    b.close()


def test_captured_clip():
    torch = _torch()
    from paper_1008_0502_amd.api import Context, Params
    H, W, T = 96, 128, 3
    frames = np.stack([synth.Clip(synth.single_ellipse_spec(H=H, W=W, T=T, seed=s)).stack()[0] for s in (1, 2)])
    clips = torch.from_numpy(frames).cuda()
    ctx = Context(H, W, Params(record_tape=T))
    ref = [ctx.run_clip(c)["pi"].clone() for c in clips]
    buf = clips[0].clone()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = ctx.run_clip(buf)["pi"]
    for i in (0, 1, 0):
        buf.copy_(clips[i])
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref[i])
        ctx.run_clip(clips[1 - i])   # eager work between the replays
        torch.cuda.synchronize()
    ctx.close()
