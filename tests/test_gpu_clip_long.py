"""Clips on both sides of the steps whose io one launch fills (256), and of two such launches: priors and
gradients as by steps, bit for bit, also captured and replayed with eager work in between."""
import pytest

from paper_1008_0502_amd import synth

from test_gpu_adjoint import _torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [255, 256, 257, 520])
def test_lengths(T):
    torch = _torch()
    from paper_1008_0502_amd.api import Context, Params
    H, W = 40, 48
    print(f"\n[case] clip of {T}", flush=True)
    frames, _ = synth.Clip(synth.single_ellipse_spec(H=H, W=W, T=T, seed=T)).stack()
    fr = torch.from_numpy(frames).cuda()
    a, b = Context(H, W, Params(record_tape=T)), Context(H, W, Params(record_tape=T))
    ref = torch.stack([a.step(fr[t], fr[t - 1] if t else None)[1] for t in range(T)])
    out = b.run_clip(fr, with_mrf=True)
    assert torch.equal(out["pi"], ref)
    g = torch.randn((T, H, W), device="cuda", generator=torch.Generator("cuda").manual_seed(T))
    for x, y in zip(a.saliency_backward(g), b.saliency_backward(g)):
        assert torch.equal(x, y)
    want = b.saliency_backward_frames(fr)
    assert torch.equal(a.saliency_backward_frames(fr), want)
    torch.cuda.synchronize()
    graph, buf = torch.cuda.CUDAGraph(), fr.clone()
    with torch.cuda.graph(graph):
        got = b.saliency_backward_frames(buf)
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(got, want)
        a.saliency_backward_frames(fr)
        torch.cuda.synchronize()
    a.close()
    b.close()
