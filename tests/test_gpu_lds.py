"""Across-scale sums whose workgroup takes nearly all of a CU's LDS (four channels of three centre
levels): every number of channels that fits is accepted, by a context, its autotuner and a batch, with
the same results; contexts of different needs take turns."""
import pytest

from paper_1008_0502_amd import synth

from test_gpu_variants import _torch

pytestmark = pytest.mark.gpu

WIDE = [dict(depth=9, centers=(2, 4), deltas=(3, 4)), dict(depth=8, centers=(2, 3, 4), deltas=(3,)),
        dict(depth=9, centers=(2, 3, 4), deltas=(4, 5)), dict(depth=6, centers=(1, 3), deltas=(3,))]
H, W = 260, 530


def _frames(torch):
    frames, _ = synth.Clip(synth.three_ellipse_spec(H=H, W=W, T=2, seed=5)).stack()
    return torch.from_numpy(frames).cuda()


@pytest.mark.parametrize("levels", WIDE)
def test_four_channels(levels):
    torch = _torch()
    from paper_1008_0502_amd.api import Batch, Context, Params
    print(f"\n[case] LDS {levels}", flush=True)
    fr = _frames(torch)
    ctx = Context(H, W, Params(**levels))
    ref = {k: v.clone() for k, v in ctx.run_clip(fr, want_C=True).items() if v is not None}
    for channels in (1, 2, 4):
        ctx.set_tune(32, True, channels)
        out = ctx.run_clip(fr, want_C=True)
        for k, v in ref.items():
            assert torch.equal(out[k], v), (k, channels)
    report = ctx.autotune(fr[1], fr[0], steps=2)
    assert "workgroup 4" in report or "workgroup 2" in report
    b = Batch([(H, W)] * 2, Params(**levels))
    for channels in (1, 2, 4):
        b.set_tune(32, True, channels)
        b.reset()
        priors = [torch.empty((H, W), device="cuda") for _ in range(2)]
        for t in range(2):
            b.step(Batch.pointer_table([fr[t], fr[t]]), Batch.pointer_table(priors))
        for p in priors:
            assert torch.equal(p, ref["pi"][1]), channels
    b.autotune(Batch.pointer_table([fr[1], fr[1]]), steps=2)
    ctx.close()
    b.close()


def test_contexts_take_turns():
    torch = _torch()
    from paper_1008_0502_amd.api import Context, Params
    fr = _frames(torch)
    ctxs = []
    for levels, channels in ((dict(depth=6, centers=(2, 3, 4), deltas=(1,)), 2), (dict(depth=6, centers=(2, 3, 4), deltas=(2,)), 2),
                             (WIDE[0], 4), (WIDE[1], 4)):
        ctx = Context(H, W, Params(**levels))
        ref = ctx.run_clip(fr)["pi"].clone()
        ctx.set_tune(32, True, channels)
        ctxs.append((ctx, ref))
    for k in (0, 3, 1, 2, 0):
        ctx, ref = ctxs[k]
        assert torch.equal(ctx.run_clip(fr)["pi"], ref), k
    for ctx, _ in ctxs:
        ctx.close()
