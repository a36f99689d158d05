"""Kernels built for a known set of pairs where they serve many streams: batches and the frame slots of
recorded clips, for every pair set and the general one, with one, two and four channels a workgroup; and
batches whose streams differ, in their pair set (frames whose depth drops a pair), in the path of their
across-scale sum, and in the kernel of their reverse step (c_max 1, 2, 3 and 4).  Saliency maps, priors
and gradients bit for bit those of a context without a tape, and of one alone."""
import pytest

from paper_1008_0502_amd import synth

from test_gpu_variants import _torch

pytestmark = pytest.mark.gpu

DEEP = dict(depth=9, centers=(2, 3, 4), deltas=(3, 4))
GENERAL = dict(depth=9, centers=(2, 3, 4), deltas=(2, 3))
MID = dict(depth=6, centers=(2, 3), deltas=(3, 4))
MID7 = dict(depth=7, centers=(2, 3), deltas=(3, 4))
FULL = dict(depth=6, centers=(1, 2), deltas=(2, 3))


def _clip(torch, H, W, T, seed):
    return torch.from_numpy(synth.Clip(synth.three_ellipse_spec(H=H, W=W, T=T, seed=seed)).stack()[0]).cuda()


def _alone(H, W, levels, clip):
    from paper_1008_0502_amd.api import Context, Params
    ctx = Context(H, W, Params(**levels))
    out = {k: v.clone() for k, v in ctx.run_clip(clip, want_C=True).items() if v is not None}
    ctx.close()
    return out


def _saliency(torch, b, i, shape):
    from paper_1008_0502_amd import _lib
    S = torch.empty(shape, device="cuda")
    _lib.hip_copy_d2d(S.data_ptr(), b.output_pointers(i)[0], S.numel() * 4, torch.cuda.current_stream().cuda_stream)
    return S


def _batch_equals(torch, sizes, levels, T, channels):
    from paper_1008_0502_amd.api import Batch, Params
    clips = [_clip(torch, h, w, T, 3 * i + 1) for i, (h, w) in enumerate(sizes)]
    ref = [_alone(h, w, levels, c) for (h, w), c in zip(sizes, clips)]
    b = Batch(sizes, Params(**levels))
    for ch in channels:
        if ch:
            b.set_tune(32, True, ch)
        b.reset()
        priors = [torch.empty(s, device="cuda") for s in sizes]
        for t in range(T):
            b.step(Batch.pointer_table([c[t] for c in clips]), Batch.pointer_table(priors))
            for i, r in enumerate(ref):
                assert torch.equal(priors[i], r["pi"][t]), ("prior", ch, t, i)
                assert torch.equal(_saliency(torch, b, i, r["S"][t].shape), r["S"][t]), ("S", ch, t, i)
    b.close()


@pytest.mark.parametrize("levels,sizes", [(DEEP, [(256, 256), (273, 531)]), (GENERAL, [(256, 256), (273, 531)]),
                                          (MID, [(97, 131), (240, 320), (259, 133)]), (MID7, [(150, 201), (240, 320)]),
                                          (FULL, [(97, 131), (120, 160)])])
def test_batches_of_one_set(levels, sizes):
    torch = _torch()
    print(f"\n[case] batch {sizes} {levels}", flush=True)
    _batch_equals(torch, sizes, levels, 2, (0, 1, 2))


@pytest.mark.parametrize("levels,sizes", [
    (dict(centers=(2, 3), deltas=(3, 4)), [(240, 320), (130, 140)]),                 # three pairs, three pairs
    (dict(centers=(2, 3), deltas=(3, 4)), [(240, 320), (300, 270), (70, 90)]),       # three, four, one
    (dict(centers=(1, 2), deltas=(2, 3)), [(120, 160), (40, 48), (24, 30)]),         # four, and small frames' fewer
    (dict(centers=(2, 3, 4), deltas=(3, 4)), [(530, 520), (600, 512)]),              # six, six
    (dict(centers=(2, 3, 4), deltas=(3, 4)), [(530, 520), (300, 256), (130, 140)])])  # six, five, three (two centres)
def test_batches_of_different_sets(levels, sizes):
    torch = _torch()
    print(f"\n[case] mixed batch {sizes} {levels}", flush=True)
    _batch_equals(torch, sizes, levels, 2, (0, 1, 2))


@pytest.mark.parametrize("levels,H,W", [(DEEP, 273, 531), (GENERAL, 256, 256), (MID, 97, 131), (MID, 240, 320),
                                        (MID7, 150, 201), (FULL, 120, 160), (dict(depth=9, centers=(2, 4), deltas=(3, 4)), 260, 270)])
@pytest.mark.parametrize("T", [2, 5])
def test_recorded_clips(levels, H, W, T):
    torch = _torch()
    from paper_1008_0502_amd.api import Context, Params
    print(f"\n[case] recorded clip {H}x{W}x{T} {levels}", flush=True)
    clip = _clip(torch, H, W, T, H)
    ref = _alone(H, W, levels, clip)
    ctx = Context(H, W, Params(record_tape=5, **levels))   # five slots: T = 2 takes a prefix of them
    for ch in (0, 1, 2, 4):
        if ch and ctx.lib.sp_set_tune(ctx._handle, 32, ch % 2, ch) != 0:
            assert ch == 4 and "LDS" in ctx.lib.sp_last_error().decode()
            continue
        out = ctx.run_clip(clip, want_C=True)
        for k in ("S", "C", "pi"):
            assert torch.equal(out[k], ref[k]), (k, ch)
    ctx.close()


@pytest.mark.parametrize("levels,sizes", [(dict(centers=(2, 3, 4), deltas=(3,)), [(300, 280), (130, 140), (70, 80)]),
                                          (dict(centers=(1, 2, 3), deltas=(3,)), [(140, 130), (72, 80), (40, 50)])])
def test_gradients_of_different_reverse_steps(levels, sizes):
    torch = _torch()
    from paper_1008_0502_amd.api import Batch, Context, Params
    print(f"\n[case] mixed gradients {sizes} {levels}", flush=True)
    T = 3
    pp = Params(record_tape=T, **levels)
    clips = [_clip(torch, h, w, T, 7 * i + 2) for i, (h, w) in enumerate(sizes)]
    gen = torch.Generator("cuda").manual_seed(9)
    grads = [torch.randn((T, h, w), device="cuda", generator=gen) for h, w in sizes]
    b = Batch(sizes, pp)
    b.steps([Batch.pointer_table([c[t] for c in clips]) for t in range(T)])
    gw, gq, gr = b.backward(grads)
    cmax = set()
    for i, (h, w) in enumerate(sizes):
        ctx = Context(h, w, pp)
        cmax.add(ctx.geometry.c_max)
        ctx.run_clip(clips[i])
        for got, want in zip((gw[i], gq[i], gr[i]), ctx.saliency_backward(grads[i])):
            assert torch.equal(got.reshape(-1), want), i
        ctx.close()
    assert len(cmax) == 3
    b.close()
