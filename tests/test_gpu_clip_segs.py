"""Segmentations and frames of a clip in the forms that run_clip takes: a tensor, a list, and a sequence
that makes each one when it is asked for, in one buffer or in a tensor that nobody else holds.  Same
results as steps with the same masks, bit for bit."""
import pytest

from paper_1008_0502_amd import synth

from test_gpu_adjoint import _torch

pytestmark = pytest.mark.gpu


class OneBuffer:
    """Every mask in the same buffer, as a decoder would."""

    def __init__(self, masks):
        self.masks, self.buf = masks, masks[0].clone()

    def __getitem__(self, t):
        return self.buf.copy_(self.masks[t])


class Fresh(OneBuffer):
    """A new tensor each time, freed by the next."""

    def __getitem__(self, t):
        return self.masks[t].clone()


class Frames:
    """Frames by index, with a shape, as a reader of a file has them."""

    def __init__(self, frames):
        self.frames, self.shape = list(frames), frames.shape

    def __getitem__(self, t):
        return self.frames[t]


@pytest.mark.parametrize("cap", [0, 5])
@pytest.mark.parametrize("form", [lambda m: m, list, tuple, OneBuffer, Fresh], ids=["tensor", "list", "tuple", "buffer", "fresh"])
def test_forms(cap, form):
    torch = _torch()
    from paper_1008_0502_amd.api import Context, Params
    H, W, T = 97, 131, 5
    print(f"\n[case] segs {form} tape {cap}", flush=True)
    frames, masks = synth.Clip(synth.single_ellipse_spec(H=H, W=W, T=T, seed=4)).stack()
    fr, mk = torch.from_numpy(frames).cuda(), torch.from_numpy(masks).cuda()
    ctx = Context(H, W, Params(record_tape=cap))
    ref = []
    for t in range(T):
        ref.append(ctx.step(fr[t], fr[t - 1] if t else None, mk[t])[1].clone())
    for frames in (fr, Frames(fr)):
        out = ctx.run_clip(frames, segs=form(mk))["pi"]
        for t in range(T):
            assert torch.equal(out[t], ref[t]), t
    ctx.close()
