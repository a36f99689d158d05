"""Pixel-level adjoint on rows of whole quads and not (levels whose widths are multiples of 4 take
16-byte accesses, pairs of pixels 2- and 8-byte ones), wavefronts on and off the levels' borders,
frames and gradients at unaligned addresses: the aligned and unaligned calls have to agree bit for bit,
and both with the FP64 oracle (test_gpu_pixel_adjoint's bar)."""
import numpy as np
import pytest

import test_gpu_pixel_adjoint as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W", [(96, 128), (95, 160), (130, 131), (97, 200), (64, 320)])
def test_unaligned_frames_and_gradients(H, W):
    torch = P._torch()
    from paper_1008_0502_amd import synth
    from paper_1008_0502_amd.api import Context, Params
    print(f"\n[case] pixel quads {H}x{W}", flush=True)
    T = 3
    frames, masks = synth.Clip(synth.single_ellipse_spec(H=H, W=W, T=T, seed=W)).stack()
    g = torch.from_numpy(np.random.default_rng(H).normal(size=(T, H, W)).astype(np.float32)).cuda()
    out = []
    for off in (0, 1):
        fr = torch.zeros(T * H * W * 3 + 1, dtype=torch.uint8, device="cuda")[off:off + T * H * W * 3].view(T, H, W, 3)
        fr.copy_(torch.from_numpy(frames))
        ctx = Context(H, W, Params(record_tape=T))
        ctx.run_clip(fr)
        ctx.saliency_backward(g)
        res = torch.zeros(T * H * W * 3 + 1, device="cuda")[off:off + T * H * W * 3]
        assert ctx.lib.saliency_backward_frames(ctx._handle, fr.data_ptr(), T, res.data_ptr()) == 0
        torch.cuda.synchronize()
        out.append(res)
        ctx.close()
    assert torch.isfinite(out[0]).all() and torch.any(out[0] != 0)
    assert torch.equal(out[0], out[1])
    P._check(frames, masks, Params(q=2e-3, r=5e-2), f"{H}x{W}")
