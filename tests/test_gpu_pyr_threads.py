"""Pyramid launches of at most 256 workgroups (1024 threads each) against larger ones (256 threads):
a stream alone and the same stream among many copies take the two kinds and have to agree bit for
bit; the stream alone is held against the FP64 oracle too (1e-4 of the conspicuity maps' peak, as in
the parity tests).  Sizes: a level of one tile, one row over, ragged rows, several down launches."""
import numpy as np
import pytest

import oracle as O
from paper_1008_0502_amd import synth

from _util import oracle_params
from test_gpu_variants import _torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,copies", [(64, 64, 48), (65, 80, 48), (97, 131, 24), (120, 160, 24), (481, 643, 3)])
def test_alone_and_among_many(H, W, copies):
    torch = _torch()
    from paper_1008_0502_amd.api import Batch, Context, Params
    print(f"\n[case] pyramid threads {H}x{W} x {copies}", flush=True)
    T = 2
    frames, _ = synth.Clip(synth.single_ellipse_spec(H=H, W=W, T=T, seed=H)).stack()
    fr = torch.from_numpy(frames).cuda()
    pp = Params()
    ctx = Context(H, W, pp)
    out = ctx.run_clip(fr, want_C=True)
    ctx.close()
    ref = O.run_clip(frames, oracle_params(pp))
    for t in range(T):
        C = out["C"][t].cpu().numpy().astype(np.float64)
        assert np.max(np.abs(C - ref["C"][t])) <= 1e-4 * max(np.max(np.abs(ref["C"][t])), 1e-12)
    b = Batch([(H, W)] * copies, pp)
    dst = [torch.empty((H, W), device="cuda") for _ in range(copies)]
    for t in range(T):
        b.step(Batch.pointer_table([fr[t]] * copies), Batch.pointer_table(dst))
        torch.cuda.synchronize()
        for d in dst:
            assert torch.equal(d, out["pi"][t])
    b.close()
