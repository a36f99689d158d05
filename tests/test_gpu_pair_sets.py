"""Across-scale sums built for a known set of pairs (three centre levels with surrounds 3 and 4 levels
above; three pairs of two centre levels) and the general ones (surrounds 2 and 3 above): one channel a
workgroup against two bit for bit, and against the FP64 oracle with the bar of the parity tests; frames
whose c_max map is below a tile, a tile and an odd remainder, several tiles."""
import numpy as np
import pytest

import oracle as O
from paper_1008_0502_amd import synth

from _util import oracle_params
from test_gpu_variants import _torch

pytestmark = pytest.mark.gpu

DEEP = dict(depth=9, centers=(2, 3, 4), deltas=(3, 4))
GENERAL = dict(depth=9, centers=(2, 3, 4), deltas=(2, 3))
MID = dict(depth=6, centers=(2, 3), deltas=(3, 4))


@pytest.mark.parametrize("levels,H,W", [(DEEP, 256, 256), (DEEP, 273, 531), (DEEP, 600, 400), (DEEP, 257, 1040),
                                        (GENERAL, 273, 531), (GENERAL, 256, 256),
                                        (MID, 97, 131), (MID, 128, 256), (MID, 240, 320), (MID, 259, 133)])
def test_known_and_general(levels, H, W):
    torch = _torch()
    from paper_1008_0502_amd.api import Context, Params
    print(f"\n[case] pair sets {H}x{W} {levels}", flush=True)
    frames, _ = synth.Clip(synth.three_ellipse_spec(H=H, W=W, T=2, seed=H)).stack()
    fr = torch.from_numpy(frames).cuda()
    pp = Params(**levels)
    out = []
    for channels in (1, 2):
        ctx = Context(H, W, pp)
        assert ctx.lib.sp_set_tune(ctx._handle, 32, 1, channels) == 0
        out.append(ctx.run_clip(fr, want_C=True))
        torch.cuda.synchronize()
        ctx.close()
    for k in ("S", "C", "pi"):
        assert torch.equal(out[0][k], out[1][k]), k
    ref = O.run_clip(frames, oracle_params(pp))
    for k in ("S", "C"):
        for t in range(2):
            r = ref[k][t]
            e = float(np.max(np.abs(out[0][k][t].cpu().numpy().astype(np.float64) - r)) / max(np.max(np.abs(r)), 1e-30))
            assert e <= 1e-4, (k, t, e)
