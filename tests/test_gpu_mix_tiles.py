"""The sum of the reduced maps at c_max on rows of whole quads and not, tiles cut to one, four and
fifteen columns or rows, and maps of more tiles than a wavefront reduces in one round (80) and in two:
conspicuity and saliency maps against the FP64 oracle with the bar of the parity tests."""
import numpy as np
import pytest

import oracle as O
from paper_1008_0502_amd import synth

from _util import oracle_params
from test_gpu_variants import _torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W", [(120, 160), (68, 208), (125, 196), (129, 252), (97, 131), (512, 704), (720, 964)])
def test_against_oracle(H, W):
    torch = _torch()
    from paper_1008_0502_amd.api import Context, Params
    print(f"\n[case] mix {H}x{W}", flush=True)
    spec = synth.three_ellipse_spec(H=H, W=W, T=2, seed=H)
    frames, _ = synth.Clip(spec).stack()
    pp = Params()
    ctx = Context(H, W, pp)
    out = ctx.run_clip(torch.from_numpy(frames).cuda(), want_C=True)
    torch.cuda.synchronize()
    ctx.close()
    ref = O.run_clip(frames, oracle_params(pp))
    for k in ("S", "C"):
        for t in range(2):
            r = ref[k][t]
            e = float(np.max(np.abs(out[k][t].cpu().numpy().astype(np.float64) - r)) / max(np.max(np.abs(r)), 1e-30))
            assert e <= 1e-4, (k, t, e)
