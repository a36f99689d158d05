"""GPU reverse step of the prior chain (one launch up to c_max 3, two above) against the FP64
oracle, on a random dL/dprior so that every pixel, border and tile edge counts: tiles of 32 with
no remainder, a remainder of one row or column, a frame below one tile, every c_max.
Tolerance: the FP32 sums of the clip's pixels against 64 bits, as for the other adjoint tests
(1e-3 of each component, components below 1e-3 of the largest against that)."""
import numpy as np
import pytest

import oracle as O
from paper_1008_0502_amd import synth

from _util import oracle_params
from test_gpu_adjoint import W8, _torch, grad_err

pytestmark = pytest.mark.gpu

LEVELS = {1: dict(depth=3, centers=(1,), deltas=(1, 2)), 2: dict(depth=5, centers=(1, 2), deltas=(2, 3)),
          3: dict(depth=5, centers=(2, 3), deltas=(1, 2)), 4: dict(depth=6, centers=(3, 4), deltas=(1, 2))}


@pytest.mark.parametrize("H,W", [(64, 96), (65, 33), (31, 130), (97, 64)])
@pytest.mark.parametrize("c_max", [1, 2, 3, 4])
def test_reverse_step(c_max, H, W):
    torch = _torch()
    from paper_1008_0502_amd.api import Batch, Context, Params
    print(f"\n[case] reverse step {H}x{W} c_max {c_max}", flush=True)
    T = 4
    pp = Params(record_tape=T, weights=tuple(W8), **LEVELS[c_max])
    spec = synth.single_ellipse_spec(H=H, W=W, T=T, seed=11)
    spec.axes = (7.0, 5.0)
    frames, _ = synth.Clip(spec).stack()
    g = np.random.default_rng(H + c_max).normal(size=(T, H, W)).astype(np.float32)
    ctx = Context(H, W, pp)
    assert ctx.geometry.c_max == c_max
    fr, gd = torch.from_numpy(frames).cuda(), torch.from_numpy(g).cuda()
    ctx.run_clip(fr)
    got = [x.cpu().numpy() for x in ctx.saliency_backward(gd)]
    ctx.close()
    op = oracle_params(pp)
    ref = O.run_clip(frames, op)
    tape = O.prior_chain_forward(ref["C"], W8, pp.q, pp.r, op, H, W, c_max)
    gw, gq, gr = O.prior_chain_backward(tape, ref["C"], g.astype(np.float64), op)
    err = grad_err(np.concatenate(got), np.concatenate([gw, [gq, gr]]))
    print(f"[grad] error {err:.2e}", flush=True)
    assert err <= 1e-3
    # the batched form beside a stream of another size: the same gradients bit for bit
    b = Batch([(H, W), (48, 80)], pp)
    other = torch.from_numpy(synth.Clip(synth.single_ellipse_spec(H=48, W=80, T=T, seed=2)).stack()[0]).cuda()
    for t in range(T):
        b.step(b.pointer_table([fr[t], other[t]]))
    bw, bq, br = b.backward([gd, torch.zeros((T, 48, 80), device="cuda")])
    for x, y in zip(got, (bw[0], bq[0], br[0])):
        assert np.array_equal(np.ravel(x), np.ravel(y.cpu().numpy()))
    b.close()
