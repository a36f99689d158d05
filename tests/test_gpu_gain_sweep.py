"""The gain recursion and the sum of the steps' weight gradients over clips of one step, one staged
chunk (256 steps) and more, against the FP64 oracle (tolerance of the other adjoint tests)."""
import pytest

from test_gpu_adjoint import W8, check, gpu_grad, oracle_grads, params, small_clip

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [2, 255, 256, 257, 520])
def test_chunks(T):
    print(f"\n[case] gain sweep over {T} steps", flush=True)
    frames, masks = small_clip(H=40, W=56, T=T, seed=T)
    pp = params()
    gpu = gpu_grad(frames, masks, pp, W8, 2e-3, 5e-2)
    check(f"T={T}", gpu, oracle_grads(frames, masks, pp, W8, 2e-3, 5e-2, fd=False))
