"""Priors copied out of a batched step: streams of one chunk of the copy (4096 pixels), a chunk
exactly, one pixel more, and larger, to aligned and unaligned buffers, nothing beyond each."""
import ctypes

import pytest

from paper_1008_0502_amd import synth

from test_gpu_batch import _torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("off", [0, 1])
def test_copied_priors(off):
    torch = _torch()
    from paper_1008_0502_amd.api import Batch, Params
    print(f"\n[case] copy out, buffers {off} elements off", flush=True)
    sizes = [(48, 64), (64, 64), (17, 241), (97, 131), (240, 320)]
    frames = [torch.from_numpy(synth.Clip(synth.single_ellipse_spec(H=H, W=W, T=1, seed=H)).stack()[0][0]).cuda()
              for H, W in sizes]
    b = Batch(sizes, Params())
    out = [torch.full((H * W + 8,), -1.0, device="cuda") for H, W in sizes]
    for _ in range(2):
        b.step(Batch.pointer_table(frames), Batch.pointer_table([o[off:] for o in out]))
    torch.cuda.synchronize()
    hip = ctypes.CDLL("libamdhip64.so.7")
    hip.hipMemcpy.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int]
    for i, (H, W) in enumerate(sizes):
        ptr = ctypes.c_void_p()
        assert b.lib.sp_batch_prior(b._handle, i, ctypes.byref(ptr)) == 0
        ref = torch.empty(H * W, device="cuda")
        assert hip.hipMemcpy(ref.data_ptr(), ptr.value, H * W * 4, 3) == 0
        torch.cuda.synchronize()
        assert torch.equal(out[i][off:off + H * W], ref)
        assert torch.all(out[i][:off] == -1.0) and torch.all(out[i][off + H * W:] == -1.0)
    b.close()
