"""The search pass with the ratios of the statistics pass carried through memory and formed again (fp32 weights, launch groups larger
than the last-level cache): the same bytes as the iterated path gives for the same settings, which always carries them."""
import pytest
import torch

from paper_2605_12245_amd import binding as B

DEV = "cuda:0"


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,rows,cols", [(torch.bfloat16, 16385, 8192), (torch.bfloat16, 2049, 4112), (torch.float32, 2049, 4112),
                                             (torch.float32, 8193, 8192)], ids=str)
def test_formed_again_equals_carried(dtype, rows, cols):
    gen = torch.Generator(device=DEV).manual_seed(rows)
    w = torch.randn((rows, cols), generator=gen, device=DEV, dtype=dtype) * 0.02
    w[:, ::256] *= 20.0
    w[7] = 0.0                                              # blocks with no code: their ratio stands for a scale
    w[11] *= 2.0 ** -30
    p = B.soar_default_params()
    p.resident = B.SOAR_RESIDENT_NEVER
    out = B.new_outputs(rows, cols, DEV)
    ws = B.new_workspace(rows, cols, p, DEV)
    want = B.new_outputs(rows, cols, DEV, 1)
    B.quantize_batch([B.make_desc(w, out)], p, ws)
    B.quantize_batch([B.make_desc(w, want)], p, ws)         # the trace selects the iterated path
    torch.cuda.synchronize()
    for f in ("codes", "scales", "global_scale", "status"):
        assert torch.equal(getattr(out, f), getattr(want, f)), f
    assert abs(out.sse.item() - want.sse.item()) <= 1e-11 * want.sse.item()       # binary64 sums of 1e7 errors in another order
