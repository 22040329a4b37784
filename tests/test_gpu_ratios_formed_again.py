"""The search pass, which forms the ratios of the statistics pass again (tensors smaller and larger than the last-level cache, both
types): the same bytes as the iterated path gives for the same settings, which carries the ratios through memory."""
import pytest
import torch

from paper_2605_12245_amd import binding as B

DEV = "cuda:0"


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,rows,cols", [(torch.bfloat16, 16385, 8192), (torch.bfloat16, 2049, 4112), (torch.float32, 2049, 4112),
                                             (torch.float32, 8193, 8192)], ids=str)
def test_formed_again_equals_the_iterated_path(dtype, rows, cols):
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


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,rows,cols", [(torch.bfloat16, 16385, 8192), (torch.float32, 2049, 4112)], ids=str)
def test_degenerate_tensors_where_the_ratios_are_formed_again(dtype, rows, cols):
    p = B.soar_default_params()
    p.resident = B.SOAR_RESIDENT_NEVER
    out, ws = B.new_outputs(rows, cols, DEV), B.new_workspace(rows, cols, p, DEV)

    def run(w):
        for t in (out.codes, out.scales):
            t.fill_(0xAA)
        ws.fill_(0xFF)                                      # the ratios, had they been read, would be NaN
        B.quantize_batch([B.make_desc(w, out)], p, ws)
        torch.cuda.synchronize()

    w = torch.zeros(rows, cols, dtype=dtype, device=DEV)
    w[rows - 1, cols - 1] = -0.0
    run(w)
    assert int(out.status.item()) == B.SOAR_STATUS_ALLZERO and out.global_scale.item() == 1.0 and out.sse.item() == 0.0
    assert bool((out.scales == 1).all()) and int(out.codes[-1, -1].item()) == 0x80 and int(out.codes.view(-1)[:-1].max().item()) == 0
    for bad in (float("nan"), float("inf"), -float("inf")):
        w.normal_(std=0.02)
        w[rows // 2, 7] = bad
        run(w)
        assert int(out.status.item()) == B.SOAR_STATUS_NONFINITE, bad
        assert int(out.scales.min().item()) >= 1 and int(out.scales.max().item()) <= 0x7E, bad
    # so small that the global scale is subnormal, with a block of zeros
    w.normal_(std=0.02)
    w[3] = 0.0
    w *= 2.0 ** -118
    run(w)
    want = B.new_outputs(rows, cols, DEV, 1)
    B.quantize_batch([B.make_desc(w, want)], p, ws)         # the trace selects the iterated path, which keeps the ratios
    torch.cuda.synchronize()
    for f in ("codes", "scales", "global_scale", "status"):
        assert torch.equal(getattr(out, f), getattr(want, f)), f
