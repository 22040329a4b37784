"""Small one-pass conversions that need no launch to clear counters (supplied maximum, MXFP4), around the sizes where the
kernels change: against the path with counters bit for bit, on workspaces holding anything, replayed from a graph."""
import math

import pytest
import torch

from paper_2605_12245_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def weights(rows, cols, dtype, pad=0):
    g = torch.Generator(device=DEV).manual_seed(rows + cols)
    w = torch.randn(rows, cols + pad, generator=g, device=DEV) * torch.exp(torch.randn(rows, 1, generator=g, device=DEV))
    return w.to(dtype)[:, :cols]


def same(a, b, what):
    assert torch.equal(a.codes, b.codes) and torch.equal(a.scales, b.scales) and torch.equal(a.status, b.status), what
    if a.global_scale is not None:
        assert torch.equal(a.global_scale.nan_to_num(-1.0), b.global_scale.nan_to_num(-1.0)), what
    # the NVFP4 sum follows the launch shape, the MXFP4 sum does not
    assert math.isclose(a.sse.item(), b.sse.item(), rel_tol=1e-12 if a.global_scale is not None else 0.0), what


def rtn(w, amax, resident, ws):
    p = B.soar_default_params(B.SOAR_METHOD_RTN, 0)
    p.resident = resident
    o = B.new_outputs(w.shape[0], w.shape[1], DEV)
    for f in (o.codes, o.scales):
        f.fill_(0x55)
    o.sse.fill_(-1.0); o.status.fill_(-1)
    B.quantize_batch([B.make_desc(w, o, amax)], p, ws)
    return o


# tiles of 256 blocks: 1, 1, 255, 256, 257 (two a workgroup from here on), 1023, 1024, 1025 (the other path)
SHAPES = [(1, 16), (3, 1040), (255, 4096), (256, 4096), (257, 4096), (1023, 4096), (1024, 4096), (1025, 4096)]


@pytest.mark.parametrize("rows,cols", SHAPES)
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "fp32"])
def test_supplied_maximum(rows, cols, dtype):
    for pad in (0, 16):
        w = weights(rows, cols, dtype, pad)
        amax = w.abs().max().float().reshape(1)
        ws = B.new_workspace(rows, cols, B.soar_default_params(B.SOAR_METHOD_RTN, 0), DEV)
        for k, factor in enumerate((1.0, 0.25, 3.0)):
            ws.fill_((0, 0xFF, 0x3C)[k])
            same(rtn(w, amax * factor, B.SOAR_RESIDENT_AUTO, ws), rtn(w, amax * factor, B.SOAR_RESIDENT_NEVER, ws), (pad, factor))
    for bad in (0.0, -1.0, float("nan"), float("inf")):
        o = rtn(w, torch.full((1,), bad, device=DEV), B.SOAR_RESIDENT_AUTO, ws)
        torch.cuda.synchronize()
        assert int(o.status.item()) == B.SOAR_STATUS_BAD_AMAX


@pytest.mark.parametrize("rows,cols", SHAPES + [(2048, 4096)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "fp32"])
def test_supplied_maximum_and_returned_scale_share_a_float(rows, cols, dtype):
    """the scale is written after the last read of the maximum, whichever path the size takes"""
    w = weights(rows, cols, dtype)
    ws = B.new_workspace(rows, cols, B.soar_default_params(B.SOAR_METHOD_RTN, 0), DEV)
    for rep in range(6):
        amax = w.abs().max().float().reshape(1) * (0.25 + rep)
        want = rtn(w, amax, B.SOAR_RESIDENT_NEVER, ws)
        for wanted in ((1, 1), (0, 1), (0, 0)):          # sse and status, status, neither
            o = B.new_outputs(rows, cols, DEV)
            o.global_scale.copy_(amax)
            d = B.make_desc(w, o, o.global_scale)
            d.d_sse, d.d_status = (d.d_sse if wanted[0] else None), (d.d_status if wanted[1] else None)
            B.quantize_batch([d], B.soar_default_params(B.SOAR_METHOD_RTN, 0), ws)
            assert torch.equal(o.codes, want.codes) and torch.equal(o.scales, want.scales), (rep, wanted)
            assert torch.equal(o.global_scale, want.global_scale), (rep, wanted)
            assert not wanted[0] or math.isclose(o.sse.item(), want.sse.item(), rel_tol=1e-12)
            assert not wanted[1] or int(o.status.item()) == 0


# tiles of 256 blocks of 32: 1, 2, 255, 256, 257, 511, 512, 513
@pytest.mark.parametrize("rows,cols", [(1, 32), (5, 3072), (510, 4096), (512, 4096), (513, 4096), (1022, 4096), (1024, 4096), (1025, 4096)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "fp32"])
def test_mxfp4(rows, cols, dtype):
    for pad in (0, 32):
        w = weights(rows, cols, dtype, pad)
        for dss in (False, True):
            got = []
            for tpw, fill in ((0, 0xFF), (2, 0)):        # a forced launch shape takes the path with counters
                p = B.soar_mx_default_params(dss=dss, n_beta=11, tiles_per_wg=tpw)
                ws = torch.full((B.soar_mxfp4_workspace_bytes(rows, cols, p),), fill, dtype=torch.uint8, device=DEV)
                got.append(B.mx_quantize(w, p, workspace=ws))
            same(*got, (pad, dss))
    w = w.clone()
    w[rows - 1, cols - 1] = float("nan")
    for dss in (False, True):
        o = B.mx_quantize(w, B.soar_mx_default_params(dss=dss, n_beta=11))
        torch.cuda.synchronize()
        assert int(o.status.item()) == B.SOAR_STATUS_NONFINITE


def test_replayed_from_a_graph_on_changing_data():
    w, amax = weights(200, 4096, torch.bfloat16).contiguous(), torch.ones(1, device=DEV)
    o, m = B.new_outputs(200, 4096, DEV), B.mx_new_outputs(200, 4096, DEV)
    p, pm = B.soar_default_params(B.SOAR_METHOD_RTN, 0), B.soar_mx_default_params(dss=False)
    ws, wm = B.new_workspace(200, 4096, p, DEV), torch.empty(B.soar_mxfp4_workspace_bytes(200, 4096, pm), dtype=torch.uint8, device=DEV)
    run = lambda: (B.quantize_rtn_amax(w, amax, ws, o), B.mx_quantize(w, pm, wm, m))  # noqa: E731
    run()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        run()
    gen = torch.Generator(device=DEV).manual_seed(1)
    for rep in range(6):
        w.copy_((torch.randn(w.shape, generator=gen, device=DEV) * (rep + 1)).to(torch.bfloat16))
        amax.copy_(w.abs().max().float().reshape(1))
        o.sse.zero_(); m.sse.zero_()
        g.replay()
        if rep % 2:
            g.replay()
        torch.cuda.synchronize()
        same(o, rtn(w, amax, B.SOAR_RESIDENT_NEVER, B.new_workspace(200, 4096, p, DEV)), rep)
        same(m, B.mx_quantize(w, B.soar_mx_default_params(dss=False, tiles_per_wg=2)), rep)


@pytest.mark.parametrize("rows", [200, 2048], ids=["path with counters", "one-launch kernel"])
def test_another_call_clears_the_workspace_between_replays(rows):
    """the captured call's words stay in the workspace: a call that clears the control words there must not bring back
    the token they carry"""
    w, amax = weights(rows, 4096, torch.bfloat16).contiguous(), torch.ones(1, device=DEV)
    o = B.new_outputs(rows, 4096, DEV)
    p = B.soar_default_params(B.SOAR_METHOD_SOAR, 0)
    never = B.soar_default_params(B.SOAR_METHOD_SOAR, 0)
    never.resident = B.SOAR_RESIDENT_NEVER
    ws = B.new_workspace(rows, 4096, p, DEV)
    small = weights(16, 64, torch.bfloat16).contiguous()
    so, ref = B.new_outputs(16, 64, DEV), B.new_outputs(rows, 4096, DEV)
    run = (lambda: B.quantize_rtn_amax(w, amax, ws, o)) if rows == 200 else (lambda: B.quantize_batch([B.make_desc(w, o)], p, ws))
    run()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        run()
    gen = torch.Generator(device=DEV).manual_seed(2)
    for rep in range(5):
        w.copy_((torch.randn(w.shape, generator=gen, device=DEV) * 2.0 ** -rep).to(torch.bfloat16))
        amax.copy_(w.abs().max().float().reshape(1))
        B.quantize_batch([B.make_desc(small, so)], never, ws)
        g.replay()
        torch.cuda.synchronize()
        if rows == 200:
            same(o, rtn(w, amax, B.SOAR_RESIDENT_NEVER, B.new_workspace(rows, 4096, p, DEV)), rep)
        else:
            B.quantize_batch([B.make_desc(w, ref)], never, B.new_workspace(rows, 4096, p, DEV))
            torch.cuda.synchronize()
            same(o, ref, rep)
