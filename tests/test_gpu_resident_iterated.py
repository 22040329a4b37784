"""The iterated path of one tensor in one launch, against the path of a launch per iteration: every launch shape
(workgroups of 256 or 1024 lanes, 1 to 16 tiles, 1 to 256 workgroups, the last one ragged), both element types, the
full method and both arms, early and late stops; degenerate tensors; workspaces holding anything; the bounded wait;
graph capture (which keeps to the other path) and two streams at once.  Everything bit for bit: both paths sum the
block errors with the same tree."""
import pytest
import torch

from paper_2605_12245_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

SHAPES = [(1, 16), (7, 272), (33, 1040), (256, 4096), (257, 4096), (1024, 4096), (2047, 4096), (4096, 4096), (5500, 4096), (7500, 8192)]


def heavy(rows, cols, seed, dtype):
    g = torch.Generator(device=DEV).manual_seed(seed)
    w = torch.randn(rows, cols, generator=g, device=DEV) * torch.exp(torch.randn(rows, 1, generator=g, device=DEV)) * 0.02
    w[:: max(1, rows // 7), 5 % cols] *= 37.0
    return w.to(dtype)


def settings(arm, **kw):
    p = B.soar_paper_params(**kw) if arm == B.SOAR_METHOD_SOAR else B.soar_arm_params(arm, **kw)
    return p


def both(w, p, ws=None):
    out = []
    for resident in (B.SOAR_RESIDENT_AUTO, B.SOAR_RESIDENT_NEVER):
        p.resident = resident
        o = B.new_outputs(w.shape[0], w.shape[1], DEV, p.iters)
        for f in (o.codes, o.scales):
            f.fill_(0x55)
        o.iters_run.fill_(-1); o.sse.fill_(-1.0); o.status.fill_(-1); o.global_scale.fill_(-1.0)
        out.append(B.quantize_iter(w, p, workspace=ws, out=o))
    torch.cuda.synchronize()
    return out


def same(a, b, what):
    for f in ("codes", "scales", "status", "iters_run"):
        assert torch.equal(getattr(a, f), getattr(b, f)), (what, f)
    for f in ("global_scale", "sse", "sse_trace"):
        assert torch.equal(getattr(a, f).nan_to_num(-2.0), getattr(b, f).nan_to_num(-2.0)), (what, f)


@pytest.mark.parametrize("rows,cols", SHAPES)
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "fp32"])
def test_equals_the_launch_per_iteration_path(rows, cols, dtype):
    w = heavy(rows, cols, rows + cols, dtype)
    B.soar_kernel_timing_enable(True)
    calls = 0
    for arm in (B.SOAR_METHOD_SOAR, B.SOAR_METHOD_CJSO_ONLY, B.SOAR_METHOD_DSS_ONLY):
        for kw in (dict(), dict(iters=5, early_stop_rel=0.0)):
            same(*both(w, settings(arm, **kw)), (arm, kw))
            calls += 1
    assert B.soar_kernel_timing_read(B.SOAR_KERNEL_RESIDENT)[1] == calls      # one launch each, and none for NEVER
    B.soar_kernel_timing_enable(False)


def test_strided_degenerate_absent_outputs_and_any_workspace():
    parent = heavy(700, 4096 + 64, 5, torch.bfloat16)
    view = parent[:, 32:32 + 4096]
    p = settings(B.SOAR_METHOD_SOAR, iters=4)
    same(*both(view, p), "strided")
    zero = torch.zeros(600, 4096, dtype=torch.bfloat16, device=DEV)
    zero[599, 4095] = -0.0
    bad = heavy(600, 4096, 6, torch.float32)
    bad[577, 123] = float("inf")
    same(*both(zero, p), "all zero")
    same(*both(bad, p), "non-finite")
    ws = B.new_batch_workspace([B.make_desc(parent, B.new_outputs(700, 4160, DEV, 4))], p, DEV)
    for fill in (0xFF, 0, 0x5A, None, None):
        for rows in (700, 33, 257, 700):
            w = parent[:rows, :4096].contiguous()
            if fill is not None:
                ws.fill_(fill)
            same(*both(w, p, ws), (fill, rows))
    # only the bytes and the scale asked for
    w = heavy(300, 4096, 8, torch.bfloat16)
    p.resident = B.SOAR_RESIDENT_AUTO
    full, o = B.quantize_iter(w, p), B.new_outputs(300, 4096, DEV)
    o.sse.fill_(-1.0); o.status.fill_(-1)
    rc = B.soar_quantize(w.data_ptr(), B.SOAR_BF16, 300, 4096, 4096, p, o.codes.data_ptr(), o.scales.data_ptr(),
                         o.global_scale.data_ptr(), 0, 0, ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert rc == B.SOAR_OK and torch.equal(o.codes, full.codes) and torch.equal(o.scales, full.scales)
    assert o.sse.item() == -1.0 and o.status.item() == -1 and o.global_scale.item() == full.global_scale.item()


def gives_up(w, p, ws, fill=None):
    """a call whose bound of one microsecond is over, and the same call on the other path.  A crossing takes two trips through
    memory, 2 us and more, but a workgroup that arrives late may find everything there: such a call is made again"""
    p.resident_wait_us = 1
    for _ in range(20):
        if fill is not None:
            ws.fill_(fill)
        got, want = both(w, p, ws)
        if int(got.status.item()) & B.SOAR_STATUS_GAVE_UP:
            break
    p.resident_wait_us = 0
    return got, want


def test_bounded_wait_gives_up_and_the_next_call_is_unaffected():
    """one microsecond is over before a crossing is complete: every workgroup says so and leaves"""
    w = heavy(2047, 4096, 9, torch.bfloat16)
    p = settings(B.SOAR_METHOD_SOAR, iters=4)
    ws = B.new_batch_workspace([B.make_desc(w, B.new_outputs(2047, 4096, DEV, 4))], p, DEV)
    for rep in range(3):
        o, _ = gives_up(w, p, ws)
        assert int(o.status.item()) == B.SOAR_STATUS_GAVE_UP
        same(*both(w, p, ws), rep)


def test_the_bound_does_not_count_the_time_of_the_loads():
    """90 MB take more than 11 us to read; the workgroups arrive within 4 us of one another"""
    w = heavy(5500, 4096, 9, torch.float32)
    p = settings(B.SOAR_METHOD_CJSO_ONLY, iters=2)
    p.resident_wait_us = 9
    ws = B.new_workspace(5500, 4096, p, DEV)
    statuses = []
    for _ in range(20):
        o = B.quantize_iter(w, p, workspace=ws)
        statuses.append(int(o.status.item()))
    assert statuses.count(0) >= 10, statuses


@pytest.mark.parametrize("rows,cols", [(65, 4096), (1024, 4096), (2047, 4096), (5500, 4096)])      # 17 to 256 workgroups, 1 to 8 tiles
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "fp32"])
def test_a_call_that_gives_up_is_finished_all_the_same(rows, cols, dtype):
    """one microsecond is over before the first crossing is complete: the last workgroup to leave does the tensor"""
    zero = torch.zeros(rows, cols, dtype=dtype, device=DEV)
    zero[rows - 1, cols - 1] = -0.0
    bad = heavy(rows, cols, 4, dtype)
    bad[rows // 2, 7] = float("nan")
    cases = [("all zero", zero, B.SOAR_METHOD_SOAR, B.SOAR_STATUS_ALLZERO), ("non-finite", bad, B.SOAR_METHOD_SOAR, B.SOAR_STATUS_NONFINITE)]
    cases += [(arm, heavy(rows, cols, rows, dtype), arm, 0) for arm in (B.SOAR_METHOD_SOAR, B.SOAR_METHOD_CJSO_ONLY, B.SOAR_METHOD_DSS_ONLY)]
    for what, w, arm, status in cases:
        p = settings(arm, iters=3)
        ws = B.new_workspace(rows, cols, p, DEV)
        for fill in (0xFF, 0):
            got, want = gives_up(w, p, ws, fill)
            assert int(got.status.item()) == B.SOAR_STATUS_GAVE_UP | status, what
            got.status.fill_(status)
            same(got, want, (what, fill))
            same(*both(w, p, ws), (what, fill, "the next call"))


def test_capture_keeps_to_the_other_path_and_two_streams_at_once():
    w = heavy(1024, 4096, 11, torch.bfloat16)
    p = settings(B.SOAR_METHOD_SOAR, iters=4)
    out = B.new_outputs(1024, 4096, DEV, 4)
    ws = B.new_batch_workspace([B.make_desc(w, out)], p, DEV)
    B.quantize_iter(w, p, workspace=ws, out=out)
    torch.cuda.synchronize()
    B.soar_kernel_timing_enable(False)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        B.quantize_iter(w, p, workspace=ws, out=out)
    for rep in range(3):
        w.copy_(heavy(1024, 4096, 20 + rep, torch.bfloat16))
        out.sse_trace.fill_(float("nan"))
        g.replay()
        eager, never = both(w, p)
        same(out, eager, rep)
        same(eager, never, rep)
    wb = heavy(3000, 4096, 12, torch.float32)
    (ra, _), (rb, _) = both(w, p), both(wb, p)
    p.resident = B.SOAR_RESIDENT_AUTO
    sa, sb = torch.cuda.Stream(), torch.cuda.Stream()
    for rep in range(3):
        with torch.cuda.stream(sa):
            oa = [B.quantize_iter(w, p) for _ in range(3)]
        with torch.cuda.stream(sb):
            ob = [B.quantize_iter(wb, p) for _ in range(3)]
        torch.cuda.synchronize()
        for o in oa:
            same(o, ra, rep)
        for o in ob:
            same(o, rb, rep)
