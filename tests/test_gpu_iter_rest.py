"""The iterations after the fourth share a launch (k_iter_rest): the bytes, traces and counts of every tensor handed over alone (one
launch of its own, or the oracle), on workspaces holding anything, twice on each, replayed from a graph."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2605_12245_amd import binding as B
from paper_2605_12245_amd import synth

DEV = "cuda:0"
FIELDS = ("codes", "scales", "global_scale", "status", "iters_run")


def params(arm):
    if arm == "closed":
        return B.soar_arm_params(B.SOAR_METHOD_CJSO_ONLY, iters=14, early_stop_rel=1e-12)
    if arm == "window":
        return B.soar_paper_params(iters=9, early_stop_rel=1e-30, n_beta=11, dd_mode=B.SOAR_DD_WINDOW, dss_radius=1)
    if arm == "every pair":
        return B.soar_paper_params(iters=9, early_stop_rel=1e-30, n_beta=3, beta_lo=0.9, beta_hi=1.1)
    return B.soar_paper_params(iters=12, early_stop_rel=1e-30, n_beta=21)


def weights_of(rows, dtype, seed, cols=48, pad=16):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    return [(torch.rand((r, cols + pad * (k % 2)), generator=gen, device=DEV) - 0.5).to(dtype)[:, :cols] for k, r in enumerate(rows)]


def outputs(ws, p):
    outs = [B.new_outputs(w.shape[0], w.shape[1], DEV, p.iters) for w in ws]
    return outs, [B.make_desc(w, o) for w, o in zip(ws, outs)]


def same(a, b, what):
    for f in FIELDS:
        assert torch.equal(getattr(a, f), getattr(b, f)), (what, f)
    assert torch.equal(a.sse_trace.nan_to_num(-1.0), b.sse_trace.nan_to_num(-1.0)), what
    assert torch.equal(a.sse.nan_to_num(-1.0), b.sse.nan_to_num(-1.0)), what


# blocks per tensor: 3 rows; one block, tiles and chunks with a remainder, several shares, more chunks than shares
@pytest.mark.gpu
@pytest.mark.parametrize("arm", ["paper", "window", "every pair", "closed"])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("rows", [(1, 853, 855), (1400, 1, 37000), (170000, 5)], ids=str)
def test_rest_equals_every_tensor_alone(rows, dtype, arm):
    p = params(arm)
    ws = weights_of(rows, dtype, sum(rows))
    outs, descs = outputs(ws, p)
    size = B.new_batch_workspace(descs, p, DEV).numel()
    alone = [B.quantize_iter(w, p) for w in ws]
    assert max(int(a.iters_run.item()) for a in alone) > 4
    for fill in (0x00, 0xFF):
        space = torch.full((size,), fill, dtype=torch.uint8, device=DEV)
        for turn in range(2):
            for o in outs:
                o.codes.fill_(0xAA)
                o.sse_trace.fill_(float("nan"))
            B.quantize_batch(descs, p, space)
            torch.cuda.synchronize()
            for k, (o, a) in enumerate(zip(outs, alone)):
                if arm == "every pair":      # alone: a launch per iteration and the rest of them, as in the batch
                    ref = oracle.quantize_iter(synth.bf16_bits(ws[k].cpu()) if dtype == torch.bfloat16 else ws[k].cpu().numpy(), iters=p.iters,
                                               n_beta=p.n_beta, beta_lo=p.beta_lo, beta_hi=p.beta_hi, dd_mode=p.dd_mode, dss_radius=p.dss_radius,
                                               early_stop_rel=p.early_stop_rel) if ws[k].shape[0] < 2000 else None
                    if ref is not None:
                        assert np.array_equal(o.codes.cpu().numpy(), ref.codes) and np.array_equal(o.scales.cpu().numpy(), ref.scales)
                        assert int(o.iters_run.item()) == ref.trace["iters_run"]
                same(o, a, (fill, turn, k))


@pytest.mark.gpu
def test_rest_beside_degenerate_and_stopped_tensors_and_in_a_graph():
    p = params("paper")
    ws = weights_of((300, 700, 90, 2600), torch.bfloat16, 3)
    ws[0] = torch.zeros_like(ws[0])
    ws[1] = ws[1].clone()
    ws[1][5, 7] = float("inf")
    ws[2] = torch.full_like(ws[2], 6.0)                      # nothing to gain: stops after one iteration
    outs, descs = outputs(ws, p)
    alone = [B.quantize_iter(w, p) for w in ws]
    space = B.new_batch_workspace(descs, p, DEV)

    def check(what):
        torch.cuda.synchronize()
        for k, (o, a) in enumerate(zip(outs, alone)):
            if k != 1:
                same(o, a, (what, k))
            else:
                assert int(o.status.item()) == B.SOAR_STATUS_NONFINITE and int(o.iters_run.item()) == 0

    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        B.quantize_batch(descs, p, space)
    check("eager")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        B.quantize_batch(descs, p, space)
    for turn in range(4):
        for o in outs:
            o.codes.fill_(0x55)
        space.random_()
        g.replay()
        check(turn)
        torch.ones(1 << 16, device=DEV).sum().item()


def without_stopping(w, p, rel):
    """what a launch per iteration gives (no early stop, as many iterations as the trace says): outputs, and how many those are"""
    q = B.soar_params.from_buffer_copy(p)
    q.early_stop_rel, q.resident = 0.0, B.SOAR_RESIDENT_NEVER
    t = B.quantize_iter(w, q).sse_trace.cpu().tolist()
    run = next((k for k in range(1, p.iters + 1) if t[k - 1] - t[k] < np.float32(rel) * t[k - 1]), p.iters)
    q.iters = run
    return B.quantize_iter(w, q), run


# tensors that stop inside the shared launch, which has as many workgroups as places; against one launch per iteration
@pytest.mark.gpu
@pytest.mark.parametrize("arm", ["paper", "every pair", "closed"])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "fp32"])
def test_rest_stops_inside_the_shared_launch(dtype, arm):
    p = params(arm)
    p.resident = B.SOAR_RESIDENT_NEVER
    ws = weights_of((170000, 113400, 900), dtype, 5)
    probe = B.quantize_iter(ws[0], p).sse_trace.cpu().tolist()
    for at in (5, 6, 8):                                     # a relative gain between those of two iterations: stops at the later one
        gains = [(probe[k - 1] - probe[k]) / probe[k - 1] for k in range(1, p.iters + 1) if probe[k] == probe[k]]
        rel = gains[at - 1] * 1.001
        p.early_stop_rel = rel
        outs, descs = outputs(ws, p)
        B.quantize_batch(descs, p, B.new_batch_workspace(descs, p, DEV))
        torch.cuda.synchronize()
        runs = []
        for k, (w, o) in enumerate(zip(ws, outs)):
            want, run = without_stopping(w, p, rel)
            runs.append(run)
            assert int(o.iters_run.item()) == run, (at, k)
            for f in ("codes", "scales", "global_scale", "status", "sse"):
                assert torch.equal(getattr(o, f), getattr(want, f)), (at, k, f)
            assert torch.equal(o.sse_trace[:run + 1], want.sse_trace[:run + 1]), (at, k)
        assert 4 < runs[0] <= at


@pytest.mark.gpu
@pytest.mark.parametrize("arm", ["paper", "every pair", "closed", "large table"])
def test_rest_on_a_stream_of_few_compute_units(arm):
    """with a large factor table in LDS some workgroups find no place, also on the whole GPU: the ones that do carry out their shares"""
    p = params("paper" if arm == "large table" else arm)
    if arm == "large table":
        p.n_beta, p.iters = 4096, 7
    p.resident = B.SOAR_RESIDENT_NEVER
    ws = weights_of((170000, 170001, 5), torch.bfloat16, 8)
    outs, descs = outputs(ws, p)
    space = B.new_batch_workspace(descs, p, DEV)
    want, wanted = outputs(ws, p)
    B.quantize_batch(wanted, p, B.new_batch_workspace(wanted, p, DEV))
    torch.cuda.synchronize()
    assert max(int(a.iters_run.item()) for a in want) > 4
    hip = ctypes.CDLL("libamdhip64.so")
    stream, mask = ctypes.c_void_p(), (ctypes.c_uint32 * 8)(*[0xFFFFFFFF, 0xFFFFFFFF, 0, 0, 0, 0, 0, 0])
    assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(stream), 8, mask) == 0
    try:
        with torch.cuda.stream(torch.cuda.ExternalStream(stream.value)):
            for turn in range(3):
                for o in outs:
                    o.codes.fill_(0xAA)
                B.quantize_batch(descs, p, space)
                torch.cuda.synchronize()
                for k, (o, a) in enumerate(zip(outs, want)):
                    same(o, a, (turn, k))
    finally:
        torch.cuda.synchronize()
        hip.hipStreamDestroy(stream)
