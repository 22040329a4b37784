"""Batches of small tensors, at the numbers of tiles (256 blocks) where their launches change shape: the bytes of a call with forced
shapes and those of every tensor handed over alone."""
import ctypes
import time

import pytest
import torch

from paper_2605_12245_amd import binding as B

DEV = "cuda:0"
FIELDS = ("codes", "scales", "global_scale", "status")


def weights_of(tiles, dtype, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    ws = [(torch.randn((t * 256 - k % 5, 16), generator=gen, device=DEV) * 0.02 * (k + 1)).to(dtype) for k, t in enumerate(tiles)]
    ws[0][::7] *= 30.0
    return ws


def run(ws, p, outs=None):
    outs = outs or [B.new_outputs(w.shape[0], w.shape[1], DEV) for w in ws]
    descs = [B.make_desc(w, o) for w, o in zip(ws, outs)]
    B.quantize_batch(descs, p, B.new_batch_workspace(descs, p, DEV))
    torch.cuda.synchronize()
    return outs


def same(got, want):
    for k, (a, b) in enumerate(zip(got, want)):
        for f in FIELDS:
            assert torch.equal(getattr(a, f), getattr(b, f)), (k, f)
        assert abs(a.sse.item() - b.sse.item()) <= 1e-12 * b.sse.item(), k       # binary64 sums in another order


# one group: 1, 1023 and 1024, 2047 and 2048, 4095 and 4096 tiles; several groups: eight tensors of 1023 to 16384 tiles in each
@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("tiles", [(1, 1), (1000, 23), (1000, 24), (2040, 7), (2047, 1), (4000, 95), (4000, 96), (127,) * 7 + (134,) * 9, (128,) * 17,
                                   (511,) * 11, (512,) * 10, (2047,) * 9, (2048,) * 9], ids=lambda t: f"{len(t)}x{t[0]}-{sum(t)}")
def test_small_groups_equal_forced_shapes(tiles, dtype):
    ws = weights_of(tiles, dtype, sum(tiles))
    for method in (B.SOAR_METHOD_SOAR, B.SOAR_METHOD_RTN):
        p = B.soar_default_params(method, 4 if method == B.SOAR_METHOD_SOAR else 0)
        got = run(ws, p)
        p.tiles_per_wg = 8
        same(got, run(ws, p))
        same([got[0], got[-1]], [B.quantize(w, method, p.dss_radius) for w in (ws[0], ws[-1])])


# ------------------------------------------------------------------ one launch for the whole batch (k_resident_batch)
def mixed(rows, dtype, seed, cols=32):
    """every other tensor a slice of wider rows"""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    return [(torch.randn((r, cols + 16 * (k % 2)), generator=gen, device=DEV) * 0.02 * (k % 3 + 1)).to(dtype)[:, :cols] for k, r in enumerate(rows)]


def launches_of(kernel, fn):
    B.soar_kernel_timing_enable(True)
    fn()
    torch.cuda.synchronize()
    n = B.soar_kernel_timing_read(kernel)[1]
    B.soar_kernel_timing_enable(False)
    return n


# rows of two blocks; workgroups of 256 x 1, 1024 x 1, x 2, x 4 blocks, full to the last place, one tensor of a single workgroup
# (no crossing), of 16 and 17, 64 and 65 (direct and grouped crossings), the most tensors a launch takes
BATCHES = [(1, 1), (128 * 100, 128 * 156), (128 * 100 + 1, 128 * 155, 5), (512 * 17, 512 * 16 - 3, 512 * 200, 7), (512 * 65, 1, 512 * 64),
           (512 * 300 - 1, 512 * 64, 512 * 65, 512 * 2), (512 * 4 * 100, 512 * 4 * 150, 512 * 4 * 6), tuple(range(1, 1600, 41))]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("rows", BATCHES, ids=lambda r: f"{len(r)}x{r[0]}-{sum(r)}")
def test_one_launch_for_a_batch_equals_several(rows, dtype):
    ws = mixed(rows, dtype, sum(rows))
    p = B.soar_default_params()
    outs = [B.new_outputs(w.shape[0], w.shape[1], DEV) for w in ws]
    assert launches_of(B.SOAR_KERNEL_RESIDENT, lambda: run(ws, p, outs)) == 1
    p.resident = B.SOAR_RESIDENT_NEVER
    want = run(ws, p)
    same(outs, want)
    p.resident = B.SOAR_RESIDENT_AUTO
    p.search_mode = B.SOAR_SEARCH_FULL
    same(run(ws, p), want)


def with_degenerate(rows, zero, bad, dtype, seed):
    """tensors of `rows` rows, an all-zero one (signed) and a non-finite one"""
    ws = mixed(tuple(rows) + (zero, bad), dtype, seed)
    ws[-2] = torch.zeros_like(ws[-2])
    ws[-2][zero - 1, 31] = -0.0
    ws[-1] = ws[-1].clone()
    ws[-1][bad // 2, 3] = float("nan")
    return ws


def same_with_degenerate(got, want):
    """but for the non-finite tensor, whose outputs are unspecified"""
    same(got[:-1], want[:-1])
    assert int(got[-2].status.item()) == B.SOAR_STATUS_ALLZERO and int(got[-1].status.item()) == B.SOAR_STATUS_NONFINITE


# workgroups of a tensor, for each of the four shapes: two-level crossings with and without a remainder, one workgroup (which waits for
# nobody), direct crossings; the degenerate ones span several
@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("unit", [128, 512, 1024, 2048], ids=["256x1", "1024x1", "1024x2", "1024x4"])
@pytest.mark.parametrize("sizes,zero,bad", [((100, 100.5, 0.1), 20.3, 17), ((16, 17, 64, 65, 0.1), 33, 19.5)], ids=["two large", "four"])
def test_a_batch_that_gives_up_is_finished(sizes, zero, bad, unit, dtype):
    """a bound of 1 us: the workgroups of the larger tensors leave, and do their tensor together"""
    ws = with_degenerate([max(1, int(unit * n)) for n in sizes], int(unit * zero), int(unit * bad), dtype, unit)
    p = B.soar_default_params()
    p.resident = B.SOAR_RESIDENT_NEVER
    want = run(ws, p)
    p.resident = B.SOAR_RESIDENT_AUTO
    several = [n for n, w in enumerate(ws) if w.shape[0] > unit]
    seen = set()
    for turn in range(12):
        p.resident_wait_us = 1
        p.search_mode = turn % 2                 # SOAR_SEARCH_AUTO and SOAR_SEARCH_FULL
        outs = [B.new_outputs(w.shape[0], w.shape[1], DEV) for w in ws]
        assert turn > 0 or launches_of(B.SOAR_KERNEL_RESIDENT, lambda: run(ws, p, outs)) == 1
        got = run(ws, p, outs)
        left = {n for n, o in enumerate(got) if int(o.status.item()) & B.SOAR_STATUS_GAVE_UP}
        assert left <= set(several)              # a single workgroup has nobody to wait for
        seen |= left
        for o in got:
            o.status &= ~B.SOAR_STATUS_GAVE_UP
        same_with_degenerate(got, want)
        if turn > 1 and seen == set(several):
            break
    assert seen == set(several)
    p.resident_wait_us = p.search_mode = 0
    same_with_degenerate(run(ws, p), want)


@pytest.mark.gpu
def test_a_batch_on_a_stream_of_few_compute_units_is_finished_by_them():
    """240 workgroups of which 64 find a place: several launches, as where there is no one launch for a batch; with a bound of the
    caller's, the one launch, which takes what the units need, not the seconds of a wait for the others.  A batch that the units hold takes one."""
    ws = with_degenerate([2048 * 100, 2048 * 100 + 1, 5], 2048 * 20, 2048 * 17, torch.bfloat16, 3)
    p = B.soar_default_params()
    p.resident = B.SOAR_RESIDENT_NEVER
    want = run(ws, p)
    p.resident = B.SOAR_RESIDENT_AUTO
    hip = ctypes.CDLL("libamdhip64.so")
    stream, mask = ctypes.c_void_p(), (ctypes.c_uint32 * 8)(*[0xFFFFFFFF, 0xFFFFFFFF, 0, 0, 0, 0, 0, 0])
    assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(stream), 8, mask) == 0
    try:
        with torch.cuda.stream(torch.cuda.ExternalStream(stream.value)):
            assert launches_of(B.SOAR_KERNEL_RESIDENT, lambda: run(ws, p)) == 0
            same_with_degenerate(run(ws, p), want)
            p.resident_wait_us = 50
            assert launches_of(B.SOAR_KERNEL_RESIDENT, lambda: run(ws, p)) == 1
            for turn in range(3):
                t = time.perf_counter()
                got = run(ws, p)
                took = time.perf_counter() - t
                left = [int(o.status.item()) & B.SOAR_STATUS_GAVE_UP for o in got]
                assert left[0] and left[1] and not left[2]
                for o in got:
                    o.status &= ~B.SOAR_STATUS_GAVE_UP
                same_with_degenerate(got, want)
                assert took < 1.0, took
            p.resident_wait_us = 0
            few = ws[:2] + ws[2:3]
            few = [w[:2048 * 25] for w in few]
            assert launches_of(B.SOAR_KERNEL_RESIDENT, lambda: run(few, p)) == 1
            p.resident = B.SOAR_RESIDENT_NEVER
            bare = run(few, p)
            p.resident = B.SOAR_RESIDENT_AUTO
            same(run(few, p), bare)
    finally:
        torch.cuda.synchronize()
        hip.hipStreamDestroy(stream)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "fp32"])
def test_one_launch_degenerate_tensors_and_workspaces_holding_anything(dtype):
    ws = mixed((513, 5000, 40, 9000, 300), dtype, 9)
    ws[0] = torch.zeros_like(ws[0])
    ws[2] = ws[2].clone()
    ws[2][3, 3] = float("nan")
    ws[4] = ws[4] * 2.0 ** -120
    p = B.soar_default_params()
    p.resident = B.SOAR_RESIDENT_NEVER
    want = run(ws, p)
    p.resident = B.SOAR_RESIDENT_AUTO
    outs = [B.new_outputs(w.shape[0], w.shape[1], DEV) for w in ws]
    descs = [B.make_desc(w, o) for w, o in zip(ws, outs)]
    space = B.new_batch_workspace(descs, p, DEV)
    for fill in (0x00, 0xFF, 0x5A, None, None):
        if fill is not None:
            space.fill_(fill)
        B.quantize_batch(descs, p, space)
        torch.cuda.synchronize()
        keep = [k for k in range(5) if k != 2]
        same([outs[k] for k in keep], [want[k] for k in keep])
        assert int(outs[2].status.item()) == B.SOAR_STATUS_NONFINITE
        never = B.soar_default_params()
        never.resident = B.SOAR_RESIDENT_NEVER
        B.quantize_batch(descs, never, space)               # the launches of the other path on the same workspace
        torch.cuda.synchronize()
        same([outs[k] for k in keep], [want[k] for k in keep])


@pytest.mark.gpu
def test_batches_that_keep_to_several_launches():
    p = B.soar_default_params()
    small = mixed((100, 200), torch.bfloat16, 1)
    both = [small[0], small[1].float()]
    many = mixed((3,) * 41, torch.bfloat16, 2)
    large = mixed((512 * 4 * 255, 512 * 4 + 1), torch.bfloat16, 3)
    for ws in (both, many, large):
        assert launches_of(B.SOAR_KERNEL_RESIDENT, lambda: run(ws, p)) == 0
        same(run(ws, p)[:2], [B.quantize(w) for w in ws[:2]])
    p.resident = B.SOAR_RESIDENT_NEVER
    assert launches_of(B.SOAR_KERNEL_RESIDENT, lambda: run(small, p)) == 0
