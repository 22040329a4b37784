"""The compiled marshalling module: the errors that the Python checks raised before, and on the GPU the same results and lifetimes
as calls with buffers of their own."""
import os
import subprocess
import sys

import pytest
import torch

from paper_2605_12245_amd import binding as B

DEV = "cuda:0"


def test_module_is_built_and_bound():
    B.lib()
    assert B._host is not None
    with pytest.raises(TypeError, match="addresses"):
        B._host.bind(1, 2)
    with pytest.raises(ValueError, match="no address"):
        B._host.bind(*([0] * 7))


def test_errors_before_anything_is_enqueued():
    w = torch.zeros(4, 32)
    for call in (lambda: B.quantize(w), lambda: B.quantize_rtn_amax(w, torch.ones(1)), lambda: B.quantize_iter(w, B.soar_paper_params()),
                 lambda: B.mx_quantize(w, B.soar_mx_default_params())):
        with pytest.raises(RuntimeError, match="must live on the GPU"):
            call()
    q = B.Quantized(w, w, w, w, w)
    for call in (lambda: B.dequantize(q, torch.float16), lambda: B.mx_dequantize_batch([q], torch.float64)):
        with pytest.raises(TypeError, match="bfloat16 or float32"):
            call()
    assert B.recon_error_batch([], []).numel() == 0


def run_python(code):
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    return subprocess.run([sys.executable, "-c", code], cwd=root, capture_output=True, text=True, timeout=300)


def test_an_exception_of_the_library_arrives_with_the_interpreter_locked(tmp_path):
    """an entry point that throws in the place of the real one; a process of its own, which may end without a word otherwise"""
    src, so = tmp_path / "throws.cpp", tmp_path / "throws.so"
    src.write_text('#include <stdexcept>\nextern "C" int throws(int, const void *, void *) { throw std::runtime_error("no memory left"); }\n')
    subprocess.run(["g++", "-shared", "-fPIC", str(src), "-o", str(so)], check=True)
    r = run_python(f"""
import ctypes
from paper_2605_12245_amd import binding as B
B.lib()
f = ctypes.cast(ctypes.CDLL({str(so)!r}).throws, ctypes.c_void_p).value
B._host.bind(*([f] * 7))
try:
    B._host.dequantize([], False, False, 0)
except RuntimeError as e:
    print("caught:", e)
print("alive")
""")
    assert r.returncode == 0 and "caught: no memory left" in r.stdout and "alive" in r.stdout, (r.returncode, r.stdout, r.stderr[-400:])


def test_the_library_is_there_without_the_module():
    """as where the module was built for another torch or Python: the raw entry points need nothing of it"""
    r = run_python("""
import sys
sys.modules["paper_2605_12245_amd.soar_host"] = None          # the import fails
import torch
from paper_2605_12245_amd import binding as B
assert B.soar_version() >= 0x00010000
assert B.soar_workspace_bytes(64, 64, B.soar_default_params()) > 0
q = B.Quantized(*[torch.zeros(2, 2)] * 5)
for call in (lambda: B.dequantize(q), lambda: B.recon_error(torch.zeros(2, 32), q)):
    try:
        call()
    except RuntimeError as e:
        assert "soar_host could not be loaded" in str(e), e
        print("refused")
""")
    assert r.returncode == 0 and r.stdout.count("refused") == 2, (r.returncode, r.stdout, r.stderr[-800:])


def test_a_build_whose_module_does_not_load_is_an_error():
    r = run_python("""
import sys
sys.modules["paper_2605_12245_amd.soar_host"] = None
import __graft_entry__, oracle.build, paper_2605_12245_amd.build
oracle.build.build = paper_2605_12245_amd.build.build = lambda **more: None       # what is there has been built
__graft_entry__.build()
""")
    assert r.returncode != 0 and "soar_host could not be loaded" in r.stderr, (r.returncode, r.stdout, r.stderr[-800:])


@pytest.mark.gpu
def test_same_as_calls_that_bring_their_buffers():
    w = (torch.randn(37, 272, device=DEV) * 0.02).to(torch.bfloat16)[:, :256]
    p = B.soar_paper_params(iters=5)
    a, b = B.quantize_iter(w, p), B.quantize_iter(w, p, out=B.new_outputs(37, 256, DEV, 5))
    m, n = B.mx_quantize(w, B.soar_mx_default_params()), B.mx_quantize(w, B.soar_mx_default_params(), out=B.mx_new_outputs(37, 256, DEV))
    c, d = B.quantize(w, dss_radius=2), B.quantize(w, dss_radius=2, out=B.new_outputs(37, 256, DEV))
    amax = w.abs().max().float().reshape(1)
    e, f = B.quantize_rtn_amax(w, amax), B.quantize_rtn_amax(w, amax, out=B.new_outputs(37, 256, DEV))
    torch.cuda.synchronize()
    for x, y in ((a, b), (m, n), (c, d), (e, f)):
        for name in ("codes", "scales", "global_scale", "sse", "status", "iters_run", "sse_trace"):
            s, t = getattr(x, name), getattr(y, name)
            assert (s is None) == (t is None), name
            if s is not None:
                assert s.dtype == t.dtype and s.shape == t.shape and s.is_contiguous() and s.device == t.device, name
                assert torch.equal(torch.nan_to_num(s, nan=-1.0) if s.is_floating_point() else s,
                                   torch.nan_to_num(t, nan=-1.0) if t.is_floating_point() else t), name
    assert torch.equal(B.dequantize(c), B.dequantize_batch((c, e))[0]) and B.dequantize(c, torch.float32).dtype == torch.float32
    assert torch.equal(B.mx_dequantize(m), B.mx_dequantize_batch([m])[0])
    assert torch.equal(B.recon_error_batch((w, w), (c, e))[:1], B.recon_error(w, c))
    # a degenerate tensor: no iteration is carried out and no entry of the trace written
    z = B.quantize_iter(torch.zeros_like(w), p)
    torch.cuda.synchronize()
    assert int(z.iters_run.item()) == 0 and bool(z.sse_trace.isnan().all())


@pytest.mark.gpu
def test_errors_with_tensors_on_the_gpu():
    w = torch.zeros(8, 64, device=DEV)
    for bad, error in ((w.half(), TypeError), (w.t(), ValueError), (w[0], ValueError)):
        for call in (lambda: B.quantize(bad), lambda: B.mx_quantize(bad, B.soar_mx_default_params()),
                     lambda: B.quantize_iter(bad, B.soar_paper_params()), lambda: B.quantize_rtn_amax(bad, torch.ones(1, device=DEV))):
            with pytest.raises(error):
                call()
    with pytest.raises(B.SoarError):
        B.quantize(torch.zeros(8, 40, device=DEV))             # columns: no multiple of 16
    with pytest.raises(B.SoarError):
        B.quantize(w, dss_radius=1000)
    for amax in (torch.ones(1), torch.ones(1, device=DEV).double(), 1.0):
        with pytest.raises(TypeError, match="amax_in"):
            B.quantize_rtn_amax(w, amax)


@pytest.mark.gpu
def test_a_maximum_that_is_missing_is_not_measured_instead():
    w = (torch.randn(16, 64, device=DEV) * 0.02).to(torch.bfloat16)
    for amax in (None, torch.empty(0, device=DEV)):
        for more in ({}, {"out": B.new_outputs(16, 64, DEV)}):
            with pytest.raises(TypeError, match="amax_in"):
                B.quantize_rtn_amax(w, amax, **more)


@pytest.mark.gpu
def test_outputs_have_storages_of_their_own():
    w = (torch.randn(64, 256, device=DEV) * 0.02).to(torch.bfloat16)
    q = B.quantize_iter(w, B.soar_paper_params(iters=5))
    outs = (q.codes, q.scales, q.global_scale, q.sse, q.status, q.iters_run, q.sse_trace)
    assert len({t.untyped_storage().data_ptr() for t in outs}) == len(outs)
    for t in outs:
        assert t.untyped_storage().nbytes() == t.numel() * t.element_size() and not t._is_view() and t.storage_offset() == 0
    q.sse_trace.resize_(2)
    assert 1 <= int(q.iters_run.item()) <= 5


@pytest.mark.gpu
def test_a_number_of_iterations_out_of_range_is_a_parameter_error():
    w = torch.zeros(8, 64, device=DEV)
    for iters in (2**31 - 1, 2**31 - 2):
        with pytest.raises(B.SoarError, match="soar_workspace_bytes"):
            B.quantize_iter(w, B.soar_paper_params(iters=iters))


@pytest.mark.gpu
def test_every_weight_has_a_stored_tensor():
    w = (torch.randn(16, 64, device=DEV) * 0.02).to(torch.bfloat16)
    q = B.quantize(w)
    with pytest.raises(ValueError, match="2 weights"):
        B.recon_error_batch([w, w], [q])
    assert torch.equal(B.recon_error_batch([w], [q, q]), B.recon_error(w, q))      # more of them: the first ones count
