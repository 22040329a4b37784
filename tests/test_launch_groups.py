"""How a batch is cut into launch groups: 208 MiB of bf16 weights where they are read three times or more, 256 MiB otherwise
and where that holds the whole call; a workspace sized once serves every method."""
import pytest
import torch

from paper_2605_12245_amd import binding as B

DEV = "cuda:0"


def desc(rows, cols, dtype):
    return B.soar_tensor_desc(16, dtype, rows, cols, cols, 16, 16, 16, None, None, None, None, None)


@pytest.mark.parametrize("shapes", [[(12288, 4096)] * 2 + [(4096, 4096)] * 3, [(7680, 8192)] * 4, [(30, 16)] * 40,
                                    [(28672, 8192)] * 2, [(1, 16)], [(13623, 8000), (1, 16), (13624, 8000), (17, 16)] + [(1664, 8192)] * 9],
                         ids=lambda s: f"{len(s)}-{s[0][0]}x{s[0][1]}")
@pytest.mark.parametrize("dtype", [B.SOAR_BF16, B.SOAR_FP32], ids=["bf16", "fp32"])
def test_one_workspace_size_for_every_method(shapes, dtype):
    descs = [desc(r, c, dtype) for r, c in shapes]
    params = [B.soar_default_params(), B.soar_default_params(B.SOAR_METHOD_RTN, 0), B.soar_paper_params(),
              B.soar_arm_params(B.SOAR_METHOD_CJSO_ONLY), B.soar_arm_params(B.SOAR_METHOD_DSS_ONLY)]
    sizes = {B.soar_batch_workspace_bytes(descs, p) for p in params}
    assert len(sizes) == 1 and sizes.pop() > 0


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,method,sizes,groups", [
    (torch.bfloat16, B.SOAR_METHOD_SOAR, [120] * 4, 4), (torch.bfloat16, B.SOAR_METHOD_SOAR, [100] * 4, 2),
    (torch.bfloat16, B.SOAR_METHOD_SOAR, [120] * 2, 1), (torch.bfloat16, B.SOAR_METHOD_RTN, [120] * 4, 2),
    (torch.float32, B.SOAR_METHOD_SOAR, [120] * 4, 2), (torch.float32, B.SOAR_METHOD_RTN, [120] * 4, 2),
    (torch.float32, B.SOAR_METHOD_SOAR, [130] * 3, 3)], ids=lambda v: str(v).replace("torch.", ""))
def test_number_of_launch_groups(dtype, method, sizes, groups):
    cols = 4096
    ws = [torch.randn(m * (1 << 20) // cols // (2 if dtype == torch.bfloat16 else 4), cols, device=DEV).to(dtype) for m in sizes]
    p = B.soar_default_params(method, 4 if method == B.SOAR_METHOD_SOAR else 0)
    outs = [B.new_outputs(w.shape[0], cols, DEV) for w in ws]
    descs = [B.make_desc(w, o) for w, o in zip(ws, outs)]
    workspace = B.new_batch_workspace(descs, B.soar_default_params(), DEV)
    B.soar_kernel_timing_enable(True)
    B.quantize_batch(descs, p, workspace)
    torch.cuda.synchronize()
    launches = B.soar_kernel_timing_read(B.SOAR_KERNEL_SEARCH)[1]
    B.soar_kernel_timing_enable(False)
    assert launches == groups
    for w, o in zip(ws[1:], outs[1:]):
        one = B.quantize(w, method, p.dss_radius)
        assert torch.equal(o.codes, one.codes) and torch.equal(o.scales, one.scales) and torch.equal(o.global_scale, one.global_scale)
