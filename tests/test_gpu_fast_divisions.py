"""Reciprocals and divisions by known reciprocals take a short exact form while the global scale is within 2^60 of one:
tensors on both sides of that line, and at magnitudes where block scales reach both ends of the E4M3 range, against the
oracle, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_12245_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def wide(dtype, scale):
    """rows from far below the smallest block scale up to the tensor's maximum, with blocks of zeros"""
    g = torch.Generator(device="cpu").manual_seed(3)
    w = torch.randn(257, 272, generator=g) * torch.exp2(torch.arange(257).float() % 29 - 28.0)[:, None]
    w[::13, 16:48] = 0.0
    return (w.double() * 2.0 ** scale).to(dtype)


def host(w):
    return w.view(torch.int16).numpy().view(np.uint16) if w.dtype == torch.bfloat16 else w.numpy()


# the maximum is about 4 * 2^scale, the global scale about 2^(scale - 9.4)
@pytest.mark.parametrize("scale", [-52, -51, -50, -30, 0, 30, 68, 69, 70, 71])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "fp32"])
def test_both_sides_of_the_line(scale, dtype):
    w = wide(dtype, scale)
    d = w.to(DEV)
    for method, K in ((B.SOAR_METHOD_SOAR, 4), (B.SOAR_METHOD_RTN, 0)):
        ref = oracle.quantize(host(w), method, K)
        for resident in (B.SOAR_RESIDENT_AUTO, B.SOAR_RESIDENT_NEVER):
            p = B.soar_default_params(method, K)
            p.resident = resident
            o = B.new_outputs(257, 272, DEV)
            B.quantize_batch([B.make_desc(d, o)], p, B.new_batch_workspace([B.make_desc(d, o)], p, DEV))
            torch.cuda.synchronize()
            assert np.array_equal(o.codes.cpu().numpy(), ref.codes) and np.array_equal(o.scales.cpu().numpy(), ref.scales)
            assert np.float32(o.global_scale.item()) == ref.global_scale
    for arm, oarm in ((B.SOAR_METHOD_CJSO_ONLY, oracle.ARM_CJSO_ONLY), (B.SOAR_METHOD_SOAR, oracle.ARM_SOAR)):
        for resident in (B.SOAR_RESIDENT_AUTO, B.SOAR_RESIDENT_NEVER):
            p = B.soar_arm_params(arm, iters=3) if arm != B.SOAR_METHOD_SOAR else B.soar_paper_params(iters=3, n_beta=9)
            p.resident = resident
            ref = oracle.quantize_iter(host(w), arm=oarm, iters=p.iters, n_beta=p.n_beta, beta_lo=p.beta_lo, beta_hi=p.beta_hi,
                                       dd_mode=p.dd_mode, dss_radius=p.dss_radius, early_stop_rel=p.early_stop_rel)
            o = B.quantize_iter(d, p)
            torch.cuda.synchronize()
            assert int(o.iters_run.item()) == ref.trace["iters_run"]
            assert np.array_equal(o.codes.cpu().numpy(), ref.codes) and np.array_equal(o.scales.cpu().numpy(), ref.scales)
            assert np.float32(o.global_scale.item()) == ref.global_scale


def test_mxfp4_reciprocals_of_every_scale():
    """blocks over the whole exponent range: 1 / 2^(e - 127) is formed from the exponent"""
    g = torch.Generator(device="cpu").manual_seed(5)
    w = torch.randn(250, 64, generator=g).double() * torch.exp2(torch.arange(250).double() - 124.0)[:, None]
    w = w.float()
    ref = oracle.mxfp4_quantize(w.numpy(), False)
    o = B.mx_quantize(w.to(DEV), B.soar_mx_default_params(dss=False))
    torch.cuda.synchronize()
    assert np.array_equal(o.codes.cpu().numpy(), ref.codes) and np.array_equal(o.scales.cpu().numpy(), ref.scales)
