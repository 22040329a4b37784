"""Batches of stored tensors, around the number that shares a launch: every tensor as when it is handed over alone."""
import pytest
import torch

from paper_2605_12245_amd import binding as B

DEV = "cuda:0"


def weights_of(n, dtype, rows=lambda k: 1 + 37 * k % 300):
    gen = torch.Generator(device=DEV).manual_seed(n)
    return [(torch.randn((rows(k), 32 * (1 + k % 3)), generator=gen, device=DEV) * 0.02 * (k + 1)).to(dtype) for k in range(n)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("n", [1, 2, 7, 8, 9, 31, 32, 33, 47, 48, 49, 97])
def test_stored_batches_equal_every_tensor_alone(n, dtype):
    ws = weights_of(n, dtype)
    qs = [B.quantize(w) for w in ws]
    mx = [B.mx_quantize(w, B.soar_mx_default_params(dss=False)) for w in ws]
    backs, mx_backs, sums = B.dequantize_batch(qs, dtype), B.mx_dequantize_batch(mx, dtype), B.recon_error_batch(ws, qs)
    for k in range(n):
        assert torch.equal(backs[k], B.dequantize(qs[k], dtype)), k
        assert torch.equal(mx_backs[k], B.mx_dequantize(mx[k], dtype)), k
        assert abs(sums[k].item() - qs[k].sse.item()) <= 1e-12 * qs[k].sse.item(), k

