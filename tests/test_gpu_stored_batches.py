"""Batches of stored tensors, around the number that shares a launch, and MXFP4 batches around the numbers of groups and tiles from which
they use two streams: every tensor as when it is handed over alone."""
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


# groups of eight: two, three below 2048 tiles, three from there on
@pytest.mark.gpu
@pytest.mark.parametrize("n,rows", [(9, 40), (16, 70000), (17, 30000), (17, 40000), (24, 22000)], ids=str)
def test_mx_batches_on_one_and_two_streams(n, rows):
    ws = weights_of(n, torch.bfloat16, lambda k: rows // (1 + k % 3) + k)
    outs = [B.mx_new_outputs(w.shape[0], w.shape[1], DEV) for w in ws]
    descs = [B.mx_make_desc(w, o) for w, o in zip(ws, outs)]
    p = B.soar_mx_default_params(n_beta=11)
    for turn in range(2):
        B.mx_quantize_batch(descs, p)
        torch.cuda.synchronize()
        for k, (w, o) in enumerate(zip(ws, outs)):
            one = B.mx_quantize(w, p)
            for f in ("codes", "scales", "sse", "status"):
                assert torch.equal(getattr(o, f), getattr(one, f)), (turn, k, f)
            o.codes.fill_(0)
