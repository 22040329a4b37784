"""Batches of small tensors, at the numbers of tiles (256 blocks) where their launches change shape: the bytes of a call with forced
shapes and those of every tensor handed over alone."""
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
